"""GPU parity of the backward pass (paper Section 2.2: gradients w.r.t. activations through frozen 8-bit
blocks) against oracle/backward.py, element by element, through the C ABI."""
import numpy as np
import pytest
import torch

import oracle
from oracle import backward as ob
from paper_2209_01188_amd import binding, synth
from tests.gpu_util import DEV, hidden_close, say, to_dev, to_np

pytestmark = pytest.mark.gpu


def _pair(cfg, nb, rows, wscale, theta=6.0):
    """The same span in the oracle and on the GPU.  wscale multiplies the N(0, 0.02) weights so that, at
    these small widths, the attention and MLP branches carry as much gradient as at full width."""
    osp = oracle.Span(nb, cfg.hidden, cfg.n_heads, cfg.F, 1e-5, theta)
    gsp = binding.Span(nb, cfg.hidden, cfg.n_heads, cfg.F, rows, 1e-5, theta, DEV)
    params = []
    for b in range(nb):
        p = synth.block_params(cfg, b)
        for n in ("w_qkv", "w_dense", "w_up", "w_down"):
            p[n] = p[n] * np.float32(wscale)
        osp.load_block(b, p)
        gsp.load_block(b, p)
        params.append(p)
    return osp, gsp, params


def grad_close(got, ref, what="gradient", rel=3e-3, max_abs=2e-2):
    """Tolerance for gradients: the hidden-state tolerance (relative L2 <= 3e-3, |diff| <= 2e-2) made relative to the
    size of the row, because a gradient row is not of order one like a hidden state (the first token of a
    sequence collects gradient from every later token): relative L2 <= 3e-3 over the tensor and over every row,
    and per element |diff| <= 2e-2 * max(1, rms of the reference row)."""
    H = ref.shape[-1]
    g, r = got.astype(np.float64).reshape(-1, H), ref.astype(np.float64).reshape(-1, H)
    d = g - r
    relerr = np.linalg.norm(d) / max(np.linalg.norm(r), 1e-30)
    assert relerr <= rel, "%s rel-L2 %.3e" % (what, relerr)
    rown = np.linalg.norm(r, axis=1)
    rowrel = np.linalg.norm(d, axis=1) / np.maximum(rown, 1e-30)
    assert (rowrel <= rel).all(), "%s row rel-L2 %.3e at row %d" % (what, rowrel.max(), rowrel.argmax())
    bound = max_abs * np.maximum(1.0, rown / np.sqrt(H))[:, None]
    bad = np.abs(d) > bound
    assert not bad.any(), "%s max-abs %.3e at %s" % (what, np.abs(d).max(), np.argwhere(bad)[:4].tolist())
    return relerr, np.abs(d).max()


def _grad(cfg, B, T, seed):
    return np.random.default_rng([cfg.seed, 77, seed]).standard_normal((B, T, cfg.hidden)).astype(np.float16)


def _check(cfg, nb, B, T, wscale, seed=0, min_branch=0.05):
    osp, gsp, params = _pair(cfg, nb, B * T, wscale)
    try:
        X = synth.hidden_states(cfg, 0, B, T)
        dY = _grad(cfg, B, T, seed)
        Y_ref, dX_ref = ob.span_backward(osp, params, X, dY)
        (say if cfg.hidden >= 8192 else print)("backward case %s nb=%d B=%d T=%d" % (cfg.name, nb, B, T))
        Y, dX = gsp.backward(to_dev(X), to_dev(dY))
        torch.cuda.synchronize()
        Y, dX = to_np(Y), to_np(dX)
        hidden_close(Y, Y_ref, "forward output")
        rel, mx = grad_close(dX, dX_ref)
        print("  gradient rel-L2 %.2e max-abs %.2e" % (rel, mx), flush=True)
        # the case exercises the branches, not just the residual path
        branch = np.linalg.norm(dX_ref.astype(np.float64) - dY.astype(np.float64)) / np.linalg.norm(dY.astype(np.float64))
        print("  branch share %.2f" % branch, flush=True)
        assert branch > min_branch, branch
        return rel, mx
    finally:
        gsp.close()
        osp.destroy()


@pytest.mark.parametrize("B,T", [(1, 1), (1, 7), (2, 16), (3, 33), (1, 70), (2, 100), (64, 2), (5, 1), (1, 128)])
def test_backward_c1_shape(B, T):
    _check(synth.CONFIGS["C1"], 2, B, T, wscale=8.0, seed=B * 100 + T)


@pytest.mark.parametrize("hidden,heads,T", [(256, 8, 45), (512, 8, 80), (1024, 8, 37), (1024, 16, 129), (512, 4, 600)])
def test_backward_head_dims_32_64_128(hidden, heads, T):
    cfg = synth.scaled(synth.CONFIGS["C2"], hidden=hidden, n_heads=heads)
    _check(cfg, 2, 2, T, wscale=1.5 / (0.02 * np.sqrt(hidden)), seed=hidden + T)


def test_backward_odd_shape_six_heads_and_an_mlp_that_is_not_four_times_wider():
    cfg = synth.scaled(synth.CONFIGS["C2"], hidden=192, n_heads=6, ffn=448, n_outlier_dims=2)
    _check(cfg, 2, 3, 21, wscale=1.5 / (0.02 * np.sqrt(192)), seed=77)


def test_backward_c2_shape_deeper_span_several_sequences():
    _check(synth.CONFIGS["C2"], 6, 4, 64, wscale=1.5 / (0.02 * 32.0), seed=5)


def test_backward_forward_output_is_the_prefill_output_bit_for_bit():
    cfg = synth.CONFIGS["C2"]
    osp, gsp, _ = _pair(cfg, 2, 2 * 50, 2.0)
    try:
        X = to_dev(synth.hidden_states(cfg, 0, 2, 50))
        dY = to_dev(_grad(cfg, 2, 50, 1))
        Y, dX = gsp.backward(X, dY)
        sessions = [gsp.open_session(50) for _ in range(2)]
        Y2 = gsp.prefill(sessions, X)
        torch.cuda.synchronize()
        assert torch.equal(Y.view(torch.int16), Y2.view(torch.int16))
        # without a buffer for the forward output the gradient is the same bits
        none, dX_only = gsp.backward(X, dY, want_output=False)
        torch.cuda.synchronize()
        assert none is None and torch.equal(dX_only.view(torch.int16), dX.view(torch.int16))
        # a second call on the same store gives the same bits (nothing carried over between calls)
        store = torch.empty(binding.petals_span_backward_bytes(gsp.cfg, 2, 50), dtype=torch.uint8, device=DEV)
        a = gsp.backward(X, dY, store=store)[1].clone()
        b = gsp.backward(X, dY, store=store)[1]
        torch.cuda.synchronize()
        assert torch.equal(a.view(torch.int16), b.view(torch.int16)) and torch.equal(a.view(torch.int16), dX.view(torch.int16))
    finally:
        gsp.close()
        osp.destroy()


def test_backward_weight_cache_gives_the_same_bits_and_follows_a_reloaded_block():
    cfg = synth.scaled(synth.CONFIGS["C2"], hidden=512, n_heads=8)
    osp, gsp, params = _pair(cfg, 2, 2 * 40, 3.0)
    try:
        X = to_dev(synth.hidden_states(cfg, 0, 2, 40))
        g = to_dev(_grad(cfg, 2, 40, 3))
        _, plain = gsp.backward(X, g)
        gsp.attach_backward_cache()
        _, first = gsp.backward(X, g)          # fills the cache
        _, second = gsp.backward(X, g)         # reads it
        torch.cuda.synchronize()
        assert torch.equal(plain.view(torch.int16), first.view(torch.int16))
        assert torch.equal(plain.view(torch.int16), second.view(torch.int16))
        # new weights in block 1: the cached tiles of that block must not be used any more
        p = dict(params[1])
        p["w_up"] = p["w_up"] * np.float32(0.5)
        gsp.load_block(1, p)
        osp.load_block(1, p)
        params[1] = p
        _, third = gsp.backward(X, g)
        torch.cuda.synchronize()
        _, ref = ob.span_backward(osp, params, to_np(X), to_np(g))
        grad_close(to_np(third), ref)
        assert not torch.equal(third.view(torch.int16), plain.view(torch.int16))
        gsp.attach_backward_cache(False)
        _, fourth = gsp.backward(X, g)
        torch.cuda.synchronize()
        assert torch.equal(third.view(torch.int16), fourth.view(torch.int16))
    finally:
        gsp.close()
        osp.destroy()


def test_backward_is_linear_in_the_incoming_gradient_and_zero_for_zero():
    cfg = synth.CONFIGS["C1"]
    osp, gsp, _ = _pair(cfg, 2, 24, 8.0)
    try:
        X = to_dev(synth.hidden_states(cfg, 0, 2, 12))
        g = to_dev(_grad(cfg, 2, 12, 2))
        _, d0 = gsp.backward(X, torch.zeros_like(g))
        _, d1 = gsp.backward(X, g)
        _, d2 = gsp.backward(X, g * 2)
        torch.cuda.synchronize()
        assert torch.count_nonzero(d0) == 0
        r = torch.linalg.norm(d2.double() - 2 * d1.double()) / torch.linalg.norm(d2.double())
        assert r < 2e-3, float(r)
    finally:
        gsp.close()
        osp.destroy()


def test_backward_argument_errors():
    cfg = synth.CONFIGS["C1"]
    osp, gsp, _ = _pair(cfg, 1, 16, 1.0)
    try:
        X = to_dev(synth.hidden_states(cfg, 0, 2, 8))
        g = torch.zeros_like(X)
        store = torch.empty(binding.petals_span_backward_bytes(gsp.cfg, 2, 8), dtype=torch.uint8, device=DEV)
        out = torch.empty_like(X)
        with pytest.raises(binding.PetalsError):                 # aliasing
            binding.petals_span_backward(gsp.handle, store, X, g, None, g)
        with pytest.raises(binding.PetalsError):                 # more rows than the span was created for
            binding.petals_span_backward_bytes(gsp.cfg, 3, 8)
        X3 = to_dev(synth.hidden_states(cfg, 0, 3, 8))
        with pytest.raises(binding.PetalsError):
            binding.petals_span_backward(gsp.handle, store, X3, torch.zeros_like(X3), None, torch.empty_like(X3))
        binding.petals_span_backward(gsp.handle, store, X, g, None, out)     # still usable afterwards
        torch.cuda.synchronize()
    finally:
        gsp.close()
        osp.destroy()


@pytest.mark.parametrize("wscale", [0.5, 1.0])
def test_backward_c4_width_one_block_ragged_rows(wscale):
    """One BLOOM-176B-shaped block, 2 sequences of 40 tokens: 80 rows take the same LDS-pipelined kernels as the
    benchmark's 4096-row calls (more than 64 rows), with a ragged last row tile.  With the recipe's weights
    (wscale 1) the dense and down linears see thousands of outlier columns (the forward pass adds them through
    exact int8 digit products); with weights half as large every linear stays at 64 outlier columns or fewer.
    The full tolerance applies either way."""
    cfg = synth.CONFIGS["C4"]
    _check(cfg, 1, 2, 40, wscale=wscale, seed=9, min_branch=0.2)


def test_backward_products_at_full_size_sampled_against_the_oracle():
    """The four backward products of a BLOOM-176B-shaped block at the benchmark's 4096 rows (8 x 512), in the launch
    configuration bench.py times: the oracle's definition dX = dY Wd evaluated for a sample of rows and columns
    (first and last tiles included)."""
    cfg = synth.CONFIGS["C4"]
    B, T = 8, 512
    M = B * T
    p = synth.block_params_device(cfg, 0, DEV)
    gsp = binding.Span(1, cfg.hidden, cfg.n_heads, cfg.F, M, 1e-5, 6.0, DEV)
    gsp.load_block(0, p)
    store = torch.empty(binding.petals_span_backward_bytes(gsp.cfg, B, T), dtype=torch.uint8, device=DEV)
    r = np.random.default_rng(21)
    gen = torch.Generator(device=DEV)
    try:
        for which, wname in ((3, "w_down"), (2, "w_up"), (0, "w_qkv"), (1, "w_dense")):
            N, K = gsp.shapes(which)
            wq, sw = oracle.quantize_weight(p[wname].cpu().numpy())
            gen.manual_seed(100 + which)
            dY = torch.empty((M, N), dtype=torch.float32, device=DEV).normal_(0.0, 1.0, generator=gen).to(torch.float16)
            dX = torch.empty((M, K), dtype=torch.float32, device=DEV)
            say("backward product of linear %d: [%d, %d] x [%d, %d]" % (which, M, N, N, K))
            binding.petals_debug_backward_product(gsp.handle, store, B, T, 0, which, dY, dX)
            torch.cuda.synchronize()
            rows = np.unique(np.concatenate([[0, 15, 16, 255, 256, M - 1], r.choice(M, 18, replace=False)]))
            cols = np.unique(np.concatenate([np.arange(16), [K - 16, K - 1], r.choice(K, 40, replace=False)]))
            Wd = ob.dequantized_weight(wq[:, cols], sw)                       # [N, len(cols)]
            ref = to_np(dY[torch.as_tensor(rows, device=DEV)]).astype(np.float64) @ Wd
            got = to_np(dX[torch.as_tensor(rows, device=DEV)][:, torch.as_tensor(cols, device=DEV)]).astype(np.float64)
            rel = np.linalg.norm(got - ref) / np.linalg.norm(ref)
            assert rel < 2e-6, (which, rel)                                   # fp32 accumulation of exact products
            assert np.abs(got - ref).max() < 1e-4 * np.sqrt((ref ** 2).mean()) * 10, (which, np.abs(got - ref).max())
            del wq, dY, dX
    finally:
        gsp.close()


def test_backward_full_size_call_is_deterministic_linear_and_keeps_the_prefill_output():
    """Properties that hold at any size, on 4096 rows (8 x 512) of two BLOOM-176B-shaped blocks: the same call twice
    gives the same bits, a zero gradient stays zero, doubling the incoming gradient doubles the result up to fp16
    rounding, and the forward output is the prefill output bit for bit."""
    cfg = synth.CONFIGS["C4"]
    B, T, nb = 8, 512, 2
    gsp = binding.Span(nb, cfg.hidden, cfg.n_heads, cfg.F, B * T, 1e-5, 6.0, DEV)
    try:
        for b in range(nb):
            gsp.load_block(b, synth.block_params_device(cfg, b, DEV))
        X = to_dev(synth.hidden_states(cfg, 0, B, T))
        gen = torch.Generator(device=DEV)
        gen.manual_seed(7)
        # the recipe's weights multiply the gradient by about 15 per block: keep it inside the fp16 range
        g = (torch.empty(X.shape, dtype=torch.float32, device=DEV).normal_(0.0, 1.0, generator=gen) * 0.05).to(torch.float16)
        store = torch.empty(binding.petals_span_backward_bytes(gsp.cfg, B, T), dtype=torch.uint8, device=DEV)
        say("full-size backward calls")
        Y, d1 = gsp.backward(X, g, store=store)
        d1 = d1.clone()
        _, d1b = gsp.backward(X, g, store=store)
        _, d0 = gsp.backward(X, torch.zeros_like(g), store=store)
        _, d2 = gsp.backward(X, g * 2, store=store)
        sessions = [gsp.open_session(T) for _ in range(B)]
        Y2 = gsp.prefill(sessions, X)
        torch.cuda.synchronize()
        assert torch.isfinite(d1.float()).all() and torch.count_nonzero(d1) > d1.numel() // 2
        assert torch.equal(d1.view(torch.int16), d1b.view(torch.int16))
        assert torch.count_nonzero(d0) == 0
        rel = torch.linalg.norm(d2.double() - 2 * d1.double()) / torch.linalg.norm(d2.double())
        assert rel < 2e-3, float(rel)
        assert torch.equal(Y.view(torch.int16), Y2.view(torch.int16))
    finally:
        gsp.close()


def test_gelu_derivative_is_as_good_as_an_fp32_tanh():
    """GeLU' where it nearly vanishes, so that fp16 storage resolves its fp32 error.  Unit weight matrices, a zero input
    and no attention branch: pre-activation = up bias exactly, and a gradient with one entry per row comes out as
    dx[row, i != j] = -dpre[row, j] / (H sqrt(eps)) with dpre = fp16(dy GeLU'(p_j)).  Bound: a tanh within one unit in
    the last place below one (2^-24), times its weight in the formula, a few fp32 roundings of the rest, two fp16 ones."""
    H = T = 64
    eps, dy = 1e-5, 2048.0
    span = binding.Span(1, H, 4, H, T, eps, 6.0, DEV)
    eye, zero = torch.eye(H, device=DEV), torch.zeros(H, dtype=torch.float16, device=DEV)
    p = dict(w_qkv=torch.zeros((3 * H, H), device=DEV), w_dense=torch.zeros((H, H), device=DEV), w_up=eye, w_down=eye,
             b_qkv=torch.zeros(3 * H, dtype=torch.float16, device=DEV), b_dense=zero, b_down=zero,
             ln1_g=zero + 1, ln1_b=zero, ln2_g=zero + 1, ln2_b=zero)
    pre = np.arange(np.float16(-6.0).view(np.uint16) - np.float16(-4.1875).view(np.uint16), dtype=np.uint16)
    pre = (np.float16(-4.1875).view(np.uint16) + pre).view(np.float16)
    pre = pre[: pre.size // H * H]
    x, g = torch.zeros((1, T, H), dtype=torch.float16, device=DEV), torch.zeros((1, T, H), dtype=torch.float16, device=DEV)
    g[0, torch.arange(T), torch.arange(T)] = dy
    got = []
    for part in pre.reshape(-1, H):
        span.load_block(0, dict(p, b_up=to_dev(part)))
        dx = to_np(span.backward(x, g, want_output=False)[1])[0].astype(np.float64)
        got.append(np.where(np.arange(H) == 0, dx[:, 1], dx[:, 0]) * -(H * np.sqrt(eps)) / dy)
    span.close()
    P = pre.astype(np.float64)
    t = np.tanh(ob._C0 * (P + ob._C1 * P ** 3))
    weight = np.abs(0.5 - P * t * ob._C0 * (1.0 + 3.0 * ob._C1 * P * P))
    err = np.abs(np.concatenate(got) - ob.gelu_grad(P))
    bound = 2.0 ** -24 * weight + 2.0 ** -22 * np.abs(ob.gelu_grad(P)) + 2.0 ** -10 * (np.abs(ob.gelu_grad(P)) + 2.0 ** -24 * weight) + 2.0 ** -24 / dy
    assert (err <= bound).all(), (err / bound).max()
