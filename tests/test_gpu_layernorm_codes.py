"""LayerNorm and row quantizer in one launch (calls of few rows): the rows tell each other their outlier columns while they run,
or work them out by themselves when they have waited too long."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
from paper_2209_01188_amd import binding, synth  # noqa: E402
from tests.gpu_util import DEV, build_pair, hidden_close, midsize, to_dev, to_np  # noqa: E402

pytestmark = pytest.mark.gpu


def _span(H, nh, M, r):
    span = binding.Span(1, H, nh, 64, M, device=DEV)
    p = {n: torch.zeros(s, dtype=torch.float32, device=DEV)
         for n, s in (("w_qkv", (3 * H, H)), ("w_dense", (H, H)), ("w_up", (64, H)), ("w_down", (H, 64)))}
    for n, s in (("b_qkv", 3 * H), ("b_dense", H), ("b_up", 64), ("b_down", H)):
        p[n] = torch.zeros(s, dtype=torch.float16, device=DEV)
    ln = {n: r.normal(1.0 if n.endswith("g") else 0.0, 0.1, H).astype(np.float16) for n in ("ln1_g", "ln1_b", "ln2_g", "ln2_b")}
    span.load_block(0, dict(p, **{n: to_dev(v) for n, v in ln.items()}))
    return span, ln


# M: the fewest rows, a full and a ragged tile, the most of the batched-decode kernel, the first of several launches' rows and the
# most of this form; H: every number of threads and of columns per thread, and their edges; out: outlier columns per row, each row's
# own (none, one, the most of a record, one more, a tenth of the row)
@pytest.mark.parametrize("M,H,nh", [(2, 64, 4), (16, 1024, 16), (17, 1088, 17), (3, 2048, 16), (40, 2112, 33), (64, 4096, 32),
                                    (65, 1024, 16), (128, 1024, 16), (128, 4096, 32), (5, 4160, 65), (9, 8192, 64), (33, 8256, 129),
                                    (7, 16384, 128)])
def test_layernorm_codes(M, H, nh):
    r = np.random.default_rng(M + H)
    span, ln = _span(H, nh, M, r)
    for out in ([0] * 5, [1, 0, 0, 2, 0], [24, 1, 0, 25, 3], [H // 10, 24, 0, 25, H // 10]):
        x = np.clip(r.standard_normal((M, H)), -2.5, 2.5)
        for t in range(M):
            n = min(out[t % 5], H // 10)
            x[t, r.choice(H, n, replace=False)] = 40.0 * r.choice([-1.0, 1.0], n)
        x = x.astype(np.float16)
        y = oracle.layernorm(x, ln["ln2_g"], ln["ln2_b"])
        mask = (np.abs(y.astype(np.float32)) >= 6.0).any(0)
        reg = np.where(mask[None], np.float32(0), y.astype(np.float32))
        s = np.abs(reg).max(1)
        with np.errstate(divide="ignore"):
            codes = np.rint(reg * np.where(s > 0, np.float32(127) / s, np.float32(0)).astype(np.float32)[:, None])
        for patience in (10000, 0):
            binding.petals_debug_norm_patience(span.handle, patience)
            with midsize("chunks"):
                got = span.debug_layernorm(0, 1, to_dev(x), want_quantized=True)
            assert np.array_equal(to_np(got["y"]).view(np.uint16), y.view(np.uint16)), (out, patience)
            assert np.array_equal(to_np(got["mask"]).astype(bool), mask), (out, patience)
            assert np.array_equal(to_np(got["sx"]), s), (out, patience)
            assert np.array_equal(to_np(got["xq"]), codes.astype(np.int8)), (out, patience)
    span.close()


@pytest.mark.parametrize("B,T,H", [(5, 1, 1024), (20, 1, 4096), (1, 100, 1024), (2, 64, 192)])
@pytest.mark.parametrize("coded", [False, True])
def test_rows_that_do_not_wait_give_the_same_calls(B, T, H, coded):
    """Two blocks, fp16 rows and 8-bit codes, with rows that wait for each other and with rows that do not; a NaN row of one
    session leaves the others as they are."""
    cfg = synth.SpanConfig("codes", 2, H, H // 64, B, T, 1, 1, (20.0, 40.0), 3)
    osp, span, _ = build_pair(cfg, max_rows=B * T)
    x = synth.hidden_states(cfg, 0, B, T)
    q, am = torch.empty(x.size, dtype=torch.uint8, device=DEV), torch.empty(-(-x.size // 64), dtype=torch.float32, device=DEV)
    if coded:
        binding.petals_hidden_quantize(to_dev(x), 64, q, am)
        decoded = torch.empty(x.shape, dtype=torch.float16, device=DEV)
        binding.petals_hidden_dequantize(q, am, 64, decoded)
        x = to_np(decoded)
    want = osp.step([osp.open_session(T) for _ in range(B)], x)
    outs = []
    for patience, poison in ((10000, False), (0, False), (10000, True), (0, True)):
        binding.petals_debug_norm_patience(span.handle, patience)
        ses = [span.open_session(T) for _ in range(B)]
        with midsize("chunks"):
            if coded:                            # poison: the maximum of a block of 64 codes of the first row
                am_i = am.clone()
                if poison:
                    am_i[0] = np.nan
                y = span.prefill_q8(ses, T, q, am_i, 64)
            else:
                xi = x.copy()
                if poison:
                    xi[0, 0, 5] = np.nan
                y = span.prefill(ses, to_dev(xi))
        outs.append(to_np(y))
        for s in ses:
            s.close()
    assert np.array_equal(outs[0].view(np.uint16), outs[1].view(np.uint16))
    assert np.array_equal(outs[2].view(np.uint16), outs[3].view(np.uint16))
    hidden_close(outs[0], want)
    assert np.isnan(outs[2][0, 0]).all()
    if B > 1:
        assert np.isfinite(outs[2][1:]).all()
    span.close(); osp.destroy()


def _us(span, x, y):
    def call():
        binding.petals_debug_layernorm(span.handle, 0, 1, x, y)
    call()
    best = 1e30
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(8):
            call()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1000 / 8)
    return best


# Rows with one outlier column more than a record holds: the same columns (all of them, every row having its own) for the linear
# behind, which is most of either call.  (128 rows of 1024 took 69 us against 40, 128 of 4096 96 against 79.)
@pytest.mark.parametrize("M,H,nh", [(128, 1024, 16), (32, 2048, 16), (128, 4096, 32)])
def test_rows_with_many_outlier_columns_cost_little_more(M, H, nh):
    r = np.random.default_rng(H)
    span, _ = _span(H, nh, M, r)
    us = []
    with midsize("chunks"):
        for n in (24, 25):
            x = np.clip(r.standard_normal((M, H)), -2.5, 2.5).astype(np.float16)
            for t in range(M):
                x[t, r.choice(H, n, replace=False)] = 60.0
            x = to_dev(x)
            us.append(_us(span, x, torch.empty_like(x)))
    span.close()
    assert us[1] - us[0] < 8.0, us


# The rows that pad a call's last token tile are cleared by workgroups of their own.  (By the call's rows: two rows cleared seven each
# behind their own work, 2 rows of 14336 took 3 us more than 16.)
@pytest.mark.parametrize("H,nh", [(12288, 96), (14336, 112)])
def test_two_rows_take_no_longer_than_sixteen(H, nh):
    r = np.random.default_rng(H)
    span, _ = _span(H, nh, 16, r)
    us = []
    for M in (2, 16):
        x = to_dev(r.standard_normal((M, H)).astype(np.float16))
        y = torch.empty_like(x)
        _us(span, x, y)
        us.append(_us(span, x, y))
    span.close()
    assert us[0] < us[1] + 1.0, us


# The runs without patience above are there for the rows that work out the outlier columns of all rows by themselves: that they do
# shows in the time of 100 rows, each of which normalises them all (many times what waiting takes, which is a few us of the call).
def test_rows_without_patience_work_the_columns_out():
    M, H = 100, 4096
    r = np.random.default_rng(1)
    span, _ = _span(H, 32, M, r)
    x = to_dev(r.standard_normal((M, H)).astype(np.float16))
    y = torch.empty_like(x)
    us = []
    with midsize("chunks"):
        for patience in (10000, 0):
            binding.petals_debug_norm_patience(span.handle, patience)
            us.append(_us(span, x, y))
    span.close()
    assert us[1] > 3.0 * us[0], us


# A span of so many blocks that the tags of its LayerNorms come round: the same as with rows that look at no record
def test_more_layernorms_than_tags():
    blocks, H = 16386, 64
    span = binding.Span(blocks, H, 1, 64, 3, device=DEV)
    g = torch.Generator(device=DEV)
    g.manual_seed(1)
    p = {n: torch.empty(s, device=DEV).normal_(0.0, 0.02, generator=g)
         for n, s in (("w_qkv", (3 * H, H)), ("w_dense", (H, H)), ("w_up", (64, H)), ("w_down", (H, 64)))}
    for n, s in (("b_qkv", 3 * H), ("b_dense", H), ("b_up", 64), ("b_down", H), ("ln1_b", H), ("ln2_b", H)):
        p[n] = torch.zeros(s, dtype=torch.float16, device=DEV)
    p["ln1_g"] = p["ln2_g"] = torch.ones(H, dtype=torch.float16, device=DEV)
    for b in range(blocks):
        binding.petals_span_load_block(span.handle, b, p)
    x = torch.empty((1, 3, H), device=DEV).normal_(generator=g).half()
    x[0, 1, 5] = 40.0
    outs = []
    for patience in (10000, 0):
        binding.petals_debug_norm_patience(span.handle, patience)
        s = span.open_session(3)
        outs.append(to_np(span.prefill([s], x)))
        s.close()
    assert np.isfinite(outs[0]).all() and np.array_equal(outs[0].view(np.uint16), outs[1].view(np.uint16))
    span.close()
