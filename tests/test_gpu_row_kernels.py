"""LayerNorm of calls of many rows (a workgroup takes several rows and flags the outlier columns of all of them once)
and the rounding of fp64 to fp16, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
from paper_2209_01188_amd import binding, synth  # noqa: E402
from tests.gpu_util import DEV, build_pair, hidden_close, to_dev, to_np  # noqa: E402

pytestmark = pytest.mark.gpu


# rows: the last call of the other form and the smallest of this one, one row per workgroup or several, a last round of few rows; hidden: every
# register-chunk count and its edges
@pytest.mark.parametrize("M,H,nh", [(512, 64, 4), (1023, 1024, 16), (1025, 2048, 16), (2049, 192, 3), (255, 4096, 32),
                                    (256, 4096, 32), (513, 4096, 32), (520, 4160, 65), (700, 8192, 64), (515, 8256, 129), (513, 16384, 128)])
def test_layernorm_of_many_rows(M, H, nh):
    r = np.random.default_rng(M + H)
    span = binding.Span(1, H, nh, 64, M, device=DEV)
    p = {n: torch.zeros(s, dtype=torch.float32, device=DEV)
         for n, s in (("w_qkv", (3 * H, H)), ("w_dense", (H, H)), ("w_up", (64, H)), ("w_down", (H, 64)))}
    for n, s in (("b_qkv", 3 * H), ("b_dense", H), ("b_up", 64), ("b_down", H)):
        p[n] = torch.zeros(s, dtype=torch.float16, device=DEV)
    host = {n: r.normal(1.0 if n.endswith("g") else 0.0, 0.3, H).astype(np.float16) for n in ("ln1_g", "ln1_b", "ln2_g", "ln2_b")}
    span.load_block(0, dict(p, **{n: to_dev(v) for n, v in host.items()}))
    x = r.standard_normal((M, H)).astype(np.float16)
    x[r.integers(0, M, 3), r.integers(0, H, 3)] = 60.0         # outliers in a few rows only
    x[M - 1, H - 1] = -90.0                                    # and in the very last value
    got = span.debug_layernorm(0, 1, to_dev(x), want_quantized=True)
    ref = oracle.layernorm(x, host["ln2_g"], host["ln2_b"])
    assert np.array_equal(to_np(got["y"]).view(np.uint16), ref.view(np.uint16))
    assert np.array_equal(to_np(got["mask"]).astype(bool), (np.abs(ref.astype(np.float32)) >= 6.0).any(0))
    span.close()


# rows: the last call whose LayerNorm flags outlier columns as bits and the first that takes bytes, both LayerNorm forms;
# columns: none, the most of the fp64 path, one more (a list in memory), all; hidden: one group of 1024 columns and a piece
@pytest.mark.parametrize("M", [64, 65, 300])
@pytest.mark.parametrize("H,nh,n_out", [(1088, 17, 0), (1088, 17, 64), (4160, 65, 65), (1088, 17, 1088), (4160, 65, 2100)])
def test_outlier_columns_of_a_layernorm_reach_the_linear(M, H, nh, n_out):
    """The gain makes n_out columns outliers; the mask and the up linear's output are those of the oracle."""
    r = np.random.default_rng(M + H + n_out)
    cols = np.sort(r.choice(H, n_out, replace=False))
    if 0 < n_out < H:
        cols[-1] = H - 1                                       # the very last column
        cols = np.unique(cols)
    cfg = synth.SpanConfig("flags", 2, H, nh, 1, M, 1, 1, (20.0, 40.0), 4)
    osp, span, params = build_pair(cfg, max_rows=M)
    # block 0 leaves its rows to block 1, whose second LayerNorm is looked at: flags are those of block and LayerNorm
    gain = np.full(H, 0.5, np.float16)
    gain[cols] = 30.0
    p = dict(params[1], ln2_g=gain, ln2_b=np.zeros(H, np.float16))
    span.load_block(1, {k: to_dev(v) for k, v in p.items()})
    x = np.clip(r.standard_normal((M, H)), -4.0, 4.0).astype(np.float16)
    got = span.debug_layernorm(1, 1, to_dev(x), want_quantized=True)
    ref = oracle.layernorm(x, gain, np.zeros(H, np.float16))
    out = (np.abs(ref.astype(np.float32)) >= 6.0).any(0)
    assert out.sum() == len(cols)
    assert np.array_equal(to_np(got["y"]).view(np.uint16), ref.view(np.uint16))
    assert np.array_equal(to_np(got["mask"]).astype(bool), out)
    wq, sw = osp.get_weight(1, 2)
    Y, dbg = oracle.linear(ref, wq, sw, params[1]["b_up"], 6.0, 1, want_debug=True)
    assert np.array_equal(to_np(got["xq"]), dbg["xq"]) and np.array_equal(to_np(got["sx"]).view(np.uint32), dbg["sx"].view(np.uint32))
    lin = span.debug_linear(1, 2, to_dev(ref), 1)
    assert np.array_equal(to_np(lin["acc"]), dbg["acc"])
    hidden_close(to_np(lin["y"]), Y, "up linear behind the LayerNorm")
    span.close(); osp.destroy()


@pytest.mark.parametrize("B,T,H,block", [(2, 256, 64, 64), (3, 171, 192, 4096), (1, 1025, 128, 1024)])
def test_codes_of_many_rows_as_span_input(B, T, H, block):
    cfg = synth.SpanConfig("rows", 2, H, H // 32, B, T, 1, 1, (20.0, 40.0), 7)
    _, span, _ = build_pair(cfg, max_rows=B * T)
    x = to_dev(synth.hidden_states(cfg, 0, B, T))
    n = x.numel()
    q, am = torch.empty(n, dtype=torch.uint8, device=DEV), torch.empty(-(-n // block), dtype=torch.float32, device=DEV)
    binding.petals_hidden_quantize(x, block, q, am)
    dec = torch.empty_like(x)
    binding.petals_hidden_dequantize(q, am, block, dec)
    a = [span.open_session(T) for _ in range(B)]
    b = [span.open_session(T) for _ in range(B)]
    want = span.prefill(a, dec)
    got = span.prefill_q8(b, T, q, am, block)
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    for s, t in zip(a, b):
        for blk in range(2):
            assert torch.equal(s.export_kv(blk).view(torch.int16), t.export_kv(blk).view(torch.int16))
    span.close()


# Attention of calls that make few workgroups: 16-query workgroups whose waves split the keys (4 waves; 8 when the
# caches are long).  T: edges of the 16-query tiles; first: tokens already cached (an empty cache, a partial key tile,
# long enough for the 8-wave form); every head_dim.
@pytest.mark.parametrize("d", [16, 32, 64, 128])
@pytest.mark.parametrize("first,T", [(0, 2), (0, 17), (5, 15), (0, 130), (33, 65), (610, 16), (530, 33)])
def test_attention_of_few_workgroups(d, first, T):
    cfg = synth.SpanConfig("few", 1, 3 * d if d >= 64 else 4 * d, 3 if d >= 64 else 4, 2, T, 1, 1, (20.0, 40.0), d + T)
    osp, span, _ = build_pair(cfg, max_rows=2 * max(first, T))
    oses, gses = [osp.open_session(first + T) for _ in range(2)], [span.open_session(first + T) for _ in range(2)]
    for call, t in enumerate([first, T]):
        if t == 0:
            continue
        x = synth.hidden_states(cfg, call, 2, t)
        ref, got = osp.step(oses, x), to_np(span.prefill(gses, to_dev(x)))
        hidden_close(got, ref, "call %d" % call)
        assert (got.view(np.uint16) == ref.view(np.uint16)).mean() > 0.999
    span.close()
    osp.destroy()


# Attention of calls that fill the GPU: scores as int8 digit products for head_dim 64 and 128.  scale: QKV weights that
# keep every query and key below 127.5 (digits), push single ones over it (the fp64 form for their tiles) and most of
# them; T: one and several 64-query blocks per workgroup, an odd count of blocks; second call onto a filled cache.
# the last two shapes make few workgroups and take the form whose waves split the keys
@pytest.mark.parametrize("d,nh,B,T", [(64, 8, 32, 17), (128, 4, 64, 20), (64, 16, 8, 140), (128, 4, 3, 21), (64, 8, 2, 70)])
@pytest.mark.parametrize("scale", [1.0, 40.0, 400.0])
def test_attention_with_digit_scores(d, nh, B, T, scale):
    H = d * nh
    cfg = synth.SpanConfig("digits", 1, H, nh, B, T, 1, 1, (20.0, 40.0), d + T, ffn=256)
    osp = oracle.Span(1, H, nh, 256, 1e-5, 6.0)
    span = binding.Span(1, H, nh, 256, B * T, 1e-5, 6.0, DEV)
    p = synth.block_params(cfg, 0)
    p["w_qkv"] = p["w_qkv"] * np.float32(scale)
    osp.load_block(0, p)
    span.load_block(0, p)
    oses, gses = [osp.open_session(2 * T) for _ in range(B)], [span.open_session(2 * T) for _ in range(B)]
    for call in range(2):
        x = synth.hidden_states(cfg, call, B, T)
        ref, got = osp.step(oses, x), to_np(span.prefill(gses, to_dev(x)))
        hidden_close(got, ref, "call %d" % call)
        assert (got.view(np.uint16) == ref.view(np.uint16)).mean() > 0.999
    span.close()
    osp.destroy()
