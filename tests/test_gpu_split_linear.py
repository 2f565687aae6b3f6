"""Prefill-size linears whose output makes few blocks: the contraction is split over workgroups and a second kernel adds
the partial sums and finishes the outputs.  Bit for bit against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
from paper_2209_01188_amd import binding, synth  # noqa: E402
from tests.gpu_util import DEV, build_pair, hidden_close, midsize, to_dev, to_np  # noqa: E402

pytestmark = pytest.mark.gpu


# ffn: 32 k-tiles (the smallest that is split), an odd count in uneven shares, eight shares; M: edges of the row tiles and
# of the 128-row blocks, and rows beyond the mid-size range; n_out: no outlier columns, the fp64 path's edges (0, 5, 64),
# the digit products, and every column (no int8 part at all)
@pytest.mark.parametrize("ffn", [2048, 2112, 8192])
@pytest.mark.parametrize("M,n_out,epilogue", [(65, 0, 0), (128, 5, 2), (129, 64, 1), (351, 65, 2), (640, 7, 0), (200, -1, 2)])
def test_split_contraction(ffn, M, n_out, epilogue):
    H, nh = 192, 3
    cfg = synth.SpanConfig("split", 1, H, nh, 1, M, 1, 1, (20.0, 40.0), ffn + M, ffn=ffn)
    osp = oracle.Span(1, H, nh, ffn, 1e-5, 6.0)
    gsp = binding.Span(1, H, nh, ffn, M, 1e-5, 6.0, DEV)
    p = synth.block_params(cfg, 0)
    osp.load_block(0, p)
    gsp.load_block(0, p)
    r = np.random.default_rng(ffn * 7 + M)
    X = np.clip(r.standard_normal((M, ffn)), -5.9, 5.9)
    cols = np.arange(ffn) if n_out < 0 else r.choice(ffn, n_out, replace=False)
    X[r.integers(0, M, len(cols)), cols] = r.uniform(6.0, 30.0, len(cols)) * r.choice([-1, 1], len(cols))
    X = X.astype(np.float16)
    resid = (r.standard_normal((M, H)) * 4).astype(np.float16) if epilogue == 2 else None
    wq, sw = osp.get_weight(0, 3)
    Y, dbg = oracle.linear(X, wq, sw, p["b_down"], 6.0, epilogue, resid, want_debug=True)
    assert dbg["mask"].sum() == len(cols)
    with midsize("blocks"):
        out = gsp.debug_linear(0, 3, to_dev(X), epilogue, None if resid is None else to_dev(resid))
        torch.cuda.synchronize()
    assert np.array_equal(to_np(out["mask"]), dbg["mask"]) and np.array_equal(to_np(out["xq"]), dbg["xq"])
    assert np.array_equal(to_np(out["sx"]).view(np.uint32), dbg["sx"].view(np.uint32))
    assert np.array_equal(to_np(out["acc"]), dbg["acc"])
    assert np.array_equal(to_np(out["y"]).view(np.uint16), Y.view(np.uint16))
    gsp.close()
    osp.destroy()


# Four waves per workgroup: 64 rows per workgroup (more than 256 workgroups, one and two panels; the smallest calls still take
# eight) and up to 32 rows where the last of several rounds of 256 workgroups is half empty (one, two and four panels); ragged
# rows, k-tile counts below, at and above the waves, outlier columns in the last tile
@pytest.mark.parametrize("ffn,hidden,nh,M", [(f, h, n, M) for f, h, n in ((7232, 192, 3), (3136, 320, 5)) for M in (33, 64, 65, 130, 200, 500)] +
                         [(f, h, n, M) for f, h, n in ((16448, 192, 3), (8256, 320, 5), (4160, 192, 3)) for M in (2, 16, 17, 32)] + [(4160, 4096, 32, 16)])
def test_four_waves_per_workgroup(ffn, hidden, nh, M):
    cfg = synth.SpanConfig("waves", 1, hidden, nh, 1, M, 1, 1, (20.0, 40.0), 3, ffn=ffn)
    osp, gsp, params = build_pair(cfg, max_rows=M)
    r = np.random.default_rng(M + ffn)
    X = np.clip(r.standard_normal((M, hidden)) * 2, -5.9, 5.9)
    X[r.integers(0, M, 20), r.choice(hidden, 20, replace=False)] = 9.0
    X[M - 1, hidden - 1] = -40.0
    X = X.astype(np.float16)
    wq, sw = osp.get_weight(0, 2)
    Y, dbg = oracle.linear(X, wq, sw, params[0]["b_up"], 6.0, 1, want_debug=True)
    with midsize("chunks"):
        out = gsp.debug_linear(0, 2, to_dev(X), 1)
        torch.cuda.synchronize()
    assert np.array_equal(to_np(out["acc"]), dbg["acc"])
    assert np.array_equal(to_np(out["y"]).view(np.uint16), Y.view(np.uint16))
    gsp.close()
    osp.destroy()


# Every form of output block (panels of 16 features x token tiles of 16): 4 x 4 (one block, and as many as it takes at most), 8 x 8,
# 12 x 12, 6 x 12, 16 x 8, 16 x 16; one to seventeen k-tiles, last blocks ragged both ways, all three tails, without outlier
# columns, with a few, with more than the fp64 path takes, with all
@pytest.mark.parametrize("ffn,hidden,nh,M,n_out,epilogue", [
    (64, 64, 1, 65, 3, 0), (4096, 192, 3, 256, 0, 1), (4096, 192, 3, 241, 70, 2), (8320, 192, 3, 77, 5, 2), (8320, 192, 3, 128, 100, 1),
    (8320, 192, 3, 113, 192, 0), (13120, 192, 3, 525, 64, 1), (13248, 192, 3, 577, 9, 2), (16576, 1088, 17, 141, 66, 2), (16576, 1088, 17, 190, 2, 1),
    (16576, 320, 5, 653, 1, 2), (16576, 1088, 17, 397, 65, 0)])
def test_every_block_form(ffn, hidden, nh, M, n_out, epilogue):
    cfg = synth.SpanConfig("forms", 1, hidden, nh, 1, M, 1, 1, (20.0, 40.0), 5, ffn=ffn)
    osp, gsp, params = build_pair(cfg, max_rows=M)
    r = np.random.default_rng(M + ffn)
    X = np.clip(r.standard_normal((M, hidden)) * 2, -5.9, 5.9)
    cols = r.choice(hidden, n_out, replace=False)
    X[r.integers(0, M, n_out), cols] = r.uniform(6.0, 30.0, n_out) * r.choice([-1, 1], n_out)
    X = X.astype(np.float16)
    resid = (r.standard_normal((M, ffn)) * 4).astype(np.float16) if epilogue == 2 else None
    wq, sw = osp.get_weight(0, 2)
    Y, dbg = oracle.linear(X, wq, sw, params[0]["b_up"], 6.0, epilogue, resid, want_debug=True)
    with midsize("blocks"):
        out = gsp.debug_linear(0, 2, to_dev(X), epilogue, None if resid is None else to_dev(resid))
        torch.cuda.synchronize()
    assert dbg["mask"].sum() == n_out and np.array_equal(to_np(out["mask"]), dbg["mask"])
    assert np.array_equal(to_np(out["acc"]), dbg["acc"])
    assert np.array_equal(to_np(out["y"]).view(np.uint16), Y.view(np.uint16))
    gsp.close()
    osp.destroy()


# 32 rows per workgroup: one panel and sixteen waves (fewer k-tiles than waves, more, an odd number), two panels and four waves (one
# round of workgroups, several); ragged last rows, one workgroup of rows that holds a single one, residual and GeLU tails
@pytest.mark.parametrize("ffn,hidden,nh,which,M,epilogue", [
    (2112, 192, 3, 3, 33, 2), (4160, 192, 3, 3, 65, 0), (4160, 192, 3, 3, 64, 2), (8256, 192, 3, 3, 130, 2),
    (8192, 320, 5, 2, 100, 1), (4160, 192, 3, 2, 200, 2), (7232, 192, 3, 2, 225, 1), (7232, 192, 3, 2, 500, 0)])
def test_32_rows_per_workgroup(ffn, hidden, nh, which, M, epilogue):
    cfg = synth.SpanConfig("rows32", 1, hidden, nh, 1, M, 1, 1, (20.0, 40.0), 4, ffn=ffn)
    osp, gsp, params = build_pair(cfg, max_rows=M)
    N, K = gsp.shapes(which)
    r = np.random.default_rng(M + ffn)
    X = np.clip(r.standard_normal((M, K)) * 2, -5.9, 5.9)
    X[r.integers(0, M, 20), r.choice(K, 20, replace=False)] = 9.0
    X[M - 1, K - 1] = -40.0
    X = X.astype(np.float16)
    resid = (r.standard_normal((M, N)) * 4).astype(np.float16) if epilogue == 2 else None
    wq, sw = osp.get_weight(0, which)
    Y, dbg = oracle.linear(X, wq, sw, params[0]["b_up" if which == 2 else "b_down"], 6.0, epilogue, resid, want_debug=True)
    with midsize("chunks"):
        out = gsp.debug_linear(0, which, to_dev(X), epilogue, None if resid is None else to_dev(resid))
        torch.cuda.synchronize()
    assert np.array_equal(to_np(out["acc"]), dbg["acc"])
    assert np.array_equal(to_np(out["y"]).view(np.uint16), Y.view(np.uint16))
    gsp.close()
    osp.destroy()


# The fused QKV linear with 32 rows per workgroup (four waves for 192 columns, sixteen for 320): the rows of a workgroup behind the
# first belong to several sessions, whose keys and values go to their caches
@pytest.mark.parametrize("H,nh", [(192, 3), (320, 5)])
@pytest.mark.parametrize("B,T", [(4, 15), (3, 23), (2, 50), (33, 2)])
def test_32_rows_per_workgroup_append_to_the_caches(H, nh, B, T):
    cfg = synth.SpanConfig("rows32", 1, H, nh, B, T, 1, 1, (20.0, 40.0), 6)
    osp, gsp, _ = build_pair(cfg, max_rows=B * T)
    oses, gses = [osp.open_session(2 * T) for _ in range(B)], [gsp.open_session(2 * T) for _ in range(B)]
    for call in range(2):                                    # the second one behind cached keys
        x = synth.hidden_states(cfg, call, B, T)
        want = osp.step(oses, x)
        with midsize("chunks"):
            got = to_np(gsp.prefill(gses, to_dev(x)))
        hidden_close(got, want)
    for o, g in zip(oses, gses):
        assert np.array_equal(to_np(g.export_kv(0)).view(np.uint16), o.export_kv(0).view(np.uint16))
    gsp.close()
    osp.destroy()


# Which form a call of 65 to 512 rows takes: the estimate behind the choice must not miss the faster one by much.
# (n_out: outlier columns.  Where the forms are equal with few, blocks do better with many.)
@pytest.mark.parametrize("H,nh,which,M,n_out", [(1024, 16, 1, 320, 4), (1024, 16, 3, 448, 4), (1536, 12, 1, 257, 4), (2048, 16, 3, 160, 4), (4096, 32, 0, 320, 4),
                                                (4096, 32, 2, 512, 4), (2048, 16, 3, 352, 4), (2048, 16, 3, 352, 4096), (1536, 12, 3, 512, 600)])
def test_the_faster_form_is_chosen(H, nh, which, M, n_out):
    span = binding.Span(1, H, nh, 4 * H, M, device=DEV)
    p = {n: torch.randn(s, device=DEV) * 0.02 for n, s in (("w_qkv", (3 * H, H)), ("w_dense", (H, H)), ("w_up", (4 * H, H)), ("w_down", (H, 4 * H)))}
    p.update({n: torch.zeros(s, dtype=torch.float16, device=DEV) for n, s in
              (("b_qkv", 3 * H), ("b_dense", H), ("b_up", 4 * H), ("b_down", H), ("ln1_g", H), ("ln1_b", H), ("ln2_g", H), ("ln2_b", H))})
    span.load_block(0, p)
    N, K = span.shapes(which)
    x = torch.randn(M, K, device=DEV).clamp_(-5.0, 5.0)
    x[:, :n_out] = 30.0
    x, y, times = x.to(torch.float16), torch.empty((M, N), dtype=torch.float16, device=DEV), {}
    for form in ("chunks", "blocks", None):
        times[form] = float("inf")
        with midsize(form):
            for _ in range(4):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                torch.cuda._sleep(2000000)           # the calls queue up behind it: their time on the device, not the host's
                a.record()
                for _ in range(10):
                    binding.petals_debug_linear(span.handle, 0, which, x, binding.EPILOGUE_NONE, None, None, None, None, None, y)
                b.record()
                b.synchronize()
                times[form] = min(times[form], a.elapsed_time(b) / 10)
    span.close()
    assert times[None] <= 1.2 * min(times["chunks"], times["blocks"]), times


# Digit tiles of the outlier columns: the rows' column by column below four in seven, in runs from there on (the line on either
# side, all but one, all); values of five digits in one tile, rows of the last token tile missing
@pytest.mark.parametrize("n_out", [271, 272, 621, 622, 1000, 1087, 1088])
@pytest.mark.parametrize("big", [False, True])
def test_digit_tiles_of_many_columns(n_out, big):
    M, hidden, nh = 203, 1088, 17
    cfg = synth.SpanConfig("tiles", 1, hidden, nh, 1, M, 1, 1, (20.0, 40.0), 5, ffn=192)
    osp, gsp, params = build_pair(cfg, max_rows=M)
    r = np.random.default_rng(n_out)
    X = np.clip(r.standard_normal((M, hidden)), -5.9, 5.9) * 2.0 ** r.integers(-18, 1, (M, hidden))
    cols = r.choice(hidden, n_out, replace=False)
    X[r.integers(0, M, n_out), cols] = r.uniform(6.0, 127.0, n_out)
    if big:
        X[M - 1, cols[-1]] = -3000.0
    X = X.astype(np.float16)
    wq, sw = osp.get_weight(0, 1)
    resid = r.standard_normal((M, hidden)).astype(np.float16)
    Y, dbg = oracle.linear(X, wq, sw, params[0]["b_dense"], 6.0, 2, resid, want_debug=True)
    assert dbg["mask"].sum() == n_out
    with midsize("blocks"):
        out = gsp.debug_linear(0, 1, to_dev(X), 2, to_dev(resid))
        torch.cuda.synchronize()
    assert np.array_equal(to_np(out["y"]).view(np.uint16), Y.view(np.uint16))
    gsp.close()
    osp.destroy()


# The int8 product over the regular columns' gathered codes: one column below the line, on it, 65, 64, 63 and 1 regular columns
@pytest.mark.parametrize("n_out", [718, 719, 1023, 1024, 1025, 1087])
def test_regular_columns_by_themselves(n_out):
    M, hidden, nh = 1030, 1088, 17
    cfg = synth.SpanConfig("regular", 1, hidden, nh, 1, M, 1, 1, (20.0, 40.0), 6, ffn=192)
    osp, gsp, params = build_pair(cfg, max_rows=M)
    r = np.random.default_rng(n_out)
    X = np.clip(r.standard_normal((M, hidden)) * 2, -5.9, 5.9)
    X[r.integers(0, M, n_out), r.choice(hidden, n_out, replace=False)] = r.uniform(6.0, 127.0, n_out) * r.choice([-1, 1], n_out)
    X = X.astype(np.float16)
    wq, sw = osp.get_weight(0, 1)
    resid = r.standard_normal((M, hidden)).astype(np.float16)
    Y, dbg = oracle.linear(X, wq, sw, params[0]["b_dense"], 6.0, 2, resid, want_debug=True)
    assert dbg["mask"].sum() == n_out
    out = gsp.debug_linear(0, 1, to_dev(X), 2, to_dev(resid))
    torch.cuda.synchronize()
    assert np.array_equal(to_np(out["acc"]), dbg["acc"])
    assert np.array_equal(to_np(out["y"]).view(np.uint16), Y.view(np.uint16))
    gsp.close()
    osp.destroy()


# Outputs so narrow that the preparation has fewer waves of gathers than the column list has groups of 1024 (12, 37 and 61 for
# 64), and just as many as it needs (65)
@pytest.mark.parametrize("hidden,nh,M", [(64, 1, 128), (64, 1, 513), (896, 7, 65), (960, 15, 65)])
@pytest.mark.parametrize("n_out", [65, 700, 20000])
def test_column_list_of_wide_inputs_and_narrow_outputs(hidden, nh, M, n_out):
    F = 65536
    sp = binding.Span(1, hidden, nh, F, M, 1e-5, 6.0, DEV)
    g = torch.Generator(device=DEV)
    g.manual_seed(M)
    p = dict(w_qkv=torch.zeros((3 * hidden, hidden), device=DEV), w_dense=torch.zeros((hidden, hidden), device=DEV),
             w_up=torch.zeros((F, hidden), device=DEV), w_down=torch.empty((hidden, F), device=DEV).normal_(0.0, 0.02, generator=g))
    for n, s in (("b_qkv", 3 * hidden), ("b_dense", hidden), ("b_up", F), ("b_down", hidden), ("ln1_g", hidden), ("ln1_b", hidden), ("ln2_g", hidden), ("ln2_b", hidden)):
        p[n] = torch.zeros(s, dtype=torch.float16, device=DEV)
    sp.load_block(0, p)
    r = np.random.default_rng(n_out)
    X = np.clip(r.standard_normal((M, F), dtype=np.float32), -5.9, 5.9)
    cols = np.unique(np.concatenate([r.choice(F - 1024, n_out - 3, replace=False), [F - 1024, F - 500, F - 1]]))   # and the last group
    X[r.integers(0, M, len(cols)), cols] = r.uniform(6.0, 100.0, len(cols))
    X = X.astype(np.float16)
    with midsize("blocks"):
        out = sp.debug_linear(0, 3, to_dev(X), 0)
        torch.cuda.synchronize()
    wq, sw = sp.export_weight(0, 3)
    rows = np.unique(np.concatenate([np.arange(16), r.integers(0, hidden, 16), [hidden - 1]]))
    Y, dbg = oracle.linear(X, to_np(wq)[rows], to_np(sw)[rows], np.zeros(len(rows), np.float16), 6.0, 0, None, want_debug=True)
    assert dbg["mask"].sum() == len(cols)
    assert np.array_equal(to_np(out["acc"])[:, rows], dbg["acc"])
    assert np.array_equal(to_np(out["y"])[:, rows].view(np.uint16), Y.view(np.uint16))
    sp.close()


# Half of the columns are fewer than five in eight, and take less time (the products alone about 0.8 of it).
def test_time_of_digit_tiles_grows_with_the_columns():
    H, F, M = 4096, 16384, 65
    g = torch.Generator(device=DEV)
    g.manual_seed(H)
    span = binding.Span(1, H, 32, F, M, device=DEV)
    p = dict(w_qkv=torch.zeros((3 * H, H), device=DEV), w_dense=torch.zeros((H, H), device=DEV), w_up=torch.zeros((F, H), device=DEV),
             w_down=torch.empty((H, F), device=DEV).normal_(0.0, 0.02, generator=g))
    for n, s in (("b_qkv", 3 * H), ("b_dense", H), ("b_up", F), ("b_down", H), ("ln1_g", H), ("ln1_b", H), ("ln2_g", H), ("ln2_b", H)):
        p[n] = torch.zeros(s, dtype=torch.float16, device=DEV)
    span.load_block(0, p)
    y = torch.empty((M, H), dtype=torch.float16, device=DEV)
    times = []
    with midsize("blocks"):
        for n_out in (F // 2, F * 5 // 8):
            X = torch.empty((M, F), device=DEV).normal_(generator=g).clamp_(-5.0, 5.0)
            cols = torch.randperm(F, generator=g, device=DEV)[:n_out]
            X[torch.randint(0, M, (n_out,), generator=g, device=DEV), cols] = 9.0
            X = X.half()
            best = 1e9
            for _ in range(6):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                torch.cuda._sleep(1000000)
                a.record()
                for _ in range(6):
                    binding.petals_debug_linear(span.handle, 0, 3, X, 0, None, None, None, None, None, y)
                b.record()
                b.synchronize()
                best = min(best, a.elapsed_time(b) / 6)
            times.append(best)
    span.close()
    assert times[0] <= 0.9 * times[1], times


# Up to 32 rows, outputs of 513 to 640 workgroups of four panels: with a little larger output each takes the other form, which
# must not be the faster one.
@pytest.mark.parametrize("H,nh,small,large,M", [(10240, 80, 40960, 41984, 8), (12288, 96, 36864, 41984, 24)])
def test_a_smaller_output_is_no_slower(H, nh, small, large, M):
    g = torch.Generator(device=DEV)
    g.manual_seed(H)
    times = []
    for F in (small, large):
        span = binding.Span(1, H, nh, F, M, device=DEV)
        p = dict(w_qkv=torch.zeros((3 * H, H), device=DEV), w_dense=torch.zeros((H, H), device=DEV), w_down=torch.zeros((H, F), device=DEV),
                 w_up=torch.empty((F, H), device=DEV).normal_(0.0, 0.02, generator=g))
        for n, s in (("b_qkv", 3 * H), ("b_dense", H), ("b_up", F), ("b_down", H), ("ln1_g", H), ("ln1_b", H), ("ln2_g", H), ("ln2_b", H)):
            p[n] = torch.zeros(s, dtype=torch.float16, device=DEV)
        span.load_block(0, p)
        del p
        X = torch.empty((M, H), device=DEV).normal_(generator=g).clamp_(-5.0, 5.0).half()
        y = torch.empty((M, F), dtype=torch.float16, device=DEV)
        best = 1e9
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda._sleep(1000000)
            a.record()
            for _ in range(10):
                binding.petals_debug_linear(span.handle, 0, 2, X, 0, None, None, None, None, None, y)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) / 10)
        times.append(best)
        span.close()
        torch.cuda.empty_cache()
    assert times[0] <= 1.03 * times[1], times


# The outlier columns of the fp64 path beyond the first eight (or, in blocks of 4 x 4, 32) come several at a time, for all token tiles of a
# wave at once: last groups of one to four columns, every block form; from 53 on the larger ones go through the digit products
@pytest.mark.parametrize("ffn,hidden,nh,M", [(64, 192, 3, 65), (4096, 192, 3, 241), (8320, 192, 3, 77), (8320, 192, 3, 113), (13248, 192, 3, 577), (16576, 320, 5, 653), (16576, 192, 3, 1025)])
@pytest.mark.parametrize("n_out", [8, 9, 13, 20, 32, 33, 41, 52, 53, 64])
def test_outlier_columns_of_the_fp64_path(ffn, hidden, nh, M, n_out):
    cfg = synth.SpanConfig("fp64", 1, hidden, nh, 1, M, 1, 1, (20.0, 40.0), 7, ffn=ffn)
    osp, gsp, params = build_pair(cfg, max_rows=M)
    r = np.random.default_rng(M + n_out)
    X = np.clip(r.standard_normal((M, hidden)) * 2, -5.9, 5.9)
    X[r.integers(0, M, n_out), r.choice(hidden, n_out, replace=False)] = r.uniform(6.0, 30.0, n_out) * r.choice([-1, 1], n_out)
    X = X.astype(np.float16)
    wq, sw = osp.get_weight(0, 2)
    Y, dbg = oracle.linear(X, wq, sw, params[0]["b_up"], 6.0, 1, want_debug=True)
    with midsize("blocks"):
        out = gsp.debug_linear(0, 2, to_dev(X), 1)
        torch.cuda.synchronize()
    assert dbg["mask"].sum() == n_out
    assert np.array_equal(to_np(out["y"]).view(np.uint16), Y.view(np.uint16))
    gsp.close()
    osp.destroy()


# ... because they cost no more there: 60 columns against 100 (in fp64 62 us, when half blocks shared the contraction, then 77).
def test_sixty_outlier_columns_cost_no_more_than_a_hundred():
    H, F, M = 3072, 9216, 192
    g = torch.Generator(device=DEV)
    g.manual_seed(H)
    span = binding.Span(1, H, 24, F, M, device=DEV)
    p = {n: torch.empty(s, device=DEV).normal_(0.0, 0.02, generator=g) for n, s in (("w_qkv", (3 * H, H)), ("w_dense", (H, H)), ("w_up", (F, H)), ("w_down", (H, F)))}
    for n, s in (("b_qkv", 3 * H), ("b_dense", H), ("b_up", F), ("b_down", H), ("ln1_g", H), ("ln1_b", H), ("ln2_g", H), ("ln2_b", H)):
        p[n] = torch.zeros(s, dtype=torch.float16, device=DEV)
    span.load_block(0, p)
    y, times = torch.empty((M, F), dtype=torch.float16, device=DEV), []
    with midsize("blocks"):
        for n_out in (60, 100):
            x = torch.empty((M, H), device=DEV).normal_(generator=g).clamp_(-5.0, 5.0)
            x[:, torch.randperm(H, generator=g, device=DEV)[:n_out]] = 20.0
            x, best = x.half(), 1e9
            for _ in range(6):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                torch.cuda._sleep(1000000)
                a.record()
                for _ in range(6):
                    binding.petals_debug_linear(span.handle, 0, 2, x, 0, None, None, None, None, None, y)
                b.record()
                b.synchronize()
                best = min(best, a.elapsed_time(b) / 6)
            times.append(best)
    span.close()
    assert times[0] <= 1.1 * times[1], times
