"""Linears of 17 to 64 rows on wide outputs whose input has many outlier columns: exact int8 digit products in the pass
over the weights (gemm_digits.h), against the oracle and, where the call falls back, against the same bits."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
from paper_2209_01188_amd import binding  # noqa: E402
from tests.gpu_util import DEV, to_dev, to_np  # noqa: E402

pytestmark = pytest.mark.gpu
H = 12288                      # the narrowest output that takes this form


@pytest.fixture(scope="module", params=[4096, 4160])      # an even and an odd number of 64-column tiles
def span(request):
    F = request.param
    sp = binding.Span(1, H, H // 128, F, 64, device=DEV)
    g = torch.Generator(device=DEV)
    g.manual_seed(F)
    w = torch.empty((H, F), dtype=torch.float32, device=DEV).normal_(0.0, 0.02, generator=g)
    w[5] = 0.0                                             # scales of zero, below fp16's normal and subnormal range,
    w[6] *= 1e-3
    w[7] *= 1e-6
    w[8] *= 2e4                                            # large ones, a weight that is just no infinity
    w[9] *= 65504.0 / w[9].abs().max()
    w[10] *= 2.0 ** torch.randint(-12, 3, (F,), generator=g, device=DEV)      # and codes mostly near zero
    p = dict(w_qkv=torch.zeros((3 * H, H), device=DEV), w_dense=torch.zeros((H, H), device=DEV),
             w_up=torch.zeros((F, H), device=DEV), w_down=w)
    for n, s in (("b_qkv", 3 * H), ("b_dense", H), ("b_up", F), ("b_down", H), ("ln1_g", H), ("ln1_b", H), ("ln2_g", H), ("ln2_b", H)):
        p[n] = torch.zeros(s, dtype=torch.float16, device=DEV)
    sp.load_block(0, p)
    del p, w
    torch.cuda.empty_cache()
    yield sp
    sp.close()


def _input(M, F, n_out, kind, seed):
    r = np.random.default_rng(seed)
    x = np.clip(r.standard_normal((M, F)), -5.9, 5.9)
    cols = np.sort(r.choice(F, n_out, replace=False))
    if n_out < F:
        cols[0], cols[-1] = 0, F - 1
    x[:, cols] *= 2.0 ** r.uniform(-20.0, 0.0, (M, n_out))              # every digit plane has work
    x[r.integers(0, M, n_out), cols] = r.uniform(6.0, 127.4, n_out) * r.choice([-1.0, 1.0], n_out)
    x = x.astype(np.float16)
    if kind == "edge":
        x[M - 1, cols[-1]], x[0, cols[0]] = 127.4375, -127.4375        # the largest value of four digits
    if kind == "big":
        x[M - 1, cols[-1]] = 127.5                                    # one more: the fp64 form
    return x


# rows: token tiles full and ragged, the smallest and largest call of both kernels; outlier columns: around the line of one
# in 16 on either side, half, all
@pytest.mark.parametrize("M", [17, 32, 33, 47, 64])
@pytest.mark.parametrize("share,kind", [(1 / 16, ""), (1 / 16, "more"), (0.5, ""), (0.5, "edge"), (0.5, "big"), (1.0, "")])
def test_linear_with_many_outlier_columns(span, M, share, kind):
    F = span.shapes(3)[1]
    n_out = int(F * share) + (kind == "more")
    x = _input(M, F, n_out, kind, M * 7 + n_out)
    res = np.random.default_rng(M).standard_normal((M, H)).astype(np.float16)
    out = span.debug_linear(0, 3, to_dev(x), 2, to_dev(res))
    torch.cuda.synchronize()
    wq, sw = span.export_weight(0, 3)
    rows = np.unique(np.concatenate([np.arange(16), np.random.default_rng(M).integers(0, H, 48), [H - 1]]))
    Y, dbg = oracle.linear(x, to_np(wq)[rows], to_np(sw)[rows], np.zeros(len(rows), np.float16), 6.0, 2, res[:, rows].copy(), want_debug=True)
    assert int(dbg["mask"].sum()) == n_out
    assert np.array_equal(to_np(out["acc"])[:, rows], dbg["acc"])
    got = to_np(out["y"])[:, rows]
    same = got.view(np.uint16) == Y.view(np.uint16)
    assert same.all(), "%d of %d outputs differ, rows %s" % ((~same).sum(), same.size, rows[np.unique(np.argwhere(~same)[:, 1])][:8])


def test_outputs_that_leave_waves_and_workgroups_over():
    """12352 outputs: 386 pairs of panels, two of them in the last of 49 workgroups."""
    N, F = 12352, 4096
    g = torch.Generator(device=DEV)
    g.manual_seed(N)
    sp = binding.Span(1, N, N // 64, F, 64, device=DEV)
    p = dict(w_qkv=torch.zeros((3 * N, N), device=DEV), w_dense=torch.zeros((N, N), device=DEV), w_up=torch.zeros((F, N), device=DEV),
             w_down=torch.empty((N, F), device=DEV).normal_(0.0, 0.02, generator=g))
    for n, s in (("b_qkv", 3 * N), ("b_dense", N), ("b_up", F), ("b_down", N), ("ln1_g", N), ("ln1_b", N), ("ln2_g", N), ("ln2_b", N)):
        p[n] = torch.zeros(s, dtype=torch.float16, device=DEV)
    sp.load_block(0, p)
    del p
    wq, sw = (to_np(v) for v in sp.export_weight(0, 3))
    rows = np.concatenate([np.arange(16), np.arange(N - 160, N)])
    for M in (17, 32, 33, 64):
        x = _input(M, F, F // 2, "", M)
        out = sp.debug_linear(0, 3, to_dev(x))
        Y, dbg = oracle.linear(x, wq[rows], sw[rows], np.zeros(len(rows), np.float16), 6.0, 0, None, want_debug=True)
        assert np.array_equal(to_np(out["acc"])[:, rows], dbg["acc"]), M
        assert np.array_equal(to_np(out["y"])[:, rows].view(np.uint16), Y.view(np.uint16)), M
    sp.close()


@pytest.mark.parametrize("M", [17, 64])
def test_every_call_adds_the_shares_in_the_same_order(span, M):
    """The workgroup that finishes an output is another one from call to call; the sums and their order are not."""
    F = span.shapes(3)[1]
    x = to_dev(_input(M, F, F // 2, "", 5))
    y = torch.empty((40, M, H), dtype=torch.float16, device=DEV)
    for i in range(len(y)):
        binding.petals_debug_linear(span.handle, 0, 3, x, 0, None, None, None, None, None, y[i])
    assert (y.view(torch.int16) == y[0].view(torch.int16)).all()


def test_calls_that_may_go_to_digits_are_no_more_launches(span):
    """One row beyond the limit: most calls have few outlier columns, and a launch that finds nothing to do costs 2 us."""
    import ctypes
    hip = ctypes.CDLL("libamdhip64.so")
    F, nodes = span.shapes(3)[1], []
    for M in (16, 17):
        x, y = to_dev(_input(M, F, 3, "", M)), torch.empty((M, H), dtype=torch.float16, device=DEV)
        call = lambda: binding.petals_debug_linear(span.handle, 0, 3, x, 0, None, None, None, None, None, y)
        call()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(graph):
            call()
        n = ctypes.c_size_t(0)
        assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
        nodes.append(n.value)
        del graph
    assert nodes[0] == nodes[1] and nodes[0] >= 3, nodes


def test_weights_that_overflow_fp16_as_in_the_other_form(span):
    """Rows with |Wd| beyond fp16: infinities and NaN exactly as the fp64 form of a 16-row call gives them."""
    F = span.shapes(3)[1]
    g = torch.Generator(device=DEV)
    g.manual_seed(1)
    w = torch.empty((H, F), dtype=torch.float32, device=DEV).normal_(0.0, 0.02, generator=g)
    w[3] *= 1e7
    w[H - 1] *= 7e4 / w[H - 1].abs().max()
    other = binding.Span(1, H, H // 128, F, 64, device=DEV)
    p = dict(w_qkv=torch.zeros((3 * H, H), device=DEV), w_dense=torch.zeros((H, H), device=DEV),
             w_up=torch.zeros((F, H), device=DEV), w_down=w)
    for n, s in (("b_qkv", 3 * H), ("b_dense", H), ("b_up", F), ("b_down", H), ("ln1_g", H), ("ln1_b", H), ("ln2_g", H), ("ln2_b", H)):
        p[n] = torch.zeros(s, dtype=torch.float16, device=DEV)
    other.load_block(0, p)
    x = _input(32, F, F // 2, "", 3)
    x[16:] = x[:16]                                        # both halves hold every outlier column of the call
    y32 = to_np(other.debug_linear(0, 3, to_dev(x))["y"])
    y16 = to_np(other.debug_linear(0, 3, to_dev(x[:16]))["y"])
    for half in (y32[:16], y32[16:]):
        assert np.array_equal(half.astype(np.float32), y16.astype(np.float32), equal_nan=True)
    assert not np.isfinite(y16[:, 3].astype(np.float32)).all()
    other.close()
