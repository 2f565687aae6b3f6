"""Values that overflowed: what one session's infinities and NaN become, and that they stay with that session."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2209_01188_amd import binding, synth  # noqa: E402
from tests.gpu_util import DEV, midsize, to_dev, to_np  # noqa: E402

pytestmark = pytest.mark.gpu


def _span(H, nh, rows, ffn=256, seed=3):
    cfg = synth.SpanConfig("nonfinite", 1, H, nh, 1, 1, 1, 1, (20.0, 40.0), seed, ffn=ffn)
    span = binding.Span(1, H, nh, ffn, rows, 1e-5, 6.0, DEV)
    span.load_block(0, synth.block_params(cfg, 0))
    return span


# Attention, one cached key whose score is NaN beside a finite value row.  T = 1: the key range in one workgroup of 4
# waves (a lane group whose only key it is), of 8 waves, and split over workgroups.  T > 1: the form whose waves split
# the keys with 4 and 8 waves, and the one with shared tiles.
@pytest.mark.parametrize("d", [16, 64, 128])
@pytest.mark.parametrize("B,L,T,at", [(2, 3, 1, 0), (2, 3, 1, 2), (2, 300, 1, 7), (2, 1000, 1, 999), (2, 9, 5, 4), (2, 610, 3, 0), (64, 20, 2, 11)])
def test_a_key_with_a_nan_score_is_not_left_out(d, B, L, T, at):
    nh, r = 4, np.random.default_rng(d + L + T)
    span = _span(nh * d, nh, B * T)
    sessions = [span.open_session(L + T) for _ in range(B)]
    for i, s in enumerate(sessions):
        kv = r.standard_normal((2, nh, L, d)).astype(np.float16)
        if i == 0:
            kv[0, 1, at, 3] = np.nan
        s.import_kv(0, to_dev(kv))
    x = to_dev(r.standard_normal((B, T, nh * d)).astype(np.float16))
    y = to_np(span.prefill(sessions, x) if T > 1 else span.decode_step(sessions, x))
    assert np.isnan(y[0]).all() and np.isfinite(y[1:]).all()
    span.close()


# GeLU behind the up linear, one row, batched decode and both prefill forms (rows through the batched-decode kernel; output blocks, there
# also with the contraction split): an infinite outlier value times a positive weight is +infinity, GeLU of it too.
@pytest.mark.parametrize("M,H,ffn,form", [(1, 64, 256, None), (8, 64, 256, None), (100, 64, 256, "chunks"), (100, 64, 256, "blocks"), (70, 2048, 256, "blocks")])
def test_gelu_of_infinity(M, H, ffn, form):
    span = _span(H, max(4, H // 64), M, ffn)
    wq = to_np(span.export_weight(0, 2)[0])
    x = torch.zeros((M, H), dtype=torch.float16, device=DEV)
    x[M // 2, 5] = float("inf")
    with midsize(form):
        plain = to_np(span.debug_linear(0, 2, x)["y"])
        y = to_np(span.debug_linear(0, 2, x, binding.EPILOGUE_GELU)["y"])
    up = wq[:, 5] > 0
    assert (plain[M // 2, up] == np.inf).all() and (y[M // 2, up] == np.inf).all()
    rest = np.delete(y, M // 2, 0)
    assert np.isfinite(rest).all()
    span.close()


# One session's row that overflowed (NaN after the first LayerNorm), beside healthy sessions: these get the bits they get
# beside a row of zeros - above all no column becomes an outlier column because of it - and the row itself stays NaN.
# Every LayerNorm form: several rows per workgroup (narrow rows; 256 rows on), one row per workgroup; fp16 rows and codes.
@pytest.mark.parametrize("B,T,H,nh,form", [(8, 1, 1024, 16, None), (3, 2, 64, 4, None), (8, 1, 4096, 32, None), (5, 60, 256, 4, "chunks"),
                                           (5, 60, 256, 4, "blocks"), (4, 70, 4096, 32, None)])
@pytest.mark.parametrize("codes", [False, True])
def test_a_row_that_overflowed_stays_with_its_session(B, T, H, nh, form, codes):
    span = _span(H, nh, B * T, 512)
    cfg = synth.SpanConfig("nonfinite", 1, H, nh, B, T, 1, 2, (20.0, 40.0), 9, ffn=512)
    x = to_dev(synth.hidden_states(cfg, 0, B, T))
    x[1] = 0
    bad = x.clone()
    bad[1, 0, 7] = float("inf")
    n, block = x.numel(), 64
    q, am = torch.empty(n, dtype=torch.uint8, device=DEV), torch.empty(n // block, device=DEV)
    binding.petals_hidden_quantize(x, block, q, am)
    am_bad = am.clone()
    am_bad[T * H // block] = float("nan")
    out, counts = [], []
    for i in range(2):
        sessions = [span.open_session(T) for _ in range(B)]
        with midsize(form):
            y = span.prefill_q8(sessions, T, q, am_bad if i else am, block) if codes else span.prefill(sessions, bad if i else x)
        out.append(to_np(y))
        counts.append(to_np(span.outlier_counts()).tolist())
    assert counts[0] == counts[1]
    rest = [0] + list(range(2, B))
    assert np.isfinite(out[0]).all() and np.array_equal(out[0][rest].view(np.uint16), out[1][rest].view(np.uint16))
    assert np.isnan(out[1][1, 0]).all()
    span.close()
