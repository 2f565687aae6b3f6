"""The LM head for several rows of hidden states: exact int8 digit products, and the fp64 form that takes over where a
value does not fit four digits.  Against fp64 sums of the exact products."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
from paper_2209_01188_amd import binding  # noqa: E402
from tests.gpu_util import to_dev  # noqa: E402

pytestmark = pytest.mark.gpu

KINDS = ["embedding", "three digits' edge", "both branches", "four digits' edge", "one large tile", "large hidden rows", "tiny"]
SMALL = 0x33e0               # fp16 bits from which on a 16 x 64 piece of the matrix takes four digits


def _matrix(kind, r, V, H):
    E = r.standard_normal((V, H)) * 0.02
    if kind in ("three digits' edge", "both branches"):
        # the whole range of three digits, its largest values in some rows and in the first and last column
        top = np.array([SMALL - 1], np.uint16).view(np.float16)[0]
        E = np.clip(r.uniform(-0.2461, 0.2461, (V, H)), -float(top), float(top)).astype(np.float16)
        E[:: 3, 0], E[1:: 3, 0], E[:: 2, H - 1], E[1:: 2, H - 1], E[V // 2] = top, -top, -top, top, top
        E[V // 3] = -top
        assert (np.abs(E).view(np.uint16) < SMALL).all()
        if kind == "both branches":          # one value in every seventh row and third piece takes its piece to four digits
            E[:: 7, 5:: 192] = np.array([SMALL], np.uint16).view(np.float16)[0]
        return E
    elif kind == "four digits' edge":
        E = r.uniform(-127.4, 127.4, (V, H))
        E[::7] *= 1e-3
    elif kind == "one large tile":
        E[V // 2, H // 2] = 127.5
        E[V - 1, H - 1] = -65504.0
        E[0, 0] = 3.0
    elif kind == "tiny":
        E *= 1e-5
    return E.astype(np.float16)


# V: ragged last tile, V % 4 != 0 (no wide stores), one and two matrix tiles per wave, several rounds of workgroups;
# H: a single 64-column piece, ragged and full chunks, both register forms of the row kernel; M: edges of the row tiles
@pytest.mark.parametrize("V,H,M", [(17, 64, 2), (1001, 192, 15), (1000, 320, 16), (4099, 256, 17), (33000, 64, 32),
                                   (66000, 128, 2), (66002, 64, 16), (300, 4160, 33), (96, 16384, 3), (70000, 64, 31)])
@pytest.mark.parametrize("kind", KINDS)
def test_lm_head_of_several_rows(V, H, M, kind):
    r = np.random.default_rng(V + H + M)
    E = _matrix(kind, r, V, H)
    gain, bias = r.normal(1.0, 0.1, H), r.normal(0.0, 0.1, H)
    if kind == "large hidden rows":
        gain = gain * 100.0                      # some rows reach 127.5, at small H most do
    gain, bias = gain.astype(np.float16), bias.astype(np.float16)
    x = (r.standard_normal((M, H)) * 2.0).astype(np.float16)
    cl = binding.Client(to_dev(E), to_dev(gain), to_dev(bias), to_dev(gain), to_dev(bias), max_rows=M)
    nxt, logits = cl.lm_head(to_dev(x), want_logits=True)
    a = oracle.layernorm(x, gain, bias).astype(np.float64)
    want = a @ E.astype(np.float64).T
    # |error| of the reference's and of the kernel's fp64 sums, and one rounding to fp32
    bound = 2.0 ** -24 * np.abs(want) + 2.0 ** -50 * (np.abs(a) @ np.abs(E.astype(np.float64)).T)
    assert (np.abs(logits.cpu().numpy() - want) <= bound).all()
    n = nxt.cpu().numpy()
    best = want.max(1)
    assert (best - want[np.arange(M), n] <= bound.max(1)).all()
    assert np.array_equal(cl.lm_head(to_dev(x)).cpu().numpy(), n)
    cl.close()


# Matrix values are moved by 1/4 before they are cut: the last ones that four digits hold, and those behind them; chunks of 128
# columns over several rounds of workgroups, one of the chunks ragged
@pytest.mark.parametrize("value", [126.9375, -126.9375, 127.0, -127.0, 127.4375, -127.4375, -127.5, 128.0])
@pytest.mark.parametrize("V,H,M", [(70003, 192, 3), (1000, 64, 17), (5000, 448, 9)])
def test_lm_head_of_matrix_values_about_the_last_of_four_digits(V, H, M, value):
    r = np.random.default_rng(V + H)
    E = (r.standard_normal((V, H)) * 0.02).astype(np.float16)
    E[V // 2, H - 1] = E[17, 0] = E[V - 1, 33] = value
    x = (r.standard_normal((M, H)) * 2.0).astype(np.float16)
    _check(E, np.ones(H, np.float16), np.zeros(H, np.float16), x)


def _check(E, gain, bias, x, finite=True):
    V, (M, H) = E.shape[0], x.shape
    cl = binding.Client(to_dev(E), to_dev(gain), to_dev(bias), to_dev(gain), to_dev(bias), max_rows=M)
    logits = cl.lm_head(to_dev(x), want_logits=True)[1].cpu().numpy()
    cl.close()
    a = oracle.layernorm(x, gain, bias).astype(np.float64)
    with np.errstate(invalid="ignore"):
        want = a @ E.astype(np.float64).T
    if not finite:
        assert np.array_equal(np.isnan(logits), np.isnan(want)) and np.array_equal(logits[np.isinf(want)], want[np.isinf(want)])
        return
    bound = 2.0 ** -24 * np.abs(want) + 2.0 ** -50 * (np.abs(a) @ np.abs(E.astype(np.float64)).T)
    assert (np.abs(logits - want) <= bound).all()


# Hidden values that need digits 4 and 5: a gain of zero and the value as bias put them into chosen columns - every
# fp16 value near the edges of the digits, the ends of the range, any finite value; one column, columns of several
# pieces (the first and last one of a piece and of the row), all columns; beside matrix pieces of three and four digits.
@pytest.mark.parametrize("V,H,M", [(33, 64, 2), (1002, 640, 16), (1000, 4160, 17), (66000, 128, 5), (80, 16384, 2)])
@pytest.mark.parametrize("where", ["one", "several", "all"])
@pytest.mark.parametrize("kind", ["embedding", "four digits' edge"])
def test_lm_head_of_hidden_values_beyond_four_digits(V, H, M, where, kind):
    r = np.random.default_rng(V + H + M)
    E = _matrix(kind, r, V, H)
    gain, bias = r.normal(1.0, 0.1, H).astype(np.float16), r.normal(0.0, 0.1, H).astype(np.float16)
    edge = np.concatenate([np.arange(0x57f0, 0x5810), np.arange(0x5bf0, 0x5c10), [0x77f8, 0x77f7, 0x7bfe, 0x7bff]]).astype(np.uint16)
    values = np.concatenate([edge, edge | 0x8000, r.integers(0, 0x7c00, 64).astype(np.uint16)]).view(np.float16)
    cols = {"one": [H - 1], "several": sorted({0, 63, H // 2, (H - 1) // 64 * 64, H - 1}), "all": list(range(H))}[where]
    gain[cols] = 0
    bias[cols] = r.permutation(np.resize(values, max(len(cols), values.size)))[:len(cols)]
    _check(E, gain, bias, (r.standard_normal((M, H)) * 2.0).astype(np.float16))


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_lm_head_of_a_nonfinite_hidden_value(value):
    r = np.random.default_rng(6)
    V, H, M = 700, 192, 3
    gain, bias = np.ones(H, np.float16), np.zeros(H, np.float16)
    gain[70], bias[70], bias[3] = 0, value, 300.0
    _check(_matrix("embedding", r, V, H), gain, bias, r.standard_normal((M, H)).astype(np.float16), finite=False)


def test_a_dominant_feature_does_not_slow_the_lm_head_down():
    """One LayerNorm output of 127.5 or more costs one more look at its 64 columns, not another form of the product."""
    V, H, M = 100000, 4096, 4
    E = (torch.randn(V, H, device="cuda") * 0.02).to(torch.float16)
    zero, x = torch.zeros(H, dtype=torch.float16, device="cuda"), torch.randn(M, H, device="cuda").to(torch.float16)
    best = []
    for gain in (1.0, 500.0):
        g = zero + 1
        g[100] = gain
        cl = binding.Client(E, g, zero, g, zero, max_rows=M)
        best.append(float("inf"))
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                cl.lm_head(x, want_logits=True)
            b.record()
            b.synchronize()
            best[-1] = min(best[-1], a.elapsed_time(b) / 4)
        cl.close()
    assert best[1] < 1.4 * best[0], best       # 2.4 times as long when the fp64 form took over


def test_lm_head_takes_rows_at_any_address():
    r = np.random.default_rng(5)
    V, H, M = 500, 128, 6
    E = _matrix("embedding", r, V, H)
    one, zero = np.ones(H, np.float16), np.zeros(H, np.float16)
    cl = binding.Client(to_dev(E), to_dev(one), to_dev(zero), to_dev(one), to_dev(zero), max_rows=M)
    x = to_dev(r.standard_normal((M, H)).astype(np.float16))
    shifted = torch.empty(M * H + 1, dtype=torch.float16, device=x.device)[1:]
    shifted.copy_(x.view(-1))
    a = cl.lm_head(x, want_logits=True)[1]
    assert torch.equal(a, cl.lm_head(shifted.view(M, H), want_logits=True)[1])
    cl.close()


def test_one_row_calls_of_clients_of_different_widths_alternate():
    """The one-row form keeps its row in local memory, whose limit is set for the function, not for the client."""
    r = np.random.default_rng(8)
    V, clients = 300, []
    for H in (16384, 64, 9216):
        E = _matrix("embedding", r, V, H)
        one, zero = np.ones(H, np.float16), np.zeros(H, np.float16)
        x = r.standard_normal((1, H)).astype(np.float16)
        want = oracle.layernorm(x, one, zero).astype(np.float64) @ E.astype(np.float64).T
        clients.append((binding.Client(to_dev(E), to_dev(one), to_dev(zero), to_dev(one), to_dev(zero), max_rows=1), to_dev(x), want))
    for i in (0, 1, 0, 2, 1, 2, 0):
        cl, x, want = clients[i]
        got = cl.lm_head(x, want_logits=True)[1].cpu().numpy()
        assert (np.abs(got - want) <= 2.0 ** -23 * np.abs(want) + 1e-10).all(), i
    for cl, _, _ in clients:
        cl.close()
