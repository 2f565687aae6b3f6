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

KINDS = ["embedding", "three digits' edge", "four digits' edge", "one large tile", "large hidden rows", "tiny"]


def _matrix(kind, r, V, H):
    E = r.standard_normal((V, H)) * 0.02
    if kind == "three digits' edge":
        E = r.uniform(-0.4985, 0.4985, (V, H))
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
