"""The codec's wide kernels (aligned buffers, one comparison per value) and its general ones (any alignment) against
the oracle, bit for bit, at the sizes where they can go wrong: ragged ends, partial blocks, every block-size class,
buffers at odd addresses, and every fp16 value there is."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
from paper_2209_01188_amd import binding  # noqa: E402
from tests.gpu_util import DEV, to_np  # noqa: E402

pytestmark = pytest.mark.gpu


def _shifted(n, dtype, shift):
    """A device buffer of n elements that starts `shift` elements past a 256-byte boundary."""
    return torch.zeros(n + shift, dtype=dtype, device=DEV)[shift:]


def _roundtrip(x, block, shift):
    n = x.size
    q, am = oracle.hidden_quantize(x, block)
    xd = _shifted(n, torch.float16, shift)
    xd.copy_(torch.from_numpy(x))
    qd, yd = _shifted(n, torch.uint8, shift), _shifted(n, torch.float16, shift)
    amd = torch.empty(am.size, dtype=torch.float32, device=DEV)
    binding.petals_hidden_quantize(xd, block, qd, amd)
    binding.petals_hidden_dequantize(qd, amd, block, yd)
    assert np.array_equal(to_np(amd), am)
    assert np.array_equal(to_np(qd), q)
    assert np.array_equal(to_np(yd).view(np.uint16), oracle.hidden_dequantize(q, am, block).view(np.uint16))


@pytest.mark.parametrize("shift", [0, 1, 8, 16])
@pytest.mark.parametrize("block", [64, 4096, 4160, 8192, 16384])
@pytest.mark.parametrize("n", [1, 7, 8, 63, 4096, 4097, 20011])
def test_codec_sizes_and_alignments(n, block, shift):
    r = np.random.default_rng(n * 31 + block + shift)
    x = (r.standard_normal(n) * np.exp(r.uniform(-6, 3, n))).astype(np.float16)
    x[:: 97] = 0.0
    _roundtrip(x, block, shift)


def test_codec_every_fp16_value():
    bits = np.arange(0x7c00, dtype=np.uint16)
    pos = bits.view(np.float16)
    x = np.concatenate([pos, -pos])
    np.random.default_rng(3).shuffle(x)
    for block in (64, 4096, 16384):
        _roundtrip(x, block, 0)
    # small values next to one large maximum: quotients down to the smallest there are
    for top in (65504.0, 1.0, 0.1, 6e-8):
        y = np.where(np.abs(x.astype(np.float64)) <= top, x, np.float16(0)).astype(np.float16)
        y[::64] = np.float16(top)
        _roundtrip(y, 64, 0)


@pytest.mark.parametrize("block", [64, 1024, 4096, 8192, 16384])
def test_codec_of_infinities_and_nan(block):
    """Blocks that hold them: aligned and odd addresses give the same codes and maxima, the largest number counts."""
    r = np.random.default_rng(block)
    n = 5 * block + 40
    x = r.standard_normal(n).astype(np.float16)
    x[3], x[block + 5], x[2 * block - 1] = np.inf, np.nan, -np.nan
    x[2 * block:3 * block] = np.nan
    x[3 * block + 1], x[3 * block + 2] = np.nan, -np.inf
    x[n - 1] = np.nan
    out = []
    for shift in (0, 1):
        xd, qd = _shifted(n, torch.float16, shift), _shifted(n, torch.uint8, shift)
        xd.copy_(torch.from_numpy(x))
        amd = torch.empty(6, dtype=torch.float32, device=DEV)
        binding.petals_hidden_quantize(xd, block, qd, amd)
        out.append((to_np(qd), to_np(amd)))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    want = [np.fmax.reduce(np.abs(x[i * block:(i + 1) * block]).astype(np.float32), initial=0.0) for i in range(6)]
    assert np.array_equal(out[0][1], np.array(want, np.float32))


def test_codec_of_infinities_takes_as_long_as_of_numbers():
    block, n = 16384, 512 * 16384
    x = torch.randn(n, device=DEV).to(torch.float16)
    q, am = torch.empty(n, dtype=torch.uint8, device=DEV), torch.empty(n // block, device=DEV)

    def time_of_one():
        best = float("inf")
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                binding.petals_hidden_quantize(x, block, q, am)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) / 5)
        return best

    numbers = time_of_one()
    x[::block] = float("inf")
    assert time_of_one() < 4.0 * numbers      # a walk through the block by every thread: a hundred times as long
