"""One token of one session through a narrow span in one launch: against the oracle, and against the same step as separate
launches (which a profiled call takes)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
from paper_2209_01188_amd import binding, synth  # noqa: E402
from tests.gpu_util import DEV, hidden_close, to_dev, to_np  # noqa: E402

pytestmark = pytest.mark.gpu


def _config(blocks, H, nh, F):
    return synth.scaled(synth.CONFIGS["C4"], name="row-%d" % H, n_blocks=blocks, hidden=H, n_heads=nh, ffn=F)


# H, F: one column tile, ragged panel groups and wave shares, the widest row of either register form, a row form that only F
# asks for, F below H; L: no cached key, one, the edges of a wave's share, several blocks of keys per wave, several key ranges
@pytest.mark.parametrize("blocks,H,nh,F,L,theta", [
    (2, 64, 1, 256, 0, 6.0), (3, 128, 1, 64, 1, 6.0), (2, 192, 3, 448, 63, 6.0), (2, 1024, 16, 4096, 64, 6.0),
    (1, 1024, 8, 4096, 400, 0.5), (2, 960, 15, 4160, 129, 6.0), (2, 1088, 17, 4352, 512, 6.0), (2, 2048, 16, 8192, 300, 6.0),
    (1, 2048, 32, 1024, 1500, 0.0), (2, 2112, 33, 8448, 70, 6.0), (2, 3072, 24, 12288, 300, 6.0), (1, 2944, 46, 9216, 1200, 6.0),
    (1, 512, 8, 12288, 20, 6.0), (2, 3136, 49, 12544, 100, 6.0), (2, 4096, 32, 16384, 64, 6.0), (1, 4096, 64, 15360, 900, 6.0),
    (1, 1024, 8, 16384, 5, 0.5), (1, 1152, 9, 8192, 2500, 6.0), (1, 128, 2, 512, 3000, 6.0),
    # several ranges in several blocks, the last range with keys and (1024 columns, 4100 keys) without
    (3, 1024, 8, 4096, 1500, 6.0), (2, 2048, 32, 8192, 2100, 6.0), (2, 4096, 32, 16384, 1100, 6.0), (2, 1024, 8, 1024, 4100, 6.0),
    # from here on three quarters of the workgroups share the keys instead of half; two blocks
    (2, 4096, 32, 16384, 3068, 6.0), (2, 4096, 64, 1024, 3072, 6.0), (2, 1024, 16, 1024, 12290, 6.0)])
def test_a_row_in_one_launch(blocks, H, nh, F, L, theta):
    cfg = _config(blocks, H, nh, F)
    spans = [binding.Span(blocks, H, nh, F, 1, 1e-5, theta, DEV) for _ in range(2)]
    osp = oracle.Span(blocks, H, nh, F, 1e-5, theta)
    for b in range(blocks):
        p = synth.block_params_device(cfg, b, DEV)
        for s in spans:
            s.load_block(b, p)
        osp.load_block(b, {k: v.cpu().numpy() for k, v in p.items()})
    ses = [s.open_session(L + 6) for s in spans]
    ose = osp.open_session(L + 6)
    if L:
        for b in range(blocks):
            kv = synth.kv_prefix_device(cfg, b, 0, L, 2.4, DEV)
            for s in ses:
                s.import_kv(b, kv)
            ose.import_kv(b, kv.cpu().numpy())
    binding.petals_span_profile_begin(spans[1].handle, 4096)
    for i in range(3):
        x = synth.hidden_states(cfg, i + 1, 1, 1)
        want = osp.step([ose], x)
        one, apart = (to_np(s.decode_step([e], to_dev(x[:, 0])))[:, None] for s, e in zip(spans, ses))
        hidden_close(one, want, "step %d" % i)
        # the same integers and fp64 sums in another order: a value moves by at most an fp16 step where its sum lies on the
        # boundary between two, which one in 1e10 does
        assert np.array_equal(one.view(np.uint16), apart.view(np.uint16))
    for b in range(blocks):
        assert torch.equal(ses[0].export_kv(b), ses[1].export_kv(b))
    # the last step again from 8-bit codes
    q = torch.empty(H, dtype=torch.uint8, device=DEV)
    am = torch.empty(-(-H // 64), dtype=torch.float32, device=DEV)
    binding.petals_hidden_quantize(to_dev(x[:, 0]), 64, q, am)
    one, apart = (to_np(s.prefill_q8([e], 1, q, am, 64)) for s, e in zip(spans, ses))
    assert np.array_equal(one.view(np.uint16), apart.view(np.uint16))
    for s in spans:
        s.close()
    osp.destroy()


def test_rows_of_two_spans_on_two_streams():
    """Two such steps share the compute units, so neither has all of its workgroups resident: both get done, with the results
    that they have alone."""
    H, nh, F, blocks = 1024, 16, 4096, 4
    cfg = _config(blocks, H, nh, F)
    spans = [binding.Span(blocks, H, nh, F, 1, 1e-5, 6.0, DEV) for _ in range(2)]
    for b in range(blocks):
        p = synth.block_params_device(cfg, b, DEV)
        for s in spans:
            s.load_block(b, p)
    xs = [to_dev(synth.hidden_states(cfg, i, 1, 1)[:, 0]) for i in range(24)]
    alone = spans[0].open_session(32)
    want = [spans[0].decode_step([alone], x).clone() for x in xs]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in spans]
    ses, got = [s.open_session(32) for s in spans], [[], []]
    for x in xs:
        for k in range(2):
            with torch.cuda.stream(streams[k]):
                got[k].append(spans[k].decode_step([ses[k]], x))
    torch.cuda.synchronize()
    for k in range(2):
        for a, b in zip(got[k], want):
            assert torch.equal(a, b)
    for s in spans:
        s.close()


# Long caches are a matter of how many compute units read them: what a step takes more with 32768 keys than with 16384 (half of the
# units: 3.2 to 4.2 TB/s, three quarters as well as the separate launches 5.8).
@pytest.mark.parametrize("H,nh", [(3072, 48), (4096, 64), (4096, 32)])
def test_long_caches_stream(H, nh):
    span = binding.Span(1, H, nh, 64, 1, 1e-5, 6.0, DEV)
    cfg = _config(1, H, nh, 64)
    span.load_block(0, synth.block_params_device(cfg, 0, DEV))
    x = to_dev(synth.hidden_states(cfg, 1, 1, 1)[:, 0])
    us = []
    for L in (16384, 32768):
        s = span.open_session(L + 64)
        s.import_kv(0, torch.zeros((2, nh, L, H // nh), dtype=torch.float16, device=DEV))
        best = 1e30
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(12):
                span.decode_step([s], x)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 1000 / 12)
        us.append(best)
        s.close()
    rate = 16384 * H * 4 / (us[1] - us[0]) * 1e-6
    assert rate > 4.8, "%.1f and %.1f us: %.1f TB/s" % (us[0], us[1], rate)
    span.close()


def _given_up():
    n = torch.zeros(1, dtype=torch.int32, device=DEV)
    binding.petals_steps_given_up(n)
    return n.item()


@pytest.mark.parametrize("H,nh,L", [(1024, 16, 40), (1024, 8, 1200), (3072, 24, 64)])
def test_a_step_that_gives_up_says_so(H, nh, L):
    """Readers that may not wait at all: the launch ends, the output is no number, the call is counted once, and the span's next
    calls are as ever."""
    cfg = _config(2, H, nh, H)
    span = binding.Span(2, H, nh, H, 1, 1e-5, 6.0, DEV)
    kv = [synth.kv_prefix_device(cfg, b, 0, L, 2.4, DEV) for b in range(2)]
    for b in range(2):
        span.load_block(b, synth.block_params_device(cfg, b, DEV))
    x, before, outs = to_dev(synth.hidden_states(cfg, 1, 1, 1)[:, 0]), _given_up(), []
    for polls, more in ((1 << 24, 0), (0, 1), (1 << 24, 1)):
        s = span.open_session(L + 2)
        for b in range(2):
            s.import_kv(b, kv[b])
        binding.petals_debug_step_patience(span.handle, polls)
        outs.append(to_np(span.decode_step([s], x)))
        assert _given_up() == before + more and s.length == L + 1
        s.close()
    assert np.isnan(outs[1]).any()
    assert np.isfinite(outs[0]).all() and np.array_equal(outs[0].view(np.uint16), outs[2].view(np.uint16))
    span.close()
