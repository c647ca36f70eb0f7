"""The shared-sum form (the route of plans without a tuning) against the oracle where it can go
wrong: the edges of its 1008- and 2016-sample tiles, partial groups and bundles, channels in
rising and in no order, odd strides, windows of several rounds of rows, and ring input."""
import numpy as np
import pytest

import fbsynth
from oracle import dedisp_oracle as orc
from tests.gpu_util import assert_rows_close, assert_stats_close, cuda

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return cuda()


@pytest.fixture(scope="module")
def dd():
    import paper_1401_8258_amd as dd
    dd.load_library()
    return dd


# nchan, MHz per channel, top MHz, ndm, step, outputs, input row padding, output row padding, order
SHAPES = [
    (128, 20.0 / 128, 428.0, 31, 0.1, 1, 0, 0, "down"),        # one output, a partial group
    (130, 20.0 / 130, 428.0, 33, 0.1, 1008, 3, 1, "down"),     # a full FP32 tile; odd paddings
    (129, 20.0 / 129, 428.0, 65, 0.1, 1009, 1, 0, "up"),       # one past it; a bundle of one channel
    (256, 20.0 / 256, 428.0, 40, 0.2, 2016, 0, 4, "down"),     # a full 8-bit tile
    (256, 20.0 / 256, 428.0, 100, 0.2, 2017, 5, 3, "up"),      # one past it
    (515, 20.0 / 515, 428.0, 70, 0.1, 5003, 7, 0, "none"),     # channels in no order, three left over
    (300, 60.0 / 300, 180.0, 64, 0.1, 3001, 1, 2, "down"),     # windows of several rounds of rows
    (160, 20.0 / 160, 428.0, 9, 6.0, 1500, 0, 0, "down"),      # delays of hundreds of samples a trial
]


def _case(nchan, df, top, ndm, step, order):
    freq = fbsynth.channel_freqs(top, df, nchan)
    if order == "up":
        freq = freq[::-1].copy()
    elif order == "none":
        freq = np.random.default_rng(3).permutation(freq)
    dm = fbsynth.dm_trials(0.0, step, ndm)
    return freq, dm, orc.delay_table(freq, dm, 51.2e-6)


def _input(rng, dtype, shape):
    x = rng.standard_normal(shape)
    if dtype == "u8":
        return np.clip(np.rint(128 + 16 * x), 0, 255).astype(np.uint8)
    return x.astype(np.float32 if dtype == "f32" else np.float16)


@pytest.mark.parametrize("dtype", ["f32", "f16", "u8"])
@pytest.mark.parametrize("shape", SHAPES)
def test_edges_equal_oracle(torch, dd, dtype, shape):
    nchan, df, top, ndm, step, nout, pad, opad, order = shape
    print(f"case: shared {dtype} {shape}", flush=True)
    freq, dm, tab = _case(nchan, df, top, ndm, step, order)
    nsamp = int(tab.max()) + nout
    full = _input(np.random.default_rng(nchan + ndm), dtype, (nchan, nsamp + pad))
    want = orc.dedisperse(full[:, :nsamp].astype(np.float64), tab)
    mean, rms = orc.series_stats(want)
    plan = dd.Plan(freq, 51.2e-6, dm, dtype=dtype)
    out = torch.full((ndm, nout + opad), -7.0, device="cuda")
    r = plan.dedisperse(torch.from_numpy(full).cuda()[:, :nsamp], out=out)
    torch.cuda.synchronize()
    got = out[:, :nout].cpu().numpy().astype(np.float64)
    assert opad == 0 or bool((out[:, nout:] == -7.0).all()), "write past nout"
    if dtype == "u8":
        np.testing.assert_array_equal(got, want)
    else:
        # a sum of nchan unit-variance samples by at most 32 + 4 + nchan / 128 FP32 additions:
        # the rounding error stays far below 1e-5 of sqrt(nchan), the series rms of long series
        assert_rows_close(got, want, np.full(ndm, np.sqrt(nchan)), what="shared")
    if nout > 1:
        assert_stats_close(r.mean.cpu().numpy(), r.rms.cpu().numpy(), mean, rms)


@pytest.mark.parametrize("dtype", ["f32", "f16", "u8"])
def test_ring_input_and_batch_equal_one_shot(torch, dd, dtype):
    """Stream windows that start anywhere in the ring (its end and mirror among them) and a batch
    equal the plain call bit for bit."""
    print(f"case: shared {dtype}, stream and batch", flush=True)
    freq, dm, tab = _case(200, 20.0 / 200, 428.0, 70, 0.1, "down")
    sizes = [2500, 2500, 901, 2500, 1, 2500, 2499, 2500, 2500]
    x = torch.from_numpy(_input(np.random.default_rng(5), dtype, (200, sum(sizes)))).cuda()
    plan = dd.Plan(freq, 51.2e-6, dm, dtype=dtype)
    whole = plan.dedisperse(x).out
    other = dd.Plan(freq[:150], 51.2e-6, dm[:33], dtype=dtype)
    res = dd.batch_dedisperse([(plan, x), (other, x[:150])])
    torch.cuda.synchronize()
    assert torch.equal(res[0].out, whole)
    assert torch.equal(res[1].out, other.dedisperse(x[:150]).out)
    st = dd.Stream(plan, 2500)
    pos = seen = 0
    for n in sizes:
        r = st.push(x[:, pos:pos + n].contiguous())
        pos += n
        if r is None:
            continue
        assert r.t0 == seen
        assert torch.equal(r.out, whole[:, seen:seen + r.out.shape[1]]), f"block at t0={r.t0} differs"
        seen += r.out.shape[1]
    assert seen == whole.shape[1]


@pytest.mark.parametrize("nchan,csub,ndm,dgroup", [(200, 32, 70, 16), (130, 64, 75, 33), (96, 8, 40, 32), (33, 32, 5, 4)])
def test_subband_steps_equal_oracle(torch, dd, nchan, csub, ndm, dgroup):
    """Both steps of a subband plan, at a short last subband (of one channel in the last case) and
    group, and on both sides of the largest group that the shared-sum form takes; batched equal."""
    print(f"case: subband {nchan}/{csub} {ndm}/{dgroup}", flush=True)
    freq, dm, _ = _case(nchan, 20.0 / nchan, 428.0, ndm, 0.1, "down")
    x = np.random.default_rng(nchan).standard_normal((nchan, 5003)).astype(np.float32)
    want = orc.subband_dedisperse(x, freq, 51.2e-6, dm, csub, dgroup)
    sp = dd.SubbandPlan(freq, 51.2e-6, dm, chans_per_sub=csub, dms_per_group=dgroup)
    dev = torch.from_numpy(x).cuda()
    res, bat = sp.dedisperse(dev, k_sigma=5.0), sp.dedisperse(dev, k_sigma=5.0, batched=True)
    torch.cuda.synchronize()
    assert [g for g, _ in res] == [(d0, d1) for d0, d1, _ in want]
    for (_, r), (_, b), (d0, _, s) in zip(res, bat, want):
        mean, rms = orc.series_stats(s)
        assert_rows_close(r.out.cpu().numpy(), s, rms, what=f"group {d0}")
        assert_stats_close(r.mean.cpu().numpy(), r.rms.cpu().numpy(), mean, rms)
        assert torch.equal(r.out, b.out) and torch.equal(r.mean, b.mean) and torch.equal(r.rms, b.rms)
