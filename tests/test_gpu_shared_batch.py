"""Batched calls of shared-sum items: one launch per input type and workgroup size over all their
units, whatever their sizes, each item equal to its own call bit for bit; and small items share
the chip, which they cannot with a launch each."""
import numpy as np
import pytest

import fbsynth
from tests.gpu_util import cuda

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return cuda()


@pytest.fixture(scope="module")
def dd():
    import paper_1401_8258_amd as dd
    dd.load_library()
    return dd


def _plan(dd, nchan, ndm, dtype, step=0.1, form="auto"):
    return dd.Plan(fbsynth.channel_freqs(428.0, 20.0 / nchan, nchan), 51.2e-6, fbsynth.dm_trials(0.0, step, ndm),
                   dtype=dtype, form=form)


def _input(torch, rng, nchan, nsamp, dtype):
    x = rng.standard_normal((nchan, nsamp))
    x = fbsynth.to_u8(x) if dtype == "u8" else x.astype(np.float32 if dtype == "f32" else np.float16)
    return torch.from_numpy(x).cuda()


# nchan, ndm, outputs, wavefronts of the workgroups: one unit, a few (fewer than the XCDs), many;
# a single item of its workgroup size among them
ITEMS = [(128, 40, 1, 16), (300, 70, 5003, 16), (256, 16, 2016, 8), (200, 100, 20011, 16), (131, 5, 3000, 4),
         (140, 15, 1009, 8), (512, 300, 9001, 16)]


@pytest.mark.parametrize("dtypes", [("f32",), ("f16",), ("u8",), ("u8", "f32", "f16")])
def test_items_equal_their_own_calls(torch, dd, dtypes):
    print(f"case: batch of shared-sum items {dtypes}", flush=True)
    rng = np.random.default_rng(17)
    jobs, want = [], []
    for i, (nchan, ndm, nout, waves) in enumerate(ITEMS * len(dtypes)):
        dtype = dtypes[i % len(dtypes)]
        plan = _plan(dd, nchan, ndm, dtype)
        assert (plan.kernel["form"], plan.kernel["waves"]) == ("shared", waves)
        jobs.append((plan, _input(torch, rng, nchan, plan.maxdelay + nout, dtype)))
    # an item of another form, and a stream's window
    lds = _plan(dd, 64, 60, dtypes[0], form="lds")
    jobs.insert(3, (lds, _input(torch, rng, 64, lds.maxdelay + 3000, dtypes[0])))
    want = [p.dedisperse(x, k_sigma=4.5) for p, x in jobs]
    plan = _plan(dd, 160, 50, dtypes[0])
    blocks = [_input(torch, rng, 160, 1500, dtypes[0]) for _ in range(plan.maxdelay // 1500 + 3)]
    alone, batched = dd.Stream(plan, 1500), dd.Stream(plan, 1500)
    for b in blocks:
        want_stream = alone.push(b, k_sigma=4.5)
    for b in blocks[:-1]:
        batched.push(b)
    jobs.append((batched, batched.append(blocks[-1])))
    for got, one in zip(dd.batch_dedisperse(jobs, k_sigma=4.5), want + [want_stream]):
        assert got.t0 == one.t0
        assert torch.equal(got.out, one.out)
        assert torch.equal(got.mean, one.mean) and torch.equal(got.rms, one.rms)
        np.testing.assert_array_equal(got.candidates(), one.candidates())


def test_small_items_share_the_chip(torch, dd):
    """16 items of a handful of workgroups each: together in well under the time of one by one (a
    quarter of it when this was written; a launch an item takes all of it)."""
    print("case: 16 small shared-sum items, timed", flush=True)
    rng = np.random.default_rng(5)
    plans = [_plan(dd, 256, 64, "u8") for _ in range(16)]
    jobs = [(p, _input(torch, rng, 256, p.maxdelay + 4000, "u8")) for p in plans]
    outs = [dd.api.alloc_outputs(64, 4000, "cuda") for _ in jobs]

    def together():
        dd.batch_dedisperse(jobs, outputs=outs)

    def one_by_one():
        for (p, x), o in zip(jobs, outs):
            p.dedisperse(x, out=o[0])

    best = {}
    for f in (together, one_by_one) * 4:
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(5):
            f()
        e1.record()
        torch.cuda.synchronize()
        best[f] = min(best.get(f, 1e9), e0.elapsed_time(e1) / 5)
    print(f"together {best[together]:.3f} ms, one by one {best[one_by_one]:.3f} ms", flush=True)
    assert best[together] < 0.6 * best[one_by_one]
