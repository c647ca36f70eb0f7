"""Shared-sum calls recorded into a graph: replays on new input, with eager work between them, equal
the eager calls (a plain call with statistics and candidates; both steps of a subband pass over its
side streams)."""
import ctypes as C

import numpy as np
import pytest

import fbsynth
from tests.gpu_util import cuda

pytestmark = pytest.mark.gpu


def _vp(t):
    return C.c_void_p(t.data_ptr())


def _record(torch, call):
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call()
    torch.cuda.current_stream().wait_stream(side)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    return g


@pytest.mark.parametrize("dtype", ["f32", "u8"])
def test_plain_call(dtype):
    torch = cuda()
    import paper_1401_8258_amd as dd
    from paper_1401_8258_amd import _lib
    print(f"case: capture {dtype}", flush=True)
    plan = dd.Plan(fbsynth.channel_freqs(428.0, 20.0 / 256, 256), 51.2e-6, fbsynth.dm_trials(0.0, 0.1, 100), dtype=dtype)
    assert plan.kernel["form"] == "shared"
    nout, cap = 5003, 4096
    nsamp = plan.maxdelay + nout
    x = torch.zeros((256, nsamp), dtype=plan.dtype, device="cuda")
    ws = plan.workspace(nsamp)
    out, mean, rms = torch.empty((100, nout), device="cuda"), torch.empty(100, device="cuda"), torch.empty(100, device="cuda")
    cand, ncand = torch.empty(cap * 24, dtype=torch.uint8, device="cuda"), torch.zeros(1, dtype=torch.int64, device="cuda")

    def call():
        st = C.c_void_p(torch.cuda.current_stream().cuda_stream)
        _lib.check(_lib.load().dd_dedisperse(plan.handle, _vp(x), nsamp, nsamp, _vp(out), nout, _vp(mean), _vp(rms), 4.0,
                                             _vp(cand), cap, _vp(ncand), _vp(ws), ws.numel(), st))

    g = _record(torch, call)
    for seed in range(4):
        v = np.random.default_rng(seed).standard_normal((256, nsamp)).astype(np.float32)
        x.copy_(torch.from_numpy(fbsynth.to_u8(v) if dtype == "u8" else v))
        out.fill_(-7.0)
        g.replay()
        torch.cuda.synchronize()
        want = plan.dedisperse(x.clone(), k_sigma=4.0)
        assert torch.equal(out, want.out) and torch.equal(mean, want.mean) and torch.equal(rms, want.rms)
        assert int(ncand.item()) == want.ncand()


def test_subband_pass():
    torch = cuda()
    import paper_1401_8258_amd as dd
    print("case: capture, subband", flush=True)
    sp = dd.SubbandPlan(fbsynth.channel_freqs(428.0, 20.0 / 256, 256), 51.2e-6, fbsynth.dm_trials(0.0, 0.1, 64),
                        chans_per_sub=32, dms_per_group=16)
    x = torch.zeros((256, 9000), device="cuda")
    keep = []
    g = _record(torch, lambda: keep.append(sp.dedisperse(x)))
    for seed in range(4):
        x.copy_(torch.from_numpy(np.random.default_rng(seed).standard_normal((256, 9000)).astype(np.float32)))
        g.replay()
        torch.cuda.synchronize()
        for (_, a), (_, b) in zip(keep[-1], sp.dedisperse(x.clone())):
            assert torch.equal(a.out, b.out) and torch.equal(a.mean, b.mean) and torch.equal(a.rms, b.rms)
