"""Streams of shared-sum plans whose ring is shorter than its mirror (short blocks, little delay):
a window then reads past the mirrored ring's end, where only outputs that are not stored look."""
import ctypes as C

import numpy as np
import pytest

import fbsynth
from tests.gpu_util import cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f16", "u8"])
@pytest.mark.parametrize("nchan,ndm,step,block", [(128, 20, 0.02, 8), (131, 40, 0.05, 100), (200, 9, 0.0, 64)])
def test_short_blocks_equal_one_shot(dtype, nchan, ndm, step, block):
    torch = cuda()
    import paper_1401_8258_amd as dd
    from paper_1401_8258_amd import _lib
    print(f"case: shared ring {dtype} {nchan} ch {ndm} x {step} block {block}", flush=True)
    plan = dd.Plan(fbsynth.channel_freqs(428.0, 20.0 / nchan, nchan), 51.2e-6, fbsynth.dm_trials(0.0, step, ndm),
                   dtype=dtype)
    assert plan.kernel["form"] == "shared"
    ring = -(-(block + plan.maxdelay) // 64) * 64
    assert ring < 1008  # samples a ring row holds, and the least its mirror does
    sizes = [block, block, 1, block - 1] * 6 + [block] * (3 + 2 * ring // block)
    x = np.random.default_rng(block).standard_normal((nchan, sum(sizes)))
    x = fbsynth.to_u8(x) if dtype == "u8" else x.astype(np.float32 if dtype == "f32" else np.float16)
    dev = torch.from_numpy(x).cuda()
    whole = plan.dedisperse(dev).out
    st = dd.Stream(plan, block)
    st.ring.fill_(0xFF)  # NaNs, or the largest code, wherever nothing is written; then the table again
    h = C.c_void_p()
    cur = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert _lib.load().dd_stream_create(plan.handle, block, C.c_void_p(st.ring.data_ptr()), st.ring.numel(), cur,
                                        C.byref(h)) == 0
    st.close()
    st._h = h
    pos = seen = 0
    for n in sizes:
        r = st.push(dev[:, pos:pos + n].contiguous())
        pos += n
        if r is None:
            continue
        assert r.t0 == seen
        assert torch.equal(r.out, whole[:, seen:seen + r.out.shape[1]]), f"block at t0={r.t0} differs"
        seen += r.out.shape[1]
    assert seen == whole.shape[1]
