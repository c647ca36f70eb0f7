"""Rounding of the shared-sum form: its series' error against FP64 must not exceed that of the LDS
form, which adds channel by channel in blocks of 32, where bundles are narrow (coarse steps, low
and unsorted bands) or channels few, for noise about zero and on a level of its own size."""
import numpy as np
import pytest

import fbsynth
from oracle import dedisp_oracle as orc
from tests.gpu_util import cuda

pytestmark = pytest.mark.gpu

# nchan, MHz per channel, top MHz, ndm, step, order, dtype
SHAPES = [
    (64, 20.0 / 64, 428.0, 128, 0.1, "down", "f16"),    # bundles of two
    (128, 20.0 / 128, 428.0, 100, 0.2, "down", "f32"),
    (160, 20.0 / 160, 428.0, 9, 6.0, "down", "f32"),    # bundles of one
    (300, 60.0 / 300, 180.0, 64, 0.1, "down", "f16"),
    (515, 20.0 / 515, 428.0, 70, 0.1, "none", "f32"),
]


@pytest.mark.parametrize("level", [0.0, 1.0])
@pytest.mark.parametrize("shape", SHAPES)
def test_error_is_no_larger_than_channel_by_channel(shape, level):
    torch = cuda()
    import paper_1401_8258_amd as dd
    nchan, df, top, ndm, step, order, dtype = shape
    print(f"case: rounding {shape} level {level}", flush=True)
    freq = fbsynth.channel_freqs(top, df, nchan)
    if order == "none":
        freq = np.random.default_rng(3).permutation(freq)
    dm = fbsynth.dm_trials(0.0, step, ndm)
    tab = orc.delay_table(freq, dm, 51.2e-6)
    x = np.random.default_rng(nchan).standard_normal((nchan, int(tab.max()) + 3000)) + level
    x = x.astype(np.float32 if dtype == "f32" else np.float16)
    want = orc.dedisperse(x.astype(np.float64), tab)
    dev = torch.from_numpy(x).cuda()

    def rms_error(form):
        plan = dd.Plan(freq, 51.2e-6, dm, dtype=dtype, form=form)
        return np.sqrt(np.mean((plan.dedisperse(dev).out.cpu().numpy() - want) ** 2))

    auto, lds = rms_error("auto"), rms_error("lds")
    print(f"rms error {auto:.3e}, channel by channel {lds:.3e}", flush=True)
    # the same additions at worst (bundles of one channel), fewer otherwise; 5% for the spread of
    # the estimates over some thousand independent samples
    assert auto <= 1.05 * lds
