"""Infinities and NaN in the input of shared-sum plans: they reach exactly the outputs whose sums
hold them, as in the definition, and every other output is as without them."""
import numpy as np
import pytest

import fbsynth
from oracle import dedisp_oracle as orc
from tests.gpu_util import cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("nchan,ndm,step,nout", [(130, 33, 0.1, 2100), (160, 9, 6.0, 1009)])
def test_special_values_stay_where_they_belong(dtype, nchan, ndm, step, nout):
    torch = cuda()
    import paper_1401_8258_amd as dd
    print(f"case: special values {dtype} {nchan} ch {ndm} x {step}", flush=True)
    freq, dm = fbsynth.channel_freqs(428.0, 20.0 / nchan, nchan), fbsynth.dm_trials(0.0, step, ndm)
    tab = orc.delay_table(freq, dm, 51.2e-6)
    nsamp = int(tab.max()) + nout
    rng = np.random.default_rng(nchan)
    x = rng.standard_normal((nchan, nsamp)).astype(np.float32 if dtype == "f32" else np.float16)
    clean = x.copy()
    for i, v in enumerate((np.nan, np.inf, -np.inf) * 4):
        x[rng.integers(nchan), rng.integers(nsamp)] = v
    x[0, 0], x[-1, -1], x[nchan // 2, nsamp - 1] = np.inf, np.nan, -np.inf  # the first and last samples
    plan = dd.Plan(freq, 51.2e-6, dm, dtype=dtype)
    assert plan.kernel["form"] == "shared"
    got = plan.dedisperse(torch.from_numpy(x).cuda()).out.cpu().numpy()
    base = plan.dedisperse(torch.from_numpy(clean).cuda()).out.cpu().numpy()
    with np.errstate(invalid="ignore"):
        want = orc.dedisperse(x.astype(np.float64), tab)
    touched = ~np.isfinite(want)
    assert touched.any() and not touched.all()
    np.testing.assert_array_equal(got[touched], want[touched].astype(np.float32))
    np.testing.assert_array_equal(got[~touched], base[~touched])
