"""Kernels whose rows may start anywhere, where their split can go wrong: detrending rows that
start 0 to 3 samples past a 16-byte boundary (a scalar head, 16-byte body and scalar tail of a
few samples each), and clipping spectra of just under, exactly and just over the channels whose
loads are issued together."""
import numpy as np
import pytest

from oracle import dedisp_oracle as orc
from tests.gpu_util import cuda

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return cuda()


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 1023, 1027, 1030])
def test_detrend_rows_at_any_offset(torch, n):
    import paper_1401_8258_amd as dd
    print(f"case: detrend n={n} at every offset", flush=True)
    nrows, stride = 8, n + (1 if n % 2 == 0 else 2)  # odd: consecutive rows take every offset
    rng = np.random.default_rng(n)
    x = (rng.standard_normal((nrows, n)) * 3 + 50 + 0.01 * np.arange(n)).astype(np.float32)
    full = np.full((nrows, stride), -7.0, np.float32)
    full[:, :n] = x
    dev = torch.from_numpy(full).cuda()
    assert len({(dev[r].data_ptr() % 16) for r in range(4)}) == 4
    rms = dd.detrend(dev[:, :n], normalise=False)
    got = dev.cpu().numpy()
    want, want_rms = orc.detrend(x.astype(np.float64), normalise=False)
    # one rounding to FP32 of a residual below 20 (2^-20), and FP64 sums far below it
    assert np.max(np.abs(got[:, :n] - want)) <= 1e-6
    np.testing.assert_allclose(rms.cpu().numpy(), want_rms, rtol=1e-6, atol=1e-6)
    assert np.all(got[:, n:] == -7.0)


@pytest.mark.parametrize("nchan,n", [(31, 63), (32, 64), (33, 65), (64, 127), (95, 1)])
def test_spectrum_clip_split(torch, nchan, n):
    import paper_1401_8258_amd as dd
    print(f"case: spectrum clip {nchan}x{n}", flush=True)
    rng = np.random.default_rng(nchan)
    x = (10.0 + rng.standard_normal((nchan, n + 1))).astype(np.float32)
    hit = (np.arange(n) % 5 == 0) & (n > 1)
    x[:, :n][:, hit] += 4.0
    dev = torch.from_numpy(x).cuda()
    fit, _, mean, _ = dd.rfi_mitigate(dev[:, :n], 1, 0.0, 0, 2.0)  # the spectrum stage and the correction
    dist = np.abs(x[:, :n].astype(np.float64).mean(axis=0) - mean)
    assert np.min(np.abs(dist - 2.0)) > 1e-3  # no decision near the threshold
    np.testing.assert_array_equal(dist > 2.0, hit)
    want = x[:, :n].astype(np.float64) - fit.astype(np.float32)[:, None]
    want[:, hit] = 0.0
    got = dev.cpu().numpy()
    # a corrected sample is one FP32 subtraction: half an ulp of a result below 16
    assert np.max(np.abs(got[:, :n] - want)) <= 2.0 ** -21
    np.testing.assert_array_equal(got[:, :n][:, hit], 0.0)
    np.testing.assert_array_equal(got[:, n], x[:, n])
