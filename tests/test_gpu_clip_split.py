"""Spectrum clipping where its split over channels can go wrong: every count below the 32 channels
whose loads are issued together, remainders of each of their halves, and series longer than a few-
channel launch has lanes. A spectrum's mean is summed in FP64 in channel order."""
import numpy as np
import pytest

from tests.gpu_util import cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nchan,n", [(k, 200) for k in range(1, 33)] + [(47, 65), (63, 64), (71, 63), (3, (1 << 20) + 67)])
def test_clipped_spectra(nchan, n):
    torch = cuda()
    import paper_1401_8258_amd as dd
    print(f"case: clip {nchan}x{n}", flush=True)
    rng = np.random.default_rng(nchan)
    x = (10.0 + 0.1 * rng.standard_normal((nchan, n + 1))).astype(np.float32)
    hit = np.arange(n) % 7 == 3
    hit[-1] = True
    x[:, :n][:, hit] += 4.0
    dev = torch.from_numpy(x).cuda()
    fit, _, mean, _ = dd.rfi_mitigate(dev[:, :n], 0, 0.0, 0, 2.0)
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
