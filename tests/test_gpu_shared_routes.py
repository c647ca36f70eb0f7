"""Each kernel of 8-bit plans on beams of its own: the shared-sum form where bundles are split,
channels in no order, windows of many rounds of rows or trials few (asserted by Plan.kernel), and
the direct-read form, asked for by name, on beams whose untuned plans run in the shared-sum form.
8-bit sums are exact, so every output equals the oracle's."""
import numpy as np
import pytest

import fbsynth
from oracle import dedisp_oracle as orc
from tests.gpu_util import assert_stats_close, compare_candidates, cuda

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return cuda()


@pytest.fixture(scope="module")
def dd():
    import paper_1401_8258_amd as dd
    dd.load_library()
    return dd


def _pairs_shuffled(freq):
    n = freq.size // 2
    return np.concatenate([freq[: 2 * n].reshape(n, 2)[np.random.default_rng(3).permutation(n)].ravel(), freq[2 * n:]])


# nchan, MHz per channel, top MHz, tsamp, ndm, step, outputs, input row padding, order, wavefronts
SHARED = [
    (515, 20.0 / 515, 428.0, 51.2e-6, 70, 0.1, 5003, 7, _pairs_shuffled, 16),  # pairs, three channels left over
    (1024, 60.0 / 1024, 180.0, 81.92e-6, 200, 0.02, 4100, 1, None, 16),         # delays of many samples a trial
    (700, 30.0 / 700, 200.0, 51.2e-6, 64, 0.03, 2017, 3, None, 16),
    (256, 20.0 / 256, 428.0, 51.2e-6, 16, 0.1, 2016, 0, None, 8),               # workgroups of 8 wavefronts
    (300, 20.0 / 300, 428.0, 51.2e-6, 7, 0.1, 6001, 5, None, 4),                # and of 4
]


@pytest.mark.parametrize("shape", SHARED)
def test_shared_sum_form_of_8bit_plans(torch, dd, shape):
    nchan, df, top, tsamp, ndm, step, nout, pad, order, waves = shape
    print(f"case: 8-bit shared-sum {nchan} ch {ndm} x {step}", flush=True)
    freq = fbsynth.channel_freqs(top, df, nchan)
    freq = order(freq) if order else freq
    dm = fbsynth.dm_trials(0.0, step, ndm)
    tab = orc.delay_table(freq, dm, tsamp)
    nsamp = int(tab.max()) + nout
    full = fbsynth.to_u8(np.random.default_rng(nchan).standard_normal((nchan, nsamp + pad)))
    plan = dd.Plan(freq, tsamp, dm, dtype="u8")
    assert (plan.kernel["form"], plan.kernel["waves"]) == ("shared", waves)
    r = plan.dedisperse(torch.from_numpy(full).cuda()[:, :nsamp])
    want = orc.dedisperse(full[:, :nsamp], tab)
    np.testing.assert_array_equal(r.out.cpu().numpy().astype(np.float64), want)
    assert_stats_close(r.mean.cpu().numpy(), r.rms.cpu().numpy(), *orc.series_stats(want))


def test_direct_form_by_name_on_config3(torch, dd):
    print("case: direct form by name, config 3", flush=True)
    b, u8, _ = fbsynth.config3()
    want = orc.dedisperse(u8, orc.delay_table(b.freq_mhz, b.dm, b.tsamp_s))
    mean, rms = orc.series_stats(want)
    x = torch.from_numpy(u8).cuda()
    p = dd.Plan(b.freq_mhz, b.tsamp_s, b.dm, dtype="u8", form="direct")
    q = dd.Plan(b.freq_mhz, b.tsamp_s, b.dm, dtype="u8")
    assert (p.kernel["form"], q.kernel["form"]) == ("direct", "shared")
    r1, r2 = p.dedisperse(x, k_sigma=4.0), q.dedisperse(x, k_sigma=4.0)
    np.testing.assert_array_equal(r1.out.cpu().numpy().astype(np.float64), want)
    assert torch.equal(r1.out, r2.out)
    assert_stats_close(r1.mean.cpu().numpy(), r1.rms.cpu().numpy(), mean, rms)
    compare_candidates(r1.candidates(), want, mean, rms, 4.0)


def test_direct_form_by_name_on_the_full_size_4096_channel_beam(torch, dd):
    specs = [sp for sp in fbsynth.config4_specs() if sp["nchan"] == 4096]
    sp = min(specs, key=lambda s: s["ndm"] * s["nsamp"])
    print(f"case: direct form by name, 4096 channels, ndm={sp['ndm']} nsamp={sp['nsamp']}", flush=True)
    b = fbsynth.make_beam(sp["name"], sp["nchan"], sp["f_top"], sp["bw"], sp["tsamp"], sp["dm0"], sp["step"],
                          sp["ndm"], sp["nsamp"], np.random.default_rng(sp["seed"]), sp["npulse"], storage="u8")
    x = torch.from_numpy(b.data).cuda()
    p = dd.Plan(b.freq_mhz, b.tsamp_s, b.dm, dtype="u8", form="direct")
    q = dd.Plan(b.freq_mhz, b.tsamp_s, b.dm, dtype="u8")
    assert (p.kernel["form"], q.kernel["form"]) == ("direct", "shared")
    r1, r2 = p.dedisperse(x), q.dedisperse(x)
    assert torch.equal(r1.out, r2.out)
    rows = [0, b.ndm // 2, b.ndm - 1]
    want = orc.dedisperse(b.data, orc.delay_table(b.freq_mhz, b.dm, b.tsamp_s), rows=rows)
    np.testing.assert_array_equal(r1.out[rows].cpu().numpy().astype(np.float64), want)
