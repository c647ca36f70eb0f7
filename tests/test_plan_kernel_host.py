"""dd_plan_kernel and dd_binned_kernel: the kernel a plan's calls run, next to the tiled form that
dd_plan_query describes. Host only."""
import ctypes as C

import numpy as np
import pytest

import fbsynth
from paper_1401_8258_amd import _lib


@pytest.fixture(scope="module")
def lib():
    try:
        return _lib.load()
    except _lib.LibraryMissing as e:  # the build step has not run in this checkout
        pytest.skip(str(e))


def _plan(lib, freq, dm, tsamp, dtype, tuning=None):
    h = C.c_void_p()
    f, d = np.ascontiguousarray(freq, np.float64), np.ascontiguousarray(dm, np.float64)
    dbl = C.POINTER(C.c_double)
    tun = C.byref(_lib.Tuning(*tuning)) if tuning else None
    rc = lib.dd_plan_create(C.byref(h), f.ctypes.data_as(dbl), f.size, tsamp, d.ctypes.data_as(dbl), d.size, dtype, tun)
    return rc, h


def _mid(nchan):
    return fbsynth.channel_freqs(428.0, 20.0 / nchan, nchan), 51.2e-6


def _low(nchan):
    return fbsynth.channel_freqs(180.0, 60.0 / nchan, nchan), 81.92e-6


F32, F16, U8 = _lib.DD_F32, _lib.DD_F16, _lib.DD_U8
LDS, DIRECT, SHARED = _lib.DD_FORM_LDS, _lib.DD_FORM_DIRECT, _lib.DD_RUNS_SHARED
TUNE_LDS, TUNE_DIRECT = (0, 0, 0, 0, 0, LDS), (0, 0, 0, 0, 0, DIRECT)


@pytest.mark.parametrize("band,ndm,step,dtype,tuning,runs,described,tile", [
    (_mid(64), 128, 0.1, F32, None, LDS, LDS, 512),
    (_mid(128), 128, 0.1, F32, None, SHARED, LDS, 1008),
    (_mid(64), 128, 0.1, F16, None, SHARED, LDS, 1008),
    (_mid(1024), 500, 0.1, F32, TUNE_LDS, LDS, LDS, 512),
    (_mid(1024), 500, 0.1, U8, None, SHARED, DIRECT, 2016),
    (_mid(1024), 500, 0.1, U8, TUNE_DIRECT, DIRECT, DIRECT, 1024),
    (_low(512), 33, 0.2, U8, None, DIRECT, DIRECT, 1024),
])
def test_plan_kernel_names_what_runs(lib, band, ndm, step, dtype, tuning, runs, described, tile):
    rc, h = _plan(lib, band[0], fbsynth.dm_trials(0.0, step, ndm), band[1], dtype, tuning)
    assert rc == 0, lib.dd_last_error()
    k, q = _lib.KernelInfo(), _lib.PlanInfo()
    assert lib.dd_plan_kernel(h, C.byref(k)) == 0
    lib.dd_plan_query(h, 1 << 20, C.byref(q))
    assert (k.form, q.kernel_form, k.tile_samples) == (runs, described, tile)
    assert k.dms_per_group == k.dms_per_wave * k.waves and 0 <= k.lds_bytes <= 160 * 1024
    if runs == SHARED:
        assert k.dms_per_wave == 2 and k.waves in (4, 8, 16) and k.producer_waves == 0 and k.lds_bytes > 0
    else:
        assert (k.dms_per_wave, k.waves, k.producer_waves) == (q.dms_per_wave, q.waves, q.producer_waves)
        assert k.lds_bytes == q.launch_lds
    lib.dd_plan_destroy(h)


def test_binned_kernel_and_errors(lib):
    (f, ts), dm = _mid(256), fbsynth.dm_trials(0.0, 0.1, 1500)
    f, dm = np.ascontiguousarray(f), np.ascontiguousarray(dm)
    dbl = C.POINTER(C.c_double)
    h, n, k = C.c_void_p(), C.c_int32(), _lib.KernelInfo()
    assert lib.dd_binned_create(C.byref(h), f.ctypes.data_as(dbl), f.size, ts, dm.ctypes.data_as(dbl), dm.size, U8, 4,
                                None) == 0
    lib.dd_binned_query(h, 0, C.byref(n), None, 0, None, None)
    assert n.value >= 2
    for i in range(n.value):
        assert lib.dd_binned_kernel(h, i, C.byref(k)) == 0
        assert (k.form, k.tile_samples) == (SHARED, 2016 if i == 0 else 1008)
    assert lib.dd_binned_kernel(h, n.value, C.byref(k)) == _lib.DD_ERR_INVALID_ARG
    assert lib.dd_binned_kernel(h, 0, None) == _lib.DD_ERR_INVALID_ARG
    lib.dd_binned_destroy(h)
    assert lib.dd_plan_kernel(None, C.byref(k)) == _lib.DD_ERR_INVALID_ARG
    # the shared-sum form is no tuning
    assert _plan(lib, f, dm, ts, F32, (0, 0, 0, 0, 0, SHARED))[0] == _lib.DD_ERR_UNSUPPORTED


def _order(freq, how):
    rng = np.random.default_rng(3)
    if how == "none":
        return rng.permutation(freq)
    if how == "halves":  # two halves of the band, channel by channel
        return np.stack([freq[: freq.size // 2], freq[freq.size // 2:]], 1).ravel()
    if how == "pairs":
        return freq.reshape(-1, 2)[rng.permutation(freq.size // 2)].ravel()
    return freq


@pytest.mark.parametrize("order,ndm,step,dtype,runs", [
    ("down", 500, 0.1, F32, SHARED),
    ("pairs", 500, 0.1, F32, SHARED),
    ("none", 500, 0.1, F32, LDS),      # neighbours share no sums: the LDS form takes two thirds of the time
    ("halves", 500, 0.1, F32, LDS),
    ("none", 2048, 0.1, F32, LDS),
    ("none", 350, 0.1, F32, SHARED),   # too few trials to fill the chip in the LDS form
    ("none", 500, 0.5, F32, SHARED),   # long windows: no 14-wavefront tiling
    ("none", 500, 0.1, F16, SHARED),   # the LDS form has no producers
    ("none", 500, 0.1, U8, DIRECT),
])
def test_beams_whose_channels_share_nothing(lib, order, ndm, step, dtype, runs):
    freq, ts = _mid(1024)
    rc, h = _plan(lib, _order(freq, order), fbsynth.dm_trials(0.0, step, ndm), ts, dtype)
    assert rc == 0, lib.dd_last_error()
    k = _lib.KernelInfo()
    assert lib.dd_plan_kernel(h, C.byref(k)) == 0
    assert k.form == runs
    lib.dd_plan_destroy(h)
