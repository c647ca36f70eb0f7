"""The scratch limit of dd_dedisperse_noalloc for 8-bit plans: what the message says of a call that
is refused. Checked before anything touches a device."""
import ctypes as C
import re

import pytest

import fbsynth
from paper_1401_8258_amd import _lib


def test_refusal_names_what_the_call_needs_and_what_it_must_leave():
    try:
        lib = _lib.load()
    except _lib.LibraryMissing as e:  # the build step has not run in this checkout
        pytest.skip(str(e))
    freq, dm = fbsynth.channel_freqs(428.0, 20.0 / 256, 256), fbsynth.dm_trials(0.0, 0.1, 64)
    h, k, dbl = C.c_void_p(), _lib.KernelInfo(), C.POINTER(C.c_double)
    assert lib.dd_plan_create(C.byref(h), freq.ctypes.data_as(dbl), freq.size, 51.2e-6, dm.ctypes.data_as(dbl), dm.size,
                              _lib.DD_U8, None) == 0
    assert lib.dd_plan_kernel(h, C.byref(k)) == 0 and k.form == _lib.DD_RUNS_SHARED
    p, nsamp = C.c_void_p(256), 1 << 17  # never dereferenced; four copies of 256 x 131,072 bytes are 128 MiB
    assert lib.dd_dedisperse_noalloc(h, p, nsamp, nsamp, p, nsamp, None, None, 0.0, None, 0, None, p,
                                     None) == _lib.DD_ERR_UNSUPPORTED
    need, leave, holds = map(int, re.findall(r"\d+", lib.dd_last_error().decode().replace("8-bit", "")))
    assert need <= holds == 96 << 20 < leave
    assert leave - need >= 4 * 256 * nsamp
    lib.dd_plan_destroy(h)
