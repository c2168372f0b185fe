"""Reading and saving a surrogate's parameters with another device current: the
kernels go to the device that holds the surrogate, and the caller's device is
current again afterwards.  The HIP runtime is stood in for by
``tests/hip_two_devices.c`` (two devices of host memory), so that the host code
runs without a GPU."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

DRIVER = r"""
import ctypes, sys
hip = ctypes.CDLL(None)
lib = ctypes.CDLL(sys.argv[1])
assert hip.test_launches() == 0
def current():
    d = ctypes.c_int(-1)
    hip.hipGetDevice(ctypes.byref(d))
    return d.value
for home in (0, 1):
    hip.hipSetDevice(home)
    s = ctypes.c_void_p(0)
    assert lib.wo_sur_create(8, None, ctypes.c_uint64(1), None, ctypes.byref(s)) == 0
    for other in (home, 1 - home):
        hip.hipSetDevice(other)
        out = (ctypes.c_float * int(sys.argv[3]))()
        for call in (lambda: lib.wo_sur_get_params(s, out), lambda: lib.wo_sur_save(s, sys.argv[2].encode())):
            hip.test_forget()
            assert call() == 0
            assert current() == other
            n = hip.test_launches()
            assert n >= 1, "no kernel"
            where = [hip.test_launch_device(i) for i in range(n)]
            assert where == [home] * n, (home, other, where)
    hip.hipSetDevice(home)
    assert lib.wo_sur_free(s) == 0
print("ok")
"""


@pytest.mark.skipif(shutil.which("gcc") is None, reason="needs gcc")
def test_parameters_are_laid_out_on_the_surrogates_device(tmp_path):
    from paper_2110_13693_amd import wo
    stub = str(tmp_path / "hip_two_devices.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", os.path.join(HERE, "hip_two_devices.c"), "-o", stub])
    r = subprocess.run([sys.executable, "-c", DRIVER, wo.lib()._name, str(tmp_path / "p.wosur"), str(wo.WO_SUR_PARAMS)],
                       capture_output=True, text=True, env=dict(os.environ, LD_PRELOAD=stub), timeout=300)
    assert r.returncode == 0 and "ok" in r.stdout, r.stdout + r.stderr
