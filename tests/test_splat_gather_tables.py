"""The tables of the splat's gather form, checked by brute force on the host: every
read in the copy's bounds, every pixel once, every set of rows within one bin (see
tests/host/splat_tables_driver.cpp, built with ASan and UBSan)."""
import math
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2410_14900_amd", "csrc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    out = str(tmp_path_factory.mktemp("splat") / "splat_tables_driver")
    cmd = [gxx, "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-D__HIP_PLATFORM_AMD__",
           "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-I/opt/rocm/include", os.path.join(CSRC, "plan_host.cpp"),
           os.path.join(ROOT, "tests", "host", "splat_tables_driver.cpp"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out


# nu, nv, dv/du, n_theta, ds/du, angles per group (None: whatever is chosen; 0: the atomic form)
CASES = [(512, 512, 1.0, 360, 1.0, 4), (620, 480, 1.0, 360, 1.0, 4), (976, 976, 1.0, 720, 1.0, 4),
         (64, 64, 1.0, 180, 1.0, None), (33, 150, 1.0, 37, 1.0, None), (5, 67, 1.0, 41, 1.0, None),
         (1, 1, 1.0, 1, 1.0, None), (61, 90, 0.8, 200, 1.0, None), (64, 64, 1.0, 360, 1.41, None),
         (90, 61, 1.0, 90, 0.9, 0), (64, 64, 1.0, 90, 1.5, 0), (70, 53, 1.0, 2, 1.0, None)]


@pytest.mark.parametrize("nu,nv,av,n_theta,ws,group", CASES)
def test_splat_gather_tables(driver, nu, nv, av, n_theta, ws, group):
    n_s = max(2, int(math.ceil(math.hypot(nu, nv) / min(ws, 1.0))))
    r = subprocess.run([driver] + [str(x) for x in (nu, nv, av, n_theta, ws, n_s)], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, (r.stdout, r.stderr[-2000:])
    got = int(r.stdout)
    print("angles per group:", got)
    assert group is None or got == group
