"""Workgroups that look at the base data of a plan: as many as the largest base has chunks for a few layers, a launch
that the device takes (and that is not mostly idle workgroups) for any plan that the other launches take."""

import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..")


@pytest.fixture(scope="module")
def groups(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    d = tmp_path_factory.mktemp("grid")
    src = d / "grid.hip"
    src.write_text('#include "vbrdf_internal.hpp"\n'
                   'extern "C" int run(long long e, int n) { return vbrdf::base_check_groups(e, n); }\n')
    so = d / "grid.so"
    subprocess.run([hipcc, "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_1707_05882_amd", "csrc"), "-o", str(so), str(src)], check=True)
    f = ctypes.CDLL(str(so)).run
    f.argtypes = [ctypes.c_longlong, ctypes.c_int]
    return f


@pytest.mark.parametrize("entries", [1, 16, 2048, 2049, 24 * 160 * 160, 64 * 128 * 128, 512 * 512 * 512])
@pytest.mark.parametrize("layers", [1, 2, 5, 64, 65, 300, 3000, 33000, 65000])
def test_launch(groups, entries, layers):
    g, chunks = groups(entries, layers), -(-entries // 2048)
    assert 1 <= g <= chunks
    assert g * layers <= max(4096, 64 * layers) < 2 ** 31 // 256
    assert g >= min(chunks, 64)  # no base is left to a handful of workgroups
    if chunks * layers <= 4096:
        assert g == chunks
