"""The engine's host code against the mock HIP runtime (tests/host/mock),
built with g++ and run under AddressSanitizer/UBSan."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("check,link", [
    ("engine_batch_check", []),
    ("engine_grid_check", []),
    ("engine_mass_check", ["-Wl,--wrap=_ZN4hhgr16launch_mass_gridEP11mock_streamidPKdPd"]),
])
def test_engine_host_logic(check, link, tmp_path):
    exe = str(tmp_path / check)
    h, src = os.path.join(ROOT, "tests/host"), os.path.join(ROOT, "paper_1506_06185_amd/csrc")
    subprocess.run(["g++", "-std=c++17", "-O0", "-g", "-fsanitize=address,undefined", "-fno-omit-frame-pointer",
                    "-I" + os.path.join(h, "mock"), "-x", "c++", os.path.join(src, "engine.hip"), "-x", "none",
                    os.path.join(src, "topology.cpp"), os.path.join(src, "mesh.cpp"), os.path.join(src, "geometry.cpp"),
                    os.path.join(h, "mock/mock_hip.cpp"), os.path.join(h, "mock/mock_kernels.cpp"),
                    os.path.join(h, check + ".cpp"), *link, "-o", exe], check=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1", UBSAN_OPTIONS="halt_on_error=1")
    out = subprocess.run([exe], capture_output=True, text=True, env=env)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "ok" in out.stdout
