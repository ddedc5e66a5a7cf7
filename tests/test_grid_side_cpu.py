"""The structured-grid kernels around the sweeps (grid.hip) on the CPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_grid_side_kernels_in_cpu_emulation(tmp_path):
    """grid.hip built for the host against a device-code emulation and run under
    AddressSanitizer: weights, closures, single tetrahedra, Neumann data,
    dJ/dk, sweeps with element counts and the FP32 one-workgroup cycle against
    their definitions; every chosen tiling."""
    exe = str(tmp_path / "gridside")
    h, src = os.path.join(ROOT, "tests/host"), os.path.join(ROOT, "paper_1506_06185_amd/csrc")
    subprocess.run(["g++", "-std=c++20", "-O1", "-g1", "-fsanitize=address", "-fno-omit-frame-pointer",
                    "-ffp-contract=off", "-pthread", "-I" + os.path.join(h, "mockgrid"), "-x", "c++",
                    os.path.join(src, "grid.hip"), "-x", "none", os.path.join(h, "grid_side_check.cpp"),
                    os.path.join(src, "topology.cpp"), "-o", exe], check=True)
    # (a workgroup's threads meet at barriers: on few CPUs they wait least)
    cpus = sorted(os.sched_getaffinity(0))[:4]
    out = subprocess.run([exe], capture_output=True, text=True, env=dict(os.environ, ASAN_OPTIONS="detect_leaks=1"),
                         preexec_fn=lambda: os.sched_setaffinity(0, cpus))
    assert out.returncode == 0, out.stdout + out.stderr
    assert "ok" in out.stdout
