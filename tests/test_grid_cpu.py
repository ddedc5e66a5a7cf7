"""The structured-grid kernels (grid.hip) on the CPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_grid_kernels_in_cpu_emulation(tmp_path):
    """grid.hip built for the host against a device-code emulation (a workgroup
    = host threads meeting at a barrier) and run under AddressSanitizer: every
    kind of sweep launch at several tile shapes, with and without frozen
    nodes, against node-by-node sweeps, interpolation, residual and
    restriction; residual and mass kernels; every chosen tiling."""
    exe = str(tmp_path / "gridcheck")
    h = os.path.join(ROOT, "tests/host")
    subprocess.run(["g++", "-std=c++20", "-O0", "-g", "-fsanitize=address", "-fno-omit-frame-pointer",
                    "-ffp-contract=off", "-pthread", "-I" + os.path.join(h, "mockgrid"), "-x", "c++",
                    os.path.join(ROOT, "paper_1506_06185_amd/csrc/grid.hip"), "-x", "none",
                    os.path.join(h, "grid_check.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, env=dict(os.environ, ASAN_OPTIONS="detect_leaks=1"))
    assert out.returncode == 0, out.stdout + out.stderr
    assert "ok" in out.stdout
