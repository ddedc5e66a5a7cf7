"""hhgr_kernel_stats on the cube: which launches are timed and the bytes that
they cannot do without."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hh():
    from paper_1506_06185_amd import hhgr

    return hhgr


# words per unknown of every timed launch of a cycle: u and b read, u written;
# from zero u is not read; per-element k reads three edge weights.  Two FP32
# sweeps from zero are one launch (k = 1).
@pytest.mark.parametrize("n_sub,level,precision,vk,nu,words", [
    (1, 4, "fp64", False, (2, 1), [3]),         # one launch runs the whole cycle
    (1, 3, "fp64", False, (1, 1), [3]),
    (2, 4, "fp64", False, (2, 2), [3, 3]),
    (1, 4, "fp64", True, (2, 1), [6, 6]),
    (2, 4, "mixed", False, (2, 1), [2]),
    (2, 4, "mixed", False, (3, 1), [2, 3]),
    (1, 4, "mixed", False, (3, 1), [2]),        # one launch runs the whole FP32 cycle
    (2, 4, "mixed", True, (3, 2), [5, 6, 6]),
    (2, 4, "fp64", False, (0, 2), []),
])
def test_timed_launches_and_bytes(hh, n_sub, level, precision, vk, nu, words):
    print(f"\n[kernel stats] {n_sub} {level} {precision} {vk} {nu}", flush=True)
    ctx = hh.Context(device="cuda:0", n_sub=n_sub, level=level, precision=precision, variable_coeff=vk,
                     nu_pre=nu[0], nu_post=nu[1])
    if vk:
        ctx.set_coeff(torch.ones(ctx.n_elems, dtype=torch.float64, device="cuda"))
    ctx.set_rhs(torch.from_numpy(np.random.default_rng(1).standard_normal(ctx.n_dofs)).cuda())
    for cycles in (3, 5):
        ctx.kernel_timing(True)
        ctx.vcycle(cycles)
        launches, mean_ms, nbytes = ctx.kernel_stats()
        ctx.kernel_timing(False)
        assert launches == cycles * len(words)
        if words:
            assert mean_ms > 0.0
            assert nbytes == pytest.approx(np.mean(words) * (4 if precision == "mixed" else 8) * ctx.n_dofs, rel=1e-12)
        else:
            assert nbytes == 0.0
    ctx.close()
