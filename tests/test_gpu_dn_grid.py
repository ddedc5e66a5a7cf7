"""Dirichlet-Neumann recovery on the cube's grid: faulty tetrahedra that share
faces, edges or vertices, every sweep count that selects other launches,
per-element k and mixed contexts, several recoveries in a row (right-hand side
and edge weights are the whole problem's again in between)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# iterates agree with the oracle to rounding, as in the other iterate tests
TOL = 1e-12


@pytest.fixture(scope="module")
def hh():
    from paper_1506_06185_amd import hhgr

    return hhgr


def T(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def rel(a, b):
    return np.abs(a - b).max() / np.abs(b).max()


@pytest.mark.parametrize("n_sub,level,vk,nu,sets", [
    (1, 4, False, (2, 1), [[1, 4], [0], [5, 2, 3]]),
    (1, 5, True, (2, 1), [[1, 4], [3]]),
    (2, 4, False, (0, 2), [[9, 25]]),
    (2, 3, True, (0, 1), [[9, 8]]),
    (2, 4, False, (2, 0), [[0, 1]]),
    (2, 4, True, (1, 0), [[3, 17]]),
    (2, 5, False, (1, 2), [[0, 1, 2, 3, 4, 5, 47, 20], [9]]),
    (3, 3, False, (3, 1), [[78, 37], [78]]),
    (3, 4, True, (2, 2), [[78, 79, 80]]),
])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_recoveries_in_a_row(hh, n_sub, level, vk, nu, sets, precision):
    import oracle

    print(f"\n[dn grid] {n_sub} {level} vk={vk} nu={nu} {sets} {precision}", flush=True)
    g = np.random.default_rng(100 * n_sub + level)
    ctx = hh.Context(device="cuda:0", n_sub=n_sub, level=level, variable_coeff=vk, precision=precision, nu_pre=nu[0],
                     nu_post=nu[1])
    k = np.exp(0.5 * g.standard_normal(ctx.n_elems)) if vk else None
    p = oracle.Problem(n_sub, level, k=k)
    b, u = g.standard_normal(p.ndof), g.standard_normal(p.ndof)
    if vk:
        ctx.set_coeff(T(k))
    ctx.set_rhs(T(b))
    ctx.set_solution(T(u))
    for tets in sets:
        for t in tets:
            ctx.inject_fault(t)
            u = p.inject_fault(t, u)
        ctx.recover_dn(tets, 2, 2)
        u = p.dn_recover(tets, u, b, n_intact=2, eta=2, nu1=nu[0], nu2=nu[1])
        assert rel(ctx.get_solution().cpu().numpy(), u) < TOL
        if precision == "fp64":
            ctx.vcycle(1)
            u, _ = p.vcycle(u, b, nu1=nu[0], nu2=nu[1])
            assert rel(ctx.get_solution().cpu().numpy(), u) < TOL
    ctx.close()
    p.close()
