"""The cube's structured-grid path (grid.hip) on the GPU against the oracle:
V-cycle iterates at grid sizes around its tile edges (8, 24, 48 and 96 cells
and powers of two), every kind of launch that a sweep count selects (two
sweeps from zero or one, sweeps in the middle of a smoothing step, none), and
the step graph when a cycle ends in the other buffer."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# operators and iterates agree with the oracle to rounding: sums of a few
# hundred terms in another order, as in the other iterate tests
TOL = 1e-12


@pytest.fixture(scope="module")
def hh():
    from paper_1506_06185_amd import hhgr

    return hhgr


def T(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def rel(a, b):
    return np.abs(a - b).max() / np.abs(b).max()


@pytest.mark.parametrize("n_sub,level,nu", [
    (1, 3, (2, 1)), (3, 3, (1, 1)), (3, 4, (2, 2)), (3, 5, (3, 1)), (1, 7, (2, 1)),
    (1, 5, (4, 2)), (2, 4, (1, 3)), (2, 3, (5, 0)), (1, 4, (0, 1)),
])
def test_iterates(hh, n_sub, level, nu):
    import oracle

    print(f"\n[grid iterates] n_sub={n_sub} level={level} nu={nu}", flush=True)
    ctx = hh.Context(device="cuda:0", n_sub=n_sub, level=level, nu_pre=nu[0], nu_post=nu[1])
    p = oracle.Problem(n_sub, level)
    g = np.random.default_rng(1000 * n_sub + 10 * level + nu[0])
    b, u = g.standard_normal(p.ndof), g.standard_normal(p.ndof)
    ctx.set_rhs(T(b))
    ctx.set_solution(T(u))
    for _ in range(3):
        r = ctx.vcycle(1)
        u, rn = p.vcycle(u, b, nu1=nu[0], nu2=nu[1])
        assert rel(ctx.get_solution().cpu().numpy(), u) < TOL
        assert abs(r * np.linalg.norm(b) - rn) <= 1e-10 * np.linalg.norm(b) * max(r, 1e-3)
    ctx.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_step_graphs_follow_the_buffers(hh, precision):
    """Graph replay equals eager cycles bit for bit over odd and even counts,
    with a fault, a local recovery and a new solution in between."""
    print(f"\n[grid graphs] {precision}", flush=True)
    out = []
    for graph in (False, True):
        ctx = hh.Context(device="cuda:0", n_sub=2, level=4, precision=precision)
        g = np.random.default_rng(3)
        ctx.set_rhs(T(g.standard_normal(ctx.n_dofs)))
        ctx.set_graph(graph)
        got = []
        for n in (1, 2, 3, 1):
            ctx.vcycle(n)
            ctx.inject_fault(7)
            ctx.recover_local(7, 2)
            got.append(ctx.get_solution().cpu().numpy())
        ctx.set_solution(T(g.standard_normal(ctx.n_dofs)))
        for n in (1, 4):
            ctx.vcycle(n)
            got.append(ctx.get_solution().cpu().numpy())
        out.append(got)
        ctx.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("n_sub,level,precision", [(1, 4, "fp64"), (2, 3, "fp64"), (3, 3, "fp64"), (3, 4, "mixed")])
def test_coarse_pcg(hh, n_sub, level, precision):
    """Cycles with a strongly varying k at 27, 343 and 1331 coarsest unknowns.
    Both sides stop their coarsest PCG at a relative residual of 1e-14, so each
    cycle's correction may differ by that times the condition number, here at
    most (2 N / pi)^2 times the contrast of the coarsest k."""
    import oracle

    print(f"\n[grid coarse pcg] n_sub={n_sub} level={level} {precision}", flush=True)
    ctx = hh.Context(device="cuda:0", n_sub=n_sub, level=level, precision=precision, variable_coeff=True)
    g = np.random.default_rng(7 * n_sub + level)
    k = np.exp(g.uniform(-1.5, 1.5, ctx.n_elems))
    cond = (8.0 * n_sub / np.pi) ** 2 * np.exp(3.0)
    p = oracle.Problem(n_sub, level, k=k)
    b, u = g.standard_normal(p.ndof), np.zeros(p.ndof)
    ctx.set_coeff(T(k))
    ctx.set_rhs(T(b))
    ctx.set_solution(None)
    if precision == "mixed":  # the FP32 cycle: only the converged solution compares
        ctx.vcycle(30)
        for _ in range(30):
            u, _ = p.vcycle(u, b)
        assert rel(ctx.get_solution().cpu().numpy(), u) < 1e-9
    else:
        for _ in range(3):
            ctx.vcycle(1)
            u, _ = p.vcycle(u, b)
            assert rel(ctx.get_solution().cpu().numpy(), u) < TOL + 2e-14 * cond
    ctx.close()


@pytest.mark.parametrize("n_sub,level", [(1, 3), (3, 4), (1, 6), (2, 6)])
def test_mass_and_vector_order(hh, n_sub, level):
    """M x and the vector order at sizes around the mass kernel's tiles (62 x
    14 nodes, 32 planes)."""
    import oracle

    print(f"\n[grid mass] n_sub={n_sub} level={level}", flush=True)
    ctx = hh.Context(device="cuda:0", n_sub=n_sub, level=level)
    x = np.random.default_rng(level).standard_normal(ctx.n_dofs)
    ctx.set_solution(T(x))
    assert np.array_equal(ctx.get_solution().cpu().numpy(), x)
    if ctx.n_dofs < 300000:
        ref = oracle.Problem(n_sub, level).apply_M(x)
    else:
        N = ctx.N
        q = np.zeros((N + 1,) * 3)
        q[1:N, 1:N, 1:N] = x.reshape((N - 1,) * 3)
        h3 = 1.0 / N ** 3

        def at(dx, dy, dz):
            return q[1 + dz:N + dz, 1 + dy:N + dy, 1 + dx:N + dx]

        ref = 0.4 * h3 * at(0, 0, 0)
        for w, ds in ((h3 / 20, ((1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 1))),
                      (h3 / 30, ((1, 1, 0), (0, 1, 1), (1, 0, 1)))):
            for d in ds:
                ref = ref + w * (at(*d) + at(-d[0], -d[1], -d[2]))
        ref = ref.reshape(-1)
    assert rel(ctx.mass_apply(T(x)).cpu().numpy(), ref) < 1e-14
    ctx.close()
