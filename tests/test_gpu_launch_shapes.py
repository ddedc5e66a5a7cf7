"""Launch shapes (workgroup size, block order, nodes per thread) where the
cube's kernels read them: the local cycles of a recovery, on one tetrahedron
(a replayed graph) and on several, and the single operators.  A shape only
moves nodes between threads, so the values equal those of the default shape;
those are checked against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hh():
    from paper_1506_06185_amd import hhgr

    return hhgr


def T(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def rel(a, b):
    return np.abs(a - b).max() / np.abs(b).max()


SHAPES = [(128, 0, 1), (128, 1, 4), (256, 0, 4), (512, 0, 1), (512, 1, 4)]


# ragged last workgroups at every size; per-element k takes other kernels
@pytest.mark.parametrize("n_sub,level,vk", [(1, 4, False), (2, 5, False), (1, 6, False), (2, 4, True)])
def test_local_cycles_and_operators(hh, n_sub, level, vk):
    import oracle

    print(f"\n[shapes] n_sub={n_sub} level={level} vk={vk}", flush=True)
    g = np.random.default_rng(10 * n_sub + level)
    nt = 6 * n_sub ** 3
    one, two = nt // 2, [1, nt - 1]
    ctx = hh.Context(device="cuda:0", n_sub=n_sub, level=level, variable_coeff=vk)
    k = np.exp(0.5 * g.standard_normal(ctx.n_elems)) if vk else None
    p = oracle.Problem(n_sub, level, k=k)
    b, u0 = g.standard_normal(p.ndof), g.standard_normal(p.ndof)
    if vk:
        ctx.set_coeff(T(k))
    ctx.set_rhs(T(b))

    def run():
        ctx.set_solution(T(u0))
        ctx.inject_fault(one)
        ctx.recover_local(one, 2)
        for t in two:
            ctx.inject_fault(t)
        ctx.recover_dd(two, 1, 3)
        out = [ctx.get_solution().cpu().numpy()]
        for l in range(3, level + 1):
            n = p.ndof_at(l)
            x, y = T(u0[:n]), T(b[:n])
            out += [hh.debug_op(ctx, op, l, x, y).cpu().numpy() for op in (0, 1, 2, 3)]
            out.append(hh.debug_op(ctx, 4, l, x).cpu().numpy())
            out.append(hh.debug_op(ctx, 5, l, T(u0[:p.ndof_at(l - 1)]), x).cpu().numpy())
        return out

    ref = run()
    u, _ = p.recover_local([one], p.inject_fault(one, u0), b, n_cycles=2)
    for t in two:
        u = p.inject_fault(t, u)
    u, _ = p.recover_local(two, p.dd_intact(two, u, b, 1), b, n_cycles=3)
    assert rel(ref[0], u) < 1e-12
    for shape in SHAPES:
        ctx.set_tuning(*shape)
        for q, (x, y) in enumerate(zip(run(), ref)):
            assert np.array_equal(x, y), (shape, q)
    ctx.close()
