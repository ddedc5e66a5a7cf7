"""Batches that are armed again with another faulty set, on meshes whose
masked steps run over a list of intact tetrahedra."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1506_06185_amd import inputs  # noqa: E402


@pytest.fixture(scope="module")
def hh():
    from paper_1506_06185_amd import hhgr

    return hhgr


def member(hh, kind, seed):
    if kind == "general":
        ctx = hh.Context(device="cuda:0", n_sub=2, level=4, general_geometry=True)
        ctx.set_geometry(inputs.perturbed_vertices(2, 5))
    elif kind == "mesh":
        v, t = inputs.box_mesh(2, 2, 1)
        ctx = hh.Context(device="cuda:0", mesh=(inputs.perturb_mesh(v, seed=0, amplitude=0.1), t), level=4)
    else:
        ctx = hh.Context(device="cuda:0", n_sub=2, level=4)
    b = np.random.default_rng(seed).uniform(-1.0, 1.0, ctx.n_dofs)
    ctx.set_rhs(torch.from_numpy(b).cuda())
    ctx.set_solution(None)
    ctx.vcycle(2)
    return ctx


@pytest.mark.parametrize("kind", ["general", "mesh", "cube"])
def test_rearmed_batch_equals_fresh_batches(hh, kind):
    """One batch, armed with one, two and one faulty tetrahedra in turn, against
    a new batch for every run: the same launches on the same data, so the same
    bits."""
    sets = [[3], [7, 3], [11]]
    out = []
    for fresh in (False, True):
        ctx = member(hh, kind, 31)
        batch, got = None, []
        for tets in sets:
            print(f"\n[batch re-armed] {kind} fresh={fresh} {tets}", flush=True)
            if fresh or batch is None:
                batch = hh.Batch([ctx])
            for t in tets:
                ctx.inject_fault(t)
            batch.arm_dd(0, tets, 1, 2)
            batch.run(1e-14, 3, raise_on_noconv=False)
            got.append(ctx.get_solution().cpu().numpy())
            if fresh:
                batch.close()
        if not fresh:
            batch.close()
        ctx.close()
        out.append(got)
    for a, b in zip(*out):
        assert np.isfinite(a).all() and np.array_equal(a, b)
