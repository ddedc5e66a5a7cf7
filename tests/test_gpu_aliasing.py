"""Calls whose output vector shares memory with their input."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hh():
    from paper_1506_06185_amd import hhgr

    return hhgr


@pytest.mark.parametrize("n_sub,level,general", [(1, 4, False), (2, 6, False), (2, 4, True)])
@pytest.mark.parametrize("shift", [0, 3, -1000])
def test_mass_in_place(hh, n_sub, level, general, shift):
    """M x written over x, or over a part of it, equals M x in a vector of its
    own, bit for bit."""
    print(f"\n[mass in place] n_sub={n_sub} level={level} general={general} shift={shift}", flush=True)
    from paper_1506_06185_amd import inputs

    ctx = hh.Context(device="cuda:0", n_sub=n_sub, level=level, general_geometry=general)
    if general:
        ctx.set_geometry(inputs.perturbed_vertices(n_sub, 5))
    n = ctx.n_dofs
    x = torch.from_numpy(np.random.default_rng(level).standard_normal(n)).cuda()
    ref = ctx.mass_apply(x)
    buf = torch.zeros(n + 2000, dtype=torch.float64, device="cuda")
    a, b = buf[1000:1000 + n], buf[1000 + shift:1000 + shift + n]
    a.copy_(x)
    torch.cuda.synchronize()
    assert hh.lib().hhgr_mass_apply(ctx.handle, a.data_ptr(), b.data_ptr()) == 0
    torch.cuda.synchronize()
    assert torch.equal(b, ref)
    ctx.close()
