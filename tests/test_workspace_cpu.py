"""Workspace of the cube's contexts: the unknowns are held on the grid alone."""
import pytest

# bytes per unknown at level 7 of 48 tetrahedra.  The vectors of all levels
# count 8/7 of the finest one's: u twice and b (8 B each, and 4 B each in mixed
# precision), two scratch vectors of 8 B, with k = 1 three bytes of element
# counts; per-element k: 6 values, 3 edge weights (FP64, in mixed precision
# FP32 too) and 3 in slot space.  Row padding and the slots' padding take up to
# a tenth more (16 places per row of 256, closures that share their faces), the
# index tables of the 534 k interface masters and the closures of 8 faulty
# tetrahedra about 12 bytes per unknown.
VECTORS = {
    ("fp64", False): 8 / 7 * (24 + 1 + 3) + 16,
    ("mixed", False): 8 / 7 * (24 + 12 + 1 + 3) + 16,
    ("fp64", True): 8 / 7 * (24 + 1 + 48 + 24 + 24) + 16,
    ("mixed", True): 8 / 7 * (24 + 12 + 1 + 48 + 24 + 12 + 24) + 16,
}


@pytest.mark.parametrize("precision,vk", list(VECTORS))
def test_cube_workspace(precision, vk):
    from paper_1506_06185_amd import hhgr

    d = hhgr.make_desc(n_sub=2, level=7, precision=precision, variable_coeff=vk)
    per = hhgr.workspace_bytes(d) / 255.0 ** 3
    assert VECTORS[precision, vk] < per < 1.1 * VECTORS[precision, vk] + 12, per
