"""rn_build_backbone in the memory it is known to take: at most 34 bytes a node of scratch, its arrays
rounded up to 256 bytes each, beside the bonds, the mask and 8 bytes a node of labels. Small lattices,
where the rounding and the levels of a hierarchy weigh most."""
import numpy as np
import pytest

from paper_1908_03301_amd import binding as B

pytestmark = pytest.mark.gpu


def up(v):
    return (v + 255) & ~255


@pytest.mark.parametrize("shape", [(3, 3), (7, 5), (20, 19), (24, 16), (45, 50), (3, 8, 5)], ids=str)
def test_backbone_in_a_tight_budget(shape):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    rng = np.random.default_rng(len(shape) * 100 + shape[0])
    g = [np.exp(rng.standard_normal(shape[::-1])) * (rng.random(shape[::-1]) < 0.8) for _ in shape]
    n, dim, V = int(np.prod(shape)), len(shape), int(np.prod(shape)) + 2
    scratch = 7 * up(4 * V) + 2 * up(V) + up(4 * (V + 40)) + 256
    budget = up(8 * dim * n) + up(n) + up(8 * n) + 256 + scratch
    mask, roomy = np.zeros(n, dtype=np.uint8), np.zeros(n, dtype=np.uint8)
    nx, ny, nz = shape + (1,) * (3 - dim)
    prob = lambda m: B.problem(dim=dim, nx=nx, ny=ny, nz=nz, axis=0, g=g, mask_out=m)
    with B.Context(0) as ctx:
        want = ctx.build_backbone(prob(roomy))
    with B.Context(0, budget) as ctx:
        got = ctx.build_backbone(prob(mask))
    assert got == want
    assert np.array_equal(mask, roomy)
