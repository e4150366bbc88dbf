"""Resident iteration loop (rn_loop.hpp): a network solved alone gives, bit for
bit, the results of one launch per pass (the graph-replayed rounds,
RN_GRAPHS=1), at the edges of its tiles, over one and several workgroups, with
every tile family it has. No tolerance: the arithmetic and its order are the
same."""
import numpy as np
import pytest

from paper_1908_03301_amd import binding as B

pytestmark = pytest.mark.gpu


def network(nx, ny, nz, seed, occupancy):
    import torch
    rng = np.random.default_rng(seed)
    shape = (ny, nx) if nz == 1 else (nz, ny, nx)
    g = [np.exp(rng.standard_normal(shape)) * (rng.random(shape) < occupancy) for _ in shape]
    return [torch.from_numpy(a).cuda() for a in g]


def solve(ctx, g, nx, ny, nz, precision, axis, periodic, tol):
    import torch
    p = torch.zeros(g[0].shape, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    r = ctx.solve(B.problem(dim=len(g), nx=nx, ny=ny, nz=nz, axis=axis, g=g, p_out=p, periodic=periodic),
                  B.opts(precision, tol))
    return (r.K, r.G, r.Q_in, r.Q_out, r.rel_resid, r.iters, r.refreshes), p


# (nx, ny, nz): below, at and past a tile (64 x 8 and 64 x 4, 128 x 16 and 128 x 8 nodes), one
# workgroup, more workgroups than sum for themselves, two tiles per workgroup
SIZES_2D = [(3, 3, 1), (16, 5, 1), (63, 7, 1), (64, 8, 1), (65, 9, 1), (128, 4, 1), (129, 33, 1), (250, 131, 1),
            (520, 515, 1), (1030, 700, 1), (1500, 1420, 1)]

# tiles of 64 x 16 x 2 and x 4 nodes: the same edges, and a last tile with fewer planes
SIZES_3D = [(3, 3, 3), (5, 4, 2), (64, 16, 2), (65, 17, 3), (63, 15, 5), (30, 18, 9), (130, 33, 8), (70, 66, 64),
            (128, 120, 99)]


@pytest.mark.parametrize("precision", [B.RN_MIXED, B.RN_FP64], ids=["mixed", "fp64"])
@pytest.mark.parametrize("size", SIZES_2D + SIZES_3D, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("axis,periodic", [(0, False), (0, True), (1, True), (2, True)])
def test_loop_bits(size, precision, axis, periodic, monkeypatch):
    import torch
    nx, ny, nz = size
    if axis == 2 and nz == 1:
        pytest.skip("2D")
    big = nx * ny * nz > 100000
    g = network(nx, ny, nz, seed=nx + 7 * ny, occupancy=0.85)
    tol = 1e-3 if big else 1e-8
    monkeypatch.setenv("RN_GRAPHS", "1")
    plain = B.Context(0)
    monkeypatch.delenv("RN_GRAPHS")
    loop = B.Context(0)
    want, p0 = solve(plain, g, nx, ny, nz, precision, axis, periodic, tol)
    for _ in range(2):                       # the second solve meets the first one's exchange memory
        got, p1 = solve(loop, g, nx, ny, nz, precision, axis, periodic, tol)
        assert got == want
        assert torch.equal(p0, p1)


@pytest.mark.parametrize("precision", [B.RN_MIXED, B.RN_FP64], ids=["mixed", "fp64"])
def test_gang_bits(precision, monkeypatch):
    """Networks that run in loops beside each other, more than the chip holds at once, of every loop
    kernel's shape, and one that fits none: each gives the bits of its own solve with one launch per pass."""
    import torch
    sizes = [(70, 60, 1), (64, 8, 1), (200, 150, 1), (520, 515, 1), (700, 600, 1), (900, 850, 1), (1030, 700, 1),
             (20, 18, 17), (200, 180, 50), (64, 48, 40), (70, 66, 64), (100, 96, 60), (128, 120, 99), (120, 128, 90)]
    nets = [(s, network(*s, seed=i, occupancy=0.9)) for i, s in enumerate(sizes)]
    monkeypatch.setenv("RN_GRAPHS", "1")
    plain = B.Context(0)
    monkeypatch.delenv("RN_GRAPHS")
    gang = B.Context(0)
    want = [solve(plain, g, *s, precision, 0, False, 1e-5) for s, g in nets]
    p = [torch.zeros(g[0].shape, dtype=torch.float64, device="cuda") for _, g in nets]
    probs = [B.problem(dim=len(g), nx=s[0], ny=s[1], nz=s[2], axis=0, g=g, p_out=q) for (s, g), q in zip(nets, p)]
    torch.cuda.synchronize()
    for _ in range(2):
        for r, q, (w, pw) in zip(gang.solve_batch(probs, B.opts(precision, 1e-5)), p, want):
            assert (r.K, r.G, r.Q_in, r.Q_out, r.rel_resid, r.iters, r.refreshes) == w
            assert torch.equal(q, pw)
