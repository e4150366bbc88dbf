"""The words that resident loops exchange live in the context's HBM budget: a
budget that leaves them no room keeps a network on one launch per pass, with the
same bits, and what they keep makes way for a request that needs it."""
import numpy as np
import pytest

from paper_1908_03301_amd import binding as B

pytestmark = pytest.mark.gpu


def network(n, seed):
    import torch
    rng = np.random.default_rng(seed)
    return [torch.from_numpy(np.exp(rng.standard_normal((n, n)))).cuda() for _ in range(2)]


def solve(ctx, n, g, p, precision):
    r = ctx.solve(B.problem(dim=2, nx=n, ny=n, nz=1, axis=0, g=g, p_out=p), B.opts(precision, 1e-8, max_iter=40),
                  check=False)
    return r.K, r.Q_in, r.rel_resid, r.iters, r.refreshes


# 2000^2 mixed exchanges 2 x 4.6 MB, more than the rounding of one allocation (2 MB)
@pytest.mark.parametrize("n,precision", [(2000, B.RN_MIXED), (1400, B.RN_FP64), (128, B.RN_MIXED)])
def test_budget_without_room(n, precision):
    import torch
    B.rn_tune_reset()
    g = network(n, 5)
    p0, p1 = (torch.zeros((n, n), dtype=torch.float64, device="cuda") for _ in range(2))
    torch.cuda.synchronize()
    with B.Context(0) as roomy:
        want = solve(roomy, n, g, p0, precision)
        assert roomy.stats()["bytes_in_use"] == 0
    budget = B.rn_footprint(B.problem(dim=2, nx=n, ny=n, nz=1, axis=0, g=g), B.opts(precision))
    for _ in range(4):                       # the HIP runtime takes memory of its own in the first ones
        with B.Context(0, budget) as tight:
            before = torch.cuda.mem_get_info()[0]
            for _ in range(2):
                got = solve(tight, n, g, p1, precision)
                assert got == want and torch.equal(p0, p1)
            used = before - torch.cuda.mem_get_info()[0]
            print(f"{used} bytes taken, budget {budget}", flush=True)
            assert tight.stats()["bytes_in_use"] == 0
    assert used <= budget + (2 << 20), (used, budget)


def test_kept_memory_makes_way():
    """What a solve left for the next is given back to a request that needs the whole budget."""
    import torch
    B.rn_tune_reset()
    small, big = network(700, 1), network(1600, 2)
    torch.cuda.synchronize()
    pb = B.problem(dim=2, nx=1600, ny=1600, nz=1, axis=0, g=big)
    o = B.opts(B.RN_MIXED, 1e-8, max_iter=40)
    ps = B.problem(dim=2, nx=700, ny=700, nz=1, axis=0, g=small)
    with B.Context(0, B.rn_footprint(pb, o)) as ctx:
        for _ in range(2):
            ctx.set_timing(True)
            r = ctx.solve(ps, o, check=False)
            n = ctx.stats()["pass_timed_launches"][B.RN_PATH_2D_FULL][B.RN_MIXED]
            ctx.set_timing(False)
            assert r.iters == 40 and n < 40          # in loops
            r = ctx.solve(pb, o, check=False)
            assert r.iters == 40 and r.status == B.RN_ENOCONV


def test_batch_in_a_budget_without_room():
    """A batch that the budget holds one network at a time."""
    import torch
    B.rn_tune_reset()
    sizes = [300, 128, 400, 200]
    nets = [(n, network(n, n)) for n in sizes]
    o = B.opts(B.RN_MIXED, 1e-6)
    probs = [B.problem(dim=2, nx=n, ny=n, nz=1, axis=0, g=g) for n, g in nets]
    torch.cuda.synchronize()
    with B.Context(0) as roomy:
        want = roomy.solve_batch(probs, o)
    with B.Context(0, max(B.rn_footprint(p, o) for p in probs)) as tight:
        got = tight.solve_batch(probs, o)
        assert tight.stats()["bytes_in_use"] == 0
    for a, b in zip(got, want):
        assert (a.K, a.iters, a.refreshes, a.status) == (b.K, b.iters, b.refreshes, b.status)
