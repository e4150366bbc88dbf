"""Which launches run a network's passes, seen from the launch counts of
rn_set_timing: resident loops where its workgroups fit the chip, of every shape
they are built for, and one launch per pass where a loop is turned away at its
gate (RN_LOOPS=2), with the bits of a context without loops (RN_LOOPS=0)."""
import numpy as np
import pytest

from paper_1908_03301_amd import binding as B

pytestmark = pytest.mark.gpu

# (nx, ny, nz), precision, and the launch plan that picks the loop kernel: path, tiles
# per workgroup, tile depth. Of the small 2D tiles, up to 32 workgroups run on one XCD.
FULL, SMALL, BLOCK = B.RN_PATH_2D_FULL, B.RN_PATH_2D_SMALL, B.RN_PATH_3D
SHAPES = [((128, 128, 1), B.RN_MIXED, (SMALL, 1, 1)), ((64, 120, 1), B.RN_FP64, (SMALL, 1, 1)),
          ((210, 160, 1), B.RN_MIXED, (SMALL, 1, 1)), ((201, 150, 1), B.RN_FP64, (SMALL, 1, 1)),
          ((520, 515, 1), B.RN_MIXED, (FULL, 1, 1)), ((520, 515, 1), B.RN_FP64, (FULL, 1, 1)),
          ((1500, 1420, 1), B.RN_MIXED, (FULL, 2, 1)), ((1390, 1400, 1), B.RN_FP64, (FULL, 2, 1)),
          ((65, 40, 33), B.RN_MIXED, (BLOCK, 1, 2)), ((65, 40, 33), B.RN_FP64, (BLOCK, 1, 2)),
          ((128, 120, 99), B.RN_MIXED, (BLOCK, 1, 4)), ((128, 120, 99), B.RN_FP64, (BLOCK, 1, 4))]


def ident(v):
    return "x".join(map(str, v)) if isinstance(v, tuple) else ("mixed" if v == B.RN_MIXED else "fp64")


def network(size, seed):
    import torch
    rng = np.random.default_rng(seed)
    shape = size[::-1] if size[2] > 1 else size[1::-1]
    return [torch.from_numpy(np.exp(rng.standard_normal(shape))).cuda() for _ in shape]


def problem(size, g, p_out=None):
    return B.problem(dim=len(g), nx=size[0], ny=size[1], nz=size[2], axis=0, g=g, p_out=p_out)


def context(monkeypatch, loops):
    monkeypatch.setenv("RN_LOOPS", loops)
    c = B.Context(0)
    monkeypatch.delenv("RN_LOOPS")
    return c


def tolerance(size):
    return 1e-8 if size[0] * size[1] * size[2] < 100000 else 1e-6


def bits(r):
    return r.K, r.G, r.Q_in, r.Q_out, r.rel_resid, r.iters, r.refreshes


def timed(ctx, prob, o):
    """The solve's result and its timed launches, all of them of its own path and precision."""
    ctx.set_timing(True)
    r = ctx.solve(prob, o)
    launches = ctx.stats()["pass_timed_launches"]
    ctx.set_timing(False)
    return r, launches


@pytest.mark.parametrize("size,precision,plan", SHAPES, ids=ident)
def test_loops_run(size, precision, plan, monkeypatch):
    import torch
    B.rn_tune_reset()
    g = network(size, 3)
    p = B.rn_plan(problem(size, g), B.opts(precision))
    assert (p["path"], p["tiles_per_wg"], p["tile_z"]) == plan
    torch.cuda.synchronize()
    with context(monkeypatch, "1") as ctx:
        r, launches = timed(ctx, problem(size, g), B.opts(precision, tolerance(size)))
    n = launches[plan[0]][precision]
    # without a loop every pass is a launch; with them a refresh and the passes up to the next one are two
    assert 0 < n < (r.iters + r.refreshes) / 2, (n, r.iters, r.refreshes)
    assert sum(map(sum, launches)) == n


@pytest.mark.parametrize("precision", [B.RN_MIXED, B.RN_FP64], ids=ident)
def test_gangs_run(precision, monkeypatch):
    """Two networks of every shape in one batch: each path's passes run in loops beside each other."""
    import torch
    B.rn_tune_reset()
    sizes = [s for s, p, _ in SHAPES if p == precision and s[0] * s[1] * s[2] < 400000]
    g = {s: network(s, 13) for s in sizes}
    o = B.opts(precision, 1e-6)
    probs = [problem(s, g[s]) for s in sizes for _ in range(2)]
    paths = [B.rn_plan(p, o)["path"] for p in probs]
    assert sorted(set(paths)) == [FULL, SMALL, BLOCK]
    torch.cuda.synchronize()
    with context(monkeypatch, "1") as ctx:
        ctx.set_timing(True)
        res = ctx.solve_batch(probs, o)
        launches = ctx.stats()["pass_timed_launches"]
    for path in (FULL, SMALL, BLOCK):
        passes = max(r.iters + r.refreshes for r, p in zip(res, paths) if p == path)
        # without loops a path's launches are at least the passes of its longest solve
        assert 0 < launches[path][precision] < passes / 2, (path, launches, passes)


@pytest.mark.parametrize("size,precision,plan", SHAPES, ids=ident)
def test_turned_away_bits(size, precision, plan, monkeypatch):
    import torch
    B.rn_tune_reset()
    g = network(size, 4)
    o = B.opts(precision, tolerance(size), max_iter=4000)
    pw, pg = (torch.zeros(g[0].shape, dtype=torch.float64, device="cuda") for _ in range(2))
    torch.cuda.synchronize()
    with context(monkeypatch, "0") as plain, context(monkeypatch, "2") as away:
        want = plain.solve(problem(size, g, pw), o, check=False)
        for _ in range(2):
            got, launches = timed(away, problem(size, g, pg), o)
            assert bits(got) == bits(want)
            assert torch.equal(pg, pw)
            # the host has noticed: every pass was a launch
            assert launches[plan[0]][precision] >= got.iters + got.refreshes


@pytest.mark.parametrize("size,precision,plan", SHAPES, ids=ident)
def test_pass_numbers_start_over(size, precision, plan, monkeypatch):
    """The tags of the words that loops exchange start over with cleared words: in the first solve or the second."""
    import torch
    B.rn_tune_reset()
    g = network(size, 5)
    o = B.opts(precision, tolerance(size))
    pw, pg = (torch.zeros(g[0].shape, dtype=torch.float64, device="cuda") for _ in range(2))
    torch.cuda.synchronize()
    with context(monkeypatch, "0") as plain, context(monkeypatch, "3") as loop:
        want = plain.solve(problem(size, g, pw), o)
        for _ in range(3):
            got, launches = timed(loop, problem(size, g, pg), o)
            assert bits(got) == bits(want)
            assert torch.equal(pg, pw)
            assert launches[plan[0]][precision] < (got.iters + got.refreshes) / 2


@pytest.mark.parametrize("precision", [B.RN_MIXED, B.RN_FP64], ids=ident)
def test_turned_away_gang_bits(precision, monkeypatch):
    import torch
    B.rn_tune_reset()
    sizes = [(70, 60, 1), (200, 150, 1), (520, 515, 1), (20, 18, 17), (70, 66, 64), (64, 48, 40), (130, 70, 1)]
    nets = [(s, network(s, 10 + i)) for i, s in enumerate(sizes)]
    pw, pg = ([torch.zeros(g[0].shape, dtype=torch.float64, device="cuda") for _, g in nets] for _ in range(2))
    o = B.opts(precision, 1e-6, max_iter=4000)
    torch.cuda.synchronize()
    with context(monkeypatch, "0") as plain, context(monkeypatch, "2") as away:
        want = [plain.solve(problem(s, g, q), o, check=False) for (s, g), q in zip(nets, pw)]
        got = away.solve_batch([problem(s, g, q) for (s, g), q in zip(nets, pg)], o, check=False)
    for a, b, qa, qb in zip(got, want, pg, pw):
        assert bits(a) == bits(b)
        assert torch.equal(qa, qb)


def test_launches_do_not_depend_on_earlier_calls(monkeypatch):
    """1,000 passes on one XCD are two loops of at most 512, before and after a batch ran the same shape
    on the whole chip."""
    import torch
    B.rn_tune_reset()
    size = (64, 120, 1)
    g = network(size, 6)
    o = B.opts(B.RN_FP64, 1e-30, max_iter=1000)
    torch.cuda.synchronize()
    with context(monkeypatch, "1") as ctx:
        first, a = timed(ctx, problem(size, g), o)
        ctx.solve_batch([problem(size, g), problem(size, g)], o, check=False)
        again, b = timed(ctx, problem(size, g), o)
    assert bits(first) == bits(again) and first.iters == 1000
    # a chunk is a pass and a loop, twice, the first with a pass more (two refreshes): all iterations
    # in the first, the last refresh in the second, and the idle chunk that is on its way by then
    assert a == b and a[SMALL][B.RN_FP64] == 5 + 4 + 4


def test_turned_away_waits_once(monkeypatch):
    """A gate gives up after 0.5 ms. The loops that were launched before the host knew (two chunks of two,
    the last of them after four iterations) do not wait again: the device is held by one such wait, not three."""
    import torch
    B.rn_tune_reset()
    size = (64, 120, 1)
    g = network(size, 7)
    o = B.opts(B.RN_FP64, 1e-30, max_iter=4)     # few passes: all else is some tens of microseconds
    torch.cuda.synchronize()

    def device_time(ctx):
        best = 1e9
        for _ in range(8):
            ctx.set_timing(True)
            ctx.solve(problem(size, g), o)
            best = min(best, sum(map(sum, ctx.stats()["pass_device_s"])))
            ctx.set_timing(False)
        return best

    with context(monkeypatch, "0") as plain, context(monkeypatch, "2") as away:
        more = device_time(away) - device_time(plain)
    print(f"turned away: {1e3 * more:.3f} ms more", flush=True)
    assert more < 1.0e-3


def test_launch_count_of_a_network_turned_away(monkeypatch):
    """rn_stats.launches of a solve that starts in loops and goes on without: each pass once, and at most
    the idle rounds of a chunk (256) more."""
    import torch
    B.rn_tune_reset()
    size = (64, 120, 1)
    g = network(size, 8)
    o = B.opts(B.RN_FP64, 1e-30, max_iter=2000)
    torch.cuda.synchronize()
    with context(monkeypatch, "2") as away:
        for k in range(1, 3):
            r = away.solve(problem(size, g), o)
            passes = r.iters + r.refreshes
            assert passes > 1000
            n = away.stats()["launches"]
            assert k * passes - 8 <= n <= k * (passes + 2 * 256), (n, k, passes)


def test_peak_counts_networks_that_run(monkeypatch):
    """Three networks of 456 workgroups each, where the chip holds 1,024 in loops: two at a time."""
    import torch
    B.rn_tune_reset()
    size = (700, 600, 1)
    g = network(size, 9)
    o = B.opts(B.RN_FP64, 1e-30, max_iter=4000)
    probs = [problem(size, g) for _ in range(3)]
    assert B.rn_plan(probs[0], o)["workgroups"] == 456
    torch.cuda.synchronize()
    with context(monkeypatch, "1") as ctx:
        ctx.solve_batch(probs, o, check=False)
        assert ctx.stats()["peak_active"] == 2
    with context(monkeypatch, "0") as ctx:
        ctx.solve_batch(probs, o, check=False)
        assert ctx.stats()["peak_active"] == 3
