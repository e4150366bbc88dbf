"""Performance cases of the library: what a user's program has it do, through the Python entry points.

A case is a plain dict; ``prepare`` makes its inputs on the GPU from a seed, ``run`` makes one call (a
solve, a batch of solves, a backbone, a generated network) and returns its whole outputs, ``exact`` gives
the same outputs from plain torch in 64 bits where that is quick enough. The networks are the families of
the repository's own workloads (i.i.d., FBM and layered log-conductances, unit conductances, bond
dilution), at their sizes, the smallest to the largest, with odd ones between. Solves run to the relative
residual 1e-8 that the benchmark uses. One context serves every call, as in a program that keeps one.
"""
import math

import torch

from paper_1908_03301_amd import binding as B
from paper_1908_03301_amd import inputs as I

TOL = 1e-8
EXACT_NODES = 1 << 21        # exact() solves networks up to this size (a torch CG of a few seconds)
_context = []


def _ctx():
    if not _context:
        _context.append(B.Context(torch.cuda.current_device()))
    return _context[0]


def _solve(name, nx, ny, nz=1, field="fbm", H=0.7, sigma=1.5, occupancy=1.0, ratio=1.0, axis=0, periodic=False,
           precision="mixed", backbone=False, compact=False, host=False):
    return dict(name=name, op="solve", nx=nx, ny=ny, nz=nz, field=field, H=H, sigma=sigma, occupancy=occupancy,
                ratio=ratio, axis=axis, periodic=periodic, precision=precision, backbone=backbone, compact=compact,
                host=host)


def listed():
    return [
        # the smallest call: one 128^2 i.i.d. network, where the latency of an iteration is the time
        _solve("iid2d_128_mixed", 128, 128, field="iid", sigma=1.0),
        # a small odd lattice in FP64 with the paper's periodic sides, flow along y
        _solve("fbm2d_201x150_fp64_periodic", 201, 150, sigma=1.0, occupancy=0.8, axis=1, periodic=True,
               precision="fp64"),
        # one member of the anisotropy study (512^2, beta_x / beta_y = 4), plain FP64 CG
        _solve("aniso2d_512_fp64", 512, 512, H=0.75, sigma=1.0, ratio=4.0, precision="fp64"),
        # the README's call: a diluted 1024^2 network in host memory, pressures and mask back to the host
        _solve("fbm2d_1024_mixed_host", 1024, 1024, occupancy=0.6, host=True),
        # the large 2D network of the benchmark
        _solve("fbm2d_2048_mixed", 2048, 2048, occupancy=0.6),
        # a small cube, as half of a batch's members are
        _solve("fbm3d_64_mixed", 64, 64, 64, H=0.7, sigma=1.0, occupancy=0.6),
        # a middle-sized ragged block in FP64, flow along z
        _solve("fbm3d_130x101x97_fp64", 130, 101, 97, H=0.75, sigma=1.0, occupancy=0.5, axis=2, precision="fp64"),
        # the largest lattice that one call sweeps: 16.8 M nodes, as the large requests of a served stream
        _solve("fbm3d_256_mixed", 256, 256, 256, H=0.75, sigma=1.5, occupancy=0.5),
        # the layered network near its threshold, on the backbone and the compact path
        _solve("strat3d_256_mixed_bb_compact", 256, 256, 256, field="strat", H=0.8, sigma=2.0, occupancy=0.27,
               backbone=True, compact=True),
        # many networks of mixed sizes in one call: a part of the 512-network batch
        dict(name="batch48_mixed", op="batch", count=48, pick=0, precision="mixed"),
        # the backbone of a random resistor network toward its threshold
        dict(name="backbone2d_2048", op="backbone", nx=2048, ny=2048, nz=1, occupancy=0.55, axis=0),
        # generation of a correlated, diluted 3D network
        dict(name="generate3d_256", op="generate", nx=256, ny=256, nz=256, H=0.75, sigma=1.5, occupancy=0.6,
             ratio=1.0, periodic=False),
    ]


def _log_int(rng, lo, hi):
    return max(2, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def _shape(rng, dim, n_lo, n_hi):
    """Extents of about log-uniform node count: a square or cube now and then, else unequal and odd sides."""
    side = _log_int(rng, n_lo ** (1.0 / dim), n_hi ** (1.0 / dim))
    cap = int(round(n_hi ** (1.0 / dim)))
    if rng.random() < 0.3:
        ext = [side] * dim
    else:
        ext = [min(cap, max(16, int(side * rng.uniform(0.6, 1.4)))) for _ in range(dim)]
    return ext + [1] * (3 - dim)


def draw(rng):
    op = rng.choice(["solve"] * 7 + ["batch", "backbone", "generate"])
    if op == "batch":
        precision = rng.choice(["mixed", "mixed", "fp64"])
        return dict(op="batch", count=rng.randint(2, 36 if precision == "mixed" else 18), pick=rng.randint(1, 10000),
                    precision=precision)
    dim = rng.choice([2, 3])
    if op == "generate":
        nx, ny, nz = _shape(rng, dim, 1e4, 2048 ** 2 if dim == 2 else 256 ** 3)
        return dict(op="generate", nx=nx, ny=ny, nz=nz, H=round(rng.uniform(0.35, 0.9), 3),
                    sigma=round(rng.uniform(0.5, 1.5), 3), occupancy=round(rng.uniform(0.3, 1.0), 3),
                    ratio=rng.choice([1.0, 1.0, 4.0]), periodic=rng.random() < 0.5)
    if op == "backbone":
        nx, ny, nz = _shape(rng, dim, 1e4, 2048 ** 2)
        return dict(op="backbone", nx=nx, ny=ny, nz=nz, axis=rng.randrange(dim),
                    occupancy=round(rng.uniform(0.55, 0.9) if dim == 2 else rng.uniform(0.3, 0.7), 3))
    nx, ny, nz = _shape(rng, dim, 1e4, 1448 ** 2 if dim == 2 else 200 ** 3)
    option = rng.random()
    c = _solve("", nx, ny, nz, field=rng.choice(["fbm", "fbm", "fbm", "iid"]), H=round(rng.uniform(0.35, 0.9), 3),
               sigma=round(rng.uniform(0.5, 1.5), 3),
               occupancy=round(rng.uniform(0.6, 1.0) if dim == 2 else rng.uniform(0.4, 1.0), 3),
               ratio=rng.choice([1.0, 1.0, 1.0, 4.0]), axis=rng.randrange(dim), periodic=rng.random() < 0.25,
               precision=rng.choice(["mixed", "mixed", "fp64"]), backbone=option < 0.12,
               compact=option < 0.06 or 0.12 <= option < 0.16, host=rng.random() < 0.2)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs (torch on the GPU)

def _field(shape, H, ratio, noise):
    """FBM node field by Fourier filtering, standardised; `ratio` scales the spectrum's x axis."""
    spec = torch.fft.rfftn(noise)
    k2 = torch.zeros((), dtype=torch.float64, device="cuda")
    for ax, n in enumerate(shape):
        last = ax == len(shape) - 1
        f = (torch.fft.rfftfreq if last else torch.fft.fftfreq)(n, dtype=torch.float64, device="cuda")
        view = [1] * len(shape)
        view[ax] = f.numel()
        k2 = k2 + (ratio if last else 1.0) * f.reshape(view) ** 2
    amp = torch.where(k2 > 0, k2.clamp_min(1e-300) ** (-(H + 0.5 * len(shape)) / 2.0), torch.zeros_like(k2))
    phi = torch.fft.irfftn(spec * amp, s=shape)
    sd = phi.std(unbiased=False)
    return (phi - phi.mean()) / sd if float(sd) > 0.0 else torch.zeros_like(phi)


def _correlated(shape, H, ratio, gen):
    """FBM node field of a network: the corner of a field on a grid of power-of-two sides, whose transforms are ready."""
    grid = [1 << (n - 1).bit_length() for n in shape]
    noise = torch.randn(grid, generator=gen, dtype=torch.float64, device="cuda")
    return _field(grid, H, ratio, noise)[tuple(slice(0, n) for n in shape)].contiguous()


def _edge(a, k, dim):
    """A view of the last plane along lattice direction k (x is the last tensor axis)."""
    return a.select(dim - 1 - k, a.shape[dim - 1 - k] - 1)


def _bonds_of(phi, sigma, periodic):
    dim = phi.dim()
    out = []
    for k in range(dim):
        g = torch.exp(sigma * 0.5 * (phi + torch.roll(phi, -1, dim - 1 - k)))
        if not periodic:
            _edge(g, k, dim).zero_()
        out.append(g.contiguous())
    return out


def _bonds(c, gen, shape):
    """Conductances of a case's network: field, then i.i.d. bond dilution."""
    dim = len(shape)
    kind, periodic = c.get("field", "fbm"), bool(c.get("periodic", False))
    rnd = dict(generator=gen, dtype=torch.float64, device="cuda")
    if kind == "iid":
        g = [torch.exp(c["sigma"] * torch.randn(shape, **rnd)) for _ in range(dim)]
    elif kind == "unit":
        g = [torch.ones(shape, dtype=torch.float64, device="cuda") for _ in range(dim)]
    elif kind == "strat":
        phi = _correlated(shape[:1], c["H"], 1.0, gen)
        layer, up = c["sigma"] * phi, c["sigma"] * 0.5 * (phi + torch.roll(phi, -1))
        g = [torch.exp(v)[:, None, None].expand(shape).contiguous() for v in (layer, layer, up)]
    else:
        g = _bonds_of(_correlated(shape, c["H"], c.get("ratio", 1.0), gen), c["sigma"], True)
    for k in range(dim):
        if not periodic:
            _edge(g[k], k, dim).zero_()
        if c["occupancy"] < 1.0:
            g[k][torch.rand(shape, **rnd) >= c["occupancy"]] = 0.0
    return g


def _dims(c):
    dim = 2 if c["nz"] == 1 else 3
    return dim, ((c["ny"], c["nx"]) if dim == 2 else (c["nz"], c["ny"], c["nx"]))


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) & 0x7FFFFFFFFFFF)


def _members(c):
    """The sizes and parameters of a batch: a part of the repository's batch recipe, picked by the case."""
    specs = I.batch_specs(count=c["count"], seed_offset=c["pick"])
    return [dict(nx=s.side, ny=s.side, nz=s.side if s.dim == 3 else 1, field="fbm", H=s.H, sigma=1.0,
                 occupancy=s.occupancy, axis=0, periodic=False) for s in specs]


def _precision(c):
    return B.RN_MIXED if c["precision"] == "mixed" else B.RN_FP64


def _device_problem(c, g, shape, p=None, mask=None):
    if p is None:
        p = torch.zeros(shape, dtype=torch.float64, device="cuda")
        mask = torch.zeros(shape, dtype=torch.uint8, device="cuda")
    prob = B.problem(dim=len(shape), nx=c["nx"], ny=c["ny"], nz=c["nz"], axis=c["axis"], g=g, p_out=p, mask_out=mask,
                     periodic=bool(c.get("periodic", False)))
    return prob, p, mask


def prepare(case, seed):
    gen = _gen(seed)
    state = dict(case=case, ctx=_ctx())
    if case["op"] == "batch":
        # the members' outputs lie end to end in one buffer each
        members = _members(case)
        total = sum(m["nx"] * m["ny"] * m["nz"] for m in members)
        p = torch.zeros(total, dtype=torch.float64, device="cuda")
        mask = torch.zeros(total, dtype=torch.uint8, device="cuda")
        probs, at = [], 0
        for m in members:
            _, shape = _dims(m)
            n = math.prod(shape)
            probs.append(_device_problem(m, _bonds(m, gen, shape), shape, p[at:at + n], mask[at:at + n])[0])
            at += n
        state.update(probs=probs, p=p, mask=mask, opts=B.opts(_precision(case), TOL))
    elif case["op"] == "backbone":
        _, shape = _dims(case)
        mask = torch.zeros(shape, dtype=torch.uint8, device="cuda")
        g = _bonds(dict(case, field="unit"), gen, shape)
        state.update(prob=B.problem(dim=len(shape), nx=case["nx"], ny=case["ny"], nz=case["nz"], axis=case["axis"], g=g,
                                    mask_out=mask), mask=mask)
    elif case["op"] == "generate":
        dim, shape = _dims(case)
        rnd = dict(generator=gen, dtype=torch.float64, device="cuda")
        state.update(noise=torch.randn(shape, **rnd), u=[torch.rand(shape, **rnd) for _ in range(dim)],
                     field=torch.empty(shape, dtype=torch.float64, device="cuda"),
                     g=[torch.empty(shape, dtype=torch.float64, device="cuda") for _ in range(dim)])
    else:
        dim, shape = _dims(case)
        g = _bonds(case, gen, shape)
        if case["host"]:
            state["net"] = I.Network(dim, case["nx"], case["ny"], case["nz"], [a.cpu().numpy() for a in g], case["axis"],
                                     {}, bool(case["periodic"]))
        else:
            state["prob"], state["p"], state["mask"] = _device_problem(case, g, shape)
            state["opts"] = B.opts(_precision(case), TOL, backbone=case["backbone"], compact=case["compact"])
    torch.cuda.synchronize()          # the context has a stream of its own: the inputs are ready before the call
    return state


def _result(r, p, mask):
    return {"K": r.K, "G": r.G, "Q_in": r.Q_in, "Q_out": r.Q_out, "n_live": int(r.n_live), "p": p, "mask": mask}


def run(state):
    case, ctx = state["case"], state["ctx"]
    if case["op"] == "batch":
        res = ctx.solve_batch(state["probs"], state["opts"])
        return {"fluxes": torch.tensor([[r.K, r.G, r.Q_in, r.Q_out] for r in res], dtype=torch.float64),
                "n_live": torch.tensor([int(r.n_live) for r in res]), "p": state["p"], "mask": state["mask"]}
    if case["op"] == "backbone":
        n_live, n_backbone = ctx.build_backbone(state["prob"])
        return {"n_live": n_live, "n_backbone": n_backbone, "mask": state["mask"]}
    if case["op"] == "generate":
        dim = len(state["g"])
        beta = [case["ratio"]] + [1.0] * (dim - 1)
        ctx.fbm_field(dim, case["nx"], case["ny"], case["nz"], case["H"], state["noise"], state["field"], beta)
        ctx.fbm_bonds(dim, case["nx"], case["ny"], case["nz"], state["field"], case["sigma"], case["periodic"],
                      state["g"], state["u"], case["occupancy"])
        return {"field": state["field"], "g": state["g"]}
    if case["host"]:
        r, p, mask = B.solve_network(ctx, state["net"], _precision(case), TOL, want_pressure=True, want_mask=True,
                                     backbone=case["backbone"], compact=case["compact"])
        return _result(r, p, mask)
    r = ctx.solve(state["prob"], state["opts"])
    return _result(r, state["p"], state["mask"])


def work(case):
    """Bytes: the inputs read once and the outputs written once. The iterations between them are not counted: their
    number depends on the conductances, and the state they need may stay on the chip. Flops: one operator application."""
    if case["op"] == "batch":
        each = [work(dict(m, op="solve")) for m in _members(case)]
        return {k: sum(w[k] for w in each) for k in ("bytes", "flops")}
    dim = 2 if case["nz"] == 1 else 3
    n = case["nx"] * case["ny"] * case["nz"]
    if case["op"] == "backbone":
        return {"bytes": n * (8 * dim + 1), "flops": 0}
    if case["op"] == "generate":
        return {"bytes": n * 8 * (1 + 1 + 2 * dim), "flops": 5 * n * math.log2(n)}
    return {"bytes": n * (8 * dim + 8 + 1), "flops": n * 3 * 2 * dim}


# ------------------------------------------------------------------ the same in plain torch, 64 bits

def _shift(a, k, up, dim, fill):
    """a at the neighbour towards +k (up) or -k, on a grid that wraps; the wrapped plane is `fill` unless None."""
    ax = dim - 1 - k
    r = torch.roll(a, -1 if up else 1, ax)
    if fill is not None:
        r.select(ax, a.shape[ax] - 1 if up else 0).fill_(fill)
    return r


def _exact_solve(c, g):
    dim = len(g)
    axis = c["axis"]
    ax = dim - 1 - axis
    na = g[0].shape[ax]
    coord = torch.arange(na, device="cuda").reshape([-1 if a == ax else 1 for a in range(dim)]).expand(g[0].shape)
    interior = (coord > 0) & (coord < na - 1)
    wrap = [bool(c.get("periodic", False)) and k != axis and g[0].shape[dim - 1 - k] >= 2 for k in range(dim)]
    up = []
    for k in range(dim):
        a = g[k].clone()
        if not wrap[k]:
            _edge(a, k, dim).zero_()
        up.append(a)
    down = [_shift(up[k], k, False, dim, None if wrap[k] else 0.0) for k in range(dim)]

    def reach(face_plane, side):
        """Interior nodes joined to a face through interior nodes."""
        gb = (up if side else down)[axis]
        on = interior & (coord == face_plane) & (gb > 0)
        for _ in range(1 << 14):
            before = on
            for _ in range(32):
                new = on
                for k in range(dim):
                    new = new | ((up[k] > 0) & _shift(on, k, True, dim, None if wrap[k] else False))
                    new = new | ((down[k] > 0) & _shift(on, k, False, dim, None if wrap[k] else False))
                on = new & interior
            if torch.equal(on, before):
                break
        return on

    to_in, to_out = reach(1, False), reach(na - 2, True)
    live = to_in & to_out
    full = torch.where(to_in & ~to_out, 1.0, 0.0).double()
    full = torch.where(coord == 0, torch.ones_like(full), full)
    lv = live.double()
    diag = sum(up) + sum(down)

    def apply(x):                     # x is zero off the live set
        y = diag * x
        for k in range(dim):
            y -= up[k] * _shift(x, k, True, dim, None if wrap[k] else 0.0)
            y -= down[k] * _shift(x, k, False, dim, None if wrap[k] else 0.0)
        return y * lv

    inlet = torch.where(coord == 1, down[axis], torch.zeros_like(full)) * lv
    b = inlet.clone()
    x = (1.0 - coord.double() / (na - 1)) * lv
    minv = torch.where(live, 1.0 / diag.clamp_min(1e-300), torch.zeros_like(diag))
    r = b - apply(x)
    z = minv * r
    p = z.clone()
    rz = (r * z).sum()
    stop = 1e-13 * float(b.norm())
    for it in range(60000):
        q = apply(p)
        alpha = rz / (p * q).sum()
        x += alpha * p
        r -= alpha * q
        if it % 64 == 63:
            if not float(r.norm()) > stop:
                break
            if it % 1024 == 1023:
                r = b - apply(x)
        z = minv * r
        new = (r * z).sum()
        p = z + (new / rz) * p
        rz = new
    pres = torch.where(live, x, full)
    drop = pres * (coord < na - 1)
    q_in = (torch.where(coord == 0, up[axis], torch.zeros_like(drop)) *
            (1.0 - _shift(drop, axis, True, dim, None)) * _shift(live, axis, True, dim, None)).sum()
    q_out = (torch.where(coord == na - 1, down[axis], torch.zeros_like(drop)) *
             _shift(pres, axis, False, dim, None) * _shift(live, axis, False, dim, None)).sum()
    G = float(q_in)
    section = pres.numel() / na
    return {"K": G * (na - 1) / section, "G": G, "Q_in": G, "Q_out": float(q_out), "n_live": None, "p": pres, "mask": None}


def exact(case, seed):
    gen = _gen(seed)
    if case["op"] == "generate":
        dim, shape = _dims(case)
        rnd = dict(generator=gen, dtype=torch.float64, device="cuda")
        noise = torch.randn(shape, **rnd)
        u = [torch.rand(shape, **rnd) for _ in range(dim)]
        phi = _field(shape, case["H"], case["ratio"], noise)
        g = _bonds_of(phi, case["sigma"], bool(case["periodic"]))
        return {"field": phi, "g": [torch.where(v < case["occupancy"], a, torch.zeros_like(a)) for a, v in zip(g, u)]}
    if case["op"] != "solve" or case["nx"] * case["ny"] * case["nz"] > EXACT_NODES:
        return None
    _, shape = _dims(case)
    out = _exact_solve(case, _bonds(case, gen, shape))
    if case["host"]:
        out["p"] = out["p"].cpu().numpy()
    return out
