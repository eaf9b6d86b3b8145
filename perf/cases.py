"""The work that programs have this library do, as cases that can be timed and
compared: binning and the cutoff sweep of one system, the pair kernels of the
paper's timing grid, time stepping, batches of many systems, and the request
server.

A case is a dict of plain values; ``prepare(case, seed)`` makes its inputs on
the GPU from the seed, ``run(state)`` is one pass through the public entry
points, ``work(case)`` the bytes and operations a pass cannot do without, and
``exact(case, seed)`` the outputs in 64 bits from plain torch.

Coordinates are multiples of a power of two, as in ``synth``, so every pair
difference is exact in float32 and neighbour counts are whole numbers that do
not depend on the organisation the tuner picks.
"""
import math
import random

import numpy as np
import torch

from paper_2406_16091_amd import device, pi, synth

# ------------------------------------------------------------------ the cases


def _sweep(name, n, dims, **more):
    return {"name": name, "op": "sweep", "n": n, "nx": dims[0], "ny": dims[1], "nz": dims[2], "cell_log2": 0, "rc": 1.0,
            "blobs": 0, "precision": "compensated", "order": "sorted", **more}


def _pair(name, n, d, kernel, precision):
    return {"name": name, "op": "pair", "n": n, "nx": d, "ny": d, "nz": d, "kernel": kernel, "precision": precision}


def listed():
    return [
        # the paper's timing grid at 8^3 cells, one particle each: the
        # smallest call, where launches and latency are all there is
        _pair("pair_lj_512", 512, 8, "lj", "plain"),
        # 32,768 uniform particles on 32^3 cells, the small benchmark system:
        # one step of a small simulation
        _sweep("sweep_32k_1ppc", 1 << 15, (32, 32, 32), cell_log2=-5),
        # the headline system: 2^24 uniform particles, one per cell
        _sweep("sweep_16m_1ppc", 1 << 24, (256, 256, 256), cell_log2=-8),
        # the same particles in wider cells, eight each
        _sweep("sweep_16m_8ppc", 1 << 24, (128, 128, 128), cell_log2=-7),
        # Gaussian blobs on a uniform background, 0 to about 75 per cell
        _sweep("sweep_8m_clustered", 1 << 23, (128, 128, 128), cell_log2=-7, blobs=64),
        # odd counts and extents, a cutoff smaller than the cell, results in
        # the caller's particle order: a user's own box
        _sweep("sweep_1m_ragged", 1234567, (97, 83, 61), rc=0.75, order="original"),
        # 64 per cell everywhere with plain sums
        _sweep("sweep_2m_64ppc_plain", 1 << 21, (32, 32, 32), cell_log2=-5, precision="plain"),
        # the densest entry of the paper's timing grid, 32^3 cells of 100
        _pair("pair_lj_3m_100ppc", 3276800, 32, "lj", "plain"),
        # the 168-FLOP kernel at 10 per cell with compensated sums
        _pair("pair_highflop_328k", 327680, 32, "highflop", "compensated"),
        # a simulation that reads its state back every fourth step
        {"name": "step_16m", "op": "step", "n": 1 << 24, "nx": 256, "ny": 256, "nz": 256, "cell_log2": -8, "steps": 4},
        # 512 independent systems of 1e3 to 2e5 particles in one call
        {"name": "batch_512", "op": "batch", "systems": 512, "n_lo": 1000, "n_hi": 200000, "sizes": 4},
        # 24 small requests through the server, each swept eight times with
        # displacements between: host arrays in, host arrays out
        {"name": "serve_24", "op": "serve", "requests": 24, "n_lo": 2000, "n_hi": 100000, "sweeps": 8, "sizes": 5},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _box(rng, cells):
    """Three extents near each other whose product is about `cells`."""
    a, b = rng.uniform(0.7, 1.4), rng.uniform(0.7, 1.4)
    g = max(1.0, cells) ** (1.0 / 3.0)
    return tuple(int(min(600, max(1, round(g * f)))) for f in (a, b, 1.0 / (a * b)))


def draw(rng):
    op = rng.choices(("sweep", "pair", "step", "batch", "serve"), (9, 4, 3, 2, 2))[0]
    if op == "sweep":
        blobs = rng.choice((0, 0, 0, rng.randint(2, 64)))
        ppc = math.exp(rng.uniform(math.log(0.5), math.log(8.0 if blobs else 64.0)))
        n = _log_uniform(rng, 1 << 12, min(1 << (23 if blobs else 24), (1 << 27) / max(1.0, ppc)))
        c = _sweep("", n, _box(rng, n / ppc), rc=rng.choice((1.0, 1.0, 0.9375, 0.75)), blobs=blobs,
                   precision=rng.choices(("compensated", "plain", "fp64acc"), (6, 2, 2))[0],
                   order=rng.choice(("sorted", "original")))
        del c["name"]
        return c
    if op == "pair":
        d, ppc = rng.randint(4, 32), math.exp(rng.uniform(0.0, math.log(100.0)))
        c = _pair("", max(2, int(d ** 3 * ppc)), d, rng.choice(("lj", "lowflop", "highflop")),
                  rng.choice(("plain", "compensated")))
        if c["kernel"] == "highflop":
            c["n"] = min(c["n"], 10 * d ** 3)
        del c["name"]
        return c
    if op == "step":
        n = _log_uniform(rng, 1 << 14, 1 << 23)
        nx, ny, nz = _box(rng, n / math.exp(rng.uniform(math.log(0.7), math.log(6.0))))
        return {"op": "step", "n": n, "nx": nx, "ny": ny, "nz": nz, "cell_log2": 0, "steps": rng.randint(1, 4)}
    if op == "batch":
        return {"op": "batch", "systems": _log_uniform(rng, 2, 512), "n_lo": 1000,
                "n_hi": _log_uniform(rng, 4000, 200000), "sizes": rng.randrange(1 << 20)}
    return {"op": "serve", "requests": rng.randint(1, 24), "n_lo": 2000, "n_hi": _log_uniform(rng, 4000, 100000),
            "sweeps": rng.randint(1, 8), "sizes": rng.randrange(1 << 20)}


# ------------------------------------------------------------------ inputs


def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _gen(seed):
    g = torch.Generator(device=_dev())
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _weights(n, g):
    """U[0.5, 1.5) on the 2^-23 lattice."""
    return 0.5 + torch.randint(0, 1 << 23, (n,), generator=g, device=_dev()).float() * 2.0 ** -23


def _lattice_log2(dims, w_log2):
    """p such that the box, in multiples of 2^-p, stays within 2^24."""
    return 24 - w_log2 - max(0, math.ceil(math.log2(max(dims))))


def _uniform(n, dims, w_log2, g):
    """n points uniform in the box of dims cells of width 2^w_log2, on its lattice."""
    p = _lattice_log2(dims, w_log2)
    return [torch.randint(0, d << (p + w_log2), (n,), generator=g, device=_dev()).float() * 2.0 ** -p for d in dims]


def _clustered(n, dims, w_log2, blobs, g):
    """Gaussian blobs truncated to the box on a 10% uniform background:
    widths U(0.04, 0.08) of the box, raised where a blob's centre would hold
    more than about 60 per cell."""
    p, dev = _lattice_log2(dims, w_log2), _dev()
    ext = torch.tensor(dims, dtype=torch.float64, device=dev)
    n_bg = n // 10
    n_bl = n - n_bg
    side = float(ext.prod()) ** (1.0 / 3.0)
    sig = (0.04 + 0.04 * torch.rand(blobs, generator=g, device=dev, dtype=torch.float64)) * side
    sig = sig.clamp(min=(n_bl / blobs / ((2.0 * math.pi) ** 1.5 * 60.0)) ** (1.0 / 3.0))
    centre = torch.rand((blobs, 3), generator=g, device=dev, dtype=torch.float64) * ext
    which = torch.randint(0, blobs, (n_bl,), generator=g, device=dev)
    pts = torch.empty((n, 3), dtype=torch.float64, device=dev)
    pts[:n_bg] = torch.rand((n_bg, 3), generator=g, device=dev, dtype=torch.float64) * ext
    todo = torch.arange(n_bl, device=dev)
    while todo.numel():
        b = which[todo]
        q = centre[b] + sig[b, None] * torch.randn((todo.numel(), 3), generator=g, device=dev, dtype=torch.float64)
        ok = ((q >= 0) & (q < ext)).all(1)
        pts[n_bg + todo[ok]] = q[ok]
        todo = todo[~ok]
    pts = pts[torch.randperm(n, generator=g, device=dev)]
    return [torch.floor(pts[:, a] * 2.0 ** (p + w_log2)).float() * 2.0 ** -p for a in range(3)]


def _system(case, seed):
    """Positions, weights, extents and cell width of a one-system case."""
    g = _gen(seed)
    dims, w_log2 = (case["nx"], case["ny"], case["nz"]), case.get("cell_log2", 0)
    if case["op"] == "pair" and not case["nx"] & (case["nx"] - 1):
        w_log2 = -(case["nx"].bit_length() - 1)  # the unit cube, as the timing grid has it
    if case.get("blobs"):
        xyz = _clustered(case["n"], dims, w_log2, case["blobs"], g)
    else:
        xyz = _uniform(case["n"], dims, w_log2, g)
    return xyz, _weights(case["n"], g), dims, 2.0 ** w_log2, g


def _velocities(n, w, g):
    """N(0, (0.05 w)^2) per axis."""
    return [0.05 * w * torch.randn(n, generator=g, device=_dev()) for _ in range(3)]


class _Shape:
    """One system's size and grid, for pi.make_system_descs."""

    def __init__(self, n, g):
        self.n, self.dims, self.origin, self.cell_w, self.rc = n, (g, g, g), (0.0, 0.0, 0.0), 1.0, 1.0


def _batch_shapes(case):
    """Sizes log-uniform in [n_lo, n_hi], 1 to 4 per cell, 10 to 58 cells a side."""
    rng = random.Random(case["sizes"])
    out = []
    for _ in range(case["systems"]):
        n = _log_uniform(rng, case["n_lo"], case["n_hi"])
        out.append(_Shape(n, int(min(58, max(10, round((n / rng.uniform(1.0, 4.0)) ** (1.0 / 3.0)))))))
    return out


def _batch_inputs(case, seed):
    shapes, g, dev = _batch_shapes(case), _gen(seed), _dev()
    count = torch.tensor([s.n for s in shapes], device=dev)
    side = torch.repeat_interleave(torch.tensor([s.dims[0] for s in shapes], device=dev), count)
    n = int(count.sum())
    xyz = [(torch.randint(0, 1 << 40, (n,), generator=g, device=dev) % (side << 18)).float() * 2.0 ** -18
           for _ in range(3)]
    return shapes, side, count, xyz, _weights(n, g)


def _requests(case, seed):
    """Requests of log-uniform size, half of them of eight blobs, 1, 2, 4 or 8 per cell."""
    rng, g = random.Random(case["sizes"]), _gen(seed)
    out = []
    for k in range(case["requests"]):
        n = _log_uniform(rng, case["n_lo"], case["n_hi"])
        side = max(1, round((n / rng.choice((1, 2, 4, 8))) ** (1.0 / 3.0)))
        dims = (side, side, side)
        xyz = _clustered(n, dims, 0, 8, g) if rng.random() < 0.5 else _uniform(n, dims, 0, g)
        # the server's lattice of 2^-16 cells
        host = [np.floor(v.cpu().numpy() * np.float32(65536.0)) * np.float32(2.0 ** -16) for v in xyz]
        s = synth.System("request", host[0], host[1], host[2], _weights(n, g).cpu().numpy(), (0.0, 0.0, 0.0), dims, 1.0,
                         1.0)
        out.append(pi.make_request(s, n_sweeps=case["sweeps"], jitter_sigma=0.1, lattice=2.0 ** -16,
                                   seed=1000 * int(seed) + k))
    return out


class _State:
    """Device arrays and the library's object of one case."""

    def __init__(self, case):
        self.case, self.ctx, self.cells, self.batch = case, device.Context.get(0).handle, None, None

    def outputs(self, n):
        dev = _dev()
        self.rho, self.gx, self.gy, self.gz = (torch.empty(n, device=dev) for _ in range(4))
        self.count = torch.empty(n, dtype=torch.int32, device=dev)

    def invariants(self, systems=1):
        self.inv = torch.zeros(pi.INV_BYTES * systems, dtype=torch.uint8, device=_dev())
        # pairs, and the two sums that do not cancel (the net force is the
        # rounding left of a sum that is zero)
        words = self.inv.view(torch.int64).view(systems, -1)
        self.pairs, self.sums = words[:, 0], words.view(torch.float64)[:, 4:6]

    def __del__(self):
        try:
            if self.cells is not None:
                pi.pi_cells_destroy(self.cells)
            if self.batch is not None:
                pi.pi_batch_destroy(self.batch)
        except Exception:
            pass


_servers = {}


def _server():
    """The one server a serving program keeps."""
    if "it" not in _servers:
        _servers["it"] = pi.pi_server_create(device.Context.get(0).handle, max_slots=64, n_streams=4)
    return _servers["it"]


def prepare(case, seed):
    s = _State(case)
    op = case["op"]
    if op == "batch":
        shapes, _, _, s.xyz, s.w = _batch_inputs(case, seed)
        s.n = s.w.numel()
        s.descs = pi.make_system_descs(shapes)
        s.batch = pi.pi_batch_create(s.ctx)
        s.opts = pi.make_opts(order="original")
        s.outputs(s.n)
        s.invariants(len(shapes))
        s.stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        return s
    if op == "serve":
        s.server, s.requests = _server(), _requests(case, seed)
        n = sum(int(r.n) for r in s.requests)
        s.host = {k: np.empty(n, np.int32 if k == "count" else np.float32)
                  for k in ("rho", "gx", "gy", "gz", "count", "x", "y", "z")}
        s.pair_sums = np.empty((len(s.requests), case["sweeps"]), np.int64)
        return s
    s.xyz, s.w, dims, w, g = _system(case, seed)
    s.n, rc = case["n"], case.get("rc", 1.0) * w
    s.grid = pi.make_grid((0.0, 0.0, 0.0), dims, w, rc)
    s.cells = pi.pi_cells_create(s.ctx)
    if op == "sweep":
        s.opts = pi.make_opts(case["precision"], "auto", case["order"])
        s.outputs(s.n)
        s.invariants()
    elif op == "pair":
        s.opts = pi.make_pairfn_opts(case["kernel"], case["precision"])
        s.v = torch.empty(s.n, device=_dev())
        s.count = torch.empty(s.n, dtype=torch.int32, device=_dev())
    else:  # step: a binned system with velocities
        s.opts = pi.make_step_opts(0.25, 0.02 * rc ** 5, 2.0 ** -_lattice_log2(dims, case["cell_log2"]))
        s.outputs(s.n)
        s.invariants()
        s.vel = _velocities(s.n, w, g)
        s.out = [torch.empty(s.n, device=_dev()) for _ in range(6)]
        pi.pi_bin(s.ctx, s.cells, *s.xyz, s.w, s.n, s.grid)
        pi.pi_state_set_velocity(s.ctx, s.cells, *s.vel)
    return s


# ------------------------------------------------------------------ one pass


def run(s):
    op = s.case["op"]
    if op == "sweep":
        pi.pi_bin(s.ctx, s.cells, *s.xyz, s.w, s.n, s.grid)
        pi.pi_interact(s.ctx, s.cells, s.opts, s.rho, s.gx, s.gy, s.gz, s.count, s.inv)
        return {"rho": s.rho, "gx": s.gx, "gy": s.gy, "gz": s.gz, "count": s.count, "pairs": s.pairs, "sums": s.sums}
    if op == "pair":
        pi.pi_bin(s.ctx, s.cells, *s.xyz, s.w, s.n, s.grid)
        pi.pi_interact_pairfn(s.ctx, s.cells, s.opts, s.v, s.count)
        return {"v": s.v, "count": s.count}
    if op == "step":
        for _ in range(s.case["steps"]):
            pi.pi_step(s.ctx, s.cells, s.opts, s.inv)
        pi.pi_state_get(s.ctx, s.cells, *s.out, s.rho, s.gx, s.gy, s.gz)
        return {"x": s.out[0], "y": s.out[1], "z": s.out[2], "vx": s.out[3], "vy": s.out[4], "vz": s.out[5],
                "rho": s.rho, "gx": s.gx, "gy": s.gy, "gz": s.gz}
    if op == "batch":
        pi.pi_batch_run(s.ctx, s.batch, s.descs, *s.xyz, s.w, s.opts, s.rho, s.gx, s.gy, s.gz, s.count, s.inv,
                        s.stream)
        return {"rho": s.rho, "gx": s.gx, "gy": s.gy, "gz": s.gz, "count": s.count, "pairs": s.pairs, "sums": s.sums}
    tickets = [pi.pi_submit(s.server, r) for r in s.requests]
    at = 0
    for k, t in enumerate(tickets):
        r = pi.pi_wait(s.server, t, copy=False)
        if r["status"] != pi.PI_OK:
            raise pi.PiError(r["status"], "request")
        for key, to in s.host.items():
            to[at:at + r["n"]] = r[key]
        s.pair_sums[k] = r["pairs_per_sweep"]
        at += r["n"]
        pi.pi_release(s.server, t)
    return dict(s.host, pairs=s.pair_sums)


# ------------------------------------------------------------------ floors

# Operations of a candidate's distance and of an accepted pair (FMA = 2), as
# bench.py counts them; of one evaluation of each pair kernel.
_CANDIDATE = 8.0
_PAIR = {"plain": 22.0, "compensated": 50.6, "fp64acc": 50.6}
_PAIRFN = {"lj": 17.0, "lowflop": 6.0, "highflop": 167.0}


def _sweep_flops(n, cells, rc, precision, dims=None, crowd=1.0):
    """One sweep of n particles: candidates of 27 cells clipped at the faces,
    and pairs in the cutoff sphere; crowd: mean density around a particle over
    the mean density."""
    clip = math.prod(1.0 - 2.0 / (3.0 * d) for d in dims) if dims else 1.0
    near = n / cells * crowd * clip
    return n * near * (27.0 * _CANDIDATE + 4.0 / 3.0 * math.pi * rc ** 3 * _PAIR[precision])


def work(case):
    op = case["op"]
    if op == "batch":
        shapes = _batch_shapes(case)
        n = sum(s.n for s in shapes)
        return {"bytes": 36.0 * n, "flops": sum(_sweep_flops(s.n, s.dims[0] ** 3, 1.0, "compensated", s.dims)
                                                for s in shapes)}
    if op == "serve":
        # positions and weights in, results and positions out; the sweeps
        rng = random.Random(case["sizes"])
        n, flops = 0, 0.0
        for _ in range(case["requests"]):
            m = _log_uniform(rng, case["n_lo"], case["n_hi"])
            ppc, clustered = rng.choice((1, 2, 4, 8)), rng.random() < 0.5
            n += m
            flops += case["sweeps"] * _sweep_flops(m, m / ppc, 1.0, "compensated", crowd=3.0 if clustered else 1.0)
        return {"bytes": 48.0 * n, "flops": flops}
    n, dims = case["n"], (case["nx"], case["ny"], case["nz"])
    cells = math.prod(dims)
    if op == "pair":
        clip = math.prod(1.0 - 2.0 / (3.0 * d) for d in dims)
        return {"bytes": 24.0 * n, "flops": n * 27.0 * clip * n / cells * _PAIRFN[case["kernel"]]}
    if op == "step":
        # per step the state (positions, velocities, weights) in and the
        # positions and velocities out; the state and the sums read back
        return {"bytes": (52.0 * case["steps"] + 80.0) * n,
                "flops": case["steps"] * _sweep_flops(n, cells, 1.0, "compensated", dims)}
    return {"bytes": 36.0 * n, "flops": _sweep_flops(n, cells, case["rc"], case["precision"], dims,
                                                     3.5 if case["blobs"] else 1.0)}


# ------------------------------------------------------------------ 64 bits


def _bin64(xyz, side, w):
    """Cell coordinates, stable cell order, and each cell's start and count.
    side: cells per axis, three numbers or three tensors with an entry per
    particle followed by the first cell of its system."""
    nx, ny, nz, base, cells = side
    i = [torch.floor(v.double() / w).long() for v in xyz]
    c = base + i[0] + nx * (i[1] + ny * i[2])
    order = torch.sort(c, stable=True).indices
    count = torch.bincount(c, minlength=cells)
    start = torch.cumsum(count, 0) - count
    return i, order, start, count


def _pairs64(xyz, w, side, width, visit):
    """Calls visit(targets, sources, dx, dy, dz) over every candidate pair of
    the 27 cells, each target at most once a call; positions in 64 bits."""
    i, order, start, count = _bin64(xyz, side, width)
    nx, ny, nz, base, _ = side
    me = torch.arange(order.numel(), device=order.device)
    p = [v.double() for v in xyz]
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                x, y, z = i[0] + dx, i[1] + dy, i[2] + dz
                ok = (x >= 0) & (x < nx) & (y >= 0) & (y < ny) & (z >= 0) & (z < nz)
                cell = torch.where(ok, base + x + nx * (y + ny * z), torch.zeros_like(x))
                left = torch.where(ok, count[cell], torch.zeros_like(x))
                first = start[cell]
                t, k = me[left > 0], 0
                del x, y, z, ok, cell
                while t.numel():
                    j = order[first[t] + k]
                    visit(t, j, *(q[t] - q[j] for q in p))
                    k += 1
                    t = t[left[t] > k]
    return order


def _spline64(xyz, w, side, width, rc):
    """rho, G, counts, A (the magnitudes of G's terms) and the cell order."""
    n, dev = w.numel(), w.device
    out = torch.zeros((5, n), dtype=torch.float64, device=dev)
    count = torch.zeros(n, dtype=torch.int32, device=dev)
    wd, sigma = w.double(), 8.0 / (math.pi * rc ** 3)

    def visit(t, j, dx, dy, dz):
        r2 = dx * dx + dy * dy + dz * dz
        at = torch.nonzero((r2 < rc * rc) & (t != j)).squeeze(1)
        t, j, dx, dy, dz, r = t[at], j[at], dx[at], dy[at], dz[at], r2[at].sqrt()
        q = r / rc
        inner = q <= 0.5
        val = torch.where(inner, sigma * (6.0 * q ** 3 - 6.0 * q ** 2 + 1.0), 2.0 * sigma * (1.0 - q) ** 3)
        der = torch.where(inner, sigma / rc * (18.0 * q ** 2 - 12.0 * q), -6.0 * sigma / rc * (1.0 - q) ** 2)
        wj = wd[j]
        f = torch.where(r > 0, wj * der / r, torch.zeros_like(r))
        for row, v in enumerate((wj * val, f * dx, f * dy, f * dz, wj * der.abs())):
            out[row].index_add_(0, t, v)
        count.index_add_(0, t, torch.ones_like(t, dtype=torch.int32))

    order = _pairs64(xyz, w, side, width, visit)
    return out, count, order


def _exact_sweep(xyz, w, side, width, rc, in_order, systems=None):
    out, count, order = _spline64(xyz, w, side, width, rc)
    wd = w.double()
    scale, rho = wd * out[4], out[0]
    if systems is None:
        sums = torch.stack([scale.sum(), rho.sum()]).view(1, 2)
        pairs = count.sum().view(1)
    else:
        owner = torch.repeat_interleave(torch.arange(systems.numel(), device=w.device), systems)
        sums = torch.zeros((systems.numel(), 2), dtype=torch.float64, device=w.device)
        sums[:, 0].index_add_(0, owner, scale)
        sums[:, 1].index_add_(0, owner, rho)
        pairs = torch.zeros(systems.numel(), dtype=torch.int64, device=w.device).index_add_(0, owner, count.long())
    at = order if in_order else slice(None)
    return {"rho": out[0][at], "gx": out[1][at], "gy": out[2][at], "gz": out[3][at], "count": count[at],
            "pairs": pairs, "sums": sums}


def _exact_pair(case, xyz, w, side, width):
    n, kernel = w.numel(), case["kernel"]
    sigma2, eps2 = (0.5 * width) ** 2, (0.25 * width) ** 2
    v = torch.zeros(n, dtype=torch.float64, device=w.device)
    count = torch.zeros(n, dtype=torch.int32, device=w.device)

    def visit(t, j, dx, dy, dz):
        if kernel == "lowflop":
            k = dx + dy + dz
        else:
            u3 = (sigma2 / (dx * dx + dy * dy + dz * dz + eps2)) ** 3
            k = 4.0 * (u3 * u3 - u3)
        other = (t != j)
        v.index_add_(0, t, torch.where(other, k, torch.zeros_like(k)))
        count.index_add_(0, t, other.to(torch.int32))

    order = _pairs64(xyz, w, side, width, visit)
    return {"v": v[order], "count": count[order]}


def _exact_step(case, xyz, w, vel, side, width, rc):
    dims, dt, kappa = side[:3], 0.25, 0.02 * rc ** 5
    lattice = 2.0 ** -_lattice_log2(dims, case["cell_log2"])
    x, v = [q.double() for q in xyz], [q.double() for q in vel]
    for _ in range(case["steps"]):
        out, _, _ = _spline64(x, w, side, width, rc)
        for a in range(3):
            top = dims[a] * width
            v[a] = v[a] - dt * kappa * out[1 + a]
            p = x[a] + (dt * v[a]).clamp(-0.5 * width, 0.5 * width)
            low, high = p < 0, p >= top
            p = torch.where(low, -p, torch.where(high, 2.0 * top - p, p))
            v[a] = torch.where(low | high, -v[a], v[a])
            x[a] = (torch.floor(p / lattice) * lattice).clamp(0.0, top - lattice)
    return {"x": x[0], "y": x[1], "z": x[2], "vx": v[0], "vy": v[1], "vz": v[2],
            "rho": out[0], "gx": out[1], "gy": out[2], "gz": out[3]}


def exact(case, seed):
    op = case["op"]
    if op == "serve":
        return None  # the displacements come from the server's own generator
    if op == "batch":
        _, side, systems, xyz, w = _batch_inputs(case, seed)
        cells = torch.tensor([s.dims[0] ** 3 for s in _batch_shapes(case)], device=w.device)
        base = torch.repeat_interleave(torch.cumsum(cells, 0) - cells, systems)
        return _exact_sweep(xyz, w, (side, side, side, base, int(cells.sum())), 1.0, 1.0, False, systems)
    xyz, w, dims, width, g = _system(case, seed)
    side = (*dims, 0, math.prod(dims))
    if op == "pair":
        return _exact_pair(case, xyz, w, side, width)
    if op == "step":
        return _exact_step(case, xyz, w, _velocities(case["n"], width, g), side, width, width)
    return _exact_sweep(xyz, w, side, width, case["rc"] * width, case["order"] == "sorted")
