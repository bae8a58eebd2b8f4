"""Performance cases of the PLAS library: the calls its users make, over the
sizes, channel counts, storages, layouts and options they make them with.

Each case is a dict of plain values; prepare() makes its inputs on the GPU,
run() is one pass through the public Python entry points, work() the bytes
and operations such a pass cannot do without, and exact() the float64 value
of the computed numbers. Case kinds:

  sort    one sort to the end of its radius schedule. inv_threshold says how
          thoroughly each radius is sorted: 10000 is the default, 1000 and
          100 the coarser thresholds of the paper's runtime experiment
          (App. C), which visit every radius of the schedule with fewer
          reorders each.
  batch   several grids sorted together (Context.sort_batch).
  serve   jobs through a Server: half are waiting when it starts, the rest
          join while the first ones run.
  energy  the energy of an arrangement (Context.grid_energy), with its own
          workspace or with the allocation-free query for small grids.
  vad     the neighbour-difference variance of an arrangement (Context.vad).

Features follow the library's benchmark inputs: 3D Gaussian Splatting
attribute vectors (position, log-scale, rotation, opacity, SH colour; 59
channels, or the first of them), or uniform RGB values for 3 channels.
"""
from __future__ import annotations

import math

import torch

import paper_2312_13299_amd as plas

SORT_SEED = 0x5EED


def listed():
    return [
        # The smallest calls: a sweep over small crops asks for the energy of
        # each (latency and launches are all there is) ...
        dict(name="energy_small", kind="energy", side=96, d=59, layout="cn", dtype="f32", storage="f32", radius=2,
             noalloc=True),
        # ... and a preview sorts one tile with every default.
        dict(name="sort_64_d59", kind="sort", side=64, d=59, layout="cn", dtype="f32", storage="f32", filter="box",
             inv_threshold=10000),
        # The paper's 512 x 512 RGB runtime experiment, with the box filter
        # at 1/1000 and with the Gaussian-like filter at 1/100.
        dict(name="sort_512_rgb", kind="sort", side=512, d=3, layout="cn", dtype="f32", storage="f32", filter="box",
             inv_threshold=1000),
        dict(name="sort_512_rgb_box3", kind="sort", side=512, d=3, layout="cn", dtype="f32", storage="f32",
             filter="box3", inv_threshold=100),
        # A mid-sized object, vector-major bfloat16 features, an odd side.
        dict(name="sort_723_d59_nc", kind="sort", side=723, d=59, layout="nc", dtype="bf16", storage="f32",
             filter="box", inv_threshold=100),
        # A scene of a million Gaussians with every attribute.
        dict(name="sort_1024_d59", kind="sort", side=1024, d=59, layout="cn", dtype="f32", storage="f32",
             filter="box", inv_threshold=100),
        # Two million Gaussians with bfloat16 working grids.
        dict(name="sort_1448_d59_bf16", kind="sort", side=1448, d=59, layout="cn", dtype="f32", storage="bf16",
             filter="box", inv_threshold=100),
        # The largest scene (4.4 million Gaussians), without the higher SH
        # coefficients.
        dict(name="sort_2091_d14", kind="sort", side=2091, d=14, layout="cn", dtype="f32", storage="f32",
             filter="box", inv_threshold=100),
        # Many objects of ragged sizes in one batch.
        dict(name="batch_12_d59", kind="batch", sides="131,163,198,223,257,301,338,389,452,511,602,724", d=59,
             layout="cn", dtype="f32", storages="f32", filter="box", inv_threshold=100),
        # A serving stream: float32 and bfloat16 jobs.
        dict(name="serve_8_d59", kind="serve", sides="256,283,341,420,487,573,660,768", d=59, layout="cn",
             dtype="f32", storages="f32,bf16", filter="box", inv_threshold=100),
        # Quality queries of a sorted scene.
        dict(name="energy_1024_d59", kind="energy", side=1024, d=59, layout="cn", dtype="f32", storage="f32", radius=1,
             noalloc=False),
        dict(name="vad_1024_d59", kind="vad", side=1024, d=59, layout="cn", dtype="f32"),
    ]


# ------------------------------------------------------------------- drawing

def _log_int(rng, lo, hi):
    return int(min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_one(rng):
    kind = rng.choice(["sort", "sort", "sort", "sort", "batch", "serve", "energy", "vad"])
    d = rng.choice([3, 14, 59, 59, rng.randint(1, 64)])
    layout = rng.choice(["cn", "cn", "nc"])
    dtype = rng.choice(["f32", "f32", "bf16"])
    storage = rng.choice(["f32", "f32", "bf16"])
    flt = rng.choice(["box", "box", "box", "box3"])
    if kind == "sort":
        return dict(kind=kind, side=_log_int(rng, 24, 2091), d=d, layout=layout, dtype=dtype, storage=storage,
                    filter=flt, inv_threshold=rng.choice([100, 100, 1000, 10000]))
    if kind == "batch":
        sides = [_log_int(rng, 64, 724) for _ in range(rng.randint(2, 16))]
        return dict(kind=kind, sides=",".join(map(str, sides)), d=d, layout=layout, dtype=dtype,
                    storages=rng.choice(["f32", "bf16", "f32,bf16"]), filter=flt, inv_threshold=100)
    if kind == "serve":
        sides = [_log_int(rng, 128, 1024) for _ in range(rng.randint(2, 8))]
        return dict(kind=kind, sides=",".join(map(str, sides)), d=d, layout=layout, dtype=dtype,
                    storages=rng.choice(["f32", "f32,bf16"]), filter=flt, inv_threshold=100)
    if kind == "energy":
        side = _log_int(rng, 16, 1448)
        return dict(kind=kind, side=side, d=d, layout=layout, dtype=dtype, storage=storage,
                    radius=rng.choice([1, 1, 2, 5, 15, 40]), noalloc=side <= 256 and rng.random() < 0.5)
    return dict(kind=kind, side=_log_int(rng, 16, 1448), d=d, layout=layout, dtype=dtype)


def draw(rng):
    """One more case of the listed ranges; none costs more than the dearest
    listed one."""
    limit = max(_cost(c) for c in listed())
    while True:
        case = _draw_one(rng)
        if _cost(case) <= limit:
            return case


def _schedule_levels(side):
    phi, levels = max(1.0, side / 2.0 - 1.0), 0
    while phi >= 1.0:
        levels += 1
        phi *= 0.95
    return levels


def _padded(d):
    dp = 4
    while dp < d:
        dp *= 2
    return dp


def _sides(case):
    return [int(s) for s in case["sides"].split(",")] if "sides" in case else [case["side"]]


def _storages(case):
    names = case["storages"].split(",") if "storages" in case else [case.get("storage", "f32")]
    return [names[i % len(names)] for i in range(len(_sides(case)))]


def _cost(case):
    """A rough duration in seconds, to keep drawn cases within the listed
    range."""
    if case["kind"] in ("energy", "vad"):
        return 10.0 * case["side"] ** 2 * _padded(case["d"]) * 4 / 1e12 + 1e-4
    per_level = {100: 4.5, 1000: 20.0, 10000: 68.0}[case["inv_threshold"]]
    passes = 7.0 if case["filter"] == "box3" else 3.0
    cells = sum(s * s * (2 if st == "bf16" else 4) for s, st in zip(_sides(case), _storages(case)))
    reorder = passes * (2.0 * cells * _padded(case["d"]) / 4e12 + max(_sides(case)) * 6e-8 + 8e-6)
    return max(_schedule_levels(s) for s in _sides(case)) * per_level * reorder


# -------------------------------------------------------------------- inputs

def _features(n, d, seed, layout, dtype):
    """n feature vectors on the GPU, [d][n] ("cn") or [n][d] ("nc")."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(k, scale=1.0, mean=0.0):
        return torch.randn(k, n, generator=gen, device="cuda") * scale + mean

    def uniform(k, lo, hi):
        return torch.rand(k, n, generator=gen, device="cuda") * (hi - lo) + lo

    if d == 3:
        f = uniform(3, 0.0, 255.0)
    else:
        centres = torch.rand(8, 3, generator=gen, device="cuda") * 4.0 - 2.0
        comp = torch.randint(0, 8, (n,), generator=gen, device="cuda")
        q = normal(4)
        q = q / q.norm(dim=0, keepdim=True).clamp_min(1e-12)
        parts = [centres[comp].t() + normal(3, 0.3), normal(3, 0.5, -4.0), q, normal(1, 2.0), uniform(3, -1.0, 1.0),
                 normal(50, 0.1)]
        f = torch.cat(parts, 0)[:d]
    if layout == "nc":
        f = f.t()
    return f.to(torch.bfloat16 if dtype == "bf16" else torch.float32).contiguous()


def _permutation(n, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed + 77)
    return torch.randperm(n, generator=gen, device="cuda", dtype=torch.int32)


def prepare(case, seed):
    kind = case["kind"]
    state = dict(case=case, ctx=plas.context(0))
    sides = _sides(case)
    state["features"] = [_features(s * s, case["d"], seed * 1000 + i, case["layout"], case["dtype"])
                         for i, s in enumerate(sides)]
    if kind in ("energy", "vad"):
        state["perm"] = _permutation(sides[0] ** 2, seed)
    else:
        state["out"] = [torch.empty(s * s, dtype=torch.int32, device="cuda") for s in sides]
        state["seeds"] = [SORT_SEED + seed * 100 + i for i in range(len(sides))]
    if kind == "serve":
        state["server"] = plas.Server(state["ctx"], 64 << 30, inv_threshold=case["inv_threshold"],
                                      filter=case["filter"])
    return state


# ----------------------------------------------------------------------- run

def _sort_outputs(perm, res):
    return perm, res.energy_fixed, res.energy, res.reorders


def run(state):
    case, ctx = state["case"], state["ctx"]
    kind = case["kind"]
    if kind == "sort":
        perm, res = ctx.sort(state["features"][0], case["side"], state["seeds"][0], case["layout"],
                             inv_threshold=case["inv_threshold"], storage=case["storage"], filter=case["filter"],
                             out=state["out"][0])
        return _sort_outputs(perm, res)
    if kind == "batch":
        perms, results, _ = ctx.sort_batch(state["features"], _sides(case), state["seeds"], case["layout"],
                                           _storages(case), inv_threshold=case["inv_threshold"],
                                           filter=case["filter"], out=state["out"])
        return [_sort_outputs(p, r) for p, r in zip(perms, results)]
    if kind == "serve":
        server, sides, storages = state["server"], _sides(case), _storages(case)

        def submit(i):
            return server.submit(state["features"][i], sides[i], state["seeds"][i], case["layout"], storages[i],
                                 out=state["out"][i])

        half = (len(sides) + 1) // 2
        jobs = [submit(i) for i in range(half)]
        done = {}
        while len(done) < len(sides):
            server.step()
            if len(jobs) < len(sides):
                jobs.append(submit(len(jobs)))
            for job, status, perm, res in server.poll():
                if status != plas.OK:
                    raise RuntimeError(f"job {job} failed with status {status}")
                done[job] = _sort_outputs(perm, res)
        return [done[j] for j in jobs]
    if kind == "energy":
        return ctx.grid_energy(state["features"][0], state["perm"], case["side"], case["radius"], case["layout"],
                               case["storage"], noalloc=case["noalloc"])
    return ctx.vad(state["features"][0], state["perm"], case["side"], case["layout"])


# ---------------------------------------------------------------------- work

def work(case):
    """Bytes and operations of one pass. A sort runs at least three reorders
    at each radius (one that improves, one that does not, one with a new
    shift that does not either); a reorder filters the grid (per axis and
    box pass: each value read and written once, one addition, one
    subtraction and one product) and assigns (grid and target read once;
    per group of four cells 16 distances)."""
    d = case["d"]
    in_bytes = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "vad":
        n = case["side"] ** 2
        return {"bytes": n * (d * in_bytes + 4), "flops": n * d * 2 * 5}
    if case["kind"] == "energy":
        n = case["side"] ** 2
        return {"bytes": n * (d * in_bytes + 4), "flops": n * d * (6 + 3)}
    passes = 6 if case["filter"] == "box3" else 2
    total_bytes = total_flops = 0
    for side, storage in zip(_sides(case), _storages(case)):
        n = side * side
        value = 2 if storage == "bf16" else 4
        reorders = 3 * _schedule_levels(side)
        total_bytes += n * (d * in_bytes + 4) + reorders * n * d * value * (2 * passes + 2)
        total_flops += reorders * n * d * (3 * passes + 12)
    return {"bytes": total_bytes, "flops": total_flops}


# --------------------------------------------------------------------- exact

def _box_mean(grid, radius, dim):
    """Mean over the window of half-width radius, clipped to the grid, along
    dim of a [side][side][d] float64 grid."""
    side = grid.shape[dim]
    total = torch.cat([torch.zeros_like(grid.narrow(dim, 0, 1)), grid.cumsum(dim)], dim)
    pos = torch.arange(side, device=grid.device)
    hi = (pos + radius + 1).clamp_max(side)
    lo = (pos - radius).clamp_min(0)
    shape = [1, 1, 1]
    shape[dim] = side
    return (total.index_select(dim, hi) - total.index_select(dim, lo)) / (hi - lo).to(grid.dtype).reshape(shape)


def exact(case, seed):
    """The energy's mean and the VAD in float64 with plain torch. A sort's
    outputs are decisions and sums of its own rounded arithmetic: no value of
    theirs is independent of it."""
    if case["kind"] not in ("energy", "vad"):
        return None
    side, d = case["side"], case["d"]
    n = side * side
    f = _features(n, d, seed * 1000, case["layout"], case["dtype"]).double()
    if case["layout"] == "cn":
        f = f.t()
    grid = f[_permutation(n, seed).long()].reshape(side, side, d)
    if case["kind"] == "vad":
        diffs = torch.cat([(grid[:, 1:] - grid[:, :-1]).abs().reshape(-1), (grid[1:] - grid[:-1]).abs().reshape(-1)])
        return float(((diffs - diffs.mean()) ** 2).mean())
    target = _box_mean(_box_mean(grid, case["radius"], 1), case["radius"], 0)
    return None, None, float(((grid - target) ** 2).sum() / n)
