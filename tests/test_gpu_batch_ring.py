"""GPU parity of batches whose blur changes kernels as the radii fall: float32
grids of a large working set whose line groups fill the chip take the ring
kernel at radii 32 to 192 and the relay kernel above and (up to 896 line
groups each) below. Every sort equals the same sort run alone, which takes
kernels of its own choice, bit for bit."""
import numpy as np
import pytest

import synthetic
from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch, plas = require_gpu()
    return torch, plas, plas.Context(0)


def _features(torch, side, d, seed):
    F = synthetic.gaussian_attributes(side * side, seed) if d > 32 else \
        synthetic.random_features(side * side, d, seed, "cn", -2.0, 2.0)
    return torch.from_numpy(np.ascontiguousarray(F[:d])).cuda()


CASES = [
    # Radii 230, 138, .., 1: relay, ring, relay. Both storages, an odd side out.
    ([905, 800, 701], [59, 59, 59], ["f32"] * 3, 230.0),
    ([905, 801, 300, 512, 700], [59, 59, 3, 59, 59], ["f32", "bf16", "f32", "f32", "f32"], 100.0),
    # Two rounds of more than 896 groups each: the ring below r = 32, too.
    ([1020, 1021], [64, 59], ["f32"] * 2, 40.0),
    # Two lines per group, and four; ragged last groups.
    ([1541, 1301], [31, 17], ["f32"] * 2, 100.0),
    ([3077], [14], ["f32"], 70.0),
]


@pytest.mark.parametrize("graph,sync,tune", [(False, 4, None), (True, 4, None), (True, 32, 4)])
@pytest.mark.parametrize("sides,ds,storages,start", CASES)
def test_batches_across_the_kernels_equal_single_sorts(env, sides, ds, storages, start, graph, sync, tune):
    torch, plas, ctx = env
    # Thresholds of 1/2 end a level after a few reorders.
    kw = dict(start_radius=start, radius_decay=0.6, inv_threshold=2, max_reorders=50)
    feats = [_features(torch, s, d, 40 + i) for i, (s, d) in enumerate(zip(sides, ds))]
    seeds = list(range(7, 7 + len(sides)))
    table = None if tune is None else [dict(side_lo=2, side_hi=5000, blur_waves_per_block=tune, assign_blocks=64)]
    perms, results, stats = ctx.sort_batch(feats, sides, seeds, storages=storages, graph=graph, tune=table,
                                           reorders_per_sync=sync, **kw)
    for f, side, seed, storage, perm, res in zip(feats, sides, seeds, storages, perms, results):
        want_perm, want = ctx.sort(f, side, seed, storage=storage, **kw)
        assert (res.reorders, res.levels, res.energy_fixed) == (want.reorders, want.levels, want.energy_fixed)
        assert res.trace == want.trace
        assert torch.equal(perm, want_perm)
    if graph and sync == 4 and start == 230.0:
        assert stats.graph_builds >= 3  # a plan for each kernel


def test_server_across_the_kernels_equals_single_sorts(env):
    torch, plas, ctx = env
    kw = dict(start_radius=100.0, radius_decay=0.6, inv_threshold=2, max_reorders=50)
    sides, storages = [840, 905, 500], ["f32", "f32", "bf16"]
    feats = [_features(torch, s, 59, 60 + s) for s in sides]
    server = plas.Server(ctx, 8 << 30, reorders_per_sync=3, **kw)
    done = {}
    jobs = [server.submit(feats[0], sides[0], 5, "cn", storages[0])]
    while len(done) < len(sides):
        server.step()
        if len(jobs) < len(sides):
            i = len(jobs)
            jobs.append(server.submit(feats[i], sides[i], 5 + i, "cn", storages[i]))
        for job, status, perm, res in server.poll():
            assert status == plas.OK
            done[job] = (perm, res)
    server.close()
    for i, job in enumerate(jobs):
        want_perm, want = ctx.sort(feats[i], sides[i], 5 + i, storage=storages[i], **kw)
        assert done[job][1].energy_fixed == want.energy_fixed and done[job][1].reorders == want.reorders
        assert torch.equal(done[job][0], want_perm)
