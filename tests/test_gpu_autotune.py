"""GPU tests of plas_autotune_batch: shapes are timed with the whole batch
running, so a bucket's choice is one for the launches it will run in."""
import ctypes

import pytest

import synthetic
from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch, plas = require_gpu()
    return torch, plas, plas.Context(0)


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("sides,ds,storages", [
    ([2, 2, 3], [3, 3, 1], ["f32", "bf16", "f32"]),  # sorts that end while they are timed
    ([2, 16, 40, 57, 90, 128], [59, 3, 59, 14, 59, 4], ["f32", "bf16", "f32", "bf16", "bf16", "bf16"]),
    ([770, 800, 33], [59, 59, 59], ["f32"] * 3),  # a large working set
])
def test_table_covers_the_sides_and_keeps_results(env, sides, ds, storages, graph):
    torch, plas, ctx = env
    feats = [torch.from_numpy(synthetic.random_features(s * s, d, 3 + i)).cuda()
             for i, (s, d) in enumerate(zip(sides, ds))]
    table = ctx.autotune_batch(feats, sides=sides, seeds=5, storages=storages, graph=graph)
    for s in sides:
        e = [t for t in table if t["side_lo"] <= s <= t["side_hi"]]
        assert len(e) >= 1
        assert e[0]["blur_waves_per_block"] in (1, 2, 4) and e[0]["assign_blocks"] in (0, 256, 1024, 16384)
    kw = dict(inv_threshold=5, max_reorders=40)
    perms, results, _ = ctx.sort_batch(feats, sides, 5, storages=storages, tune=table, graph=graph, **kw)
    for f, side, storage, perm, res in zip(feats, sides, storages, perms, results):
        want_perm, want = ctx.sort(f, side, 5, storage=storage, **kw)
        assert res.energy_fixed == want.energy_fixed and res.trace == want.trace
        assert torch.equal(perm, want_perm)


def test_errors_are_reported_and_leave_the_handle_usable(env):
    torch, plas, ctx = env
    f = torch.from_numpy(synthetic.gaussian_attributes(64, 1)).cuda()
    bad = f.clone()
    bad[3, 9] = float("inf")
    with pytest.raises(plas.PlasError) as e:
        ctx.autotune_batch([f, bad], sides=[8, 8])
    assert e.value.status == plas.ERR_NONFINITE
    with pytest.raises(plas.PlasError) as e:
        ctx.autotune_batch([f], sides=[9])
    assert e.value.status == plas.ERR_INVALID_ARGUMENT
    assert ctx.autotune_batch([f], sides=[8])


def test_every_item_runs_before_a_shape_is_timed(env):
    """A bad item of the last side bucket is found before the first bucket's
    shapes are timed (with the whole batch), so no entry is written."""
    torch, plas, ctx = env
    good = torch.from_numpy(synthetic.gaussian_attributes(64, 1)).cuda()
    bad = torch.from_numpy(synthetic.gaussian_attributes(4096, 2)).cuda()
    bad[3, 9] = float("nan")
    items, keep = ctx._batch_items([good, bad], [8, 64], 5, "cn", "f32", None, None)
    table, entries = (plas.TuneEntry * 4)(), ctypes.c_int32(-1)
    status = plas.library().plas_autotune_batch(ctx._h, items, 2, None, 0, table, 4, ctypes.byref(entries))
    assert status == plas.ERR_NONFINITE and entries.value == 0
    assert keep
