"""GPU parity of the assignment where its items can go wrong: every number of
lanes per item (channel widths, both storages), waves that end in the middle
of the groups, packs of four ungrouped cells with one to three left over, odd
blocks with a left-over cell, grids that are mostly ungrouped, and costs too
large for the packed (cost, ordering) keys. Integer results and moved cells
equal the oracle's."""
import numpy as np
import pytest

import synthetic
from gpu_util import bits, from_working_layout, require_gpu, to_working_layout

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env(ref):
    torch, plas = require_gpu()
    return torch, plas, plas.Context(0), ref


def _check(env, side, d, storage, beta, shift_boost=0):
    torch, plas, ctx, ref = env
    N = side * side
    F = np.random.default_rng(side * 100 + d + beta).standard_normal((N, d)).astype(np.float32)
    if storage == "bf16":
        F = torch.from_numpy(F).to(torch.bfloat16).float().numpy()
    st, s, _ = ref.scale_shift(np.ascontiguousarray(F.T))
    s += shift_boost
    P = synthetic.random_permutation(N, side + beta)
    G = np.ascontiguousarray(F[P])
    T = ref.blur(G, side, max(1, beta // 2), storage_bf16=storage == "bf16")
    keys = ref.draw(0x5EED, 1, side + beta)
    dp = plas.padded_channels(d)
    g_dev = to_working_layout(torch, G, dp, storage)
    p_dev = torch.from_numpy(P.copy()).cuda()
    dy, dx = (7 * beta) % side, (3 * beta + 1) % side
    E, moved = ctx.stage_assign(g_dev, to_working_layout(torch, T, dp, storage), p_dev, side, beta, dy, dx, keys, s)
    G_ref, P_ref = G.copy(), P.copy()
    E_ref, moved_ref = ref.assign(G_ref, T, P_ref, side, beta, dy, dx, keys, s)
    assert (E, moved) == (E_ref, moved_ref)
    assert np.array_equal(p_dev.cpu().numpy(), P_ref)
    assert np.array_equal(bits(from_working_layout(g_dev, d)), bits(G_ref))


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("d", [3, 8, 14, 31, 59])
@pytest.mark.parametrize("side,beta", [(2, 2), (3, 2), (3, 3), (5, 4), (7, 5), (16, 16), (17, 16), (18, 16),
                                       (19, 17), (33, 16), (40, 21), (61, 31), (64, 33), (96, 47), (131, 66)])
def test_assign_edges(env, side, beta, d, storage):
    _check(env, side, d, storage, beta)


# Costs from 2^57 on (a scale larger than the library's own): the packed keys
# do not hold them.
@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("d", [3, 8, 14, 31, 59])
def test_assign_large_costs(env, d, storage):
    _check(env, 20, d, storage, 9, shift_boost=7)
