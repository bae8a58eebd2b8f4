"""GPU test of a sort's host loop, which queues part of the next chunk of
reorders before it reads the last one's state: the result is that of any other
chunk length, at every place of the stop within a chunk."""
import numpy as np
import pytest

import synthetic
from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("filter", ["box", "box3"])
@pytest.mark.parametrize("max_reorders", [0, 1, 4, 5, 31, 32, 33, 36, 65])
def test_every_chunk_length_gives_the_same_sort(ref, filter, max_reorders):
    torch, plas = require_gpu()
    ctx = plas.Context(0)
    side, d = 24, 5
    F = synthetic.random_features(side * side, d, 4, "cn")
    f = torch.from_numpy(F).cuda()
    want = ref.sort(F, side, 9, max_reorders=max_reorders, filter=filter)
    assert max_reorders == 0 or want.reorders == max_reorders
    for per_sync in (1, 3, 4, 5, 0, 200):
        for profile in (False, True):
            perm, res = ctx.sort(f, side, 9, max_reorders=max_reorders, reorders_per_sync=per_sync, filter=filter,
                                 profile=profile)
            assert (res.reorders, res.energy_fixed, res.levels) == (want.reorders, want.energy, want.levels)
            assert np.array_equal(perm.cpu().numpy(), want.perm)
