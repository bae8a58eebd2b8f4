"""GPU parity of the large float32 blur passes by the way they take: the ring
kernel with 128 rows (769 to 1024 line groups of 64 / dp lines, over 128 MiB),
the ring kernel with 64 rows (1025 to 2048 groups, over 256 MiB, radii 32 to
64, or over 288 MiB, radii of 2/5 of a side and more) and the relay kernel
with streaming stores (over 1024 groups and 384 MiB, below r = 32 640 MiB).
Radii lie on both sides of every limit of the ring (r = 15, 47), its register
slots (64, 192) and the second load stream, windows beyond half a line
included; sides give ragged last chunks and, with several lines per group,
ragged last groups. Results are equal to the oracle's bit for bit."""
import numpy as np
import pytest

import synthetic
from gpu_util import bits, from_working_layout, require_gpu, to_working_layout

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env(ref):
    torch, plas = require_gpu()
    return torch, plas, plas.Context(0), ref


CASES = [
    # ring of 128 rows: 771, 771 (two lines each, the last group one) and 769 groups (four, the last three)
    (771, 59, [1, 15, 16, 17, 46, 47, 48, 49, 50, 63, 64, 190, 191, 192, 193, 194, 300, 385, 386, 400, 770]),
    (1541, 31, [31, 47, 48, 191, 192, 193, 770, 771, 1500]),
    (3075, 14, [47, 192, 1600]),
    # ring of 64 rows: 1045 groups, 1026 (the last of one line) and 1025 (the last of three)
    (1045, 59, [31, 32, 33, 47, 48, 49, 63, 64, 65]),
    (1101, 59, [32, 64, 440, 441, 550, 551, 1000, 1100]),
    (2051, 31, [32, 63, 64, 820, 821, 1030, 2050]),
    (4099, 14, [1640]),
    # relay with streaming stores, rows and columns, ragged last column blocks
    (1451, 59, [65, 100, 500]), (1641, 59, [1, 31]), (2051, 31, [65, 400]), (2051, 59, [40]),
]


@pytest.mark.parametrize("side,d,radii", CASES)
def test_blur_of_large_grids(env, side, d, radii):
    torch, plas, ctx, ref = env
    rng = np.random.default_rng(side + d)
    G = rng.standard_normal((side * side, d), dtype=np.float32) * rng.uniform(0.01, 10, d).astype(np.float32)
    g = to_working_layout(torch, G, plas.padded_channels(d))
    for r in radii:
        got = from_working_layout(ctx.stage_blur(g, side, r), d)
        assert np.array_equal(bits(got), bits(ref.blur(G, side, r))), (side, d, r)


def test_sort_across_the_kernels_does_not_depend_on_when_the_host_looks(env):
    """The host chooses a pass's kernel by the radius it last saw: after every
    reorder, every 32, or once. 1100 line groups, radii from the relay's through
    the 64-row ring's to the relay's."""
    torch, plas, ctx, ref = env
    side, d = 1100, 59
    F = torch.from_numpy(synthetic.gaussian_attributes(side * side, 11)[:d]).cuda()
    results = []
    for sync in (1, 32, 500):
        perm, res = ctx.sort(F, side, 9, start_radius=80.0, radius_decay=0.7, inv_threshold=20, max_reorders=400,
                             reorders_per_sync=sync)
        results.append((perm.cpu().numpy(), res.reorders, res.levels, res.energy_fixed))
    assert results[0][2] >= 3  # radii 80, 56, 39, ..
    for perm, *rest in results[1:]:
        assert np.array_equal(perm, results[0][0]) and rest == list(results[0][1:])
