"""GPU parity of the ring blur kernel (float32, over 128 MiB, 769 to 1024 line
groups of 64 / dp lines). Radii lie on both sides of the limits of the ring (r =
47), its register slots (192) and the second load stream, windows beyond half a
line included; sides give ragged last chunks and, with several lines per group,
ragged last groups. Results are equal to the oracle's bit for bit."""
import numpy as np
import pytest

from gpu_util import bits, from_working_layout, require_gpu, to_working_layout

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env(ref):
    torch, plas = require_gpu()
    return torch, plas, plas.Context(0), ref


CASES = [
    # 771, 771 (two lines each, the last group one) and 769 groups (four, the last three)
    (771, 59, [1, 15, 16, 17, 46, 47, 48, 49, 50, 63, 64, 190, 191, 192, 193, 194, 300, 385, 386, 400, 770]),
    (1541, 31, [31, 47, 48, 191, 192, 193, 770, 771, 1500]),
    (3075, 14, [47, 192, 1600]),
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
