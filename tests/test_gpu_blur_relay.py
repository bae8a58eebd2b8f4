"""GPU parity of the relay blur (loading, summing and storing waves) where its
steps can go wrong: sides around the chunk of 16 positions and around whole
line groups, radii around the chunk, the ring's limit (r = 31 | 32) and whole
lines, column blocks of several line groups, zeros of both signs. The kernel
and the oracle evaluate the same operations in the same order, so the results
are equal bit for bit."""
import numpy as np
import pytest

from gpu_util import bits, from_working_layout, require_gpu, to_working_layout

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env(ref):
    torch, plas = require_gpu()
    return torch, plas, plas.Context(0), ref


def _grid(torch, side, d, storage, seed):
    rng = np.random.default_rng(seed)
    G = rng.standard_normal((side * side, d)).astype(np.float32) * rng.uniform(0.01, 10, d).astype(np.float32)
    G[rng.random(G.shape) < 0.1] = 0.0
    G[rng.random(G.shape) < 0.1] = -0.0
    if storage == "bf16":
        G = torch.from_numpy(G).to(torch.bfloat16).float().numpy()
    return G


def _check(env, side, d, storage, radii):
    torch, plas, ctx, ref = env
    G = _grid(torch, side, d, storage, side * 100 + d)
    g = to_working_layout(torch, G, plas.padded_channels(d), storage)
    for r in radii:
        T = from_working_layout(ctx.stage_blur(g, side, r), d)
        want = ref.blur(G, side, r, storage_bf16=storage == "bf16")
        assert np.array_equal(bits(T), bits(want)), (side, d, storage, r)


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("d", [3, 8, 14, 31, 59])
@pytest.mark.parametrize("side", [2, 15, 16, 17, 31, 32, 33, 49, 64, 65, 129, 161])
def test_relay_edges(env, side, d, storage):
    radii = {1, 7, 8, 15, 16, 23, 24, 30, 31, 32, 33, 39, 40, 47, 48, 63, 64, 65,
             side // 2 - 1, side // 2, side - 2, side - 1, side, side + 17, 1 << 30}
    _check(env, side, d, storage, sorted(r for r in radii if r > 0))


# More than 128 MiB: column blocks of three line groups (bfloat16; float32 of
# at most 768 groups) and of two (float32 of more than 1024), ragged last
# blocks among them.
@pytest.mark.parametrize("side,d,storage,radii", [
    (1030, 59, "bf16", [1, 31, 32, 400]), (2057, 14, "bf16", [15, 40]),
    (733, 59, "f32", [31, 32, 300]), (1450, 14, "f32", [16, 33]), (1027, 59, "f32", [31, 32, 513]),
])
def test_relay_column_blocks(env, side, d, storage, radii):
    _check(env, side, d, storage, radii)
