"""GPU parity of radii beyond the line in every blur kernel: every window of
half-width side - 1 or more is the whole line, so the result is that of radius
side - 1, bit for bit, up to the largest radius an entry point takes."""
import numpy as np
import pytest

import synthetic
from gpu_util import bits, from_working_layout, require_gpu, to_working_layout

pytestmark = pytest.mark.gpu

BEYOND = [0, 1, 17, (1 << 30) - 1, 1 << 30, (1 << 31) - 16, (1 << 31) - 1]  # added to, or (from 2^30) as the radius


@pytest.fixture(scope="module")
def env(ref):
    torch, plas = require_gpu()
    return torch, plas, plas.Context(0), ref


def _radii(side):
    return [side - 1 + r if r < 1 << 29 else r for r in BEYOND]


# The register kernel (bfloat16 cells of 8 bytes), the relay kernel, and the
# ring kernel (float32, more than 128 MiB, 769 to 1024 line groups) with one
# and with two lines per group.
@pytest.mark.parametrize("side,d,storage", [(2, 3, "bf16"), (33, 3, "bf16"), (130, 4, "bf16"), (33, 59, "f32"),
                                            (49, 14, "bf16"), (785, 59, "f32"), (1541, 31, "f32")])
def test_blur_of_radii_beyond_the_line(env, side, d, storage):
    torch, plas, ctx, ref = env
    G = np.random.default_rng(side).standard_normal((side * side, d)).astype(np.float32)
    if storage == "bf16":
        G = torch.from_numpy(G).to(torch.bfloat16).float().numpy()
    g = to_working_layout(torch, G, plas.padded_channels(d), storage)
    want = bits(ref.blur(G, side, side - 1, storage_bf16=storage == "bf16"))
    target = torch.empty_like(g)
    for r in _radii(side):
        target.fill_(-7.0)  # a pass that writes nothing shows
        assert np.array_equal(bits(from_working_layout(ctx.stage_blur(g, side, r, target), d)), want), (side, d, r)


@pytest.mark.parametrize("side,d,storage,noalloc", [(40, 3, "bf16", False), (40, 3, "bf16", True),
                                                    (40, 59, "f32", True), (785, 59, "f32", False)])
def test_energy_of_radii_beyond_the_line(env, side, d, storage, noalloc):
    torch, plas, ctx, ref = env
    F = torch.from_numpy(synthetic.random_features(side * side, d, side)).cuda()
    want = ctx.grid_energy(F, None, side, side - 1, storage=storage, noalloc=noalloc)
    for r in _radii(side):
        assert ctx.grid_energy(F, None, side, r, storage=storage, noalloc=noalloc) == want, r


@pytest.mark.parametrize("side,d,storage", [(24, 3, "bf16"), (24, 14, "f32")])
def test_sort_from_a_radius_beyond_the_grid(env, side, d, storage):
    torch, plas, ctx, ref = env
    F = synthetic.random_features(side * side, d, 5)
    bf16 = storage == "bf16"
    for start in (side + 0.5, 2.0e9):
        perm, res = ctx.sort(torch.from_numpy(F).cuda(), side, 3, storage=storage, start_radius=start,
                             radius_decay=0.5, max_reorders=400)
        want = ref.sort(F, side, 3, start_radius=start, radius_decay=0.5, max_reorders=400, storage_bf16=bf16)
        assert (res.reorders, res.levels, res.energy_fixed) == (want.reorders, want.levels, want.energy)
        assert np.array_equal(perm.cpu().numpy(), want.perm)
