"""GPU tests of the features' way into the working grid: the permutation check,
the ingest in arranged order with the features' range and energy scale, and
the fixed-point energy, all through the energy query, whose whole-number
results equal the oracle's; and which calls it refuses, in which order."""
import numpy as np
import pytest

import synthetic
from gpu_util import require_gpu

pytestmark = pytest.mark.gpu

# Tiles hold 4096 / dp cells (dp 4: 1024, 8: 512, 16: 256, 32: 128, 64: 64):
# part of one tile, just under and over whole tiles, and more tiles than the
# 512 blocks of a launch (d 59 from side 182, d 16 from side 363).
SHAPES = [(2, 59), (7, 64), (8, 59), (9, 33), (32, 3), (33, 3), (45, 8), (46, 5), (64, 59), (127, 16), (181, 59),
          (182, 57), (183, 64), (257, 20), (363, 14), (725, 4)]


@pytest.fixture(scope="module")
def env():
    torch, plas = require_gpu()
    return torch, plas, plas.Context(0)


@pytest.mark.parametrize("layout", ["cn", "nc"])
@pytest.mark.parametrize("dtype,storage", [("f32", "f32"), ("f32", "bf16"), ("bf16", "f32"), ("bf16", "bf16")])
@pytest.mark.parametrize("side,d", SHAPES)
def test_energy_equals_the_oracle(env, ref, side, d, dtype, storage, layout):
    torch, plas, ctx = env
    n = side * side
    F = synthetic.random_features(n, d, side * 100 + d, layout, -3.0, 5.0)
    if dtype == "bf16":
        F = ref.round_bf16(F)
    f = torch.from_numpy(F).cuda()
    if dtype == "bf16":
        f = f.to(torch.bfloat16)
    perm = synthetic.random_permutation(n, side) if side % 2 else None
    p = None if perm is None else torch.from_numpy(perm).cuda()
    E, s, mean = ctx.grid_energy(f, p, side, 1, layout, storage=storage)
    assert (ref.OK, E, s, mean) == ref.grid_energy(F, perm, side, 1, layout, storage == "bf16")


@pytest.mark.parametrize("side,d", [(8, 59), (183, 59), (300, 3)])
@pytest.mark.parametrize("fault", ["twice", "negative", "n", "far"])
def test_a_permutation_that_is_none_is_refused(env, side, d, fault):
    torch, plas, ctx = env
    n = side * side
    f = torch.from_numpy(synthetic.random_features(n, d, 3, "cn")).cuda()
    good = synthetic.random_permutation(n, 5)
    want = ctx.grid_energy(f, torch.from_numpy(good).cuda(), side, 1)
    for at in (0, n // 2, n - 1):
        bad = good.copy()
        bad[at] = {"twice": good[at - 1], "negative": -1, "n": n, "far": 2**31 - 1}[fault]
        p = torch.from_numpy(bad).cuda()
        for call in (lambda: ctx.grid_energy(f, p, side, 1), lambda: ctx.vad(f, p, side),
                     lambda: ctx.sort(f, side, 1, init_perm=p)):
            with pytest.raises(plas.PlasError) as e:
                call()
            assert e.value.status == plas.ERR_INVALID_ARGUMENT
        # The scratch a refused call leaves does not make the next one pass or fail.
        assert ctx.grid_energy(f, torch.from_numpy(good).cuda(), side, 1) == want


@pytest.mark.parametrize("layout", ["cn", "nc"])
@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("side,d", [(9, 59), (190, 59), (190, 3)])
def test_a_value_that_is_not_finite_is_refused_before_a_bad_permutation(env, side, d, value, layout):
    torch, plas, ctx = env
    n = side * side
    F = synthetic.random_features(n, d, 3, layout)
    p = torch.zeros(n, dtype=torch.int32, device="cuda")
    for at in (0, n * d // 2, n * d - 1):
        bad = F.copy()
        bad.reshape(-1)[at] = value
        for perm in (None, p):
            with pytest.raises(plas.PlasError) as e:
                ctx.grid_energy(torch.from_numpy(bad).cuda(), perm, side, 1, layout)
            assert e.value.status == plas.ERR_NONFINITE


def test_values_that_round_to_infinity_in_bfloat16_are_refused_there(env):
    torch, plas, ctx = env
    F = synthetic.random_features(400, 5, 3, "cn")
    F[2, 77] = np.float32(3.4e38)
    f = torch.from_numpy(F).cuda()
    with pytest.raises(plas.PlasError) as e:
        ctx.grid_energy(f, None, 20, 1, storage="bf16")
    assert e.value.status == plas.ERR_NONFINITE
