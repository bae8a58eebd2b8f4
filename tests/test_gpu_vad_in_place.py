"""GPU tests of plas_vad's way on a device without room for the arranged grid:
the permutation check, the results' clearing and reading, and the in-place
kernels, against the oracle's float64 VAD."""
import math

import numpy as np
import pytest

import synthetic
from gpu_util import require_gpu

pytestmark = pytest.mark.gpu

# As for the arranged way: all summands are of one sign, so any order of N of
# them is off by a share of at most N 2^-53 (N <= 2 x 130^2 x 59 here).
REL = 1e-9


@pytest.fixture(scope="module")
def env():
    torch, plas = require_gpu()
    return torch, plas, plas.Context(0)


@pytest.mark.parametrize("layout", ["cn", "nc"])
@pytest.mark.parametrize("side,d,dtype", [(2, 1, "f32"), (3, 59, "bf16"), (16, 14, "f32"), (65, 3, "bf16"),
                                          (130, 59, "f32")])
def test_in_place_vad_equals_the_oracle(env, ref, side, d, dtype, layout):
    torch, plas, ctx = env
    n = side * side
    F = synthetic.random_features(n, d, side + d, layout, -3.0, 3.0)
    if dtype == "bf16":
        F = ref.round_bf16(F)
    f = torch.from_numpy(F).cuda().to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    perm = synthetic.random_permutation(n, side)
    for p in (perm, None, perm[::-1].copy()):  # the scratch holds the inverse of another permutation by then
        dev = None if p is None else torch.from_numpy(p).cuda()
        want = ref.vad(F, p, side, layout)
        assert ctx.stage_vad_in_place(f, dev, side, layout) == pytest.approx(want, rel=REL, abs=1e-14)
        assert ctx.vad(f, dev, side, layout) == pytest.approx(want, rel=REL, abs=1e-14)


@pytest.mark.parametrize("at,value", [(0, 1), (899, -1), (450, 900), (17, 2**31 - 1), (5, -(2**31))])
def test_in_place_vad_refuses_what_is_no_permutation(env, at, value):
    torch, plas, ctx = env
    side = 30
    f = torch.from_numpy(synthetic.random_features(side * side, 3, 1)).cuda()
    good = np.arange(side * side, dtype=np.int32)
    bad = good.copy()
    bad[at] = value
    for call in (ctx.stage_vad_in_place, ctx.vad):
        want = call(f, torch.from_numpy(good).cuda(), side)
        with pytest.raises(plas.PlasError) as e:
            call(f, torch.from_numpy(bad).cuda(), side)
        assert e.value.status == plas.ERR_INVALID_ARGUMENT
        assert call(f, torch.from_numpy(good).cuda(), side) == want  # the flag does not stay set
        assert call(f, None, side) == want


def test_in_place_vad_of_a_value_that_is_not_finite_is_nan(env):
    torch, plas, ctx = env
    F = synthetic.random_features(33 * 33, 5, 3, "cn")
    for value in (np.nan, np.inf):
        F[2, 500] = value
        assert math.isnan(ctx.stage_vad_in_place(torch.from_numpy(F).cuda(), None, 33))
