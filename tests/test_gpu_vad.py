"""GPU tests of the VAD kernels against the oracle's float64 VAD: chunk edges
of the walk over an arranged grid, every cell width, values whose mean is far
from their spread, values that are not finite, and the way without a grid."""
import ctypes
import math

import numpy as np
import pytest

import synthetic
from gpu_util import require_gpu

pytestmark = pytest.mark.gpu

# All summands are of one sign, so a sum of N of them in any order is off by
# at most a share N 2^-53, in the mean and in the deviations, here and in the
# oracle: 4 x 2 x 200^2 x 64 x 2^-53 < 3e-9 for the largest case, in the worst
# order; pairwise and blocked sums like these grow with the depth alone.
REL = 1e-10


@pytest.fixture(scope="module")
def env():
    torch, plas = require_gpu()
    return torch, plas, plas.Context(0)


def _case(torch, ref, side, d, layout, dtype, shift=0.0):
    n = side * side
    F = synthetic.random_features(n, d, 10 * side + d, layout, -3.0, 3.0) + np.float32(shift)
    if dtype == "bf16":
        F = ref.round_bf16(F)
    f = torch.from_numpy(F).cuda()
    if dtype == "bf16":
        f = f.to(torch.bfloat16)
    return F, f, synthetic.random_permutation(n, side)


# Chunks are 16 rows by 4 (d 59), 8 (d 32), 16 (d 16), 32 (d 8) or 64 (d 3) columns.
@pytest.mark.parametrize("layout", ["cn", "nc"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [1, 3, 8, 13, 32, 59, 64])
@pytest.mark.parametrize("side", [2, 3, 15, 16, 17, 33, 64, 65, 200])
def test_vad_equals_the_oracle(env, ref, side, d, dtype, layout):
    torch, plas, ctx = env
    F, f, perm = _case(torch, ref, side, d, layout, dtype)
    for p in (None, perm):
        got = ctx.vad(f, None if p is None else torch.from_numpy(p).cuda(), side, layout)
        assert got == pytest.approx(ref.vad(F, p, side, layout), rel=REL, abs=1e-14)


def test_vad_of_a_large_common_offset_and_of_a_ramp(env, ref):
    torch, plas, ctx = env
    F, f, perm = _case(torch, ref, 65, 14, "cn", "f32", shift=1.0e5)
    assert ctx.vad(f, torch.from_numpy(perm).cuda(), 65) == pytest.approx(ref.vad(F, perm, 65), rel=REL)
    # A ramp: every difference is 0 or 1 but for one far cell, which dominates.
    ramp = np.tile(np.arange(80, dtype=np.float32), 80)[None].copy()
    ramp[0, 80 * 77 + 3] = 1.0e6
    assert ctx.vad(torch.from_numpy(ramp).cuda(), None, 80) == pytest.approx(ref.vad(ramp, None, 80), rel=REL)
    # All differences equal: no variance at all.
    flat = np.zeros((3, 400), dtype=np.float32)
    assert ctx.vad(torch.from_numpy(flat).cuda(), None, 20) == 0.0


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_vad_of_a_value_that_is_not_finite_is_nan(env, value):
    torch, plas, ctx = env
    F = synthetic.random_features(33 * 33, 5, 3, "cn")
    for at in (0, 32, 500, 33 * 33 - 1):
        bad = F.copy()
        bad[4, at] = value
        assert math.isnan(ctx.vad(torch.from_numpy(bad).cuda(), None, 33))


@pytest.mark.parametrize("side,d,layout,dtype", [(7, 3, "cn", "f32"), (65, 59, "nc", "f32"), (64, 14, "cn", "bf16")])
def test_vad_without_a_grid_equals_the_oracle(env, ref, side, d, layout, dtype):
    """The way taken when the device has no room for an arranged grid, called
    as the library calls it then."""
    torch, plas, ctx = env
    F, f, perm = _case(torch, ref, side, d, layout, dtype)
    p = torch.from_numpy(perm).cuda()
    part = torch.empty(4096, dtype=torch.float64, device="cuda")
    out = torch.empty(2, dtype=torch.float64, device="cuda")
    fn = plas.library()["_ZN4plas19launch_vad_in_placeEPKviPKiliiiPdS4_P12ihipStream_t"]
    fn.restype = ctypes.c_int
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    torch.cuda.synchronize()
    assert fn(ptr(f), ctypes.c_int(dtype == "bf16"), ptr(p), ctypes.c_int64(side * side), ctypes.c_int(d),
              ctypes.c_int(side), ctypes.c_int(0 if layout == "cn" else 1), ptr(part), ptr(out), None) == 0
    torch.cuda.synchronize()
    assert out[1].item() == pytest.approx(ref.vad(F, perm, side, layout), rel=REL, abs=1e-14)
