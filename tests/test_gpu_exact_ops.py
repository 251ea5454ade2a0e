"""The range-limited square root and division the step's fast path uses, and
the line between that path and the general one (GPU).

madd_check_exact_ops compares the operations with the general ones: the
square root and the reciprocal on every fp32 of their ranges, the quotient on
every denominator significand with 1024 numerators, and madd_check_quotients on
slices of them with all.  The step test mixes weights, gradients and
moments from the denormals to the largest values, zeros of both signs,
infinities and NaN within each group of four and expects the oracle's bits;
most such groups take the general path (test_gpu_step_path.py places one
operand at a time next to a bound and asserts which path its group takes).
"""
import ctypes

import numpy as np
import pytest
import torch

from gpu_parity_util import DevState, HostState, assert_state_equal, gpu_step, oracle_step, to_dev
from paper_2607_10611_amd import _build
from paper_2607_10611_amd import binding as B
from paper_2607_10611_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_range_limited_operations_match_the_general_ones():
    B.lib()
    L = ctypes.CDLL(_build.PROBE_LIB)
    L.madd_check_exact_ops.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    L.madd_check_exact_ops.restype = ctypes.c_int32
    c = torch.zeros(4, dtype=torch.int64, device="cuda")
    assert L.madd_check_exact_ops(c.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert c.tolist() == [0, 0, 0, 2**32]


def test_quotients_of_whole_slices_of_significands():
    """Every numerator over 1024 denominators next to 1, 1.5 and 2 and in between
    (all 2^23 denominators: 128 calls of 65536, half a minute)."""
    L = ctypes.CDLL(_build.PROBE_LIB)
    L.madd_check_quotients.argtypes = [ctypes.c_int32, ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p]
    L.madd_check_quotients.restype = ctypes.c_int32
    c = torch.zeros(2, dtype=torch.int64, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    firsts = (0, 1234567, (1 << 22) - 512, 7654321, (1 << 23) - 1024)
    for first in firsts:
        assert L.madd_check_quotients(first, 1024, c.data_ptr(), stream) == 0
    assert L.madd_check_quotients((1 << 23) - 1023, 1024, c.data_ptr(), stream) == -1
    torch.cuda.synchronize()
    assert c.tolist() == [0, len(firsts) * 1024 * 2**23]


EXPS = (-149, -140, -127, -126, -125, -110, -101, -100, -99, -90, -82, -71, -70, -64, -63, -60,
        -50, -47, -46, -41, -40, -39, -30, -27, -10, -6, -1, 0, 3, 20, 24, 30, 48, 49, 59, 60, 61,
        64, 100, 125, 126, 127)


def spread(rng, n, signed=True):
    """Magnitudes on and next to the bounds, plus ordinary ones; zeros of both
    signs, infinities and NaN among them."""
    e = rng.choice(EXPS, n).astype(np.float64)
    x = np.exp2(e) * np.where(rng.random(n) < 0.3, 1.0, 1.0 + rng.random(n))
    x = np.where(rng.random(n) < 0.4, rng.normal(0, 0.02, n), x)
    x = np.where(rng.random(n) < 0.1, 0.0, x)
    with np.errstate(over="ignore"):
        x = np.minimum(x, 3.4e38).astype(np.float32)
    x = np.where(rng.random(n) < 0.005, np.float32(np.inf), x)
    x = np.where(rng.random(n) < 0.005, np.float32(np.nan), x)
    if signed:
        return np.where(rng.random(n) < 0.5, -x, x).astype(np.float32)
    return np.abs(x)


@pytest.mark.parametrize("wfmt", ["fp32", "bf16"])
@pytest.mark.parametrize("change", [
    {}, {"eps": 2.0**-38}, {"eps": 2.0**-38 * (1 - 2.0**-20)}, {"eps": 0.0}, {"eps": 2.0**20},
    {"tau": 2.0**-40}, {"tau": 2.0**-41}, {"tau": 2.0**60}, {"lr_mul": 0.0}, {"lr_mul": 2.0**-61},
    {"lr_mul": 2.0**19}, {"lr_mul": 2.0**21}, {"lr_add": 0.0}, {"lr_add": 1e30},
    {"r_max": 1 - 2.0**-20}, {"r_max": 1 - 2.0**-22}, {"r_max": 2.0**-30},
    {"g_max": 1.0, "w_max": 2.0}, {"g_max": 1e-30}, {"bias_correction": 0},
    {"beta2": 0.0}, {"beta2": 1 - 2.0**-24}, {"step": 100000}],
    ids=lambda c: ",".join(f"{k}={v:.9g}" for k, v in c.items()) or "default")
def test_step_on_both_sides_of_every_bound(wfmt, change):
    n = 3 * 2048 + 40
    rng = np.random.default_rng(2607)
    hp = dict(dict(W.DEFAULT_HPARAMS, rounding="sr", seed=5, step=7), **change)
    w = spread(rng, n)
    codes = w.view(np.uint32) if wfmt == "fp32" else (w.view(np.uint32) >> 16).astype(np.uint16)
    codes = np.where(np.isnan(w), 0x7FC00000 if wfmt == "fp32" else 0x7FC0, codes).astype(codes.dtype)
    g = spread(rng, n)
    hs = HostState(codes, n)
    hs.m, hs.v, hs.ve = spread(rng, n), spread(rng, n, False), spread(rng, n, False)
    # rows without a gradient for a long time, states of -0 and negative v
    g[:512] = 0.0
    hs.v[1000:1064], hs.ve[1032:1100] = 0.0, 0.0
    hs.m[1040:1050], hs.v[1050:1055], hs.v[2000] = -0.0, -0.0, -1e-40
    ds = DevState(wfmt, codes, n)
    ds.m, ds.v, ds.ve = to_dev(hs.m), to_dev(hs.v), to_dev(hs.ve)
    with np.errstate(all="ignore"):
        oracle_step(wfmt, hs, g, hp)
    gpu_step(ds, to_dev(g), hp)
    torch.cuda.synchronize()
    got = ds.host()
    assert_state_equal(f"{wfmt} {change}", got[0], hs.w, got[1], hs.m, got[2], hs.v, got[3], hs.ve,
                       max_ulp=0)
