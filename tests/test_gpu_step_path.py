"""Which arithmetic a group of four elements takes, and that both give the same
bits (GPU).

The step takes the range-limited square root and division where its guard
vouches for all four elements, else the general ones.  Every group here holds
ordinary operands except for one operand, or one intermediate, placed on one
side of one bound, in one lane or in all four.  The probe runs the kernels' own
functions and says which form each group took, so a group meant to be just
inside a bound is known to have been computed by the range-limited form; its
bits are compared with the general form's and, through madd_step, with the
oracle's."""
import ctypes

import numpy as np
import pytest
import torch

from gpu_parity_util import DevState, HostState, assert_state_equal, gpu_step, oracle_step, to_dev
from paper_2607_10611_amd import _build
from paper_2607_10611_amd import binding as B
from paper_2607_10611_amd import workloads as W

pytestmark = pytest.mark.gpu

BASE = dict(W.DEFAULT_HPARAMS, rounding="rne", step=7)
QUADS = 1000
IBC2 = 1 / (1 - 0.999**7)  # bias corrections at step 7
SA = 1e-3 / (1 - 0.9**7)
ROOT1 = np.sqrt(0.999 * IBC2)  # sqrt(v IBC2) from v = 1 without a gradient


def log2_uniform(rng, n, lo, hi):
    return np.exp2(rng.uniform(lo, hi, n))


def sign(rng, n):
    return np.where(rng.random(n) < 0.5, -1.0, 1.0)


def ordinary(rng, n):
    """Operands whose every intermediate is far from every bound."""
    return dict(w=sign(rng, n) * log2_uniform(rng, n, -10, -3), g=sign(rng, n) * log2_uniform(rng, n, -14, -8),
                m=sign(rng, n) * log2_uniform(rng, n, -14, -10), v=log2_uniform(rng, n, -26, -20),
                ve=log2_uniform(rng, n, -38, -32))


def operands(rng, special, quads=QUADS):
    """Groups of ordinary operands with `special` (a function of rng and n that
    replaces some of them) in lane 0, 1, 2, 3 or all four, in turn."""
    n = 4 * quads
    a = ordinary(rng, n)
    at = (np.arange(n) % 4 == np.arange(n) // 4 % 5) | (np.arange(n) // 4 % 5 == 4)
    for k, x in special(rng, n).items():
        a[k] = np.where(at, x, a[k])
    with np.errstate(over="ignore"):
        return {k: x.astype(np.float32) for k, x in a.items()}


def probe(a, hp):
    """(new weights as the kernels compute them, the general form's, groups that fell back)"""
    L = ctypes.CDLL(_build.PROBE_LIB)
    P = ctypes.c_void_p
    L.madd_probe_step_path.argtypes = [P] * 5 + [ctypes.c_int64, P, ctypes.c_int32, P, P, P, P]
    L.madd_probe_step_path.restype = ctypes.c_int32
    n = a["w"].size
    d = [to_dev(a[k]) for k in ("w", "g", "m", "v", "ve")]
    sc = torch.frombuffer(bytearray(B.prepare_scalars(hp)), dtype=torch.uint8).cuda()
    got, general = torch.empty(n, device="cuda"), torch.empty(n, device="cuda")
    took = torch.empty(n // 4, dtype=torch.uint8, device="cuda")
    clamp = int(np.isfinite(hp["g_max"]) or np.isfinite(hp["w_max"]))
    assert L.madd_probe_step_path(*(t.data_ptr() for t in d), n // 4, sc.data_ptr(), clamp,
                                  got.data_ptr(), general.data_ptr(), took.data_ptr(),
                                  torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    return got.cpu().numpy(), general.cpu().numpy(), took.cpu().numpy()


def check(a, hp, falls_back):
    got, general, took = probe(a, hp)
    both_nan = np.isnan(got) & np.isnan(general)
    bad = np.nonzero((got.view(np.uint32) != general.view(np.uint32)) & ~both_nan)[0]
    assert bad.size == 0, (bad[:5], got[bad[:5]], general[bad[:5]])
    assert (took == falls_back).all(), f"{int((took != falls_back).sum())} of {took.size} groups"
    n = a["w"].size
    codes = np.where(np.isnan(a["w"]), np.uint32(0x7FC00000), a["w"].view(np.uint32))
    hs, ds = HostState(codes, n), DevState("fp32", codes, n)
    hs.m, hs.v, hs.ve = a["m"].copy(), a["v"].copy(), a["ve"].copy()
    ds.m, ds.v, ds.ve = to_dev(hs.m), to_dev(hs.v), to_dev(hs.ve)
    with np.errstate(all="ignore"):
        oracle_step("fp32", hs, a["g"].copy(), hp)
    gpu_step(ds, to_dev(a["g"]), hp)
    torch.cuda.synchronize()
    h = ds.host()
    assert_state_equal("step", h[0], hs.w, h[1], hs.m, h[2], hs.v, h[3], hs.ve, max_ulp=0)
    same = (h[0] == got.view(np.uint32)) | (np.isnan(got) & (h[0] == 0x7FC00000))
    assert same.all()


def still(rng, n, **over):
    """No gradient and no first moment: the weight stays as it is."""
    z = np.zeros(n)
    return dict(dict(g=z, m=z), **over)


def near_cancelled(rng, n, target):
    """w' = target from a 2^-97 weight and an additive update of its size."""
    w = sign(rng, n) * log2_uniform(rng, n, -97, -96)
    return still(rng, n, w=w, v=np.ones(n), m=(w - target) * ROOT1 / (SA * 0.9))


# name: (hyper-parameters, special operands, whether groups with them fall back)
BIG_Q = dict(lr_mul=2.0**19, tau=2.0**-40, eps=2.0**-38, lr_add=0.0)
CASES = {
    "ordinary": ({}, lambda r, n: {}, False),
    # |w'| against 2^-100 and 2^60
    "w' from 2^-100": ({}, lambda r, n: still(r, n, w=sign(r, n) * np.where(
        r.random(n) < 0.2, 2.0**-100, log2_uniform(r, n, -100, -96))), False),
    "w' below 2^-100": ({}, lambda r, n: still(r, n, w=sign(r, n) * np.where(
        r.random(n) < 0.2, 2.0**-100 * (1 - 2.0**-24), log2_uniform(r, n, -104, -100.001))), True),
    "w' from 2^-100, cancelled": ({}, lambda r, n: near_cancelled(
        r, n, sign(r, n) * log2_uniform(r, n, -99.9, -98)), False),
    "w' below 2^-100, cancelled": ({}, lambda r, n: near_cancelled(
        r, n, sign(r, n) * log2_uniform(r, n, -104, -100.1)), True),
    "w' below 2^60": ({}, lambda r, n: still(r, n, w=sign(r, n) * np.where(
        r.random(n) < 0.2, 2.0**60 * (1 - 2.0**-24), log2_uniform(r, n, 56, 60))), False),
    "w' from 2^60": ({}, lambda r, n: still(r, n, w=sign(r, n) * np.where(
        r.random(n) < 0.2, 2.0**60, log2_uniform(r, n, 60.001, 127.9))), True),
    # |ut / rho| against 2^60: from a fresh v_e the quotient is 2^19 2.642 / |w|
    "quotient below 2^60": (BIG_Q, lambda r, n: dict(
        w=sign(r, n) * log2_uniform(r, n, -39.5, -37), g=np.full(n, 2.0**15), ve=np.zeros(n)), False),
    "quotient from 2^60": (BIG_Q, lambda r, n: dict(
        w=sign(r, n) * log2_uniform(r, n, -40, -39.75), g=np.full(n, 2.0**15), ve=np.zeros(n)), True),
    # roots: arguments too small to be normal, and up to the largest before the scaling overflows
    "denormal v": ({}, lambda r, n: dict(g=np.zeros(n), v=log2_uniform(r, n, -149, -133),
                                         m=sign(r, n) * log2_uniform(r, n, -36, -32)), False),
    "denormal v_e": ({}, lambda r, n: dict(g=sign(r, n) * log2_uniform(r, n, -64, -60),
                                           ve=log2_uniform(r, n, -149, -133)), False),
    "v up to 2^48 / IBC2": ({}, lambda r, n: dict(g=np.zeros(n), m=sign(r, n) * log2_uniform(r, n, 5, 20),
                                                 v=log2_uniform(r, n, 45, 47.999) / (0.999 * IBC2)), False),
    "v from 2^48 / IBC2": ({}, lambda r, n: dict(g=np.zeros(n), m=sign(r, n) * log2_uniform(r, n, 5, 20),
                                                v=log2_uniform(r, n, 48.001, 50) / (0.999 * IBC2)), True),
    "v_e up to 2^48 / IBC2": ({}, lambda r, n: dict(ve=log2_uniform(r, n, 45, 47.999) / (0.999 * IBC2)), False),
    "v_e from 2^48 / IBC2": ({}, lambda r, n: dict(ve=log2_uniform(r, n, 48.001, 50) / (0.999 * IBC2)), True),
    "zero v and v_e": ({}, lambda r, n: still(r, n, v=np.zeros(n), ve=np.where(r.random(n) < 0.5, -0.0, 0.0)), False),
    "negative v": ({}, lambda r, n: still(r, n, v=-log2_uniform(r, n, -149, 10)), True),
    "negative v_e": ({}, lambda r, n: still(r, n, ve=-log2_uniform(r, n, -149, 10)), True),
    # numerators
    "SA m below 2^64": ({}, lambda r, n: dict(g=np.zeros(n), v=np.full(n, 2.0**40),
                                             m=sign(r, n) * log2_uniform(r, n, 60, 63.999) / (SA * 0.9)), False),
    "SA m from 2^64": ({}, lambda r, n: dict(g=np.zeros(n), v=np.full(n, 2.0**40),
                                            m=sign(r, n) * log2_uniform(r, n, 64.001, 66) / (SA * 0.9)), True),
    "tiny m": ({}, lambda r, n: dict(g=np.zeros(n), m=sign(r, n) * log2_uniform(r, n, -149, -100)), False),
    "tiny m over a large v": ({}, lambda r, n: dict(g=np.zeros(n), v=np.full(n, 2.0**38),
                                                   m=sign(r, n) * log2_uniform(r, n, -149, -90)), False),
    "tiny g": ({}, lambda r, n: dict(g=sign(r, n) * log2_uniform(r, n, -149, -70)), False),
    "tiny g, fresh v_e": ({}, lambda r, n: dict(g=sign(r, n) * log2_uniform(r, n, -149, -70),
                                               ve=np.zeros(n)), False),
    "u_a alone, from 2^-126": ({}, lambda r, n: dict(w=np.where(r.random(n) < 0.5, -0.0, 0.0), g=np.zeros(n), v=np.ones(n),
                               m=sign(r, n) * log2_uniform(r, n, -125.99, -96) * ROOT1 / (SA * 0.9)), False),
    "denormal u_a alone": ({}, lambda r, n: dict(w=np.where(r.random(n) < 0.5, -0.0, 0.0), g=np.zeros(n), v=np.ones(n),
                           m=sign(r, n) * log2_uniform(r, n, -139, -126.01) * ROOT1 / (SA * 0.9)), True),
    "denormal u_a alone, clamps": ({"g_max": 1.0, "w_max": 2.0**-140}, lambda r, n: dict(
        w=np.where(r.random(n) < 0.5, -0.0, 0.0), g=np.zeros(n), v=np.ones(n),
        m=sign(r, n) * log2_uniform(r, n, -139, -126.01) * ROOT1 / (SA * 0.9)), True),
    "u_a alone rounds to 0": ({}, lambda r, n: dict({k: np.where(r.random(n) < 0.5, -0.0, 0.0) for k in ("w", "g")},
                              v=np.full(n, 2.0**40), m=sign(r, n) * log2_uniform(r, n, -139, -124)), True),
    "u_a alone rounds to 0, eta_m < 0": ({"lr_mul": -1e-3}, lambda r, n: dict(
        {k: np.where(r.random(n) < 0.5, -0.0, 0.0) for k in ("w", "g")},
        v=np.full(n, 2.0**40), m=sign(r, n) * log2_uniform(r, n, -139, -124)), True),
    "u_a of a denormal SA m": ({}, lambda r, n: dict(w=np.where(r.random(n) < 0.5, -0.0, 0.0), g=np.zeros(n),
                               v=log2_uniform(r, n, -46, -40), m=sign(r, n) * log2_uniform(r, n, -133, -125)), False),
    # zero weights that nothing moves (padding rows, pruned weights): zeros of the right sign
    "zero w and m": ({}, lambda r, n: {k: np.where(r.random(n) < 0.5, -0.0, 0.0) for k in ("w", "g", "m")}, False),
    "zero w and m, no v": ({}, lambda r, n: dict({k: np.where(r.random(n) < 0.5, -0.0, 0.0) for k in ("w", "g", "m")},
                                                 v=np.zeros(n), ve=np.zeros(n)), False),
    "zero w, SA m rounds to 0": ({"lr_add": 2.0**-30}, lambda r, n: dict(
        w=np.where(r.random(n) < 0.5, -0.0, 0.0), g=np.zeros(n), m=sign(r, n) * log2_uniform(r, n, -149, -124)), False),
    "zero w without additive rate": ({"lr_add": 0.0}, lambda r, n: dict(
        w=np.where(r.random(n) < 0.5, -0.0, 0.0)), False),
    "zero w, clamps": ({"g_max": 1.0, "w_max": 2.0}, lambda r, n: still(r, n, w=np.zeros(n)), False),
    "zero w and m, infinite v": ({}, lambda r, n: still(r, n, w=np.zeros(n), v=np.full(n, np.inf)), True),
    # denominators of the relative update
    "w at tau": ({}, lambda r, n: dict(w=sign(r, n) * 1e-8 * log2_uniform(r, n, -2, 2)), False),
    "w at tau = 2^-40": ({"tau": 2.0**-40}, lambda r, n: dict(w=sign(r, n) * log2_uniform(r, n, -42, -38)), False),
    # clips
    "u_m at a bound next to 1": ({"r_max": 1 - 2.0**-20, "lr_mul": 16.0}, lambda r, n: dict(
        g=sign(r, n) * log2_uniform(r, n, -2, 2), ve=np.zeros(n)), False),
    "g_max met": ({"g_max": 1.0, "w_max": 2.0}, lambda r, n: dict(
        g=sign(r, n) * log2_uniform(r, n, -2, 2), ve=np.zeros(n)), False),
    "w_max met": ({"w_max": 2.0**-6}, lambda r, n: {}, False),
    "g_max of 2^100": ({"g_max": 2.0**100}, lambda r, n: {}, False),
    # no element's business
    "infinite operands": ({}, lambda r, n: {k: np.where(np.arange(n) // 20 % 5 == j, np.inf, x) for j, (k, x) in
                                            enumerate(ordinary(r, n).items())}, True),
    "NaN operands": ({}, lambda r, n: {k: np.where(np.arange(n) // 20 % 5 == j, np.nan, x) for j, (k, x) in
                                       enumerate(ordinary(r, n).items())}, True),
}


@pytest.mark.parametrize("name", list(CASES))
def test_groups_next_to_one_bound(name):
    change, special, falls_back = CASES[name]
    hp = dict(BASE, **change)
    check(operands(np.random.default_rng(len(name) * 7919 + QUADS), special), hp, falls_back)


def test_exactly_cancelled_weights_fall_back():
    rng = np.random.default_rng(5)
    a = operands(rng, lambda r, n: dict(g=np.zeros(n), w=np.zeros(n), m=sign(r, n) * log2_uniform(r, n, -14, -10)))
    ua = probe(a, BASE)[1]
    a["w"] = np.where(a["w"] == 0, -ua, a["w"])  # w + 0 w + u_a = 0
    got = probe(a, BASE)[0]
    assert (got == 0).sum() >= QUADS
    check(a, BASE, True)


INSIDE = [{"eps": 2.0**-38}, {"eps": 2.0**20 * (1 - 2.0**-23)}, {"tau": 2.0**-40}, {"tau": 2.0**60 * (1 - 2.0**-23)},
          {"lr_mul": 0.0}, {"lr_mul": 2.0**-60}, {"lr_mul": 2.0**20 * (1 - 2.0**-23)}, {"lr_mul": -0.01}, {"lr_add": 0.0},
          {"r_max": 1 - 2.0**-20}, {"bias_correction": 0}, {"beta2": 0.0}, {"beta2": 1 - 2.0**-24, "step": 1},
          {"beta2": 1 - 2.0**-39, "step": 1}, {"step": 100000}]
OUTSIDE = [{"eps": 2.0**-38 * (1 - 2.0**-23)}, {"eps": 0.0}, {"eps": 2.0**20}, {"tau": 2.0**-40 * (1 - 2.0**-23)},
           {"tau": 2.0**60}, {"lr_mul": 2.0**-60 * (1 - 2.0**-23)}, {"lr_mul": -2.0**-100}, {"lr_mul": 2.0**20},
           {"r_max": 1 - 2.0**-21}, {"beta2": 1 - 2.0**-41, "step": 1}]


@pytest.mark.parametrize("change,falls_back", [(c, False) for c in INSIDE] + [(c, True) for c in OUTSIDE],
                         ids=lambda c: ",".join(f"{k}={v:.9g}" for k, v in c.items()) if isinstance(c, dict) else str(c))
def test_hyper_parameters_on_both_sides_of_the_window(change, falls_back):
    check(operands(np.random.default_rng(11), lambda r, n: {}), dict(BASE, **change), falls_back)
