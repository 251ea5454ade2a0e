"""Block-scaled tensors whose index base is not a multiple of eight (GPU):
whole and partial tiles, every storage of the moments, with and without a
compute copy, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_parity_util import (DevState, HostState, assert_copy_equal, assert_state_equal,
                             encode_nv_current, gpu_step, oracle_step, to_dev, to_host)
from paper_2607_10611_amd import workloads as W

pytestmark = pytest.mark.gpu

BLOCK = {"e4m3": 128, "e5m2": 128, "mxfp4": 32, "nvfp4": 16, "nvfp4_current": 16}
ENCODE = {"mxfp4": oracle.encode_mx, "nvfp4": oracle.encode_nv, "nvfp4_current": encode_nv_current}


@pytest.mark.parametrize("base", [0, 1, 4, 7, 2**33 + 3])
@pytest.mark.parametrize("sfmt", ["fp32", "bf16", "bf16_sr"])
@pytest.mark.parametrize("wfmt", list(BLOCK))
def test_any_index_base(wfmt, sfmt, base):
    blk = BLOCK[wfmt]
    for n in (blk, 2048, 3 * 2048 + 5 * blk):
        rng = np.random.default_rng(n + base % 97)
        x = rng.normal(0, 0.02, n).astype(np.float32)
        codes, scales = ENCODE[wfmt](x) if wfmt in ENCODE else oracle.encode_block(wfmt, x)
        copy = bool((base + n // blk) % 2)
        hs = HostState(codes, n, scales, sfmt=sfmt, copy=copy)
        ds = DevState(wfmt, codes, n, scales, sfmt=sfmt, copy=copy)
        for t, rounding in ((1, "sr"), (2, "sr"), (3, "rne")):
            g = rng.normal(0, 1e-3, n).astype(np.float32)
            hp = dict(W.DEFAULT_HPARAMS, rounding=rounding, step=t, lr_mul=5e-3)
            gpu_step(ds, to_dev(g), hp, index_base=base)
            oracle_step(wfmt, hs, g, hp, index_base=base)
        torch.cuda.synchronize()
        tag = f"{wfmt} n={n} base {base} {sfmt}"
        h = ds.host()
        assert_state_equal(tag, h[0], hs.w, h[1], hs.m, h[2], hs.v, h[3], hs.ve, max_ulp=0)
        assert (to_host(ds.scales).view(hs.scales.dtype) == hs.scales).all(), tag
        assert_copy_equal(tag, ds, hs)


@pytest.mark.parametrize("n", [16, 1040, 2048, 2048 + 272])
def test_current_scaling_takes_the_largest_weight_from_any_wave(n):
    rng = np.random.default_rng(n)
    for at in sorted({0, 15, 255, 256, 700, 1023, 1024, 1300, 2047, 2048, n - 1}):
        if at >= n:
            continue
        x = rng.normal(0, 0.02, n).astype(np.float32)
        x[at] = -3.0
        codes, scales = encode_nv_current(x)
        hs, ds = HostState(codes, n, scales), DevState("nvfp4_current", codes, n, scales)
        g = rng.normal(0, 1e-3, n).astype(np.float32)
        hp = dict(W.DEFAULT_HPARAMS, rounding="sr", step=1)
        gpu_step(ds, to_dev(g), hp)
        oracle_step("nvfp4_current", hs, g, hp)
        torch.cuda.synchronize()
        assert (to_host(ds.scales) == hs.scales).all(), at
        assert (ds.host()[0] == hs.w).all(), at
