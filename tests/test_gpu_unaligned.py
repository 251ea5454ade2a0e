"""Unscaled tensors that start anywhere (GPU): every phase of the global index
and of the buffers, sizes that end inside a quad or a tile, against the oracle;
nothing next to the tensor is written (the neighbours hold a pattern that a
step on zeros does not leave), and the gradients not at all."""
import numpy as np
import pytest
import torch

import oracle
from gpu_parity_util import STATE_NP, to_dev, to_host
from paper_2607_10611_amd import binding as B
from paper_2607_10611_amd import workloads as W

pytestmark = pytest.mark.gpu

PAD = 16
FILL = 0xA5


@pytest.mark.parametrize("wfmt,gfmt,sfmt,rounding", [
    ("bf16", "fp32", "fp32", "sr"), ("e4m3", "bf16", "bf16", "sr"), ("e5m2", "fp32", "bf16_sr", "sr"),
    ("fp32", "bf16", "bf16_sr", "rne"), ("bf16", "bf16", "bf16", "rne"), ("e4m3", "fp32", "fp32", "rne")])
@pytest.mark.parametrize("n", [1, 3, 7, 1021, 2048, 4099])
def test_any_start(wfmt, gfmt, sfmt, rounding, n):
    rng = np.random.default_rng(n)
    x = rng.normal(0, 0.02, n).astype(np.float32)
    g = rng.normal(0, 1e-3, n).astype(np.float32)
    gc = oracle.encode_array("bf16", g) if gfmt == "bf16" else g
    codes = oracle.encode_array(wfmt, x)
    cases = [(p, p, p, p) for p in range(8)] + [(0, 0, 0, 5), (0, 0, 0, 2), (3, 1, 2, 0), (1, 6, 0, 7)]
    for pw, pg, pm, base in cases:
        def put(a, at):  # the tensor inside a buffer of FILL bytes, `at` elements in
            dt = to_dev(a[:1]).dtype
            t = torch.full(((n + 2 * PAD) * dt.itemsize,), FILL, dtype=torch.uint8, device="cuda").view(dt)
            t[at:at + n] = to_dev(a)
            return t, t[at:at + n]
        st = [np.zeros(n, STATE_NP[sfmt]) for _ in range(3)]
        bw, w = put(codes, pw)
        bg, gd = put(gc, pg)
        bs = [put(a, pm) for a in st]
        bc, cp = put(np.zeros(n, np.uint16), pg)
        hw, hc = codes.copy(), np.zeros(n, np.uint16)
        for t in (1, 2):
            hp = dict(W.DEFAULT_HPARAMS, rounding=rounding, step=t)
            B.madd_step(w, wfmt, gd, *(v for _, v in bs), hp, gfmt=gfmt, index_base=base + 8 * t,
                        sfmt=sfmt, copy=cp)
            oracle.step(wfmt, hw, gc, *st, hp, gfmt=gfmt, index_base=base + 8 * t, sfmt=sfmt, copy=hc)
        torch.cuda.synchronize()
        tag = f"{wfmt} n={n} phases {pw},{pg},{pm} base {base}"
        for name, buf, at, ref in [("w", bw, pw, hw), ("copy", bc, pg, hc), ("g", bg, pg, gc)] + [
                (k, b, pm, r) for k, (b, _), r in zip(("m", "v", "ve"), bs, st)]:
            got = to_host(buf).view(ref.dtype)
            assert (got[at:at + n] == ref).all(), f"{tag}: {name}"
            outside = np.concatenate([got[:at], got[at + n:]]).view(np.uint8)
            assert (outside == FILL).all(), f"{tag}: outside {name}"
