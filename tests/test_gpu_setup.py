"""Set-up kernels at the edges of their lanes (GPU): encoding and zeroing
buffers that start at any element (not only on 16-byte boundaries) and end
inside a quad, a tile or a block group, with non-finite and all-zero blocks,
against the oracle; nothing outside the buffers is written."""
import numpy as np
import pytest
import torch

import oracle
from gpu_parity_util import to_host
from paper_2607_10611_amd import binding as B

pytestmark = pytest.mark.gpu

BLOCK = {"e4m3": 128, "e5m2": 128, "mxfp4": 32, "nvfp4": 16, "nvfp4_current": 16}


def values(rng, n, blk):
    x = rng.normal(0, 0.02, n).astype(np.float32)
    x[rng.random(n) < 0.02] = 0.0
    x[rng.random(n) < 0.01] *= 1e4
    if blk and n >= 4 * blk:
        x[blk:2 * blk] = 0.0
        x[2 * blk + 3] = np.inf
        x[3 * blk + 1] = np.nan
    return x


def guarded(nbytes, at):
    """A byte buffer of 0xA5 and the `nbytes` of it that start `at` bytes in."""
    t = torch.full((nbytes + at + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    return t, t[at:at + nbytes]


def assert_guards(t, nbytes, at):
    h = t.cpu().numpy()
    assert (h[:at] == 0xA5).all() and (h[at + nbytes:] == 0xA5).all()


@pytest.mark.parametrize("shift", [0, 1, 3])
@pytest.mark.parametrize("wfmt", ["bf16", "e4m3", "e5m2", "fp32"])
@pytest.mark.parametrize("n", [1, 5, 1023, 1024, 4099])
def test_encode_at_any_element(wfmt, n, shift):
    rng = np.random.default_rng(n + shift)
    x = values(rng, n, 0)
    es = int(B.CODE_BYTES[wfmt])
    buf, w = guarded(n * es, shift * es)
    xd = torch.zeros(n + shift, device="cuda")
    xd[shift:] = torch.from_numpy(x).cuda()
    B.madd_encode_weights(xd[shift:], w, wfmt)
    torch.cuda.synchronize()
    ref = oracle.encode_array(wfmt, x)
    assert (to_host(w).view(ref.dtype) == ref).all()
    assert_guards(buf, n * es, shift * es)


@pytest.mark.parametrize("shift", [0, 1, 3])
@pytest.mark.parametrize("wfmt", list(BLOCK))
@pytest.mark.parametrize("blocks", [1, 7, 8, 9, 64, 65, 300])
def test_encode_blocks_at_any_byte(wfmt, blocks, shift):
    blk = BLOCK[wfmt]
    n = blocks * blk
    rng = np.random.default_rng(blocks * 8 + shift)
    x = values(rng, n, blk)
    xd = torch.zeros(n + shift, device="cuda")
    xd[shift:] = torch.from_numpy(x).cuda()
    nb = int(n * B.CODE_BYTES[wfmt])
    buf, w = guarded(nb, shift)
    sb = B.scale_bytes(wfmt, n)
    sbuf, scales = guarded(sb, 4)
    B.madd_encode_weights(xd[shift:], w, wfmt, scales=scales)
    torch.cuda.synchronize()
    enc = {"mxfp4": oracle.encode_mx, "nvfp4": oracle.encode_nv, "nvfp4_current": oracle.encode_nv}
    q, s = enc[wfmt](x) if wfmt in enc else oracle.encode_block(wfmt, x)
    got = to_host(scales)
    if wfmt == "nvfp4_current":  # tensor scale, amax word (cleared), block codes
        assert (got[4:8] == 0).all()
        got = np.concatenate([got[:4], got[8:]])
    assert (to_host(w).view(q.dtype) == q).all()
    assert (got.view(s.dtype) == s).all()
    assert_guards(buf, nb, shift)
    assert_guards(sbuf, sb, 4)


@pytest.mark.parametrize("sfmt", ["fp32", "bf16"])
@pytest.mark.parametrize("n", [1, 3, 7, 8, 9, 4096, 8191, 70001])
def test_zero_state_at_any_element(sfmt, n):
    es = B.STATE_BYTES[sfmt]
    bufs = [guarded(n * es, at * es) for at in (0, 1, 7)]
    views = [b.view(torch.float32 if es == 4 else torch.int16) for _, b in bufs]
    B.madd_init_state(*views, sfmt=sfmt)
    torch.cuda.synchronize()
    for (t, b), at in zip(bufs, (0, 1, 7)):
        assert not b.any()
        assert_guards(t, n * es, at * es)
