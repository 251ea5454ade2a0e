"""Parity of the HIP step (through the C ABI) with the CPU oracle, on the same
seeded inputs.  Bar: weight codes bit-exact; fp32 moments within 2 ulp.

Small cases are compared element by element in full (sizes spanning several
workgroup tiles and ragged tails); the full-size parameter lists run in the
benchmark's launch configuration and are compared on sampled elements, whose
trajectories the oracle recomputes one by one (the step is elementwise and its
random draws are keyed by global index, so a sample is exact).
"""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2607_10611_amd import binding as B
from paper_2607_10611_amd import workloads as W
from gpu_parity_util import (CODE_NP, DevState, HostState, assert_copy_equal, assert_state_equal,
                             free_device_bytes, gpu_step, oracle_step, to_dev, to_host)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    B.lib()  # the HIP library must be built
    yield
    torch.cuda.synchronize()


def hp(**kw):
    h = dict(W.DEFAULT_HPARAMS)
    h.update(kw)
    return h


def random_weights(rng, n, wfmt):
    x = rng.normal(0, 0.02, n).astype(np.float32)
    x[rng.random(n) < 0.02] = 0.0
    big = rng.random(n) < 0.01
    x[big] = rng.normal(0, 3.0, big.sum())
    tiny = rng.random(n) < 0.01
    x[tiny] = rng.normal(0, 1e-6, tiny.sum())
    if wfmt in ("e4m3", "e5m2"):
        lim = 448.0 if wfmt == "e4m3" else 57344.0
        x = np.clip(x, -lim, lim)
    return x


def random_grad(rng, n):
    g = (rng.normal(0, 1, n) * 10.0 ** rng.uniform(-6, -1, n)).astype(np.float32)
    g[rng.random(n) < 0.05] = 0.0
    out = rng.random(n) < 0.001
    g[out] *= 100.0
    return g


def encode_both(wfmt, x, block=False):
    """Initial codes by the oracle and by madd_encode_weights; must agree."""
    xd = torch.from_numpy(x).cuda()
    n = x.size
    if block:
        q_ref, s_ref = oracle.encode_block(wfmt, x)
        q = torch.empty(n, dtype=torch.uint8, device="cuda")
        s = torch.empty(n // 128, dtype=torch.int16, device="cuda")
        B.madd_encode_weights(xd, q, wfmt, scales=s)
        torch.cuda.synchronize()
        assert (to_host(q) == q_ref).all() and (to_host(s, np.uint16) == s_ref).all()
        return q_ref, s_ref
    ref = oracle.encode_array(wfmt, x)
    out = torch.empty(n, dtype={"bf16": torch.int16, "e4m3": torch.uint8, "e5m2": torch.uint8,
                                "fp32": torch.int32}[wfmt], device="cuda")
    B.madd_encode_weights(xd, out, wfmt)
    torch.cuda.synchronize()
    got = to_host(out, CODE_NP[wfmt])
    assert (got == ref).all(), f"encode {wfmt}: {np.nonzero(got != ref)[0][:5]}"
    return ref


def run_pair(wfmt, n, steps, seed, hpkw, gfmt="fp32", index_base=0, block=False, sfmt="fp32",
             copy=False):
    rng = np.random.default_rng(seed)
    x = random_weights(rng, n, wfmt)
    enc = encode_both(wfmt, x, block)
    codes, scales = (enc if block else (enc, None))
    ds = DevState(wfmt, codes, n, scales, sfmt=sfmt, copy=copy)
    hs = HostState(codes, n, scales, sfmt=sfmt, copy=copy)
    for t in range(1, steps + 1):
        g = random_grad(rng, n)
        if gfmt == "bf16":
            g = oracle.encode_array("bf16", g)
        h = hp(step=t, **hpkw)
        gpu_step(ds, to_dev(g), h, gfmt=gfmt, index_base=index_base)
        oracle_step(wfmt, hs, g, h, gfmt=gfmt, index_base=index_base)
        torch.cuda.synchronize()
        w_g, m_g, v_g, ve_g = ds.host()
        assert_state_equal(f"{wfmt} n={n} t={t}", w_g, hs.w, m_g, hs.m, v_g, hs.v, ve_g, hs.ve)
        assert_copy_equal(f"{wfmt} n={n} t={t}", ds, hs)
        if block:
            assert (to_host(ds.scales, np.uint16) == hs.scales).all(), f"scales t={t}"


# ---------------------------------------------------------------------------
# full element-by-element parity at small sizes
# ---------------------------------------------------------------------------

def test_config1_full_trajectory():
    """1024x1024 bf16, N(0, 0.02) weights, fresh N(0, 1e-3) gradients, RNE, as
    many steps as the benchmark runs on this tensor by default (3 + 20)."""
    n = 1024 * 1024
    x = W.init_fp32("c1", 0)
    codes = encode_both("bf16", x)
    ds, hs = DevState("bf16", codes, n), HostState(codes, n)
    for t in range(1, 24):
        g = W.grad_fp32("c1", 0, t)
        h = W.hparams("c1", step=t)
        gpu_step(ds, to_dev(g), h)
        oracle_step("bf16", hs, g, h)
        torch.cuda.synchronize()
        assert_state_equal(f"c1 t={t}", *[a for pair in zip(ds.host(), (hs.w, hs.m, hs.v, hs.ve))
                                          for a in pair])


@pytest.mark.parametrize("bias_correction", [1, 0])
def test_fp32_passthrough_unrounded_step_is_bit_exact(bias_correction):
    """No rounding into a storage format: the fp32 new weights themselves match."""
    run_pair("fp32", 3 * 2048 + 77, 6, 11, dict(rounding="rne", bias_correction=bias_correction))


@pytest.mark.parametrize("n", [1, 7, 8, 9, 127, 1023, 1025, 2047, 2049, 8191, 8193, 65536 + 13])
def test_ragged_sizes_sr(n):
    run_pair("bf16", n, 3, 100 + n, dict(rounding="sr", seed=77), index_base=12345)


@pytest.mark.parametrize("index_base", [0, 3, 8, 2 ** 33 + 5])
def test_index_base_keys_the_draws(index_base):
    run_pair("bf16", 4096 + 40, 2, 5, dict(rounding="sr", seed=2 ** 40 + 1), index_base=index_base)


@pytest.mark.parametrize("wfmt", ["e4m3", "e5m2"])
@pytest.mark.parametrize("rounding", ["rne", "sr"])
def test_fp8_storage(wfmt, rounding):
    run_pair(wfmt, 3 * 8192 + 24, 4, 21, dict(rounding=rounding, lr_add=3e-3, lr_mul=5e-3))


@pytest.mark.parametrize("wfmt", ["e4m3", "e5m2"])
@pytest.mark.parametrize("rounding", ["rne", "sr"])
def test_block_scaled_fp8(wfmt, rounding):
    run_pair(wfmt, 5 * 8192 + 3 * 128, 4, 31, dict(rounding=rounding), block=True)


def test_bf16_gradients():
    run_pair("bf16", 20000, 3, 41, dict(rounding="sr"), gfmt="bf16")


@pytest.mark.parametrize("wfmt", ["bf16", "e4m3", "fp32"])
@pytest.mark.parametrize("n", [9, 2049, 3 * 8192 + 24])
def test_bf16_moments(wfmt, n):
    run_pair(wfmt, n, 4, 43 + n, dict(rounding="sr", lr_mul=5e-3), sfmt="bf16", index_base=16)


@pytest.mark.parametrize("wfmt", ["bf16", "e4m3"])
@pytest.mark.parametrize("n,base", [(1036, 0), (2047, 8), (4095, 2 ** 33 + 16),
                                    (3 * 2048 + 1024 + 20, 64), (1024 + 20, 8), (516, 0)])
def test_aligned_ragged_tails_split_lane_pairs(wfmt, n, base):
    """Aligned index bases with a last tile that ends inside a lane pair's
    group of sub-tile A or B: both lanes draw (they share Philox blocks), and
    the quad over the end is loaded and stored element by element."""
    run_pair(wfmt, n, 3, 70 + n, dict(rounding="sr", seed=91), index_base=base)


@pytest.mark.parametrize("wfmt", ["bf16", "e4m3", "fp32"])
@pytest.mark.parametrize("n,base", [(9, 16), (2047, 16), (3 * 8192 + 24, 16), (5000, 3)])
def test_bf16_sr_moments(wfmt, n, base):
    run_pair(wfmt, n, 4, 60 + n, dict(rounding="sr", lr_mul=5e-3), sfmt="bf16_sr", index_base=base)


def test_bf16_sr_moments_with_nearest_weights_and_bf16_gradients():
    run_pair("bf16", 3 * 8192 + 100, 3, 62, dict(rounding="rne", seed=5), gfmt="bf16",
             sfmt="bf16_sr", index_base=8)


@pytest.mark.parametrize("wfmt", ["e4m3", "e5m2"])
def test_block_scaled_fp8_bf16_sr_moments(wfmt):
    run_pair(wfmt, 2 * 8192 + 5 * 128, 3, 63, dict(rounding="sr"), block=True, copy=True,
             sfmt="bf16_sr")


@pytest.mark.parametrize("wfmt", ["bf16", "e4m3", "e5m2", "fp32"])
@pytest.mark.parametrize("n", [13, 2048 + 4, 2 * 8192 + 40])
def test_compute_copy(wfmt, n):
    run_pair(wfmt, n, 3, 46 + n, dict(rounding="sr"), copy=True, index_base=8 * (n % 3) + n % 2)


@pytest.mark.parametrize("wfmt", ["e4m3", "e5m2"])
@pytest.mark.parametrize("sfmt", ["fp32", "bf16"])
def test_block_scaled_compute_copy(wfmt, sfmt):
    run_pair(wfmt, 2 * 8192 + 7 * 128, 3, 47, dict(rounding="sr"), block=True, copy=True,
             sfmt=sfmt)


def test_bf16_moments_bf16_gradients_misaligned_base():
    run_pair("bf16", 10000, 3, 44, dict(rounding="sr"), gfmt="bf16", sfmt="bf16", index_base=5)


@pytest.mark.parametrize("wfmt", ["e4m3", "e5m2"])
def test_block_scaled_fp8_bf16_moments(wfmt):
    run_pair(wfmt, 3 * 8192 + 5 * 128, 3, 45, dict(rounding="sr"), block=True, sfmt="bf16")


@pytest.mark.parametrize("kw", [dict(g_max=0.5), dict(d_mult_max=0.05), dict(w_max=0.03),
                                dict(eps0=0.2), dict(bias_correction=0),
                                dict(lr_add=0.0), dict(lr_mul=0.0), dict(lr_add=0.0, lr_mul=0.0),
                                dict(beta1=0.0, beta2=0.0)])
def test_algorithm2_options(kw):
    run_pair("bf16", 10000, 3, 51, {**dict(rounding="sr", lr_mul=5e-3), **kw})


def test_last_step_counters():
    """t = 2^32 - 2 and 2^32 - 1, the largest step counters: the bias
    corrections are 1 in fp32 and the Philox counter's step word is all ones."""
    n = 2 * 8192 + 40
    rng = np.random.default_rng(64)
    codes = encode_both("bf16", random_weights(rng, n, "bf16"))
    ds, hs = DevState("bf16", codes, n), HostState(codes, n)
    for t in (2 ** 32 - 2, 2 ** 32 - 1):
        g = random_grad(rng, n)
        h = hp(step=t, rounding="sr", seed=2 ** 63 + 11)
        gpu_step(ds, to_dev(g), h, index_base=8)
        oracle_step("bf16", hs, g, h, index_base=8)
        torch.cuda.synchronize()
        w_g, m_g, v_g, ve_g = ds.host()
        assert_state_equal(f"t={t}", w_g, hs.w, m_g, hs.m, v_g, hs.v, ve_g, hs.ve)


def test_unaligned_buffers_take_the_scalar_path():
    n = 5000
    rng = np.random.default_rng(61)
    x = random_weights(rng, n + 1, "bf16")
    codes = encode_both("bf16", x)
    wbuf = to_dev(codes)
    mbuf, vbuf, vebuf = (torch.zeros(n + 1, device="cuda") for _ in range(3))
    hs = HostState(codes[1:], n)
    for t in range(1, 4):
        g = random_grad(rng, n + 1)
        gd = to_dev(g)
        h = hp(step=t, rounding="sr")
        # element offset 1: every pointer is 2 or 4 bytes off a 16-byte boundary
        B.madd_step(wbuf[1:], "bf16", gd[1:], mbuf[1:], vbuf[1:], vebuf[1:], h, index_base=7)
        oracle_step("bf16", hs, np.ascontiguousarray(g[1:]), h, index_base=7)
        torch.cuda.synchronize()
        assert_state_equal(f"unaligned t={t}", to_host(wbuf, np.uint16)[1:], hs.w,
                           to_host(mbuf)[1:], hs.m, to_host(vbuf)[1:], hs.v, to_host(vebuf)[1:],
                           hs.ve)
        assert to_host(mbuf)[0] == 0.0  # untouched neighbour


def test_unaligned_buffers_bf16_sr_moments():
    # the moment draws (streams 1-3) of quads at any address
    n = 3000
    rng = np.random.default_rng(62)
    codes = encode_both("bf16", random_weights(rng, n + 1, "bf16"))
    wbuf = to_dev(codes)
    mbuf, vbuf, vebuf = (torch.zeros(n + 1, dtype=torch.int16, device="cuda") for _ in range(3))
    hs = HostState(codes[1:], n, sfmt="bf16_sr")
    for t in range(1, 4):
        g = random_grad(rng, n + 1)
        gd = to_dev(g)
        h = hp(step=t, rounding="sr", seed=99)
        B.madd_step(wbuf[1:], "bf16", gd[1:], mbuf[1:], vbuf[1:], vebuf[1:], h, index_base=8,
                    sfmt="bf16_sr")
        oracle_step("bf16", hs, np.ascontiguousarray(g[1:]), h, index_base=8)
        torch.cuda.synchronize()
        assert_state_equal(f"unaligned bf16_sr t={t}", to_host(wbuf, np.uint16)[1:], hs.w,
                           to_host(mbuf, np.uint16)[1:], hs.m, to_host(vbuf, np.uint16)[1:], hs.v,
                           to_host(vebuf, np.uint16)[1:], hs.ve)


def test_nonfinite_gradients():
    n = 4096
    rng = np.random.default_rng(71)
    for wfmt in ("bf16", "e4m3", "e5m2", "fp32"):
        x = random_weights(rng, n, wfmt)
        codes = encode_both(wfmt, x)
        ds, hs = DevState(wfmt, codes, n), HostState(codes, n)
        g = random_grad(rng, n)
        g[::97] = np.nan
        g[1::89] = np.inf
        g[2::83] = -np.inf
        h = hp(rounding="sr")
        gpu_step(ds, to_dev(g), h)
        oracle_step(wfmt, hs, g, h)
        torch.cuda.synchronize()
        w_g, m_g, v_g, ve_g = ds.host()
        assert_state_equal(f"nonfinite {wfmt}", w_g, hs.w, m_g, hs.m, v_g, hs.v, ve_g, hs.ve)


def test_multi_tensor_mixed_list_matches_oracle_and_single_calls():
    rng = np.random.default_rng(81)
    layout = [("bf16", 3000, False), ("e4m3", 8192, True), ("fp32", 17, False),
              ("bf16", 20480, False), ("e5m2", 1024, False), ("e5m2", 384, True),
              ("bf16", 0, False), ("e4m3", 5000, False)]
    devs, hosts, singles = [], [], []
    for wfmt, n, blk in layout:
        x = random_weights(rng, n, wfmt)
        enc = encode_both(wfmt, x, blk) if n else ((np.zeros(0, CODE_NP[wfmt]),
                                                    np.zeros(0, np.uint16)) if blk else
                                                   np.zeros(0, CODE_NP[wfmt]))
        codes, scales = (enc if blk else (enc, None))
        cp = wfmt in ("e4m3", "e5m2")  # compute copies for the FP8 tensors
        devs.append(DevState(wfmt, codes, n, scales, copy=cp))
        singles.append(DevState(wfmt, codes, n, scales, copy=cp))
        hosts.append(HostState(codes, n, scales, copy=cp))
    base = 1000
    for t in range(1, 4):
        gs = [random_grad(rng, n) for _, n, _ in layout]
        gds = [to_dev(g) for g in gs]
        h = hp(step=t, rounding="sr", seed=314)
        tl = B.TensorList([d.w for d in devs], [d.wfmt for d in devs], gds, [d.m for d in devs],
                          [d.v for d in devs], [d.ve for d in devs],
                          scales=[d.scales for d in devs], copies=[d.copy for d in devs])
        B.madd_multi_tensor_step(tl, h, index_base=base)
        off = base
        for (wfmt, n, blk), d1, hs, g, gd in zip(layout, singles, hosts, gs, gds):
            if n:
                gpu_step(d1, gd, h, index_base=off)
                oracle_step(wfmt, hs, g, h, index_base=off)
            off += n
        torch.cuda.synchronize()
        for (wfmt, n, blk), d, d1, hs in zip(layout, devs, singles, hosts):
            if not n:
                continue
            w_g, m_g, v_g, ve_g = d.host()
            assert_state_equal(f"multi {wfmt} n={n} t={t}", w_g, hs.w, m_g, hs.m, v_g, hs.v,
                               ve_g, hs.ve)
            for a, b in zip(d.host(), d1.host()):
                assert a.tobytes() == b.tobytes()
            assert_copy_equal(f"multi {wfmt} n={n} t={t}", d, hs)
            if blk:
                assert (to_host(d.scales, np.uint16) == hs.scales).all()


def test_descriptor_table_cache_eviction():
    """More distinct tensor lists than the library caches (32): each new list
    uploads a table, the least recently used one is evicted after the device
    drains, and a list whose table was evicted is uploaded again on its next
    call.  Every step must still match single calls."""
    rng = np.random.default_rng(83)
    lists = []
    for k in range(40):
        sizes = (256 + 8 * k, 1000 + k)
        devs, singles = [], []
        for j, n in enumerate(sizes):
            codes = oracle.encode_array("bf16", random_weights(rng, n, "bf16"))
            devs.append(DevState("bf16", codes, n))
            singles.append(DevState("bf16", codes, n))
        gs = [to_dev(random_grad(rng, n)) for n in sizes]
        tl = B.TensorList([d.w for d in devs], ["bf16"] * 2, gs, [d.m for d in devs],
                          [d.v for d in devs], [d.ve for d in devs])
        lists.append((sizes, devs, singles, gs, tl))
    order = list(range(40)) + [0, 1, 39, 5]
    steps = {}
    for k in order:
        sizes, devs, singles, gs, tl = lists[k]
        t = steps[k] = steps.get(k, 0) + 1
        h = hp(step=t, rounding="sr", seed=k)
        B.madd_multi_tensor_step(tl, h, index_base=64)
        off = 64
        for d1, g, n in zip(singles, gs, sizes):
            gpu_step(d1, g, h, index_base=off)
            off += n
    torch.cuda.synchronize()
    for sizes, devs, singles, gs, tl in lists:
        for d, d1 in zip(devs, singles):
            for a, b in zip(d.host(), d1.host()):
                assert a.tobytes() == b.tobytes()


def test_init_state_zeroes():
    n = 70001
    ts = [torch.full((n + 1,), 3.0, device="cuda") for _ in range(3)]
    B.madd_init_state(*[t[:n] for t in ts])
    hs = [torch.full((n + 1,), 7, dtype=torch.int16, device="cuda") for _ in range(3)]
    B.madd_init_state(*[t[:n] for t in hs])
    torch.cuda.synchronize()
    assert all(float(t[:n].abs().max()) == 0.0 and float(t[n]) == 3.0 for t in ts)
    assert all(int(t[:n].abs().max()) == 0 and int(t[n]) == 7 for t in hs)


def test_encode_weights_all_formats():
    rng = np.random.default_rng(91)
    x = random_weights(rng, 128 * 333, "bf16")
    x[:5] = [np.nan, np.inf, -np.inf, 1e38, -3e38]
    for wfmt in ("bf16", "e4m3", "e5m2", "fp32"):
        encode_both(wfmt, x)
    for wfmt in ("e4m3", "e5m2"):
        encode_both(wfmt, np.nan_to_num(x, nan=0.0, posinf=1.0, neginf=-1.0), block=True)


# ---------------------------------------------------------------------------
# full-size parameter lists, sampled
# ---------------------------------------------------------------------------

def sample_indices(n, rng, k=4096):
    if n <= 3 * k:
        return np.arange(n)
    head, tail = np.arange(k), np.arange(n - k, n)
    mid = np.sort(rng.choice(np.arange(k, n - k), size=k, replace=False))
    return np.concatenate([head, mid, tail])


def run_list_sampled(cfg, steps, wfmt=None, per_tensor=4096, sfmt="fp32"):
    """Whole list on the GPU with one multi-tensor call per step (the benchmark
    launch); the oracle follows sampled elements of every tensor."""
    specs = W.specs(cfg)
    wfmt = wfmt or W.CONFIGS[cfg]["wfmt"]
    rng = np.random.default_rng(7)
    ws, ms, vs, ves, gs, samples, hosts = [], [], [], [], [], [], []
    offsets = np.cumsum([0] + [s.numel for s in specs])
    for i, s in enumerate(specs):
        x = W.init_fp32_device(cfg, i)
        w = torch.empty(s.numel, dtype={"bf16": torch.int16, "e4m3": torch.uint8,
                                        "e5m2": torch.uint8}[wfmt], device="cuda")
        B.madd_encode_weights(x, w, wfmt)
        idx = sample_indices(s.numel, rng, per_tensor)
        idx_t = torch.from_numpy(idx).cuda()
        x_s = to_host(x[idx_t])
        codes_ref = oracle.encode_array(wfmt, x_s)
        assert (to_host(w[idx_t], CODE_NP[wfmt]) == codes_ref).all(), f"encode {s.name}"
        del x
        ws.append(w)
        st = torch.float32 if sfmt == "fp32" else torch.int16
        ms.append(torch.zeros(s.numel, dtype=st, device="cuda"))
        vs.append(torch.zeros(s.numel, dtype=st, device="cuda"))
        ves.append(torch.zeros(s.numel, dtype=st, device="cuda"))
        gs.append(torch.empty(s.numel, device="cuda"))
        samples.append((idx, idx_t))
        hosts.append(HostState(codes_ref, idx.size, sfmt=sfmt))
    tl = B.TensorList(ws, [wfmt] * len(ws), gs, ms, vs, ves, sfmt=sfmt)
    for t in range(1, steps + 1):
        for i in range(len(specs)):
            W.grad_fp32_device_(cfg, i, t, gs[i])
        h = W.hparams(cfg, step=t)
        B.madd_multi_tensor_step(tl, h)
        for i, (idx, idx_t) in enumerate(samples):
            g_s = to_host(gs[i][idx_t])
            oracle_step(wfmt, hosts[i], g_s, h, gidx=idx + offsets[i])
        if t == steps or t % 5 == 0:
            torch.cuda.synchronize()
            sn = np.float32 if sfmt == "fp32" else np.uint16
            for i, (idx, idx_t) in enumerate(samples):
                hs = hosts[i]
                assert_state_equal(f"{cfg} {specs[i].name} t={t}",
                                   to_host(ws[i][idx_t], CODE_NP[wfmt]), hs.w,
                                   to_host(ms[i][idx_t], sn), hs.m, to_host(vs[i][idx_t], sn),
                                   hs.v, to_host(ves[i][idx_t], sn), hs.ve)
    return offsets[-1]


def test_one_tensor_past_2pow32_elements():
    """Maximum sizes: one madd_step call over 2^32 + 4196 elements (byte offsets
    past 16 GiB, chunk indices past 2^21), checked on samples at the start,
    across element 2^32 and at the ragged end."""
    n = 2 ** 32 + 4196
    free = free_device_bytes()
    assert free > n * 24 + (1 << 30), "needs about 100 GiB of device memory"
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    w = torch.empty(n, dtype=torch.int16, device="cuda")
    x = torch.randn(n, device="cuda", generator=gen).mul_(0.02)
    B.madd_encode_weights(x, w, "bf16")
    del x
    m, v, ve = (torch.zeros(n, device="cuda") for _ in range(3))
    idx = np.concatenate([np.arange(0, 3000), np.arange(2 ** 32 - 1500, 2 ** 32 + 1500),
                          np.arange(n - 3000, n)])
    idx_t = torch.from_numpy(idx).cuda()
    hs = HostState(to_host(w[idx_t], np.uint16), idx.size)
    base = 2 ** 20
    for t in (1, 2):
        g = torch.randn(n, device="cuda", generator=gen).mul_(1e-3)
        h = hp(step=t, rounding="sr", seed=17)
        B.madd_step(w, "bf16", g, m, v, ve, h, index_base=base)
        oracle_step("bf16", hs, to_host(g[idx_t]), h, gidx=idx + base)
        torch.cuda.synchronize()
        assert_state_equal(f"2^32+ t={t}", to_host(w[idx_t], np.uint16), hs.w, to_host(m[idx_t]),
                           hs.m, to_host(v[idx_t]), hs.v, to_host(ve[idx_t]), hs.ve)
        del g


def test_config2_gpt2_small_100_steps_sampled():
    assert run_list_sampled("c2", 100, per_tensor=1024) == 124_439_808


def test_config3_llama_1b_sampled():
    # every step the benchmark runs on this list at its defaults: 3 + 20
    assert run_list_sampled("c3", 23) == 1_100_048_384


@pytest.mark.parametrize("wfmt", ["e4m3", "e5m2"])
def test_config4_llama_1b_fp8_sampled(wfmt):
    assert run_list_sampled("c4", 23, wfmt=wfmt) == 1_100_048_384


def test_config3_llama_1b_bf16_moments_sampled():
    assert run_list_sampled("c3", 10, sfmt="bf16") == 1_100_048_384


def test_config3_llama_1b_bf16_sr_moments_sampled():
    assert run_list_sampled("c3", 10, sfmt="bf16_sr") == 1_100_048_384


def test_config5_llama_7b_sampled():
    free = free_device_bytes()
    need = 6_738_415_616 * 18 + (1 << 30)
    assert free > need, f"config 5 needs {need / 2**30:.0f} GiB of device memory"
    # every step the benchmark runs: 5 warm-up and 20 timed steps
    assert run_list_sampled("c5", 25, per_tensor=2048) == 6_738_415_616


def test_config5_llama_7b_bf16_moments_sampled():
    free = free_device_bytes()
    need = 6_738_415_616 * 12 + (1 << 30)
    assert free > need, f"needs {need / 2**30:.0f} GiB of device memory"
    assert run_list_sampled("c5", 10, per_tensor=1024, sfmt="bf16") == 6_738_415_616


# ---------------------------------------------------------------------------
# the paper's FP8-master setting on the full 7B list, sampled
# ---------------------------------------------------------------------------

def test_fp8_master_llama7b_sampled():
    """Attention and MLP linear weights block-scaled E4M3 with bf16 compute
    copies, embeddings / norms / head in bf16 (Section 4.2), one multi-tensor
    call per step; the oracle follows sampled whole 128-element blocks."""
    cfg = "c5"
    specs = W.specs(cfg)
    plan = W.fp8_master_plan(cfg)
    rng = np.random.default_rng(9)
    offsets = np.cumsum([0] + [s.numel for s in specs])
    dev = dict(w=[], sc=[], cp=[], m=[], v=[], ve=[], g=[])
    samples, hosts = [], []
    for i, (s, (wfmt, blk, cp)) in enumerate(zip(specs, plan)):
        x = W.init_fp32_device(cfg, i)
        w = torch.empty(s.numel, dtype=torch.uint8 if blk else torch.int16, device="cuda")
        sc = torch.empty(s.numel // 128, dtype=torch.int16, device="cuda") if blk else None
        B.madd_encode_weights(x, w, wfmt, scales=sc)
        nb = s.numel // 128
        bidx = np.unique(np.concatenate([np.arange(4), np.arange(nb - 4, nb),
                                         rng.choice(nb, size=min(nb, 24), replace=False)]))
        idx = (bidx[:, None] * 128 + np.arange(128)[None, :]).ravel()
        idx_t = torch.from_numpy(idx).cuda()
        x_s = to_host(x[idx_t])
        if blk:
            q_ref, s_ref = oracle.encode_block(wfmt, x_s)
            assert (to_host(w[idx_t], np.uint8) == q_ref).all()
            assert (to_host(sc[torch.from_numpy(bidx).cuda()], np.uint16) == s_ref).all()
            hs = HostState(q_ref, idx.size, s_ref, copy=cp)
        else:
            codes = oracle.encode_array(wfmt, x_s)
            assert (to_host(w[idx_t], np.uint16) == codes).all()
            hs = HostState(codes, idx.size, copy=cp)
        del x
        dev["w"].append(w)
        dev["sc"].append(sc)
        dev["cp"].append(torch.zeros(s.numel, dtype=torch.int16, device="cuda") if cp else None)
        for k in ("m", "v", "ve"):
            dev[k].append(torch.zeros(s.numel, device="cuda"))
        dev["g"].append(torch.empty(s.numel, device="cuda"))
        samples.append((idx, idx_t, bidx))
        hosts.append(hs)
    tl = B.TensorList(dev["w"], [p[0] for p in plan], dev["g"], dev["m"], dev["v"], dev["ve"],
                      scales=dev["sc"], copies=dev["cp"])
    for t in range(1, 11):
        for i in range(len(specs)):
            W.grad_fp32_device_(cfg, i, t, dev["g"][i])
        h = W.hparams(cfg, step=t)
        B.madd_multi_tensor_step(tl, h)
        for i, (idx, idx_t, bidx) in enumerate(samples):
            oracle_step(plan[i][0], hosts[i], to_host(dev["g"][i][idx_t]), h,
                        gidx=idx + offsets[i])
        torch.cuda.synchronize()
        for i, (idx, idx_t, bidx) in enumerate(samples):
            hs, (wfmt, blk, cp) = hosts[i], plan[i]
            tag = f"fp8-master {specs[i].name} t={t}"
            assert_state_equal(tag, to_host(dev["w"][i][idx_t], CODE_NP[wfmt]), hs.w,
                               to_host(dev["m"][i][idx_t]), hs.m, to_host(dev["v"][i][idx_t]),
                               hs.v, to_host(dev["ve"][i][idx_t]), hs.ve)
            if blk:
                got = to_host(dev["sc"][i][torch.from_numpy(bidx).cuda()], np.uint16)
                assert (got == hs.scales).all(), tag
            if cp:
                assert (to_host(dev["cp"][i][idx_t], np.uint16) == hs.copy).all(), tag


def test_binding_checks_buffer_sizes_before_launch():
    """The binding refuses tensors too small for the call, non-contiguous
    ones and short scale arrays, so no kernel touches memory past a buffer."""
    n = 4096
    w = torch.zeros(n, dtype=torch.int16, device="cuda")
    g, m, v, ve = (torch.zeros(n, device="cuda") for _ in range(4))
    with pytest.raises(ValueError, match="bytes"):
        B.madd_step(w[:n - 8], "bf16", g, m, v, ve, hp())
    with pytest.raises(ValueError, match="bytes"):
        B.madd_step(w, "bf16", g[:n - 4], m, v, ve, hp())
    with pytest.raises(ValueError, match="contiguous"):
        B.madd_step(w, "bf16", torch.zeros(2 * n, device="cuda")[::2], m, v, ve, hp())
    q = torch.zeros(n // 2, dtype=torch.uint8, device="cuda")
    with pytest.raises(ValueError, match="scales"):
        B.madd_step(q, "nvfp4", g, m, v, ve, hp(),
                    scales=torch.zeros(n // 16, dtype=torch.uint8, device="cuda"))
    with pytest.raises(ValueError, match="copy"):
        B.madd_step(w, "bf16", g, m, v, ve, hp(), copy=w[:10])
    with pytest.raises(ValueError, match="bytes"):
        B.TensorList([w], ["bf16"], [g], [m], [v[:100]], [ve])
    tl = B.TensorList([w], ["bf16"], [g[:n // 2]], [m], [v], [ve])
    with pytest.raises(ValueError, match="bytes"):
        B.madd_multi_tensor_step(tl, hp())
    torch.cuda.synchronize()
    assert (m == 0).all() and (w == 0).all()


def test_adjacent_slices_of_one_buffer_step_like_separate_buffers():
    """Disjoint buffers may sit back to back in one allocation (m, v, v_e as
    consecutive slices, the gradient right after the weights): the step takes
    them and gives the same bits as separate allocations; slices that overlap
    by one element are rejected (MADD_EINVAL) before any device work."""
    n = 3 * 2048 + 520
    rng = np.random.default_rng(91)
    x = random_weights(rng, n, "bf16")
    codes = oracle.encode_array("bf16", x)
    h = hp(step=1, rounding="sr", seed=5)
    results = []
    for packed in (False, True):
        grads = [random_grad(np.random.default_rng(7 + t), n) for t in (1, 2)]
        if packed:
            state = torch.zeros(3 * n, device="cuda")
            m, v, ve = state[:n], state[n:2 * n], state[2 * n:]
            wg = torch.zeros(n + 2 * n, dtype=torch.int16, device="cuda")  # w, then g (fp32)
            w, g = wg[:n], wg[n:].view(torch.float32)
        else:
            m, v, ve = (torch.zeros(n, device="cuda") for _ in range(3))
            w = torch.zeros(n, dtype=torch.int16, device="cuda")
            g = torch.zeros(n, device="cuda")
        w.copy_(torch.from_numpy(codes.view(np.int16)).cuda())
        for t, gh in enumerate(grads, start=1):
            g.copy_(torch.from_numpy(gh).cuda())
            B.madd_step(w, "bf16", g, m, v, ve, dict(h, step=t))
        torch.cuda.synchronize()
        results.append([to_host(a) for a in (w, m, v, ve)])
    for a, b in zip(*results):
        assert np.array_equal(a.view(np.uint8), b.view(np.uint8))
    state = torch.zeros(3 * n, device="cuda")
    w = torch.zeros(n, dtype=torch.int16, device="cuda")
    g = torch.zeros(n, device="cuda")
    with pytest.raises(B.MaddError, match="EINVAL"):
        B.madd_step(w, "bf16", g, state[:n], state[n - 1:2 * n - 1], state[2 * n:], h)
    with pytest.raises(B.MaddError, match="EINVAL"):
        B.madd_init_state(state[:n], state[:n], state[2 * n:])
    torch.cuda.synchronize()
    assert (state == 0).all()
