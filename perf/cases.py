"""Timed cases of the M+Adam step: the calls a training program makes, through
the public entry points (binding.madd_*, optim.MAdam), over the formats and
sizes the library is used at.

Every case keeps a tensor list the way fused optimizers do, one flat buffer
per role with the tensors as views in list order, so that a pass returns whole
buffers.  The update is specified to the bit (one fixed fp32 operation order
with correctly rounded divisions and square roots, draws keyed by seed, step
and global index), so every tolerance is "exact".

A pass advances the step counter, as a training loop does.  Gradients are not
rewritten between passes, except by the NVFP4 current-scaling step, which
leaves the updated weights in them; the next pass then steps with those.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2607_10611_amd import binding as B
from paper_2607_10611_amd.optim import MAdam

HP = dict(lr_add=1e-3, lr_mul=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, tau=1e-8, r_max=0.75)
TOY_HP = dict(HP, lr_add=10.0, lr_mul=10.0, rounding="rne", step=1)  # the diagnostic's rate
SEED = 0x4D414444
T0 = 100  # steps already taken when a case starts

CODE = {"bf16": 2, "e4m3": 1, "e5m2": 1, "fp32": 4, "mxfp4": 0.5, "nvfp4": 0.5,
        "nvfp4_current": 0.5}
CODE_DTYPE = {"bf16": torch.int16, "fp32": torch.int32}  # others: bytes
GRAD = {"fp32": torch.float32, "bf16": torch.bfloat16}
MOMENT = {"fp32": torch.float32, "bf16": torch.bfloat16, "bf16_sr": torch.bfloat16}
BLOCK = {"e4m3": 128, "e5m2": 128, "mxfp4": 32, "nvfp4": 16, "nvfp4_current": 16}


# ---------------------------------------------------------------------------
# The lists
# ---------------------------------------------------------------------------

def _llama(c):
    """(elements, is a linear layer) of every tensor of a Llama-shaped list."""
    d, ff, kv = c["d"], c["ff"], c["kv"]
    layer = [(d * d, True), (kv * d, True), (kv * d, True), (d * d, True), (ff * d, True),
             (ff * d, True), (d * ff, True), (d, False), (d, False)]
    return [(c["vocab"] * d, False)] + layer * c["layers"] + [(d, False), (c["vocab"] * d, False)]


def _gpt2(c):
    d = c["d"]
    layer = [(d, False), (d, False), (3 * d * d, True), (3 * d, False), (d * d, True), (d, False),
             (d, False), (d, False), (4 * d * d, True), (4 * d, False), (4 * d * d, True),
             (d, False)]
    return [(c["vocab"] * d, False), (c["context"] * d, False)] + layer * c["layers"] + [(d, False)] * 2


def _ragged(c):
    r = random.Random(c["mix"])
    top = math.log(c["largest"])
    sizes = [max(1, int(math.exp(r.uniform(0.0, top)))) for _ in range(c["tensors"] - 1)]
    sizes.insert(r.randrange(len(sizes) + 1), c["largest"])
    return [(n, False) for n in sizes]


def _tensors(c):
    return {"llama": _llama, "gpt2": _gpt2, "ragged": _ragged,
            "one": lambda c: [(c["n"], True)]}[c["list"]](c)


def _format(c, linear):
    """(weight format, block-scaled) of one tensor: in a "-master" list the
    linear layers are block-scaled, the rest bf16."""
    w = c["weights"]
    if not w.endswith("-master"):
        return w, False
    return (w[:-len("-master")], True) if linear else ("bf16", False)


class _Layout:
    """Where each tensor starts in the flat buffers.  Separately allocated
    parameters are aligned; packed ones follow each other without gaps."""

    def __init__(self, c):
        self.tensors = [(n,) + _format(c, lin) for n, lin in _tensors(c)]
        gap = 1 if c.get("packed") else 128
        self.at, o = [], int(c.get("shift", 0))
        for n, _, _ in self.tensors:
            self.at.append(o)
            o += -(-n // gap) * gap
        self.total = o


def _inputs(c, seed, lay):
    """Initial fp32 weights, gradients and moments of a run T0 steps old, in
    the layout's flat buffers.  Gradients N(0, s) with s log-uniform per
    tensor in [1e-5, 1e-2], 5% exact zeros and 0.1% outliers x100; moments of
    the matching sizes."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 1000003 + 17)
    host = random.Random(int(seed))
    N = lay.total

    def noise():
        return torch.randn(N, generator=gen, device="cuda")

    x, g, m, v, ve = noise().mul_(0.02), noise(), noise(), noise().abs_(), noise().abs_()
    u = torch.rand(N, generator=gen, device="cuda")
    g.masked_fill_(u < 0.05, 0.0)
    g.mul_(torch.where(u > 0.999, 100.0, 1.0))
    del u
    end = 0
    for (n, _, _), o in zip(lay.tensors, lay.at):
        for a in (x, g, m, v, ve):
            a[end:o].zero_()  # between two tensors
        end = o + n
        s = math.exp(host.uniform(math.log(1e-5), math.log(1e-2)))
        g[o:o + n].mul_(s)
        m[o:o + n].mul_(0.3 * s)
        v[o:o + n].mul_(0.1 * s * s)
        ve[o:o + n].mul_(0.1 * (0.014 * s) ** 2)
    for a in (x, g, m, v, ve):
        a[end:].zero_()
    dt = MOMENT[c["moments"]]
    return x, g.to(GRAD[c["grads"]]), m.to(dt), v.to(dt), ve.to(dt)


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def listed():
    llama1b = dict(kind="step", list="llama", d=2048, ff=5632, layers=22, vocab=32000, kv=256,
                   rounding="sr")
    return [
        # Appendix B's diagnostic, one iteration of its loop: 4096 entries, the
        # smallest calls, where launches and their gaps are the time.
        dict(name="diagnostic-4096", kind="toy", n=4096, batch=4096, weights="bf16"),
        # One 1024x1024 weight matrix, the smallest benchmarked step.
        dict(name="matrix-1024x1024", kind="one", list="one", n=1024 * 1024, base=0, weights="bf16",
             moments="fp32", grads="fp32", rounding="rne"),
        # GPT-2-small (148 tensors) from a PyTorch training loop: the torch.optim front end,
        # bf16 parameters, gradients and moments.
        dict(name="gpt2-madam-bf16", kind="madam", list="gpt2", d=768, layers=12, vocab=50257,
             context=1024, weights="bf16", moments="bf16", grads="bf16", rounding="sr"),
        # The 1.1B list with bf16 weights and fp32 gradients and moments: the headline
        # workload's kernel.
        dict(llama1b, name="llama1b-bf16", weights="bf16", moments="fp32", grads="fp32"),
        # bf16 moments, stochastically rounded: half the optimizer state.
        dict(llama1b, name="llama1b-bf16sr-moments", weights="bf16", moments="bf16_sr",
             grads="fp32"),
        # The same list stored in FP8.
        dict(llama1b, name="llama1b-e4m3", weights="e4m3", moments="fp32", grads="fp32"),
        # FP8 master weights with their bf16 compute copies, bf16 gradients and moments.
        dict(llama1b, name="llama1b-fp8-master", weights="e4m3-master", moments="bf16",
             grads="bf16"),
        # 4-bit master weights (NVFP4) in the same setting.
        dict(llama1b, name="llama1b-nvfp4-master", weights="nvfp4-master", moments="bf16",
             grads="bf16"),
        # NVFP4 with its tensor scale derived anew every step.
        dict(llama1b, name="llama1b-nvfp4cs-master", weights="nvfp4_current-master",
             moments="fp32", grads="fp32"),
        # A model with odd-sized tensors (biases of one element, odd vocabularies, small
        # convolutions), each parameter allocated by itself: global indices that are not
        # multiples of eight.
        dict(name="ragged-bf16", kind="step", list="ragged", tensors=96, largest=15999989, mix=7,
             packed=False, weights="bf16", moments="fp32", grads="fp32", rounding="sr"),
        # Such a model packed into flat buffers without gaps, as sharded optimizers do: its
        # tensors are not 16-byte aligned either.
        dict(name="ragged-packed-e4m3", kind="step", list="ragged", tensors=64, largest=9999991,
             mix=11, packed=True, weights="e4m3", moments="bf16", grads="bf16", rounding="sr"),
        # Setting up 4-bit masters for the 11008x4096 matrix of a 7B model: state zeroed,
        # weights encoded (also how a kept tensor scale is refreshed).
        dict(name="setup-nvfp4-11008x4096", kind="setup", list="one", n=11008 * 4096,
             weights="nvfp4-master", moments="bf16"),
    ]


def _log(r, lo, hi):
    return int(math.exp(r.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    moments, grads = rng.choice(["fp32", "bf16", "bf16_sr"]), rng.choice(["fp32", "bf16"])
    rounding = rng.choice(["sr", "sr", "rne"])
    kind = rng.choice(["llama", "llama", "ragged", "one", "one", "madam", "setup", "toy"])
    plain = rng.choice(["bf16", "bf16", "e4m3", "e5m2", "fp32"])
    master = rng.choice(["e4m3", "e5m2", "mxfp4", "nvfp4", "nvfp4_current"])
    opts = dict(moments=moments, grads=grads, rounding=rounding)
    if kind in ("llama", "madam"):
        d = 128 * rng.randint(2, 16)
        c = dict(kind="step" if kind == "llama" else "madam", list="llama", d=d,
                 ff=rng.randint(2 * d, 4 * d) // 2 * 2, kv=64 * rng.randint(1, d // 64),
                 vocab=_log(rng, 1000, 32000), layers=_log(rng, 1, 22), **opts)
        c["weights"] = (master + "-master") if rng.random() < 0.6 and kind == "llama" else plain
        if c["weights"].startswith("nvfp4_current"):
            c["grads"] = "fp32"
        if kind == "madam":
            c["weights"] = rng.choice(["bf16", "fp32"])
            c["grads"] = "fp32" if c["weights"] == "fp32" else "bf16"
        while sum(n for n, _ in _tensors(c)) > 1000000000:
            c["layers"] -= 1
        return c
    if kind == "ragged":
        return dict(kind="step", list="ragged", tensors=_log(rng, 2, 128),
                    largest=_log(rng, 2000, 16000000), mix=rng.randrange(1 << 30),
                    packed=rng.random() < 0.5, weights=plain, **opts)
    if kind == "one":
        if rng.random() < 0.5:
            w = master + "-master"
            n = BLOCK[master] * _log(rng, 8, 300000000 // BLOCK[master])
            if master == "nvfp4_current":
                opts["grads"] = "fp32"
            return dict(kind="one", list="one", n=n, base=rng.choice([0, 8 * rng.randrange(1 << 30),
                        rng.randrange(1 << 33)]), weights=w, **opts)
        base = rng.choice([0, 8 * rng.randrange(1 << 30), rng.randrange(1 << 33)])
        shift = rng.choice([0, 0, 1, 8, rng.randrange(64)])
        top = 30000000 if base % 8 or shift else 300000000
        return dict(kind="one", list="one", n=_log(rng, 500, top), base=base, shift=shift,
                    weights=plain, **opts)
    if kind == "setup":
        if rng.random() < 0.7:
            return dict(kind="setup", list="one", weights=master + "-master", moments=moments,
                        n=BLOCK[master] * _log(rng, 32, 300000000 // BLOCK[master]))
        return dict(kind="setup", list="one", weights=plain, moments=moments,
                    n=_log(rng, 2000, 300000000))
    return dict(kind="toy", n=_log(rng, 256, 4000000), batch=_log(rng, 256, 1000000),
                weights=plain)


# ---------------------------------------------------------------------------
# Preparing, running
# ---------------------------------------------------------------------------

def _codes(fmt, n):
    dt = CODE_DTYPE.get(fmt, torch.uint8)
    return torch.empty(math.ceil(n * CODE[fmt] / dt.itemsize), dtype=dt, device="cuda")


def _code_view(flat, fmt, o, n):
    if CODE[fmt] == 0.5:
        return flat[o // 2:(o + n) // 2]
    return flat[o:o + n]


def _as_values(codes, fmt):
    return codes.view({"bf16": torch.bfloat16, "fp32": torch.float32}.get(fmt, codes.dtype))


def _prepare_toy(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 1000003 + 29)
    n = c["n"]
    target = torch.randn(n, generator=gen, device="cuda")
    w0 = target + 0.5 * torch.randn(n, generator=gen, device="cuda")
    w = _codes(c["weights"], n)
    B.madd_encode_weights(w0, w, c["weights"])
    return dict(case=c, w=w, target=target, c=torch.ones(n, device="cuda"),
                idx=torch.randint(0, n, (c["batch"],), generator=gen, device="cuda"),
                counts=torch.empty(n, dtype=torch.int32, device="cuda"),
                g=torch.empty(n, device="cuda"))


def prepare(case, seed):
    c = dict(case)
    if c["kind"] == "toy":
        return _prepare_toy(c, seed)
    lay = _Layout(c)
    if c["kind"] == "setup":
        gen = torch.Generator(device="cuda")
        gen.manual_seed(int(seed) * 1000003 + 41)
        n, fmt, blk = lay.tensors[0]
        x = torch.randn(n, generator=gen, device="cuda").mul_(0.02)
        w = _codes(fmt, n)
        sc = torch.zeros(B.scale_bytes(fmt, n), dtype=torch.uint8, device="cuda") if blk else None
        mom = [torch.empty(n, dtype=MOMENT[c["moments"]], device="cuda") for _ in range(3)]
        return dict(case=c, x=x, w=w, scales=sc, mom=mom, fmt=fmt,
                    sfmt=c["moments"])
    x, g, m, v, ve = _inputs(c, seed, lay)
    fmts = sorted({f for _, f, _ in lay.tensors})
    flat = {f: _codes(f, lay.total).zero_() for f in fmts}
    copy = torch.zeros(lay.total, dtype=torch.int16, device="cuda") if c["weights"].endswith("-master") else None
    sizes = [-(-B.scale_bytes(f, n) // 16) * 16 if blk else 0 for n, f, blk in lay.tensors]
    scales = torch.zeros(max(1, sum(sizes)), dtype=torch.uint8, device="cuda")
    ws, scs, cps, so = [], [], [], 0
    for (n, f, blk), o, k in zip(lay.tensors, lay.at, sizes):
        w = _code_view(flat[f], f, o, n)
        sc = scales[so:so + B.scale_bytes(f, n)] if blk else None
        so += k
        B.madd_encode_weights(x[o:o + n], w, f, scales=sc)
        ws.append(w)
        scs.append(sc)
        cps.append(copy[o:o + n] if blk else None)
    del x
    cut = lambda t: [t[o:o + n] for (n, _, _), o in zip(lay.tensors, lay.at)]  # noqa: E731
    out = {"m": m, "v": v, "ve": ve, "w": [_as_values(flat[f], f) for f in fmts]}
    if copy is not None:
        out["copy"], out["scales"] = copy, scales
    if c["weights"].startswith("nvfp4_current"):
        out["new"] = g
    s = dict(case=c, t=T0, out=out, gfmt=c["grads"], sfmt=c["moments"],
             hp=dict(HP, rounding=c["rounding"], seed=SEED))
    if c["kind"] == "madam":
        params = []
        for w, gi in zip(ws, cut(g)):
            p = torch.nn.Parameter(_as_values(w, c["weights"]))
            p.grad = gi
            params.append(p)
        opt = MAdam(params, lr_add=HP["lr_add"], lr_mul=HP["lr_mul"], rounding=c["rounding"],
                    seed=SEED, state_format=c["moments"])
        raw = (lambda t: t) if c["moments"] == "fp32" else (lambda t: t.view(torch.int16))
        for p, a, b, e in zip(params, cut(raw(m)), cut(raw(v)), cut(raw(ve))):  # resumed
            opt.state[p].update(step=T0, m=a, v=b, ve=e)
        s["opt"] = opt
    elif c["kind"] == "one":
        s["args"] = (ws[0], lay.tensors[0][1], cut(g)[0], cut(m)[0], cut(v)[0], cut(ve)[0])
        s["more"] = dict(gfmt=c["grads"], sfmt=c["moments"], scales=scs[0], copy=cps[0],
                         index_base=c["base"])
    else:
        blocks = any(blk for _, _, blk in lay.tensors)
        s["tl"] = B.TensorList(ws, [f for _, f, _ in lay.tensors], cut(g), cut(m), cut(v), cut(ve),
                               scales=scs if blocks else None, sfmt=c["moments"],
                               copies=cps if blocks else None)
    return s


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "toy":
        B.madd_toy_gradient(s["w"], c["weights"], s["target"], s["c"], s["idx"], s["counts"], s["g"])
        B.madd_plain_step(s["w"], c["weights"], s["g"], TOY_HP)
        return {"w": _as_values(s["w"], c["weights"]), "g": s["g"], "counts": s["counts"]}
    if c["kind"] == "setup":
        B.madd_init_state(*s["mom"], sfmt=s["sfmt"])
        B.madd_encode_weights(s["x"], s["w"], s["fmt"], scales=s["scales"])
        return {"w": _as_values(s["w"], s["fmt"]), "scales": s["scales"], "mom": s["mom"]}
    if c["kind"] == "madam":
        s["opt"].step()
        return s["out"]
    s["t"] += 1
    hp = dict(s["hp"], step=s["t"])
    if c["kind"] == "one":
        B.madd_step(*s["args"], hp, **s["more"])
    else:
        B.madd_multi_tensor_step(s["tl"], hp, gfmt=s["gfmt"])
    return s["out"]


# ---------------------------------------------------------------------------
# What a pass cannot do without; how exact it is
# ---------------------------------------------------------------------------

def _scale_bytes(fmt, n):
    return {"mxfp4": n / 32, "nvfp4": 4 + n / 16, "nvfp4_current": 4 + n / 16}.get(fmt, n / 64)


def work(case):
    c = case
    if c["kind"] == "toy":
        w, n = CODE[c["weights"]], c["n"]
        # idx; target, c, w read and w written; the gradient and the counts written
        return {"bytes": 8 * c["batch"] + n * (8 + 2 * w + 8), "flops": 16 * n}
    bytes_ = flops = 0.0
    for n, f, blk in _Layout(c).tensors:
        mom = MOMENT[c["moments"]].itemsize
        if c["kind"] == "setup":
            bytes_ += n * (4 + CODE[f] + 3 * mom) + (_scale_bytes(f, n) if blk else 0)
            flops += 4 * n
        else:
            bytes_ += n * (2 * CODE[f] + GRAD[c["grads"]].itemsize + 6 * mom + (2 if blk else 0))
            bytes_ += 2 * _scale_bytes(f, n) if blk else 0
            flops += 40 * n
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    # The step fixes its fp32 operation order and the rounding of every
    # operation, and codes and scales are whole numbers: one right answer.
    return "exact"


def _e2m1(x):
    a = x.abs().clamp(max=6.0)
    step = torch.where(a < 2, 0.5, torch.where(a < 4, 1.0, 2.0))
    return torch.copysign(torch.round(a / step) * step, x)


def _stored(x, fmt, blk):
    """The values that fp32 x has once stored in a format."""
    if fmt == "fp32":
        return x
    if fmt == "bf16":
        return x.bfloat16().float()
    fp8 = {"e4m3": torch.float8_e4m3fn, "e5m2": torch.float8_e5m2}
    top = {"e4m3": 448.0, "e5m2": 57344.0}
    if not blk:
        return x.clamp(-top[fmt], top[fmt]).to(fp8[fmt]).float()
    b = x.view(-1, BLOCK[fmt])
    amax = b.abs().amax(1, keepdim=True)
    if fmt in fp8:
        s = (amax / top[fmt]).half().clamp(min=2.0 ** -24).float()
        s = torch.where(amax == 0, 1.0, s)
        return ((b / s).clamp(-top[fmt], top[fmt]).to(fp8[fmt]).float() * s).view(-1)
    if fmt == "mxfp4":
        s = torch.ldexp(torch.ones_like(amax), torch.frexp(amax)[1] - 3)
        return (_e2m1(b / s) * s).view(-1)
    st = amax.amax() / 2688.0
    den = (amax / (6.0 * st)).clamp(max=448.0).to(torch.float8_e4m3fn).float() * st
    return (_e2m1(torch.where(den == 0, 0.0, b / den)) * den).view(-1)


def exact(case, seed):
    """The pass in 64 bits: unrounded new weights and moments, without draws."""
    c = dict(case)
    if c["kind"] == "toy":
        gen = torch.Generator(device="cuda")
        gen.manual_seed(int(seed) * 1000003 + 29)
        n = c["n"]
        target = torch.randn(n, generator=gen, device="cuda")
        w0 = target + 0.5 * torch.randn(n, generator=gen, device="cuda")
        idx = torch.randint(0, n, (c["batch"],), generator=gen, device="cuda")
        w = _stored(w0, c["weights"], False).double()
        g = 4.0 / c["batch"] * torch.bincount(idx, minlength=n).double() * (w - target.double()) ** 3
        ge = math.log(2) * w * g
        um = (-TOY_HP["lr_mul"] * ge / w.abs().clamp(min=HP["tau"])).clamp(-HP["r_max"], HP["r_max"])
        new = w + w * um - TOY_HP["lr_add"] * g
        return {"w": new if c["weights"] in CODE_DTYPE else None, "g": g, "counts": None}
    if c["kind"] == "setup":
        if c["weights"] not in CODE_DTYPE:
            return None
        gen = torch.Generator(device="cuda")
        gen.manual_seed(int(seed) * 1000003 + 41)
        x = torch.randn(c["n"], generator=gen, device="cuda").mul_(0.02)
        return {"w": x.double(), "scales": None, "mom": None}
    lay = _Layout(c)
    x, g, m, v, ve = _inputs(c, seed, lay)
    t = T0 + 1
    sa = HP["lr_add"] / (1 - HP["beta1"] ** t)
    ibc2 = 1 / (1 - HP["beta2"] ** t)
    b1, b2, eps = HP["beta1"], HP["beta2"], HP["eps"]
    new = torch.zeros(lay.total, dtype=torch.float64, device="cuda")
    M, V, E = (a.double() for a in (m, v, ve))
    for (n, f, blk), o in zip(lay.tensors, lay.at):
        at = slice(o, o + n)
        w, gd = _stored(x[at], f, blk).double(), g[at].double()
        M[at] = b1 * M[at] + (1 - b1) * gd
        V[at] = b2 * V[at] + (1 - b2) * gd * gd
        ge = math.log(2) * w * gd
        E[at] = b2 * E[at] + (1 - b2) * ge * ge
        ua = -sa * M[at] / ((V[at] * ibc2).sqrt() + eps)
        ut = -HP["lr_mul"] * ge / ((E[at] * ibc2).sqrt() + eps)
        um = (ut / w.abs().clamp(min=HP["tau"])).clamp(-HP["r_max"], HP["r_max"])
        new[at] = w + w * um + ua
    out = {"m": M, "v": V, "ve": E}
    fmts = sorted({f for _, f, _ in lay.tensors})
    out["w"] = [new if f in CODE_DTYPE and len(fmts) == 1 else None for f in fmts]
    if c["weights"].endswith("-master"):
        out["copy"] = out["scales"] = None
    if c["weights"].startswith("nvfp4_current"):
        out["new"] = None if len(fmts) > 1 else new
    return out
