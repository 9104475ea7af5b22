"""Performance cases: the work a user of this library has it do, through its public calls.

Kinds of case (a case is a dict of plain values with a "kind"):

  linear   one training step of a quantization-aware linear layer: qlinear_fwd, then
           qlinear_bwd_ste (Y, dX, dW).  M tokens, W [N, K].  wfmt nvfp4 / mxfp4 / q4k, afmt
           none / nvfp4 (running amax updated first) / mxfp4; saved: the forward leaves its
           packed operands for the backward (else the backward quantizes again); keep_ws: the
           workspace survives from forward to backward (QF_FLAG_REUSE_WS).
  forward  one forward call that allocates nothing (qlinear_fwd_noalloc), as a serving or
           evaluation loop makes it.
  grouped  one training step of a mixture-of-experts linear layer: qlinear_grouped_fwd and
           qlinear_grouped_bwd_ste over rows routed with Zipf(1.1) expert popularity.
  lora     one training step of a linear layer with a rank-r adapter on a frozen weight:
           qlinear_lora_fwd and qlinear_lora_bwd_ste (Y, dX, dA, dB).
  kl       the distillation loss of L tokens over a vocabulary of V, with its gradient.
  export   engine-native codes and scales of a fused projection (export_fused), or the Q4_K
           blocks of a weight (fakequant_q4k).

Inputs follow the layers they stand for: weights N(0, 0.02), activations N(0, 1) times a
heavy-tailed per-channel factor, upstream gradients N(0, 1), peaked next-token logits.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2609_39223_amd as qf

DEV = "cuda"


def listed():
    return [
        # One small layer (a test-sized or draft model): launches and latency count.
        dict(name="linear_small_nvfp4", kind="linear", M=256, N=512, K=512, wfmt="nvfp4",
             afmt="none", saved=True, keep_ws=False),
        # A few rows through a 4096-wide projection with quantization simulated on the fly: one
        # decode step of a rollout or evaluation loop that must not allocate.
        dict(name="forward_decode_nvfp4", kind="forward", M=32, N=4096, K=4096, wfmt="nvfp4",
             afmt="none"),
        # The attention output projection of a 9B-class layer on a 2K-token micro-batch.
        dict(name="linear_2k_o_nvfp4", kind="linear", M=2048, N=4096, K=4096, wfmt="nvfp4",
             afmt="none", saved=True, keep_ws=False),
        # The fused QKV projection on packed sequences whose token count is odd.
        dict(name="linear_ragged_qkv_nvfp4", kind="linear", M=1777, N=6144, K=4096, wfmt="nvfp4",
             afmt="none", saved=True, keep_ws=False),
        # The fused gate/up projection of a 9B-class layer on one 32K-token sequence, the
        # workspace kept for the backward: the largest layer call of the main workload.
        dict(name="linear_32k_gate_up_nvfp4", kind="linear", M=32768, N=24576, K=4096,
             wfmt="nvfp4", afmt="none", saved=True, keep_ws=True),
        # An 8B-class MLP up-projection with weights and activations both in MXFP4, 8K tokens.
        dict(name="linear_8k_mlp_up_mxfp4_w4a4", kind="linear", M=8192, N=14336, K=4096,
             wfmt="mxfp4", afmt="mxfp4", saved=True, keep_ws=False),
        # Training towards a llama.cpp checkpoint: a Q4_K weight on 4K tokens.
        dict(name="linear_4k_mlp_up_q4k", kind="linear", M=4096, N=14336, K=4096, wfmt="q4k",
             afmt="none", saved=True, keep_ws=False),
        # 128 experts' down projection, 32K tokens routed to 8 experts each.
        dict(name="moe_32k_down_nvfp4", kind="grouped", E=128, tokens=32768, topk=8, N=3072,
             K=1536, wfmt="nvfp4", afmt="none"),
        # The same experts' fused gate/up projection on a small micro-batch: most experts see
        # fewer than 128 rows, some none.
        dict(name="moe_2k_gate_up_nvfp4", kind="grouped", E=128, tokens=2048, topk=8, N=3072,
             K=3072, wfmt="nvfp4", afmt="none"),
        # Adapter distillation: a rank-16 adapter on a frozen MLP up-projection, 8K tokens.
        dict(name="lora_8k_mlp_up_nvfp4_r16", kind="lora", M=8192, N=14336, K=4096, r=16,
             wfmt="nvfp4", afmt="none"),
        # The distillation loss and its gradient over a 152K-token vocabulary.
        dict(name="kl_4k_v152k", kind="kl", L=4096, V=151936),
        # Weight sync: the fused QKV projection's NVFP4 codes and scales (tied tensor scale).
        dict(name="export_qkv_nvfp4", kind="export", rows="4096,1024,1024", K=4096, fmt="nvfp4"),
    ]


_MAX_FLOPS = 6.0 * 32768 * 24576 * 4096
_NOALLOC_BYTES = 64 << 20


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi, step):
    return max(step, _log(rng, lo, hi) // step * step)


def _kstep(wfmt, rng):
    # mostly multiples of the GEMM's usual depths, sometimes just of the format's own block
    block = {"nvfp4": 16, "mxfp4": 32, "q4k": 256}[wfmt]
    return max(block, rng.choice([256, 128, 64, 32, 16]))


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "forward", "grouped", "grouped", "lora", "kl",
                       "export"])
    while True:
        if kind == "linear":
            wfmt, afmt = rng.choice([("nvfp4", "none"), ("nvfp4", "none"), ("mxfp4", "none"),
                                     ("q4k", "none"), ("nvfp4", "nvfp4"), ("mxfp4", "mxfp4")])
            step = max(_kstep(wfmt, rng), 32 if afmt == "mxfp4" else 16)
            c = dict(kind=kind, M=_log(rng, 16, 32768), N=_width(rng, 512, 24576, rng.choice([8, 64, 256])),
                     K=_width(rng, 512, 14336, step), wfmt=wfmt, afmt=afmt,
                     saved=rng.random() < 0.75, keep_ws=rng.random() < 0.3)
        elif kind == "forward":
            wfmt = rng.choice(["nvfp4", "mxfp4", "q4k"])
            c = dict(kind=kind, M=_log(rng, 1, 1024), N=_width(rng, 256, 8192, rng.choice([8, 64, 256])),
                     K=_width(rng, 512, 8192, _kstep(wfmt, rng)), wfmt=wfmt,
                     afmt="mxfp4" if wfmt == "mxfp4" and rng.random() < 0.5 else "none")
            if 2 * c["K"] * (c["N"] + c["M"]) + 1024 > _NOALLOC_BYTES:
                continue
        elif kind == "grouped":
            wfmt = rng.choice(["nvfp4", "nvfp4", "mxfp4", "q4k"])
            c = dict(kind=kind, E=rng.choice([8, 16, 32, 64, 128]), tokens=_log(rng, 128, 32768),
                     topk=rng.choice([2, 4, 8]), N=_width(rng, 768, 3072, 64),
                     K=_width(rng, 768, 3072, _kstep(wfmt, rng)), wfmt=wfmt,
                     afmt="mxfp4" if wfmt == "mxfp4" and rng.random() < 0.5 else "none")
            if c["afmt"] == "mxfp4" and c["K"] % 32:
                continue
        elif kind == "lora":
            wfmt = rng.choice(["nvfp4", "mxfp4"])
            c = dict(kind=kind, M=_log(rng, 256, 8192), N=_width(rng, 1024, 14336, 64),
                     K=_width(rng, 1024, 8192, 64), r=rng.choice([4, 16, 24, 64]), wfmt=wfmt,
                     afmt="mxfp4" if wfmt == "mxfp4" and rng.random() < 0.5 else "none")
        elif kind == "kl":
            c = dict(kind=kind, L=_log(rng, 64, 8192), V=_width(rng, 32000, 151936, 8))
        else:
            fmt = rng.choice(["nvfp4", "mxfp4", "q4k"])
            rows = [_width(rng, 512, 12288, 64) for _ in range(rng.choice([1, 2, 3]) if fmt != "q4k" else 1)]
            c = dict(kind=kind, rows=",".join(map(str, rows)), K=_width(rng, 1024, 12288, 256), fmt=fmt)
        if work(c)["flops"] <= _MAX_FLOPS:
            return c


# ---------------------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) % (1 << 62))
    return g


def _normal(g, shape, std=1.0, cols=None, rows=None):
    z = torch.randn(shape, generator=g, device=DEV)
    if std != 1.0:
        z.mul_(std)
    if cols is not None:
        z.mul_(cols[None, :])
    if rows is not None:
        z.mul_(rows[:, None])
    return z.to(torch.bfloat16)


def _acts(g, M, K):
    # per-channel magnitudes |Student-t(3)|: a few channels are many times the typical one
    z = torch.randn(4, K, generator=g, device=DEV)
    tau = (z[0] / (z[1:].square().sum(0) / 3).sqrt()).abs()
    return _normal(g, (M, K), cols=tau)


def _weight(g, N, K, wfmt):
    rows = None
    if wfmt == "q4k":      # rows of different magnitude
        rows = torch.exp(0.5 * torch.randn(N, generator=g, device=DEV))
    return _normal(g, (N, K), 0.02, rows=rows)


def _routing(g, tokens, E, topk):
    """Offsets [E+1] of the rows sorted by expert: Gumbel-top-k over Zipf(1.1) popularity."""
    rank = torch.randperm(E, generator=g, device=DEV).double() + 1
    gum = -torch.log(-torch.log(torch.rand(tokens, E, generator=g, device=DEV).double().clamp(1e-12, 1 - 1e-12)))
    choice = (gum - 1.1 * torch.log(rank)[None, :]).topk(min(topk, E), dim=1).indices
    counts = torch.bincount(choice.reshape(-1), minlength=E)
    off = torch.zeros(E + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(counts, 0)
    return off


def _inputs(case, seed):
    g = _gen(seed)
    k = case["kind"]
    if k in ("linear", "forward", "lora"):
        M, N, K = case["M"], case["N"], case["K"]
        out = {"X": _acts(g, M, K), "W": _weight(g, N, K, case["wfmt"])}
        if k != "forward":
            out["dY"] = _normal(g, (M, N))
        if k == "lora":
            r = case["r"]
            out["A"] = torch.randn(r, K, generator=g, device=DEV) / math.sqrt(K)
            out["B"] = torch.randn(N, r, generator=g, device=DEV) * (0.001 * math.sqrt(K / r))
        return out
    if k == "grouped":
        E, N, K = case["E"], case["N"], case["K"]
        off = _routing(g, case["tokens"], E, case["topk"])
        T = case["tokens"] * min(case["topk"], E)
        return {"off": off, "X": _normal(g, (T, K)), "W": _weight(g, E * N, K, case["wfmt"]),
                "dY": _normal(g, (T, N))}
    if k == "kl":
        L, V = case["L"], case["V"]
        t = torch.randn(L, V, generator=g, device=DEV) * 2
        hot = torch.randint(0, V, (L, 3), generator=g, device=DEV)
        t.scatter_add_(1, hot, torch.rand(L, 3, generator=g, device=DEV) * 8 + 6)
        zt = t.to(torch.bfloat16)
        t += torch.randn(L, V, generator=g, device=DEV) * 0.5
        return {"zt": zt, "zs": t.to(torch.bfloat16)}
    return {"members": [_weight(g, n, case["K"], case["fmt"]) for n in _rows_of(case)]}


def _rows_of(case):
    return [int(v) for v in case["rows"].split(",")]


def _empty(shape, dtype):
    return torch.empty(shape, dtype=dtype, device=DEV)


def prepare(case, seed):
    s = _inputs(case, seed)
    s["kind"] = k = case["kind"]
    bf, f32 = torch.bfloat16, torch.float32
    if k == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        s["a_amax"] = torch.zeros(1, dtype=f32, device=DEV) if case["afmt"] == "nvfp4" else None
        s["d"] = qf.qlinear_desc(M, N, K, case["wfmt"], case["afmt"], a_amax=s["a_amax"],
                                 flags=qf.FLAG_REUSE_WS if case["keep_ws"] else 0)
        s["ws"] = qf.workspace(s["d"])
        s["saved"] = qf.saved_buffer(s["d"]) if case["saved"] else None
        s["Y"], s["dX"], s["dW"] = _empty((M, N), bf), _empty((M, K), bf), _empty((N, K), f32)
    elif k == "forward":
        s["d"] = qf.qlinear_desc(case["M"], case["N"], case["K"], case["wfmt"], case["afmt"])
        s["Y"] = _empty((case["M"], case["N"]), bf)
    elif k == "grouped":
        E, N, K, T = case["E"], case["N"], case["K"], s["X"].shape[0]
        s["d"] = qf.grouped_desc(E, T, N, K, case["wfmt"], case["afmt"])
        s["ws"], s["saved"] = qf.grouped_workspace(s["d"]), qf.grouped_saved_buffer(s["d"])
        s["Y"], s["dX"], s["dW"] = _empty((T, N), bf), _empty((T, K), bf), _empty((E, N, K), f32)
    elif k == "lora":
        M, N, K, r = case["M"], case["N"], case["K"], case["r"]
        s["lo"] = qf.lora(s["A"], s["B"], 2.0)
        s["d"] = qf.qlinear_desc(M, N, K, case["wfmt"], case["afmt"])
        s["ws"] = qf.lora_workspace(s["d"], s["lo"])
        s["Y"], s["dX"] = _empty((M, N), bf), _empty((M, K), bf)
        s["dA"], s["dB"] = _empty((r, K), f32), _empty((N, r), f32)
    elif k == "kl":
        L, V = case["L"], case["V"]
        s["kl"], s["loss"], s["agree"] = _empty(L, f32), _empty(1, f32), _empty(L, torch.int32)
        s["grad"] = _empty((L, V), bf)
    else:
        N, K, fmt = sum(_rows_of(case)), case["K"], case["fmt"]
        s["fmt"] = fmt
        if fmt == "q4k":
            s["packed"] = _empty((N, K // 256, 144), torch.uint8)
        else:
            s["codes"] = _empty((N, K // 2), torch.uint8)
            s["scales"] = _empty((N, K // (16 if fmt == "nvfp4" else 32)), torch.uint8)
            s["amax"], s["scale2"] = _empty(1, f32), _empty(1, f32)
    return s


# ------------------------------------------------------------------------------------- runs
def run(s):
    k = s["kind"]
    if k == "linear":
        out = {"Y": s["Y"], "dX": s["dX"], "dW": s["dW"]}
        if s["a_amax"] is not None:
            qf.amax(s["X"], s["a_amax"], accumulate=True)
            out["a_amax"] = s["a_amax"]
        qf.qlinear_fwd(s["d"], s["X"], s["W"], s["Y"], s["ws"], saved=s["saved"])
        qf.qlinear_bwd_ste(s["d"], s["dY"], s["X"], s["W"], s["dX"], s["dW"], s["ws"],
                           saved=s["saved"])
        return out
    if k == "forward":
        return {"Y": qf.qlinear_fwd_noalloc(s["d"], s["X"], s["W"], s["Y"])}
    if k == "grouped":
        qf.qlinear_grouped_fwd(s["d"], s["off"], s["X"], s["W"], s["Y"], s["ws"], saved=s["saved"])
        qf.qlinear_grouped_bwd_ste(s["d"], s["off"], s["dY"], s["X"], s["W"], s["dX"], s["dW"],
                                   s["ws"], saved=s["saved"])
        return {"Y": s["Y"], "dX": s["dX"], "dW": s["dW"]}
    if k == "lora":
        qf.qlinear_lora_fwd(s["d"], s["lo"], s["X"], s["W"], s["Y"], s["ws"])
        qf.qlinear_lora_bwd_ste(s["d"], s["lo"], s["dY"], s["X"], s["W"], s["dX"], s["dA"],
                                s["dB"], s["ws"])
        return {"Y": s["Y"], "dX": s["dX"], "dA": s["dA"], "dB": s["dB"]}
    if k == "kl":
        qf.qad_kl(s["zt"], s["zs"], s["kl"], loss=s["loss"], grad=s["grad"], agree=s["agree"])
        return {"kl": s["kl"], "loss": s["loss"], "grad": s["grad"], "agree": s["agree"]}
    if s["fmt"] == "q4k":
        qf.fakequant_q4k(s["members"][0], s["packed"], None)
        return {"packed": s["packed"]}
    nv = s["fmt"] == "nvfp4"
    qf.export_fused(s["members"], s["fmt"], s["codes"], s["scales"],
                    w_amax=s["amax"] if nv else None, weight_scale_2=s["scale2"] if nv else None)
    out = {"codes": s["codes"], "scales": s["scales"]}
    if nv:
        out.update(amax=s["amax"], scale2=s["scale2"])
    return out


def work(case):
    k = case["kind"]
    if k in ("linear", "forward", "lora"):
        M, N, K = case["M"], case["N"], case["K"]
        gemm = 2.0 * M * N * K
        fwd = 2 * (M * K + N * K + M * N)
        if k == "forward":
            return {"bytes": fwd, "flops": gemm}
        if k == "linear":
            return {"bytes": fwd + 2 * (M * N + M * K) + 4 * N * K, "flops": 3 * gemm}
        r = case["r"]
        return {"bytes": fwd + 2 * (M * N + M * K) + 2 * 4 * r * (N + K),
                "flops": 2 * gemm + 2.0 * r * (N * K + 2 * M * K + 2 * M * N)}
    if k == "grouped":
        E, N, K, T = case["E"], case["N"], case["K"], case["tokens"] * min(case["topk"], case["E"])
        return {"bytes": 2 * (2 * T * K + 2 * T * N + E * N * K) + 4 * E * N * K,
                "flops": 6.0 * T * N * K}
    if k == "kl":
        n = case["L"] * case["V"]
        return {"bytes": 6 * n, "flops": 12.0 * n}
    n = sum(_rows_of(case)) * case["K"]
    out = {"nvfp4": 0.5 + 1 / 16, "mxfp4": 0.5 + 1 / 32, "q4k": 144 / 256}[case["fmt"]]
    return {"bytes": int(n * (2 + out)), "flops": 8.0 * n}


def tolerance(case):
    """bf16 results carry a rounding of up to 2^-9 relative each (1.66e-3 over a whole output,
    measured against exact()); codes, scales and scalars of an export are whole values."""
    if case["kind"] == "export":
        return "exact"
    if case["kind"] == "kl":
        # the agreement flags are whole values; the gradient is the bf16 output
        return {"rel": 7e-3, "max": 2e-2, "differ": 0.0}
    return {"rel": 7e-3, "max": 2e-2}


# ---------------------------------------------------------- the same results in 64 bits
# Scale and code decisions are the formats' own 32-bit steps (a code is a whole number, not a
# rounded one); everything that is summed is summed in float64.  Divisions use device scalars:
# a division by a Python number may be evaluated as a multiplication by its reciprocal.
def _c(v):
    return torch.tensor(v, dtype=torch.float32, device=DEV)


def _e2m1(u):
    """Code 0..7 of the nearest E2M1 magnitude to u >= 0, ties to the even code."""
    m = (u > 0.25).to(torch.uint8)
    for t, tie in ((0.75, 1), (1.25, 0), (1.75, 1), (2.5, 0), (3.5, 1), (5.0, 0)):
        m += (u >= t) if tie else (u > t)
    return m


def _e2m1_value(m):
    return torch.tensor([0, 0.5, 1, 1.5, 2, 3, 4, 6], device=DEV)[m.long()]


def _nibbles(code):
    return code[:, 0::2] | (code[:, 1::2] << 4)


def _nvfp4(x, g=None):
    R, K = x.shape
    x = x.float()
    g = x.abs().max() if g is None else g.reshape(())
    S = g / _c(2688.0)
    b = x.view(R, K // 16, 16)
    t = (b.abs().amax(-1) / (_c(6.0) * S)).clamp(max=448.0)
    sb = torch.where(S == 0, torch.zeros_like(t), t).to(torch.float8_e4m3fn)
    D = S * sb.float()
    r = torch.where(D != 0, _c(1.0) / D, torch.zeros_like(D))
    m = _e2m1((b.abs() * r[..., None]).nan_to_num(0.0))
    xh = torch.copysign(_e2m1_value(m) * D[..., None], b).to(torch.bfloat16).view(R, K)
    codes = _nibbles((m | (torch.signbit(b).to(torch.uint8) << 3)).view(R, K))
    return xh, codes, sb.view(torch.uint8), g, S


def _mxfp4(x):
    R, K = x.shape
    b = x.float().view(R, K // 32, 32)
    a = b.abs().amax(-1)
    p = torch.where(a == 0, torch.full_like(a, -127).int(), (torch.frexp(a).exponent - 3).clamp(-127, 127))
    sc = torch.ldexp(torch.ones_like(a, dtype=torch.float64), p)
    m = _e2m1(b.abs().double() / sc[..., None])
    xh = torch.copysign(_e2m1_value(m) * sc[..., None], b.double()).to(torch.bfloat16).view(R, K)
    codes = _nibbles((m | (torch.signbit(b).to(torch.uint8) << 3)).view(R, K))
    return xh, codes, (p + 127).to(torch.uint8)


def _q4k(x):
    """x_hat and the packed 144-byte blocks."""
    R, K = x.shape
    b = x.float().view(R, K // 256, 8, 32) + 0.0
    lo, hi = b.amin(-1).clamp(max=0.0), b.amax(-1)
    a, mu = (hi - lo) / _c(15.0), _c(0.0) - lo
    dh = (a.amax(-1) / _c(63.0)).clamp(max=65504.0).half()
    mh = (mu.amax(-1) / _c(63.0)).clamp(max=65504.0).half()
    d, dm = dh.float()[..., None], mh.float()[..., None]
    ls = torch.where(d != 0, torch.round(a / d).clamp(0, 63), torch.zeros_like(a))
    lm = torch.where(dm != 0, torch.round(mu / dm).clamp(0, 63), torch.zeros_like(mu))
    t1, t2 = (d * ls)[..., None], (dm * lm)[..., None]
    q = torch.where(t1 != 0, torch.round((b + t2) / t1).clamp(0, 15), torch.zeros_like(b))
    xh = (t1 * q - t2).to(torch.bfloat16).view(R, K)
    ls, lm, q = ls.to(torch.uint8), lm.to(torch.uint8), q.to(torch.uint8)
    hd = torch.stack([dh, mh], -1).view(torch.uint8).view(R, K // 256, 4)
    sc = torch.cat([ls[..., :4] | ((ls[..., 4:] >> 4) << 6), lm[..., :4] | ((lm[..., 4:] >> 4) << 6),
                    (ls[..., 4:] & 15) | ((lm[..., 4:] & 15) << 4)], -1)
    qs = (q[:, :, 0::2] | (q[:, :, 1::2] << 4)).reshape(R, K // 256, 128)
    return xh, torch.cat([hd, sc, qs], -1)


def _hat(x, fmt, g=None):
    if fmt == "none":
        return x
    if fmt == "nvfp4":
        return _nvfp4(x, g)[0]
    return (_mxfp4 if fmt == "mxfp4" else _q4k)(x)[0]


def _merged(W, A, B, scale):
    """bf16(W + scale B A), the sum over the rank in rising order in 32 bits."""
    acc = torch.zeros_like(W, dtype=torch.float32)
    for j in range(A.shape[0]):
        acc = (acc.double() + B[:, j:j + 1].double() * A[j:j + 1].double()).float()
    return (W.float() + _c(scale) * acc).to(torch.bfloat16)


def exact(case, seed):
    s = _inputs(case, seed)
    k = case["kind"]
    if k in ("linear", "forward", "lora"):
        W = s["W"] if k != "lora" else _merged(s["W"], s["A"], s["B"], 2.0)
        Wh = _hat(W, case["wfmt"]).double()
        g = s["X"].float().abs().max() if case["afmt"] == "nvfp4" else None
        Xh = _hat(s["X"], case["afmt"], g).double()
        out = {"Y": Xh @ Wh.t()}
        if k == "forward":
            return out
        dY = s["dY"].double()
        out["dX"] = dY @ Wh
        del Wh
        dW = dY.t() @ Xh
        if k == "lora":
            out["dA"] = 2.0 * (s["B"].double().t() @ dW)
            out["dB"] = 2.0 * (dW @ s["A"].double().t())
            return out
        out["dW"] = dW
        if g is not None:
            out["a_amax"] = g.double().reshape(1)
        return out
    if k == "grouped":
        E, N, K = case["E"], case["N"], case["K"]
        X, dY, T = _hat(s["X"], case["afmt"]), s["dY"], s["X"].shape[0]
        out = {"Y": _empty((T, N), torch.float64), "dX": _empty((T, K), torch.float64),
               "dW": torch.zeros((E, N, K), dtype=torch.float64, device=DEV)}
        off = s["off"].tolist()
        for e in range(E):
            a, b = off[e], off[e + 1]
            if a == b:
                continue
            Wh = _hat(s["W"][e * N:(e + 1) * N], case["wfmt"]).double()
            x, dy = X[a:b].double(), dY[a:b].double()
            out["Y"][a:b] = x @ Wh.t()
            out["dX"][a:b] = dy @ Wh
            out["dW"][e] = dy.t() @ x
        return out
    if k == "kl":
        L, V = case["L"], case["V"]
        kl, grad = _empty(L, torch.float64), _empty((L, V), torch.float64)
        agree = _empty(L, torch.int32)
        idx = torch.arange(V, device=DEV)
        for r in range(0, L, 512):
            t, z = s["zt"][r:r + 512].double(), s["zs"][r:r + 512].double()
            lt, lz = t.log_softmax(-1), z.log_softmax(-1)
            p = lt.exp()
            kl[r:r + 512] = (p * (lt - lz)).sum(-1)
            grad[r:r + 512] = (lz.exp() - p) / L
            first = [torch.where(v == v.amax(-1, keepdim=True), idx, V).amin(-1) for v in (t, z)]
            agree[r:r + 512] = (first[0] == first[1]).int()
        return {"kl": kl, "loss": kl.mean().reshape(1), "grad": grad, "agree": agree}
    W = torch.cat(s["members"])
    if case["fmt"] == "q4k":
        return {"packed": _q4k(W)[1]}
    if case["fmt"] == "mxfp4":
        _, codes, scales = _mxfp4(W)
        return {"codes": codes, "scales": scales}
    _, codes, scales, g, S = _nvfp4(W)
    return {"codes": codes, "scales": scales, "amax": g.double().reshape(1), "scale2": S.double().reshape(1)}
