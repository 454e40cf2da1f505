"""What the Hadamard Linear Attention operator is used for, as a list of cases to time: each is one
pass through the public binding (`paper_2602_12128_amd`), a forward or a forward and a backward, with
the inputs and the handle a user's program has at hand.

Sizes are those of the repository's own configurations (`workloads.py`: the paper's video-DiT token
counts, 12 heads of 128 channels), of its tests, or generic; values follow the recipes of the same
file.  `listed` names the cases, `draw` makes more of the same ranges.
"""
from __future__ import annotations

import math

import torch

import paper_2602_12128_amd as hla
from paper_2602_12128_amd import workloads as wl

EPS = 1e-6

# Plain description of a case; every field has a value in every case.
#   dtype       "bf16" (matrix-core kernels for d = 64, 128) or "fp32"
#   B, H, N, d  batch rows, heads, tokens per batch row, head dim
#   lens        "" for a dense batch, else the packed sequences' lengths, comma separated (their sum is N)
#   F, d_phi    Hadamard degree and feature count: (3, 6) or (2, 12), the paper's two forms
#   features    Q and K are already feature-mapped (no feature-map weights)
#   static      hla_forward_static instead of a handle (features, forward only)
#   backward    forward + backward; weight_grads: with the gradients of every registered weight
#   vmod        value modulation; causal, decay: the causal variant
#   values      how the vectors of Q, K, V are drawn: "gauss" or "unit" (each vector of unit norm), "lowrank" (unit, tokens correlated)
_BASE = dict(dtype="bf16", B=1, H=12, N=4096, d=128, lens="", F=3, d_phi=6, features=False, static=False,
             backward=True, weight_grads=False, vmod=False, causal=False, decay=1.0, values="unit")


def _case(**kw):
    return {**_BASE, **kw}


def listed():
    return [
        # smallest fp32 call: a check of a few hundred tokens, all latency
        _case(name="tiny_fp32_fwd", dtype="fp32", H=2, N=256, d=32, backward=False, values="gauss"),
        # one latent frame (30 x 52 patches) of a 480p video: inference on a single image, launches count
        _case(name="frame_fwd", N=1560, backward=False),
        # features computed by the caller, no handle: a serving loop that may not allocate (ragged token count)
        _case(name="features_static_fwd", N=8190, features=True, static=True, backward=False),
        # training in full precision, weights included
        _case(name="fp32_d64_train", dtype="fp32", N=4095, d=64, weight_grads=True, values="gauss"),
        # mid-size batch with 64-channel heads
        _case(name="mid_d64_fwdbwd", B=2, N=4096, d=64, values="gauss"),
        # training step at the lower video resolution, feature-map weights included
        _case(name="dit320p_train", N=12600, weight_grads=True),
        # the headline step: 480p video, gradients of the inputs
        _case(name="dit480p_fwdbwd", N=32760),
        # the two-factor form at the same shape
        _case(name="dit480p_2factor_fwdbwd", N=32760, F=2, d_phi=12),
        # training step with the value modulation: every weight's gradient
        _case(name="dit480p_vmod_train", N=32760, vmod=True, weight_grads=True),
        # causal variant with a decay factor
        _case(name="dit480p_causal_fwdbwd", N=32760, causal=True, decay=0.99),
        # sequences of different lengths packed into one call
        _case(name="packed_fwdbwd", N=90090, lens="8190,16380,32760,32760", values="gauss"),
        # inference on 720p video with the wide model's 40 heads
        _case(name="dit720p_fwd", H=40, N=75600, backward=False, values="lowrank"),
    ]


def _log(rng, lo, hi):
    """An integer of [lo, hi], evenly spread over its logarithm (odd ones included)."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["fp32_fwd", "fp32_train", "fwd", "static", "fwdbwd", "train", "packed", "vmod", "causal"])
    form = rng.choice([dict(F=3, d_phi=6), dict(F=3, d_phi=6), dict(F=2, d_phi=12)])
    d = rng.choice([64, 128, 128])
    values = rng.choice(["gauss", "unit"])
    if kind == "fp32_fwd":
        return _case(dtype="fp32", H=rng.choice([1, 2, 5, 12]), N=_log(rng, 200, 8190), d=rng.choice([32, 64, 128]),
                     backward=False, values=values, **form)
    if kind == "fp32_train":
        return _case(dtype="fp32", H=rng.choice([1, 2, 4]), N=_log(rng, 200, 6000), d=rng.choice([32, 64, 128]),
                     weight_grads=rng.random() < 0.5, values=values, **form)
    if kind == "fwd":
        return _case(B=1, H=rng.choice([1, 8, 12, 16, 40]), N=_log(rng, 256, 75600), d=d, backward=False,
                     values=rng.choice(["gauss", "unit", "lowrank"]), **form)
    if kind == "static":
        return _case(B=rng.choice([1, 2]), H=rng.choice([1, 3, 8, 12]), N=_log(rng, 256, 7000), d=d, features=True,
                     static=True, backward=False, **form)
    N = _log(rng, 700, 32760)
    H = rng.choice([3, 8, 12])
    B = rng.choice([1, 1, 2]) if N < 8000 else 1
    if kind == "packed":
        lens = [_log(rng, 300, 16380) for _ in range(rng.randint(2, 5))]
        return _case(H=H, N=sum(lens), lens=",".join(str(n) for n in lens), d=d, values=values, **form)
    if kind == "vmod":
        return _case(B=B, H=H, N=N, d=d, vmod=True, weight_grads=rng.random() < 0.5, values=values, **form)
    if kind == "causal":
        return _case(B=B, H=H, N=N, d=d, causal=True, decay=rng.choice([1.0, 0.99, 0.999]), values=values, **form)
    return _case(B=B, H=H, N=N, d=d, weight_grads=kind == "train", values=values, **form)


def _draw_values(case, gen, shape, dtype):
    x = torch.randn(shape, generator=gen, device="cuda")
    d = shape[-1]
    if case["values"] == "gauss":
        return (x / math.sqrt(d)).to(dtype)
    if case["values"] == "lowrank":  # rank 16 shared by the tokens of a head, amplitude 0.5
        basis = torch.randn((*shape[:2], 16, d), generator=gen, device="cuda")
        coef = torch.randn((*shape[:3], 16), generator=gen, device="cuda") / 4.0
        for h in range(shape[1]):
            x[0, h].addmm_(coef[0, h], basis[0, h], alpha=0.5)
    x /= x.square().sum(dim=-1, keepdim=True).sqrt()
    return x.to(dtype)


def prepare(case, seed):
    """Inputs, weights, output buffers and the handle of one case."""
    dtype = torch.float32 if case["dtype"] == "fp32" else torch.bfloat16
    io = hla.HLA_F32 if case["dtype"] == "fp32" else hla.HLA_BF16
    B, H, N, d, F, d_phi = (case[k] for k in ("B", "H", "N", "d", "F", "d_phi"))
    gen = torch.Generator("cuda").manual_seed(seed)
    cpu_gen = torch.Generator("cpu").manual_seed(seed)
    shape = (B, H, N, d)
    t = {}
    if case["features"]:
        t["Q"] = torch.randn((B, H, N, d_phi), generator=gen, device="cuda").abs().to(dtype)
        t["K"] = torch.randn((B, H, N, F * d_phi), generator=gen, device="cuda").abs().to(dtype)
        t["V"] = torch.randn(shape, generator=gen, device="cuda").to(dtype)
    else:
        for k in ("Q", "K", "V"):
            t[k] = _draw_values(case, gen, shape, dtype)
    t["O"] = torch.empty_like(t["V"])
    if case["backward"]:
        t["dO"] = torch.randn(shape, generator=gen, device="cuda").to(dtype)
        for k in ("Q", "K", "V"):
            t["d" + k] = torch.empty_like(t[k])
    state = {"case": case, "t": t, "io": io, "cu": None, "wgrads": [], "op": None}
    if case["static"]:
        return state
    cu = None
    if case["lens"]:
        cu = [0]
        for n in case["lens"].split(","):
            cu.append(cu[-1] + int(n))
    op = hla.HLA(head_dim=d, feature_dim=d_phi, degree=F, eps=EPS, io_dtype=io,
                 phi_mode=hla.HLA_PHI_NONE if case["features"] else hla.HLA_PHI_MLP, max_heads=H,
                 max_tokens=B * N, max_seqs=B if cu is None else len(cu) - 1, causal=case["causal"],
                 decay=case["decay"])
    phi = wl.draw_phi_weights(cpu_gen, d, d_phi, 1 + F, dtype)
    op.set_phi_weights([{k: v.cuda() for k, v in m.items()} for m in phi])
    wgrads = []
    if case["weight_grads"]:
        wgrads += [{"d" + k: torch.empty(v.shape, device="cuda") for k, v in m.items()} for m in phi]
        op.set_phi_weight_grads(wgrads)
    if case["vmod"]:
        vm = wl.draw_vmod_weights(cpu_gen, d, dtype)
        op.set_value_modulation([{k: v.cuda() for k, v in m.items()} for m in vm])
        if case["weight_grads"]:
            vg = [{"d" + k: torch.empty(v.shape, device="cuda") for k, v in m.items()} for m in vm]
            op.set_value_modulation_grads(vg)
            wgrads += vg
    state.update(op=op, cu=cu, wgrads=wgrads)
    return state


def run(state):
    """One forward, or one forward and its backward."""
    t, op = state["t"], state["op"]
    if op is None:
        case = state["case"]
        hla.hla_forward_static(t["Q"], t["K"], t["V"], t["O"], feature_dim=case["d_phi"], degree=case["F"],
                               eps=EPS, io_dtype=state["io"])
        return t["O"]
    op.forward(t["Q"], t["K"], t["V"], t["O"], cu_seqlens=state["cu"])
    if "dO" not in t:
        return t["O"]
    op.backward(t["Q"], t["K"], t["V"], t["O"], t["dO"], t["dQ"], t["dK"], t["dV"], cu_seqlens=state["cu"])
    return {"O": t["O"], "dQ": t["dQ"], "dK": t["dK"], "dV": t["dV"], "weights": state["wgrads"]}


def work(case):
    """Bytes: the operator's inputs read once and its outputs written once.  Operations (2 per
    multiply-add): the feature maps' layers, the contractions over the distinct monomials of the
    symmetric state (C(d_phi + F - 1, F) of them) with d channels and the normaliser, and the
    modulation's layers; a backward costs the two products of every forward product, less those
    for weight gradients that are not asked for; nothing is counted twice for being recomputed."""
    d, F, d_phi = case["d"], case["F"], case["d_phi"]
    th = case["B"] * case["H"] * case["N"]
    elem = 4 if case["dtype"] == "fp32" else 2
    qk = (1 + F) * d_phi if case["features"] else 2 * d
    nbytes = th * elem * (qk + 2 * d)
    phi = 0 if case["features"] else (1 + F) * 2 * d * (d + d_phi)
    core = 2 * 2 * math.comb(d_phi + F - 1, F) * (d + 1)
    vmod = 2 * 2 * 2 * d * d if case["vmod"] else 0
    flops = phi + core + vmod
    if case["backward"]:
        nbytes += th * elem * (qk + 2 * d)  # dO in; dQ, dK, dV out
        flops += phi + 2 * core + vmod + (phi + vmod if case["weight_grads"] else 0)
    return {"bytes": nbytes, "flops": th * flops}


def tolerance(case):
    """Measured against the same operator in 64-bit arithmetic (2-norm of the difference over that
    of the result, worst output of several seeds): fp32 O, dV 4e-7, dQ 2e-6, weight gradients 8e-6
    (bias gradients are sums of random-sign terms).  bf16 O 1.8e-3 (modulated 3e-3), dV 2-4e-3, dK
    4e-3 and dQ 1e-2 on the tokens whose ReLUs have a clear sign; a feature whose pre-activation lies
    within rounding of zero may take either branch, which moves single rows of dQ and dK by their
    own size and the 2-norms to 1-2e-2."""
    if case["dtype"] == "fp32":
        return {"rel": 3e-5}
    if case["backward"]:
        return {"rel": 2e-2, "max": 1.0}
    return {"rel": 7e-3, "max": 0.1}
