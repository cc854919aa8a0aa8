"""The work that programs have this library do, as cases that can be timed and compared.

A case is one call (or one whole optimizer step) of 1.5-SPSA over a model's weights: the perturb
theta + eps z_k, the transition from one probe to the next (two probes in one pass), the
update theta - lr sum_k c_k z_k with or without the last restore merged in, over one flat buffer,
over a shard of one, or over a list of separate tensors. Model shapes are those of
`workloads`; weights and losses are synthetic, as everywhere in this repository.

Fields of a case:
  op       "perturb", "transition", "update", "update_restore" or "step" (Algorithm 1 on one
           device in 2K + 1 sweeps: +eps, -2 eps, transitions, the update with the last restore)
  dtype    "bf16" or "f32"
  n        weights the call covers
  K        probes per step (for a perturb or transition: the step it belongs to)
  offset   global index of the first weight (a shard of a larger model)
  layout   "flat" or "tensors" (separate tensors, each with its global offset)
  model    name of the workload whose tensor list is used ("tensors" only; "" for a ragged list)
  tensors  number of tensors of a ragged list ("tensors" only)
"""

import math
import random

import numpy as np
import torch

import paper_2609_38095_amd as zo
import workloads

EPS = 1e-3
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
SEGMENT_ALIGN = 512  # bytes between the starts of separate tensors, as torch's allocator rounds


def _case(op, dtype, n, K, offset=0, layout="flat", model="", tensors=0):
    return {"op": op, "dtype": dtype, "n": n, "K": K, "offset": offset, "layout": layout, "model": model,
            "tensors": tensors}


def listed():
    W = workloads.WORKLOADS
    n13, n30 = W["opt13b"].n, W["opt30b"].n
    n1, n125 = W["opt1.3b"].n, W["opt125m"].n
    third = -(-n1 // 3)
    named = {
        # a whole step of a small model: nine short launches and the coefficients, bound by latency
        "tiny_step": _case("step", "f32", W["tiny"].n, 4),
        # a small model kept as separate tensors (196 of them): the pass between two probes
        "opt125m_tensors_transition": _case("transition", "bf16", n125, 16, layout="tensors", model="opt125m"),
        # the same model as one flat buffer: the update that ends a step
        "opt125m_update_k16": _case("update", "bf16", n125, 16),
        # a mid-sized model in 32-bit weights: the most frequent call, and its update
        "opt1.3b_f32_perturb": _case("perturb", "f32", n1, 32),
        "opt1.3b_f32_update_k32": _case("update", "f32", n1, 32),
        # many probes per step: 64, and 96 as in the paper's timing table
        "opt1.3b_update_k64": _case("update", "bf16", n1, 64),
        "opt1.3b_update_k96": _case("update", "bf16", n1, 96),
        # the paper's Qwen3 runs (60 probes) with the model as separate tensors, last restore merged in
        "qwen3_1.7b_tensors_update_k60": _case("update_restore", "bf16", W["qwen3-1.7b"].n, 60, layout="tensors",
                                               model="qwen3-1.7b"),
        # the second of three uneven shards, which starts at an odd global index
        "opt1.3b_odd_shard_update_k16": _case("update", "bf16", min(third, n1 - third), 16, offset=third),
        # the headline model: the perturb a step makes most of, and its update with the last restore
        "opt13b_perturb": _case("perturb", "bf16", n13, 16),
        "opt13b_update_k16": _case("update_restore", "bf16", n13, 16),
        # one of eight equal shards of the largest model, 32 probes
        "opt30b_shard_update_k32": _case("update", "bf16", n30 // 8, 32, offset=3 * (n30 // 8)),
    }
    return [dict(c, name=name) for name, c in named.items()]


def draw(rng):
    """One more case: any operation, 2^18 to 2^31 weights, 1 to 128 probes, whole buffers, shards at even
    and odd indices, and lists of 2 to 300 ragged tensors."""
    op = rng.choice(["perturb", "transition", "update", "update", "update_restore", "update_restore", "step"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    layout = rng.choice(["flat", "flat", "tensors"])
    place = rng.choice(["whole", "whole", "shard", "odd"]) if layout == "flat" else "whole"
    top = 27 if op == "step" else 29 if place == "odd" else 31 if layout == "flat" else 30
    n = int(2 ** rng.uniform(18, top))
    n -= n % rng.choice([1, 8, 1024])
    if op == "step":
        K = rng.choice([4, 8, 16])
    else:
        K = rng.choice([rng.randint(1, 16), 8, 16, 32, 60, 64, rng.randint(17, 128)])
    offset = {"whole": 0, "shard": 8 * rng.randrange(1 << 30), "odd": 2 * rng.randrange(1 << 32) + 1}[place]
    tensors = rng.randint(2, 300) if layout == "tensors" else 0
    return _case(op, dtype, n, K, offset=offset, layout=layout, tensors=tensors)


def _spans(case):
    """[(start in the arena, weights)] of a list of separate tensors, in order: the model's own
    tensors, or a ragged list with a few large tensors and many small ones."""
    if case["model"]:
        sizes = [sz for _, sz, _ in workloads.model_tensors(workloads.WORKLOADS[case["model"]])]
    else:
        r = random.Random(case["n"] * 1009 + case["tensors"])
        part = [math.exp(r.uniform(0, 8)) for _ in range(case["tensors"])]
        sizes = [max(1, int(case["n"] * p / sum(part))) for p in part]
        sizes[-1] += max(0, case["n"] - sum(sizes))
    step = SEGMENT_ALIGN // (2 if case["dtype"] == "bf16" else 4)
    spans, at = [], 0
    for sz in sizes:
        spans.append((at, sz))
        at += -(-sz // step) * step
    return spans


def _host(case, seed):
    """The draws that both the library and the 64-bit evaluation use: step seed and number, the probe
    indices of a perturb or transition, the losses."""
    r = random.Random(1_000_003 * seed + 17)
    K = case["K"]
    k = r.randrange(K)
    losses = workloads.synthetic_losses(K, seed % (1 << 31))
    return {"seed": r.getrandbits(64), "step": r.getrandbits(20), "k": k, "k_next": (k + 1) % K, "losses": losses}


def _weights(case, seed):
    """Weights ~ N(0, 0.02) on the device. A list of tensors is laid out in one arena whose gaps are 0."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    if case["layout"] == "flat":
        return torch.empty(case["n"], device="cuda", dtype=DTYPES[case["dtype"]]).normal_(0.0, 0.02, generator=g)
    spans = _spans(case)
    arena = torch.zeros(spans[-1][0] + spans[-1][1], device="cuda", dtype=DTYPES[case["dtype"]])
    for at, sz in spans:
        arena[at:at + sz].normal_(0.0, 0.02, generator=g)
    return arena


def prepare(case, seed):
    h = _host(case, seed)
    theta = _weights(case, seed)
    lp, lm, l0 = h["losses"]
    s = {"case": case, "theta": theta, "lp": lp, "lm": lm, "l0": l0, "seed": h["seed"], "step": h["step"],
         "k": h["k"], "k_next": h["k_next"], "c": zo.zo_probe_coeffs(lp, lm, l0, EPS)}
    if case["layout"] == "tensors":
        spans = _spans(case)
        s["tensors"] = [theta[at:at + sz] for at, sz in spans]
        s["offsets"] = [case["offset"] + int(o) for o in np.cumsum([0] + [sz for _, sz in spans[:-1]])]
    return s


def run(s):
    """One call through the public entry points (for "step": one whole step). The weights are updated in
    place and returned."""
    case, seed, step = s["case"], s["seed"], s["step"]
    op, K, offset, th = case["op"], case["K"], case["offset"], s["theta"]
    if case["layout"] == "tensors":
        ts, os_ = s["tensors"], s["offsets"]
        if op == "step":
            zo.zo_perturb_segments(ts, os_, 0, EPS, 0, 0.0, seed, step)
            for k in range(K):
                zo.zo_perturb_segments(ts, os_, k, -2 * EPS, 0, 0.0, seed, step)
                if k + 1 < K:
                    zo.zo_perturb_segments(ts, os_, k, EPS, k + 1, EPS, seed, step)
            c = zo.zo_probe_coeffs(s["lp"], s["lm"], s["l0"], EPS)
            zo.zo_update_segments(ts, os_, c, EPS, seed, step, K - 1, EPS)
        elif op == "perturb":
            zo.zo_perturb_segments(ts, os_, s["k"], EPS, 0, 0.0, seed, step)
        elif op == "transition":
            zo.zo_perturb_segments(ts, os_, s["k"], EPS, s["k_next"], EPS, seed, step)
        elif op == "update":
            zo.zo_update_segments(ts, os_, s["c"], EPS, seed, step)
        else:
            zo.zo_update_segments(ts, os_, s["c"], EPS, seed, step, K - 1, EPS)
        return th
    if op == "step":
        zo.zo_perturb(th, 0, EPS, seed, step, offset)
        for k in range(K):
            zo.zo_perturb(th, k, -2 * EPS, seed, step, offset)
            if k + 1 < K:
                zo.zo_perturb2(th, k, EPS, k + 1, EPS, seed, step, offset)
        c = zo.zo_probe_coeffs(s["lp"], s["lm"], s["l0"], EPS)
        zo.zo_update_restore(th, c, EPS, seed, step, K - 1, EPS, offset)
    elif op == "perturb":
        zo.zo_perturb(th, s["k"], EPS, seed, step, offset)
    elif op == "transition":
        zo.zo_perturb2(th, s["k"], EPS, s["k_next"], EPS, seed, step, offset)
    elif op == "update":
        zo.zo_update_ex(th, s["c"], EPS, seed, step, offset)
    else:
        zo.zo_update_restore(th, s["c"], EPS, seed, step, K - 1, EPS, offset)
    return th


def work(case):
    """One read and one write of every weight per sweep; one multiply-add per weight and probe applied."""
    n = sum(sz for _, sz in _spans(case)) if case["layout"] == "tensors" else case["n"]
    size = 2 if case["dtype"] == "bf16" else 4
    K = case["K"]
    sweeps = 2 * K + 1 if case["op"] == "step" else 1
    probes = {"perturb": 1, "transition": 2, "update": K, "update_restore": K + 1, "step": 4 * K}[case["op"]]
    return {"bytes": 2 * size * n * sweeps, "flops": 2 * n * probes}


def tolerance(case):
    """Perturbs and transitions are one (exactly defined) addition per weight. An update's sum may be taken in
    another order in 32 bits; in bf16 that moves a few results to the neighbouring value (at most 2^-7 of it).
    Measured on 4 M weights, 8 to 128 probes, the probe groups' sums in reverse order: at most 6.6e-6 of the norm
    in bf16, 1.7e-8 (and 1.2e-7 of a single value) in f32. A whole step holds one update, and single
    moved values weigh more in the smallest buffers."""
    if case["op"] in ("perturb", "transition"):
        return "exact"
    return {"rel": 4e-5, "max": 0.02} if case["dtype"] == "bf16" else {"rel": 2e-7, "max": 1e-6}


# The same in 64 bits, in plain torch.
_M32 = 0xFFFFFFFF


def _blocks(t, group, seed, step):
    """Philox4x32-10 of the tiles t (int64): [len(t), 16] probe bytes, element order."""
    x0, x1 = t & _M32, (t >> 32) & _M32
    x2, x3 = torch.full_like(t, step), torch.full_like(t, group)
    k0, k1 = seed & _M32, (seed >> 32) & _M32
    for _ in range(10):
        p0, p1 = x0 * 0xD2511F53, x2 * 0xCD9E8D57
        x0, x2 = ((p1 >> 32) & _M32) ^ x1 ^ k0, ((p0 >> 32) & _M32) ^ x3 ^ k1
        x1, x3 = p1 & _M32, p0 & _M32
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    words = torch.stack([x0, x1, x2, x3], 1)
    shifts = torch.tensor([0, 8, 16, 24], device=t.device)
    return ((words[:, :, None] >> shifts) & 0xFF).reshape(-1, 16)


def _add_probes(out, offset, weights, seed, step):
    """out[i] += sum_k weights[k] z_k[offset + i], piece by piece."""
    b = np.arange(256)
    tables = {}
    for k, w in weights.items():
        sign = np.where((b >> (k % 8)) & 1, 1.0, -1.0)
        tables[k // 8] = tables.get(k // 8, 0.0) + w * sign
    n, piece = out.numel(), 1 << 21  # tiles per piece
    for t0 in range(offset // 16, (offset + n - 1) // 16 + 1, piece):
        t1 = min(t0 + piece, (offset + n - 1) // 16 + 1)
        t = torch.arange(t0, t1, device=out.device, dtype=torch.int64)
        lo, hi = max(offset, 16 * t0), min(offset + n, 16 * t1)
        total = 0
        for g, tab in tables.items():
            total = total + torch.from_numpy(tab).to(out.device)[_blocks(t, g, seed, step)].reshape(-1)
        out[lo - offset:hi - offset] += total[lo - 16 * t0:hi - 16 * t0]


def exact(case, seed):
    h = _host(case, seed)
    op, K = case["op"], case["K"]
    if op == "perturb":
        w = {h["k"]: float(np.float32(EPS))}
    elif op == "transition":
        w = {h["k"]: float(np.float32(EPS))}
        w[h["k_next"]] = w.get(h["k_next"], 0.0) + float(np.float32(EPS))
    else:
        lp, lm, l0 = h["losses"]
        chat = ((lp - 2.0 * l0) + lm) / (EPS * EPS)
        c = ((lp - lm) / np.maximum(np.abs(chat) ** 0.1, 1.0)) / (2.0 * K * EPS)
        w = {k: -float(np.float32(EPS)) * float(np.float32(c[k])) for k in range(K)}
        if op == "update_restore":
            w[K - 1] += float(np.float32(EPS))
    out = _weights(case, seed).double()
    if case["layout"] == "flat":
        _add_probes(out, case["offset"], w, h["seed"], h["step"])
    else:
        o = case["offset"]
        for at, sz in _spans(case):
            _add_probes(out[at:at + sz], o, w, h["seed"], h["step"])
            o += sz
    return out
