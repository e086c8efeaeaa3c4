"""The work whose speed is watched: what a program built on this library has it do.

A program keeps every linear of a model resident at several bit-widths, decodes token by token with
the bit-width of each linear picked from device memory, processes prompts of any length, scores
logits, and quantizes weights when the model is loaded.  The cases go through the package's public
calls; shapes are those of the Llama-7B, -13B and -70B shaped stacks of ``synth`` and of the tests.
Weights and activations are normal (optionally with one entry in a thousand 20 times larger, as in
the 13B stack); a weight's deviation is 1 / sqrt(K), so that a chain of linears keeps its scale.
"""
from __future__ import annotations

import math
import random

import torch

import paper_2506_12024_amd as fq

DEV = "cuda:0"
GROUP = 128
# hidden, FFN, width of the key and value projections
STACKS = {"7b": (4096, 11008, 4096), "13b": (5120, 13824, 5120), "70b": (8192, 28672, 1024)}


def listed():
    return [
        # one projection of one token by itself: launch and latency
        {"name": "linear_m1", "kind": "linear", "M": 1, "N": 4096, "K": 4096, "bits": 4, "outliers": False},
        # a whole token of the 7B-shaped stack in the order a decoder issues it, one launch
        {"name": "token_7b_staged", "kind": "plan", "mode": "staged", "stack": "7b", "layers": 32, "M": 1,
         "choices": "4,8", "pattern": 1},
        # a batch of 16 sequences through eight decoder layers: four plans per layer (q/k/v, o, gate/up, down)
        {"name": "layers_7b_batch16", "kind": "plan", "mode": "stages", "stack": "7b", "layers": 8, "M": 16,
         "choices": "4,8", "pattern": 2},
        # the widest batch of the decode kernels, linears that do not depend on each other, three widths
        {"name": "plan_7b_batch32", "kind": "plan", "mode": "independent", "stack": "7b", "layers": 16, "M": 32,
         "choices": "4,8,16", "pattern": 3},
        # a short prompt (or a chunk of one) through the 7B down projection
        {"name": "prompt_100", "kind": "linear", "M": 100, "N": 4096, "K": 11008, "bits": 4, "outliers": False},
        # a prompt of some hundred tokens through the 7B gate projection at the higher width
        {"name": "prompt_515", "kind": "linear", "M": 515, "N": 11008, "K": 4096, "bits": 8, "outliers": False},
        # a long prompt through a 70B-shaped linear
        {"name": "prompt_2048", "kind": "linear", "M": 2048, "N": 28672, "K": 8192, "bits": 4, "outliers": False},
        # 8-bit activations: a few hundred tokens through the 13B down projection, groups of 128
        {"name": "w8a8_300", "kind": "w8a8", "M": 300, "N": 5120, "K": 13824, "per_row": False, "outliers": True},
        # 8-bit activations, one scale per weight row: a long prompt through the 70B down projection
        {"name": "w8a8_row_2048", "kind": "w8a8", "M": 2048, "N": 8192, "K": 28672, "per_row": True,
         "outliers": False},
        # entropy and KL of a prompt's logits over a large vocabulary (offline analysis, threshold from the prefill)
        {"name": "entropy_kl_2048", "kind": "entropy", "R": 2048, "V": 128256, "kl": True, "half": False},
        # the output layer with the entropy and the token of a decode step
        {"name": "lm_head_m1", "kind": "lm_head", "M": 1, "V": 32000, "K": 4096, "logits": True},
        # loading a model: one 7B-shaped weight to its packed 4-bit copy
        {"name": "quantize_w4", "kind": "quantize", "N": 11008, "K": 4096, "bits": 4, "form": "asym",
         "outliers": True},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng, most):
    """Rows (any number, every other time a multiple of 128) and a row length for at most `most` weights."""
    K = max(4, _log(rng, 512, 28672) // GROUP) * GROUP
    N = _log(rng, 512, min(28672, most // K))
    return (N if rng.random() < 0.5 else max(GROUP, N // GROUP * GROUP)), K


def draw(rng):
    kind = rng.choice(["linear_decode", "linear_prompt", "linear_prompt", "staged", "stages", "stages", "independent",
                       "w8a8", "w8a8", "entropy", "lm_head", "quantize"])
    outliers = rng.random() < 0.3
    if kind == "linear_decode":
        N, K = _shape(rng, 28672 * 8192)
        return {"kind": "linear", "M": _log(rng, 1, 32), "N": N, "K": K, "bits": rng.choice([2, 3, 4, 4, 8, 8, 16]),
                "outliers": outliers}
    if kind == "linear_prompt":
        N, K = _shape(rng, 28672 * 8192)
        M = _log(rng, 33, 2048)
        return {"kind": "linear", "M": M, "N": N, "K": K,
                "bits": rng.choice([2, 4, 4, 8, 8, 16] if M > 128 else [2, 3, 4, 4, 8, 8, 16]), "outliers": outliers}
    if kind in ("staged", "stages", "independent"):
        stack = rng.choice(["7b", "7b", "13b", "70b"])
        most = {"7b": 16, "13b": 10, "70b": 3}[stack]
        if kind == "stages":
            most = {"7b": 8, "13b": 5, "70b": 2}[stack]
        M = 1 if kind == "staged" else _log(rng, 2, 32) if kind == "stages" else _log(rng, 1, 32)
        return {"kind": "plan", "mode": kind, "stack": stack, "layers": rng.randint(1, most), "M": M,
                "choices": rng.choice(["4,8", "4,8", "4", "8", "2,4,8", "3,4,8", "4,8,16"]), "pattern": rng.randint(0, 999)}
    if kind == "w8a8":
        N, K = _shape(rng, 28672 * 8192)
        return {"kind": "w8a8", "M": _log(rng, 16, 2048), "N": N, "K": K, "per_row": rng.random() < 0.5,
                "outliers": outliers}
    if kind == "entropy":
        R = _log(rng, 1, 2048)
        return {"kind": "entropy", "R": R, "V": rng.choice([32000, 32001, 128256, _log(rng, 1000, 128256)]),
                "kl": rng.random() < 0.6, "half": rng.random() < 0.4}
    if kind == "lm_head":
        K = 512 * rng.randint(2, 16)
        M = rng.randint(1, min(4, 32768 // K))
        return {"kind": "lm_head", "M": M, "V": rng.choice([32000, 128256, _log(rng, 8000, 128256)]), "K": K,
                "logits": rng.random() < 0.5}
    N, K = _shape(rng, 28672 * 4096)
    form = rng.choice(["asym", "asym", "sym", "fake", "row"])
    bits = 8 if form == "row" else rng.randint(2, 8) if form == "fake" else rng.choice([2, 3, 4, 8])
    return {"kind": "quantize", "N": N, "K": K, "bits": bits, "form": form, "outliers": outliers}


# ---- inputs -------------------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _weight(g, N, K, outliers=False):
    w = torch.randn(N, K, generator=g, dtype=torch.float16, device=DEV)
    w *= K ** -0.5
    if outliers:
        i = torch.randint(0, N * K, (max(1, N * K // 1000),), generator=g, device=DEV)
        w.view(-1)[i] *= 20.0
    return w


def _x(g, M, K):
    return torch.randn(M, K, generator=g, dtype=torch.float16, device=DEV)


def _packed(w, bits, group=GROUP, sym=False):
    N, K = w.shape
    cb, sb, zb = fq.fq_packed_sizes(N, K, bits, group)
    c = torch.empty(cb, dtype=torch.uint8, device=DEV)
    s = torch.empty(sb // 4, dtype=torch.float32, device=DEV)
    z = torch.empty(zb, dtype=torch.uint8, device=DEV)
    (fq.fq_quantize_sym if sym else fq.fq_quantize)(w, N, K, bits, group, c, s, z)
    return c, s, z


def _attach(w, widths, group=GROUP):
    N, K = w.shape
    layer = fq.Layer(N, K, group)
    for b in widths:
        layer.attach(b, *((w,) if b == 16 else _packed(w, b, group)))
    return layer


def _entries(case):
    """(stage, name, K, N, entry whose y is this entry's x or None) of a plan's linears."""
    hidden, ffn, kv = STACKS[case["stack"]]
    chained = case["mode"] != "independent"
    out = []
    for li in range(case["layers"]):
        b = 7 * li
        prev = b - 1 if chained and li else None
        out += [(4 * li, "q", hidden, hidden, prev), (4 * li, "k", hidden, kv, prev), (4 * li, "v", hidden, kv, prev),
                (4 * li + 1, "o", hidden, hidden, b if chained else None),
                (4 * li + 2, "gate", hidden, ffn, b + 3 if chained else None),
                (4 * li + 2, "up", hidden, ffn, b + 3 if chained else None),
                (4 * li + 3, "down", ffn, hidden, b + 4 if chained else None)]
    return out


def _bits(case, n):
    rng = random.Random(case["pattern"])
    choices = [int(b) for b in case["choices"].split(",")]
    return [rng.choice(choices) for _ in range(n)]


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    if kind == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        w = _weight(g, N, K, case["outliers"])
        return {"case": case, "layer": _attach(w, [case["bits"]]), "x": _x(g, M, K),
                "y": torch.empty(M, N, dtype=torch.float16, device=DEV)}
    if kind == "plan":
        M, ents = case["M"], _entries(case)
        widths = sorted({int(b) for b in case["choices"].split(",")})
        # every linear's result is a run of one buffer, as a program that sizes its memory once keeps them
        out = torch.empty(M * sum(e[3] for e in ents), dtype=torch.float16, device=DEV)
        layers, xs, ys, at = [], [], [], 0
        for st, _, K, N, src in ents:
            x = xs[-1] if src is None and xs and st == last and case["mode"] != "independent" else \
                _x(g, M, K) if src is None else ys[src]
            layers.append(_attach(_weight(g, N, K), widths))
            xs.append(x)
            ys.append(out[at:at + M * N].view(M, N))
            at += M * N
            last = st
        bits = torch.tensor(_bits(case, len(ents)), dtype=torch.int32, device=DEV)
        plans = []
        if case["mode"] == "staged":
            st = [e[0] for e in ents]
            ws = torch.empty(fq.StagedPlan.workspace_bytes(len(ents), st[-1] + 1), dtype=torch.uint8, device=DEV)
            plans.append((fq.StagedPlan(layers, xs, ys, st, M, ws), bits))
        else:
            cuts = [0, len(ents)]
            if case["mode"] == "stages":
                cuts = [i for i in range(len(ents)) if i == 0 or ents[i][0] != ents[i - 1][0]] + [len(ents)]
            for a, b in zip(cuts, cuts[1:]):
                ws = torch.empty(fq.Plan.workspace_bytes(b - a), dtype=torch.uint8, device=DEV)
                plans.append((fq.Plan(layers[a:b], xs[a:b], ys[a:b], M, ws), bits[a:b]))
        return {"case": case, "plans": plans, "out": out}
    if kind == "w8a8":
        M, N, K = case["M"], case["N"], case["K"]
        w = _weight(g, N, K, case["outliers"])
        return {"case": case, "layer": _attach(w, [8], K if case["per_row"] else GROUP), "x": _x(g, M, K),
                "xq": torch.empty(M, K, dtype=torch.int8, device=DEV),
                "sx": torch.empty(M, dtype=torch.float32, device=DEV),
                "xsum": torch.empty(K // GROUP, M, dtype=torch.int32, device=DEV),
                "y": torch.empty(M, N, dtype=torch.float16, device=DEV)}
    if kind == "entropy":
        R = case["R"]
        p, q = _logits(case, g)
        return {"case": case, "p": p, "q": q, "H": torch.empty(R, dtype=torch.float32, device=DEV),
                "KL": torch.empty(R, dtype=torch.float32, device=DEV) if case["kl"] else None}
    if kind == "lm_head":
        M, V, K = case["M"], case["V"], case["K"]
        return {"case": case, "w": _weight(g, V, K), "x": _head_x(g, M, K),
                "logits": torch.empty(M, V, dtype=torch.float32, device=DEV) if case["logits"] else None,
                "H": torch.empty(M, dtype=torch.float32, device=DEV),
                "argmax": torch.empty(M, dtype=torch.int32, device=DEV)}
    N, K, bits = case["N"], case["K"], case["bits"]
    w = _weight(g, N, K, case["outliers"])
    if case["form"] == "fake":
        return {"case": case, "w": w, "out": torch.empty_like(w)}
    group = K if case["form"] == "row" else GROUP
    cb, sb, zb = fq.fq_packed_sizes(N, K, bits, group)
    return {"case": case, "w": w, "group": group, "codes": torch.empty(cb, dtype=torch.uint8, device=DEV),
            "scales": torch.empty(sb // 4, dtype=torch.float32, device=DEV),
            "zeros": torch.empty(zb, dtype=torch.uint8, device=DEV)}


def _logits(case, g):
    R, V = case["R"], case["V"]
    p = torch.randn(R, V, generator=g, dtype=torch.float32, device=DEV)
    p *= 3.0
    q = None
    if case["kl"]:
        q = torch.randn(R, V, generator=g, dtype=torch.float32, device=DEV)
        q *= 0.1
        q += p
    if case["half"]:
        p, q = p.half(), None if q is None else q.half()
    return p, q


def _head_x(g, M, K):
    return _x(g, M, K) * 3.0


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "linear":
        fq.fq_linear(state["layer"], case["bits"], state["x"], case["M"], state["y"])
        return state["y"]
    if kind == "plan":
        for plan, bits in state["plans"]:
            plan.run(bits)
        return state["out"]
    if kind == "w8a8":
        fq.fq_quantize_act(state["x"], case["M"], case["K"], state["xq"], state["sx"], state["xsum"])
        fq.fq_linear_w8a8(state["layer"], state["xq"], state["sx"], state["xsum"], case["M"], state["y"])
        return state["y"]
    if kind == "entropy":
        call = fq.fq_entropy_kl_f16 if case["half"] else fq.fq_entropy_kl
        call(state["p"], state["q"], case["R"], case["V"], state["H"], state["KL"])
        return [state["H"], state["KL"]] if case["kl"] else state["H"]
    if kind == "lm_head":
        fq.fq_lm_head_entropy(state["x"], state["w"], case["M"], case["V"], case["K"], state["logits"], state["H"],
                              state["argmax"])
        return [state["H"], state["argmax"]] + ([state["logits"]] if case["logits"] else [])
    if case["form"] == "fake":
        fq.fq_fake_quantize(state["w"], case["N"], case["K"], case["bits"], GROUP, False, state["out"])
        return state["out"]
    call = fq.fq_quantize_sym if case["form"] == "sym" else fq.fq_quantize
    call(state["w"], case["N"], case["K"], case["bits"], state["group"], state["codes"], state["scales"], state["zeros"])
    return [state["codes"], state["scales"], state["zeros"]]


# ---- what a pass cannot do without ----------------------------------------------------------------

def _copy_bytes(N, K, bits, group=GROUP):
    return 2 * N * K if bits == 16 else N * K * bits // 8 + N * (K // group) * 5


def work(case):
    kind = case["kind"]
    if kind == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": _copy_bytes(N, K, case["bits"]) + 2 * M * (N + K), "flops": 2 * M * N * K}
    if kind == "plan":
        M, ents = case["M"], _entries(case)
        nbytes = flops = 0
        for (st, name, K, N, src), b in zip(ents, _bits(case, len(ents))):
            # q, k, v and gate, up read one x; in a plan of independent linears each has its own
            shared = case["mode"] != "independent" and name in ("k", "v", "up")
            nbytes += _copy_bytes(N, K, b) + 2 * M * (N + (0 if shared else K))
            flops += 2 * M * N * K
        return {"bytes": nbytes, "flops": flops}
    if kind == "w8a8":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": _copy_bytes(N, K, 8, K if case["per_row"] else GROUP) + 2 * M * (N + K), "flops": 2 * M * N * K}
    if kind == "entropy":
        n = case["R"] * case["V"] * (2 if case["kl"] else 1)
        return {"bytes": n * (2 if case["half"] else 4) + 4 * case["R"] * (2 if case["kl"] else 1), "flops": 8 * n}
    if kind == "lm_head":
        M, V, K = case["M"], case["V"], case["K"]
        return {"bytes": 2 * V * K + 2 * M * K + (4 * M * V if case["logits"] else 0), "flops": 2 * M * V * K}
    N, K = case["N"], case["K"]
    if case["form"] == "fake":
        return {"bytes": 4 * N * K, "flops": 6 * N * K}
    return {"bytes": 2 * N * K + _copy_bytes(N, K, case["bits"], K if case["form"] == "row" else GROUP), "flops": 6 * N * K}


def tolerance(case):
    # about four times what was seen against exact(): 2.1e-4 is the rounding of the results to fp16
    kind = case["kind"]
    if kind == "linear":
        # above 32 rows the matrix-core product takes weights that were rounded to fp16 twice: 3.7e-4
        return {"rel": 1e-3, "max": 4e-3} if case["M"] <= 32 else {"rel": 1.5e-3, "max": 1e-2}
    if kind == "plan":
        # a chain rounds to fp16 at every link: 1.6e-3 after 128, 8.5e-4 after 32
        links = 1 if case["mode"] == "independent" else 4 * case["layers"]
        return {"rel": max(1e-3, 6e-4 * math.sqrt(links)), "max": max(4e-3, 3e-3 * math.sqrt(links))}
    if kind == "w8a8":
        return {"rel": 1e-3, "max": 4e-3}
    if kind == "entropy":
        # the KL of near distributions is the small difference of sums: 1.7e-5
        return {"rel": 7e-5}
    if kind == "lm_head":
        return {"rel": 2e-6}
    return "exact"


# ---- the same in 64 bits ---------------------------------------------------------------------------

def _div(a, b):
    """a / b in binary32; by a tensor, since torch multiplies by the reciprocal of a plain number."""
    return a / torch.full_like(a, float(b))


def _quant(w, bits, group=GROUP, sym=False):
    """Codes, scales and zero points of asymmetric (or symmetric) quantization: the definition fixes
    binary32 with one rounding per operation, so that is what this computes in."""
    N, K = w.shape
    v = w.float().view(N, K // group, group)
    if sym:
        s = _div(2.0 * v.abs().amax(2, keepdim=True), 2 ** bits - 2)
        s = torch.where(s == 0, torch.ones_like(s), s)
        top = float(2 ** (bits - 1) - 1)
        return torch.round(v / s).clamp_(-top, top) + 2.0 ** (bits - 1), s, torch.full_like(s, 2.0 ** (bits - 1))
    lo = v.amin(2, keepdim=True).clamp_(max=0.0)
    hi = v.amax(2, keepdim=True).clamp_(min=0.0)
    top = float(2 ** bits - 1)
    s = _div(hi - lo, top)
    zero = s == 0
    s = torch.where(zero, torch.ones_like(s), s)
    z = torch.round(-lo / s).clamp_(0.0, top)
    return torch.round(v / s + z).clamp_(0.0, top), s, z


def _dense(w, bits, group=GROUP):
    """The weights a copy of `bits` stands for, binary64."""
    if bits == 16:
        return w.double()
    N, K = w.shape
    q, s, z = _quant(w, bits, group)
    return ((q.double() - z.double()) * s.double()).view(N, K)


def _pack(q, bits):
    q = q.to(torch.int32).reshape(q.shape[0], -1)
    N, K = q.shape
    if bits == 8:
        return q.to(torch.uint8).view(-1)
    if bits == 3:
        c = q.view(N, K // 32, 32).to(torch.int64)
        words = []
        for j in range(3):
            word = torch.zeros(N, K // 32, dtype=torch.int64, device=q.device)
            for h in range(2):
                for p in range(5):
                    word |= c[:, :, 10 * j + 5 * h + p] << (16 * h + 3 * p)
                word |= ((c[:, :, 30 + h] >> j) & 1) << (16 * h + 15)
            words.append(word)
        w = torch.stack(words, 2)
        return torch.stack([(w >> (8 * i)) & 255 for i in range(4)], 3).to(torch.uint8).reshape(-1)
    per = 8 // bits
    q = q.view(N, K // per, per)
    out = torch.zeros(N, K // per, dtype=torch.int32, device=q.device)
    for i in range(per):
        out |= q[:, :, i] << (bits * i)
    return out.to(torch.uint8).view(-1)


def exact(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    if kind == "linear":
        w = _weight(g, case["N"], case["K"], case["outliers"])
        return _x(g, case["M"], case["K"]).double() @ _dense(w, case["bits"]).t()
    if kind == "plan":
        ents = _entries(case)
        ys, x, last = [], None, None
        for (st, _, K, N, src), b in zip(ents, _bits(case, len(ents))):
            if src is not None:
                x = ys[src]
            elif not (x is not None and st == last and case["mode"] != "independent"):
                x = _x(g, case["M"], K).double()
            ys.append(x @ _dense(_weight(g, N, K), b).t())
            last = st
        return torch.cat([y.reshape(-1) for y in ys])
    if kind == "w8a8":
        w = _weight(g, case["N"], case["K"], case["outliers"])
        x = _x(g, case["M"], case["K"]).float()
        s = _div(2.0 * x.abs().amax(1, keepdim=True), 254)
        s = torch.where(s == 0, torch.ones_like(s), s)
        xq = torch.round(x / s).clamp_(-127.0, 127.0)
        return (xq.double() * s.double()) @ _dense(w, 8, case["K"] if case["per_row"] else GROUP).t()
    if kind == "entropy":
        p, q = _logits(case, g)
        H, KL = [], []
        for i in range(0, case["R"], 256):
            lp = torch.log_softmax(p[i:i + 256].double(), 1)
            H.append(-(lp.exp() * lp).sum(1))
            if q is not None:
                KL.append((lp.exp() * (lp - torch.log_softmax(q[i:i + 256].double(), 1))).sum(1))
        return torch.cat(H) if q is None else [torch.cat(H), torch.cat(KL)]
    if kind == "lm_head":
        w = _weight(g, case["V"], case["K"])
        logits = _head_x(g, case["M"], case["K"]).double() @ w.double().t()
        lp = torch.log_softmax(logits, 1)
        return [-(lp.exp() * lp).sum(1), logits.argmax(1).to(torch.int32)] + ([logits] if case["logits"] else [])
    w = _weight(g, case["N"], case["K"], case["outliers"])
    if case["form"] == "fake":
        q, s, z = _quant(w, case["bits"])
        return ((q - z) * s).half().view(case["N"], case["K"])
    group = case["K"] if case["form"] == "row" else GROUP
    q, s, z = _quant(w, case["bits"], group, case["form"] == "sym")
    return [_pack(q, case["bits"]), s.reshape(-1), z.to(torch.uint8).reshape(-1)]
