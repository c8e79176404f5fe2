"""Performance cases of the multi-LoRA layer: what its users have it do, from the smallest layer to the largest.

A case is one pass of a training (or validation) program over one segmentation of the flat token buffer, through the public
binding.  Every buffer, the plan and the workspace are made once per state, as such a program keeps them; gradients,
parameters and optimizer state of all adapters live in flat buffers with one view per adapter.

Fields of a case: kind (what one pass does, see `run`), dtype, k, n, tokens, adapters, ranks (cycled over the adapters), alpha
(scale = alpha / rank; 0: the scale 2 that alpha = 2 * rank gives), lens ("equal", "ragged" or the segment lengths
themselves) and lens_seed (which ragged lengths)."""
import math
import random

import torch

from paper_2604_05426_amd import binding as ml
from paper_2604_05426_amd.workloads import LLAMA8B_BLOCK

HPARAMS = (1e-4, 0.9, 0.999, 1e-8, 0.01)      # lr, beta1, beta2, eps, weight decay


def _case(name, kind, dtype, k, n, tokens, adapters, ranks, alpha=0, lens="equal", lens_seed=0):
    c = {"kind": kind, "dtype": dtype, "k": k, "n": n, "tokens": tokens, "adapters": adapters, "ranks": ranks, "alpha": alpha,
         "lens": lens, "lens_seed": lens_seed}
    return {"name": name, **c} if name else c


HETERO_RANKS = "128,8,4,8,16,64,16,4,16,32,64,64,128,8,128,4"
HETERO_LENS = "2343,1219,927,2737,1341,2359,1160,723,3101,1845,2821,2784,3879,1806,1000,2641"


def listed():
    return [
        # the smallest job: four fp32 adapters of 64 tokens each, bound by launches (benchmark config 1)
        _case("tiny_fp32", "step", "f32", 256, 256, 256, 4, "4,8,8,16"),
        # single-precision training of a 1B-model attention projection, ragged segments
        _case("fp32_proj", "step", "f32", 2048, 2048, 2048, 8, "8,16,32,64", lens="ragged", lens_seed=1),
        # a short bf16 step: four adapters with one short sequence each, on a narrow (key / value) projection
        _case("short_kv", "step", "bf16", 2048, 512, 230, 4, "8,16", lens="ragged", lens_seed=2),
        # the fine-tuning microbenchmark shape: 32 adapters, one 256-token sequence each, 1B-model width
        _case("many_adapters", "step", "bf16", 2048, 2048, 8192, 32, "16,32,64"),
        # gradient accumulation over two micro-batches on the 8B key / value projection
        _case("kv_accumulate", "accumulate", "bf16", 4096, 1024, 3000, 8, "8,16,32,64", alpha=16, lens="ragged", lens_seed=3),
        # 8B query projection, 8 adapters x 2048 tokens (benchmark config 2)
        _case("q_proj", "step", "bf16", 4096, 4096, 16384, 8, "8,8,16,16,32,32,64,64", alpha=16),
        # heterogeneous jobs: lengths 723 .. 3879, ranks 4 .. 128 (benchmark config 3)
        _case("hetero", "step", "bf16", 4096, 4096, 32686, 16, HETERO_RANKS, alpha=16, lens=HETERO_LENS),
        # a validation pass (forward alone) through the 8B down projection
        _case("down_eval", "forward", "bf16", 14336, 4096, 4001, 8, "16,64", lens="ragged", lens_seed=4),
        # 70B MLP, 16 adapters x 2048 tokens (benchmark config 5, the headline workload)
        _case("mlp_70b", "step", "bf16", 8192, 28672, 32768, 16, "16,32,64,128", alpha=16),
        # a head whose output width is no multiple of 8
        _case("odd_head", "step", "bf16", 2048, 1001, 1500, 6, "4,7,16,33", lens="ragged", lens_seed=5),
        # the decoupled form: frozen-weight products first, the LoRA terms added in place
        _case("decoupled", "decoupled", "bf16", 4096, 4096, 8192, 8, "8,16,32,64", alpha=16),
        # a whole training step of an 8B block, 8 adapters with about 128 tokens each: every projection forward and
        # backward over shared tables, then the grouped AdamW update
        _case("block_step", "block", "bf16", 4096, 4096, 1024, 8, "8,8,16,16,32,32,64,64", lens="ragged", lens_seed=6),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    w = _log_uniform(rng, lo, hi)
    step = rng.choice([256, 256, 256, 64, 64, 8])
    return max(step, w // step * step)


def draw(rng):
    adapters = rng.choice([1, 2, 3, 4, 6, 8, 8, 12, 16, 24, 32])
    ranks = rng.choice(["16", "64", "8,16", "16,32,64", "8,16,32,64", "16,32,64,128", "4,8,16,32,64,128", "128", "4,7,16,33,100"])
    alpha = rng.choice([0, 16])
    lens = rng.choice(["equal", "ragged", "ragged"])
    lens_seed = rng.randrange(1 << 20)
    kind = rng.choice(["step"] * 4 + ["forward", "accumulate", "decoupled", "f32", "f32", "odd", "block"])
    if kind in ("f32", "odd"):
        k, n = _log_uniform(rng, 64, 4096), _log_uniform(rng, 64, 4096)
        if kind == "odd":
            n += 1 if n % 8 == 0 else 0
        elif rng.random() < 0.7:
            k, n = max(8, k // 8 * 8), max(8, n // 8 * 8)
        tokens = min(_log_uniform(rng, 64, 8192), int(3e10) // (k * n))
        return _case("", "step", "bf16" if kind == "odd" else "f32", k, n, max(tokens, adapters), adapters, ranks, alpha, lens, lens_seed)
    if kind == "block":
        return _case("", "block", "bf16", 4096, 4096, max(_log_uniform(rng, 64, 8192), adapters), adapters, ranks, alpha, lens, lens_seed)
    k, n = _width(rng, 256, 14336), _width(rng, 256, 14336)
    tokens = _log_uniform(rng, 64, 16384 if kind == "accumulate" else 32768)
    return _case("", kind, "bf16", k, n, max(tokens, adapters), adapters, ranks, alpha, lens, lens_seed)


# ---- segmentation ------------------------------------------------------------------------------------------------------------

def _segments(case):
    """(ranks, scales, offsets) of a case."""
    N, T = case["adapters"], case["tokens"]
    cyc = [int(r) for r in case["ranks"].split(",")]
    ranks = [cyc[i % len(cyc)] for i in range(N)]
    scales = [case["alpha"] / r if case["alpha"] else 2.0 for r in ranks]
    if case["lens"] == "equal":
        lens = [T // N + (1 if i < T % N else 0) for i in range(N)]
    elif case["lens"] == "ragged":      # shares between a quarter and seven quarters of the mean, one token at least
        r = random.Random(case["lens_seed"])
        share = [r.uniform(0.25, 1.75) for _ in range(N)]
        lens = [1 + int((T - N) * x / sum(share)) for x in share]
        lens[-1] += T - sum(lens)
    else:
        lens = [int(x) for x in case["lens"].split(",")]
    off = [0]
    for t in lens:
        off.append(off[-1] + t)
    assert off[-1] == T and min(lens) > 0
    return ranks, scales, off


def _layers(case):
    return [(k, n) for _, k, n in LLAMA8B_BLOCK] if case["kind"] == "block" else [(case["k"], case["n"])]


def _flat(sizes, dtype):
    """One zeroed flat buffer and a view per size, each starting at a multiple of 64 elements."""
    starts, at = [], 0
    for s in sizes:
        starts.append(at)
        at += (s + 63) // 64 * 64
    buf = torch.zeros(max(at, 64), dtype=dtype, device="cuda")
    return buf, [buf[a:a + s] for a, s in zip(starts, sizes)]


# ---- states ------------------------------------------------------------------------------------------------------------------

def _tensors(case, seed):
    """Seeded inputs of every layer: X, dY ~ N(0, 1), W ~ N(0, 0.02^2), A ~ N(0, 1 / k), B ~ N(0, 0.02^2)."""
    ranks, scales, off = _segments(case)
    T = case["tokens"]
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(shape, sigma):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).mul_(sigma).to(dt)

    micro = 2 if case["kind"] == "accumulate" else 1
    out = []
    for k, n in _layers(case):
        L = {"k": k, "n": n, "W": normal((k, n), 0.02)}
        L["A_flat"], A = _flat([k * r for r in ranks], dt)
        L["B_flat"], B = _flat([r * n for r in ranks], dt)
        for a in A:
            a.copy_(normal(a.shape, 1.0 / math.sqrt(k)))
        for b in B:
            b.copy_(normal(b.shape, 0.02))
        L["A"], L["B"] = [a.view(k, r) for a, r in zip(A, ranks)], [b.view(r, n) for b, r in zip(B, ranks)]
        L["X"] = [normal((T, k), 1.0) for _ in range(micro)]
        L["dY"] = [normal((T, n), 1.0) for _ in range(micro)] if case["kind"] != "forward" else []
        out.append(L)
    return dt, ranks, scales, off, out


def prepare(case, seed):
    dt, ranks, scales, off, layers = _tensors(case, seed)
    T, kind = case["tokens"], case["kind"]
    stream = torch.cuda.current_stream().cuda_stream
    R1 = sum((off[i + 1] - off[i]) * r for i, r in enumerate(ranks))
    dtype = ml.F32 if case["dtype"] == "f32" else ml.BF16
    for L in layers:
        k, n = L["k"], L["n"]
        if L is layers[0]:
            L["plan"] = ml.Plan(dtype, T, k, n, ranks, scales, off, stream=stream)
        else:
            L["plan"] = ml.Plan.like(layers[0]["plan"], k, n, stream=stream)
        L["ws"] = torch.empty(max(L["plan"].workspace_bytes(), 256), dtype=torch.uint8, device="cuda")
        L["Y"] = [torch.empty((T, n), dtype=dt, device="cuda") for _ in L["X"]]
        L["S"] = [torch.empty(R1, dtype=dt, device="cuda") for _ in L["X"]]
        if kind != "forward":
            L["dX"] = [torch.empty((T, k), dtype=dt, device="cuda") for _ in L["X"]]
            L["dA_flat"], L["dA"] = _flat([k * r for r in ranks], dt)
            L["dB_flat"], L["dB"] = _flat([r * n for r in ranks], dt)
        if kind == "block":
            L["sA_flat"], L["sA"] = _flat([3 * k * r for r in ranks], torch.float32)
            L["sB_flat"], L["sB"] = _flat([3 * r * n for r in ranks], torch.float32)
            ml.multi_lora_adamw_init(L["plan"], L["A"], L["B"], L["sA"], L["sB"], stream)
    return {"kind": kind, "layers": layers, "stream": stream, "step": 0, "N": len(ranks)}


def _fwd(L, j, flags, stream):
    ml.multi_lora_fwd(L["plan"], L["X"][j], L["W"], L["A"], L["B"], L["Y"][j], L["S"][j], L["ws"], flags, stream)


def _bwd(L, j, flags, stream):
    ml.multi_lora_bwd(L["plan"], L["dY"][j], L["X"][j], L["W"], L["A"], L["B"], L["S"][j], L["dX"][j], L["dA"], L["dB"], L["ws"],
                      flags, stream)


def run(state):
    kind, stream, layers = state["kind"], state["stream"], state["layers"]
    L = layers[0]
    if kind == "forward":
        _fwd(L, 0, 0, stream)
        return {"Y": L["Y"][0], "S": L["S"][0]}
    if kind == "step":
        _fwd(L, 0, 0, stream)
        _bwd(L, 0, 0, stream)
    elif kind == "decoupled":
        _fwd(L, 0, ml.FLAG_BASE_ONLY, stream)
        _fwd(L, 0, ml.FLAG_LORA_ONLY, stream)
        _bwd(L, 0, ml.FLAG_BASE_ONLY, stream)
        _bwd(L, 0, ml.FLAG_LORA_ONLY, stream)
    elif kind == "accumulate":
        for j in range(2):
            _fwd(L, j, 0, stream)
            _bwd(L, j, ml.FLAG_ACCUM_GRADS if j else 0, stream)
    else:
        for L in layers:
            _fwd(L, 0, 0, stream)
        for L in reversed(layers):
            _bwd(L, 0, 0, stream)
        state["step"] += 1
        hp = [HPARAMS + (state["step"],)] * state["N"]
        for L in layers:
            ml.multi_lora_adamw_step(L["plan"], L["A"], L["B"], L["dA"], L["dB"], L["sA"], L["sB"], hp, stream)
        return [{"Y": L["Y"][0], "S": L["S"][0], "dX": L["dX"][0], "dA": L["dA_flat"], "dB": L["dB_flat"], "A": L["A_flat"],
                 "B": L["B_flat"], "stateA": L["sA_flat"], "stateB": L["sB_flat"]} for L in layers]
    return {"Y": L["Y"], "S": L["S"], "dX": L["dX"], "dA": L["dA_flat"], "dB": L["dB_flat"]}


# ---- what a pass cannot do without, and how exact its results are --------------------------------------------------------------

def work(case):
    ranks, _, off = _segments(case)
    T, kind = case["tokens"], case["kind"]
    e = 4 if case["dtype"] == "f32" else 2
    R1 = sum((off[i + 1] - off[i]) * r for i, r in enumerate(ranks))
    Sr = sum(ranks)
    nbytes = flops = 0
    for k, n in _layers(case):
        fwd_bytes = (T * k + k * n + Sr * (k + n) + T * n + R1) * e                  # X, W, A, B in, Y, S out
        if kind == "forward":
            nbytes += fwd_bytes
            flops += 2 * T * k * n + 2 * R1 * (k + n)
            continue
        # inputs once (X, W, A, B, dY), outputs once (Y, S, dX, dA, dB)
        m = 2 if kind == "accumulate" else 1
        nbytes += (m * (2 * T * k + 2 * T * n + R1) + k * n + 2 * Sr * (k + n)) * e
        flops += m * (4 * T * k * n + 6 * R1 * (k + n))
        if kind == "block":      # parameters out, optimizer state in and out (12 bytes a parameter)
            nbytes += Sr * (k + n) * (e + 24)
            flops += 16 * Sr * (k + n)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # bf16: rounded S / dS / outputs; fp32: sums of up to a few thousand products in another order
    return {"rel": 1e-5, "max": 2e-4} if case["dtype"] == "f32" else {"rel": 1e-2, "max": 6e-2}


def exact(case, seed):
    dt, ranks, scales, off, layers = _tensors(case, seed)
    kind = case["kind"]
    d = torch.float64
    result = []
    for L in layers:
        k, n = L["k"], L["n"]
        W, A, B = L["W"].to(d), [a.to(d) for a in L["A"]], [b.to(d) for b in L["B"]]
        Ys, Ss, dXs = [], [], []
        dA_flat, dA = _flat([k * r for r in ranks], d)
        dB_flat, dB = _flat([r * n for r in ranks], d)
        for j, X in enumerate(L["X"]):
            X = X.to(d)
            Y, S = X @ W, []
            for i, r in enumerate(ranks):
                rows = slice(off[i], off[i + 1])
                S.append(X[rows] @ A[i])
                Y[rows] += scales[i] * (S[i] @ B[i])
            Ys.append(Y)
            Ss.append(torch.cat([s.reshape(-1) for s in S]))
            if kind == "forward":
                continue
            dY = L["dY"][j].to(d)
            dX = dY @ W.T.contiguous()
            for i, r in enumerate(ranks):
                rows = slice(off[i], off[i + 1])
                dS = scales[i] * (dY[rows] @ B[i].T.contiguous())
                dX[rows] += dS @ A[i].T.contiguous()
                dA[i] += (X[rows].T.contiguous() @ dS).reshape(-1)
                dB[i] += (scales[i] * (S[i].T.contiguous() @ dY[rows])).reshape(-1)
            dXs.append(dX)
            del dY, X
        if kind == "forward":
            return {"Y": Ys[0], "S": Ss[0]}
        if kind != "block":
            return {"Y": Ys, "S": Ss, "dX": dXs, "dA": dA_flat, "dB": dB_flat}
        lr, b1, b2, eps, wd = HPARAMS
        out = {"Y": Ys[0], "S": Ss[0], "dX": dXs[0], "dA": dA_flat, "dB": dB_flat}
        for name, params, grads in (("A", A, dA), ("B", B, dB)):
            p_flat, p_new = _flat([p.numel() for p in params], d)
            s_flat, s_new = _flat([3 * p.numel() for p in params], d)
            for p, g, pn, sn in zip(params, grads, p_new, s_new):
                p = p.reshape(-1)
                m, v = (1 - b1) * g, (1 - b2) * g * g
                pn.copy_(p - lr * ((m / (1 - b1)) / ((v / (1 - b2)).sqrt() + eps) + wd * p))
                sn.copy_(torch.cat([pn, m, v]))
            out[name], out["state" + name] = p_flat, s_flat
        result.append(out)
    return result
