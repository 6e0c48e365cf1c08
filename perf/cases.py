"""The work this library is used for, as measurable cases: packing weights, unpacking them, and the
matmul over packed weights from one activation row (decode) through serving batches to prefill.

A case names an operation, the weight tensors it runs over and the number of activation rows:

  op        quantize / quantize_sub   fp32 weights -> packed (the 100-byte and the 116-byte format)
            dequantize                packed -> fp32 or fp16 weights
            matmul                    one stage after another of a layer; the tensors of a stage read the
                                      same activations and go into one grouped call
            matmul_sub                the same over the 116-byte format, one call per tensor
  layers    how many times the stages are there, each time with weights of their own
  stages    "KxN+N+N,KxN": stages separated by commas, the rows N of a stage's tensors by plus signs
  M         activation rows
  out       "f32" or "f16", the type of the results
  graph     true: the calls are captured once in a HIP graph and run() replays it, as a decode loop
            does; false: run() makes the calls one by one
  pad       extra elements in the row strides of activations and results (a slice of a larger buffer)

Layer shapes are those of paper_2603_27914_amd/synth.py.  Weights are 0.02 x Student-t (4 degrees of
freedom) with 0.1 % of the input channels times 20, activations N(0, 1) rounded to fp16 with 0.5 % of
the channels times 10: the value distributions of that file, drawn on the device.
"""
import math

import torch

from paper_2603_27914_amd import binding

LAYER_7B = "4096x4096+4096+4096,4096x4096,4096x11008+11008,11008x4096"
LAYER_70B = "8192x8192+1024+1024,8192x8192,8192x28672+28672,28672x8192"
MLP_8B = "4096x14336+14336,14336x4096"

T_STAR = 0.7979  # scale of the ternary grid over the deviation of a rotated block


def listed():
    return [
        # one projection of a small model for one token, called directly: the smallest call there is
        dict(name="gemv_2048", op="matmul", layers=1, stages="2048x2048", M=1, out="f32", graph=False, pad=0),
        # decode of one token, 7B shapes: short launches (6 to 35 MB each), four layers of a replayed step
        dict(name="decode_7b_m1", op="matmul", layers=4, stages=LAYER_7B, M=1, out="f32", graph=True, pad=0),
        # decode of one token, 70B shapes: long launches next to short ones (26 to 184 MB)
        dict(name="decode_70b_m1", op="matmul", layers=1, stages=LAYER_70B, M=1, out="f16", graph=True, pad=0),
        # a few tokens at once: speculative decoding, or four users
        dict(name="decode_7b_m4", op="matmul", layers=4, stages=LAYER_7B, M=4, out="f16", graph=True, pad=0),
        # a full decode batch of sixteen users on the large shapes
        dict(name="decode_70b_m16", op="matmul", layers=1, stages=LAYER_70B, M=16, out="f16", graph=True, pad=0),
        # a serving batch between decode and prefill
        dict(name="batch_7b_m48", op="matmul", layers=2, stages=LAYER_7B, M=48, out="f16", graph=True, pad=0),
        # a short prompt, odd length, results and activations as slices of wider buffers, ragged row counts
        dict(name="prompt_ragged_m149", op="matmul", layers=1, stages="4096x4100+1032,11008x4090", M=149, out="f16", graph=False, pad=64),
        # prefill of a chunk of 512 tokens through a whole 7B layer
        dict(name="prefill_7b_m512", op="matmul", layers=1, stages=LAYER_7B, M=512, out="f16", graph=False, pad=0),
        # the largest: prefill of 2048 tokens through an MLP
        dict(name="prefill_mlp_m2048", op="matmul", layers=1, stages=MLP_8B, M=2048, out="f16", graph=False, pad=0),
        # the 116-byte format, a decode batch
        dict(name="sub_m8", op="matmul_sub", layers=3, stages="4096x11008+11008,11008x4096", M=8, out="f16", graph=True, pad=0),
        # packing the weights of an MLP projection (offline, over every tensor of a checkpoint)
        dict(name="quantize_11008", op="quantize", layers=1, stages="4096x11008", M=0, out="", graph=False, pad=0),
        # unpacking a tensor to half precision for a consumer that wants it dense
        dict(name="dequantize_11008", op="dequantize", layers=1, stages="4096x11008", M=0, out="f16", graph=False, pad=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["matmul"] * 7 + ["matmul_sub", "quantize", "quantize_sub", "dequantize", "dequantize"])
    K = 256 * _log_int(rng, 4, 112)
    N = _log_int(rng, 300, 28672)
    while N * K > 28672 * 8192:
        K -= 256
    if rng.random() < 0.4:
        N = N // 16 * 16
    if op in ("quantize", "quantize_sub", "dequantize"):
        return dict(op=op, layers=1, stages="%dx%d" % (K, N), M=0, out=rng.choice(["f32", "f16"]) if op == "dequantize" else "", graph=False, pad=rng.choice([0, 0, 8, 64]))
    M = rng.choice([1, 1, 2, 3, 4, _log_int(rng, 5, 16), _log_int(rng, 17, 64), _log_int(rng, 17, 64), _log_int(rng, 65, 512), _log_int(rng, 65, 2048)])
    if op == "matmul_sub":
        M = min(M, 1024)
    Ns = [N]
    for _ in range(rng.choice([0, 0, 1, 2])):
        Ns.append(rng.choice([N, max(16, N // 8)]))
    while sum(Ns) * K * M > 3 * 14336 * 4096 * 2048 or sum(Ns) * K > 57344 * 8192:
        if len(Ns) > 1:
            Ns.pop()
        else:
            M = M // 2
    return dict(op=op, layers=1, stages="%dx%s" % (K, "+".join(map(str, Ns))), M=M, out=rng.choice(["f32", "f16", "f16"]),
                graph=M <= 64, pad=rng.choice([0, 0, 0, 8, 40]))


# ---- inputs


def _stages(case):
    """[(K, [N, ...])] over all layers."""
    one = []
    for s in case["stages"].split(","):
        k, ns = s.split("x")
        one.append((int(k), [int(n) for n in ns.split("+")]))
    return one * case["layers"]


def _weights(gen, N, K, pad=0):
    """fp32 [N, K] (row stride K + pad)."""
    W = torch.empty((N, K + pad), device="cuda")
    for n0 in range(0, N, 4096):  # in slabs: the temporaries stay small
        n = min(4096, N - n0)
        z = torch.randn((n, K), generator=gen, device="cuda")
        chi = torch.rand((n, K), generator=gen, device="cuda").clamp_min_(1e-12).log_()
        chi += torch.rand((n, K), generator=gen, device="cuda").clamp_min_(1e-12).log_()  # -2 (log u + log v): chi-square, 4 degrees of freedom
        W[n0 : n0 + n, :K] = 0.02 * z * torch.rsqrt(-0.5 * chi)
    cols = torch.randperm(K, generator=gen, device="cuda")[: int(round(0.001 * K))]
    W[:, cols] *= 20.0
    return W[:, :K]


def _activations(gen, M, K, pad):
    X = torch.zeros((M, K + pad), device="cuda")
    X[:, :K] = torch.randn((M, K), generator=gen, device="cuda")
    cols = torch.randperm(K, generator=gen, device="cuda")[: int(round(0.005 * K))]
    X[:, cols] *= 10.0
    return X.half()[:, :K]


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(1000003 * seed + 20260327)


def _dtype(case):
    return {"f32": torch.float32, "f16": torch.float16}[case["out"]]


def prepare(case, seed):
    gen = _generator(seed)
    op, pad = case["op"], case["pad"]
    flags = torch.zeros(1, dtype=torch.int32, device="cuda")
    if op in ("quantize", "quantize_sub", "dequantize"):
        (K, (N,)), = _stages(case)
        W = _weights(gen, N, K, pad)
        if op == "quantize":
            return dict(op=op, W=W, packed=binding.alloc_packed(N, K), flags=flags)
        if op == "quantize_sub":
            sub = torch.empty(binding.itq3s_subscales_bytes(N, K) // 4, dtype=torch.int32, device="cuda")
            return dict(op=op, W=W, packed=binding.alloc_packed(N, K) + (sub,), flags=flags)
        out = torch.zeros((N, K + pad), dtype=_dtype(case), device="cuda")[:, :K]
        return dict(op=op, N=N, K=K, packed=binding.itq3s_quantize(W), out=out, flags=flags)
    M, calls, ws_bytes = case["M"], [], 256
    for K, Ns in _stages(case):
        X = _activations(gen, M, K, pad)
        weights, outs = [], []
        for N in Ns:
            W = _weights(gen, N, K)
            weights.append((binding.itq3s_quantize_sub(W) if op == "matmul_sub" else binding.itq3s_quantize(W)) + (N,))
            del W
            outs.append(torch.zeros((M, N + pad), dtype=_dtype(case), device="cuda")[:, :N])
            rows = min(M, 16) if op == "matmul_sub" else M
            ws_bytes = max(ws_bytes, binding.itq3s_matmul_workspace_bytes(rows, N, K))
        calls.append((K, X, weights, outs))
    state = dict(op=op, calls=calls, workspace=torch.empty(ws_bytes, dtype=torch.uint8, device="cuda"), flags=flags, outs=[o for c in calls for o in c[3]])
    if case["graph"]:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _matmuls(state)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            _matmuls(state)
        state["graph"] = graph
    return state


def _matmuls(state):
    ws, flags = state["workspace"], state["flags"]
    for K, X, weights, outs in state["calls"]:
        if state["op"] == "matmul_sub":
            for (codes, scales, subscales, N), out in zip(weights, outs):
                binding.itq3s_matmul_sub(codes, scales, subscales, N, K, X, out=out, workspace=ws, status_flags=flags)
        elif len(weights) == 1:
            codes, scales, N = weights[0]
            binding.itq3s_matmul(codes, scales, N, K, X, out=outs[0], workspace=ws, status_flags=flags)
        else:
            binding.itq3s_matmul_grouped(weights, K, X, outs=outs, workspace=ws, status_flags=flags)


def run(state):
    op, flags = state["op"], state["flags"]
    if op == "quantize":
        codes, scales = state["packed"]
        binding.itq3s_quantize(state["W"], codes, scales, status_flags=flags)
        return {"codes": codes, "scales": scales, "flags": flags}
    if op == "quantize_sub":
        codes, scales, subscales = binding.itq3s_quantize_sub(state["W"], out=state["packed"], status_flags=flags)
        return {"codes": codes, "scales": scales, "subscales": subscales, "flags": flags}
    if op == "dequantize":
        codes, scales = state["packed"]
        binding.itq3s_dequantize(codes, scales, state["N"], state["K"], out=state["out"], status_flags=flags)
        return {"W": state["out"], "flags": flags}
    if "graph" in state:
        state["graph"].replay()
    else:
        _matmuls(state)
    return {"Y": state["outs"], "flags": flags}


def work(case):
    nbytes, flops, M = 0, 0, case["M"]
    block = 116 if case["op"].endswith("_sub") else 100
    size = {"f32": 4, "f16": 2, "": 0}[case["out"]]
    for K, Ns in _stages(case):
        nbytes += 2 * M * K
        for N in Ns:
            nbytes += N * (K // 256) * block + M * N * size
            flops += 2 * M * N * K
            if case["op"] in ("quantize", "quantize_sub"):
                nbytes += 4 * N * K
            if case["op"] == "dequantize":
                nbytes += size * N * K
            if M == 0:  # the 256-point transform: 8 additions per weight; on encode two sums, two comparisons and a square besides
                flops += N * K * (8 if case["op"] == "dequantize" else 13)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["op"] in ("quantize", "quantize_sub"):
        return "exact"
    if case["op"] == "dequantize":  # one rounding to fp32, one more to fp16
        return {"rel": 2.4e-7, "max": 1e-6} if case["out"] == "f32" else {"rel": 8e-4, "max": 2e-3}
    # one rounding to fp16 of the rotated activations (or of the reconstructed weights), 2^-11 / sqrt(3) each at most,
    # fp32 sums, and for fp16 results one more rounding
    return {"rel": 1.2e-3, "max": 1e-2}


# ---- the same results in 64 bits


def _hadamard(device):
    i = torch.arange(256, device=device)
    bits = i[:, None] & i[None, :]
    for s in (4, 2, 1):
        bits = bits ^ (bits >> s)
    return (1.0 - 2.0 * (bits & 1).double()) / 16.0


def _reconstruct(W, sub):
    """H d (s q - z) over the blocks of W, by the format's definition, in float64."""
    N, K = W.shape
    H = _hadamard(W.device)
    out = torch.empty((N, K), dtype=torch.float64, device=W.device)
    for n0 in range(0, N, 4096):
        w = W[n0 : n0 + 4096].double().reshape(-1, 256) @ H
        mu = w.mean(dim=1, keepdim=True)
        d = (T_STAR * (w - mu).square().mean(dim=1, keepdim=True).sqrt()).clamp_max(65504.0).float().half().double()
        safe = torch.where(d > 0, d, torch.ones_like(d))
        z = (0.0 - torch.floor(mu / safe + 0.5)).clamp(-2048, 2048)
        s = torch.ones_like(w)
        if sub:
            sj = T_STAR * (w - mu).square().reshape(-1, 8, 32).mean(dim=2).sqrt() / safe
            s = sj.clamp_max(65504.0).float().half().double().repeat_interleave(32, dim=1)
        q = (w >= (0.5 * s - z) * d).double() - (w < (-0.5 * s - z) * d).double()
        q = torch.where(s > 0, q, torch.zeros_like(q))
        rows = torch.where(d > 0, d * (s * q - z), torch.zeros_like(w)) @ H
        out[n0 : n0 + 4096] = rows.reshape(-1, K)
    return out


def exact(case, seed):
    gen = _generator(seed)
    op, pad = case["op"], case["pad"]
    if op in ("quantize", "quantize_sub"):
        return None  # whole numbers: compared bit by bit
    if op == "dequantize":
        (K, (N,)), = _stages(case)
        return {"W": _reconstruct(_weights(gen, N, K, pad), False), "flags": None}
    ys = []
    for K, Ns in _stages(case):
        X = _activations(gen, case["M"], K, pad).double()
        for N in Ns:
            ys.append(X @ _reconstruct(_weights(gen, N, K), op == "matmul_sub").T)
    return {"Y": ys, "flags": None}
