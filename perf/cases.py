"""The calls that the performance of this framework is judged on.

A program that serves or prepares a MosaicQuant model makes these calls:

* ``linear``: one layer call from fp16 activations (quantisation and fused
  GEMM), from one token to a long prefill;
* ``step``: the four linear operators of several decoder layers at decode
  batch sizes, captured once in a HIP graph and replayed for every token;
* ``shared``: activations quantised once and multiplied with the weights of
  several layers that read the same input (q, k and v projections);
* ``a8``: the W4A8 layer (INT8 activations), decode and prefill;
* ``prepare``: offline preparation of one layer's weight (base quantisation,
  block scores, selection, residual quantisation) by either criterion.

Layer shapes are those of the synthetic workloads and tests (LLaMA3 / Qwen3
layers); drawn cases add generic multiples of 128.  Weights of the layer calls
come from a synthetic checkpoint in the canonical interchange layout (two's
complement nibbles), repacked once as a loader would.
"""
from __future__ import annotations

import math

import torch

import paper_2606_15652_amd as mq

BLOCK = 128
# (K, N): attention and MLP projections of the workload families
SHAPES = [(1024, 1024), (4096, 4096), (4096, 6144), (4096, 14336), (14336, 4096), (4096, 24576), (12288, 4096),
          (5120, 5120), (5120, 1024), (5120, 25600), (25600, 5120), (8192, 28672), (28672, 8192)]
# the concatenated operators of one decoder layer: qkv, o, gate_up, down
STEP_OPS = [(4096, 6144), (4096, 4096), (4096, 24576), (12288, 4096)]
DENSITIES = [0, 5, 10, 20]          # residual blocks, per cent
LARGEST = 2.2 * 8192 * 8192 * 28672  # operations of the largest listed case


def listed():
    return [
        # one token through one attention projection: the smallest call, eager
        {"name": "linear_m1", "kind": "linear", "M": 1, "K": 4096, "N": 4096, "density": 10, "skew": False},
        # a decode batch of 8 through four decoder layers, replayed from a graph
        {"name": "step_m8", "kind": "step", "M": 8, "layers": 4, "density": 10, "skew": False},
        # speculative or small-batch decode through the widest MLP layer
        {"name": "linear_wide_m4", "kind": "linear", "M": 4, "K": 8192, "N": 28672, "density": 10, "skew": False},
        # a large decode batch or a short prompt
        {"name": "linear_m256", "kind": "linear", "M": 256, "K": 4096, "N": 4096, "density": 10, "skew": False},
        # a long prompt through an attention projection
        {"name": "linear_m4096", "kind": "linear", "M": 4096, "K": 4096, "N": 4096, "density": 10, "skew": False},
        # a prompt of no round length through an MLP layer
        {"name": "linear_ragged", "kind": "linear", "M": 1157, "K": 4096, "N": 14336, "density": 5, "skew": False},
        # q, k and v projections of one prompt, residual blocks in hot rows
        {"name": "qkv_m2048", "kind": "shared", "M": 2048, "K": 5120, "N": 5120, "N2": 1024, "density": 10,
         "skew": True},
        # the largest prefill of the workload families
        {"name": "linear_m8192", "kind": "linear", "M": 8192, "K": 8192, "N": 28672, "density": 10, "skew": False},
        # W4A8, a decode batch
        {"name": "a8_m16", "kind": "a8", "M": 16, "K": 14336, "N": 4096, "density": 10, "skew": False},
        # W4A8, a prompt
        {"name": "a8_m2048", "kind": "a8", "M": 2048, "K": 4096, "N": 14336, "density": 10, "skew": False},
        # weight preparation by residual norm
        {"name": "prepare_frob", "kind": "prepare", "K": 4096, "N": 14336, "density": 10, "criterion": "frob",
         "tokens": 0},
        # weight preparation by the Delta-Hessian score, with calibration tokens
        {"name": "prepare_dhessian", "kind": "prepare", "K": 4096, "N": 4096, "density": 10,
         "criterion": "dhessian", "tokens": 2048},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _shape(rng):
    if rng.random() < 0.6:
        return rng.choice(SHAPES)
    return BLOCK * _log_int(rng, 4, 160), BLOCK * _log_int(rng, 4, 200)


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "step", "shared", "a8", "a8", "prepare"])
    density = rng.choice(DENSITIES)
    skew = rng.random() < 0.4
    if kind == "step":
        return {"kind": kind, "M": _log_int(rng, 1, 32), "layers": rng.randint(1, 4), "density": density, "skew": skew}
    K, N = _shape(rng)
    if kind == "prepare":
        while K * N > 4096 * 14336:
            K, N = _shape(rng)
        return {"kind": kind, "K": K, "N": N, "density": max(density, 1),
                "criterion": rng.choice(["frob", "dhessian"]), "tokens": _log_int(rng, 128, 2048)}
    most = int(LARGEST / (2.4 * K * N))
    if kind == "a8":
        most = min(most // 4, 4096)
    case = {"kind": kind, "M": _log_int(rng, 1, max(1, min(8192, most))), "K": K, "N": N, "density": density,
            "skew": skew}
    if kind == "shared":
        case["M"] = max(1, case["M"] // 2)
        case["N2"] = BLOCK * max(1, N // BLOCK // rng.choice([1, 4, 5, 8]))
    return case


# ------------------------------------------------------------------ inputs --
def _generator(seed, stream):
    return torch.Generator(device="cuda").manual_seed(1000003 * int(seed) + stream)


def _blocks(N, K, density):
    return (density * (N // BLOCK) * (K // BLOCK) + 50) // 100


def _weight(N, K, seed, stream):
    """fp32 weight: N(0, 0.02), 0.5 % outliers of 20 times the size."""
    g = _generator(seed, stream)
    w = torch.randn((N, K), generator=g, device="cuda") * 0.02
    return torch.where(torch.rand((N, K), generator=g, device="cuda") < 0.005, w * 20, w)


def _tokens(M, K, seed, stream):
    """fp16 activations: N(0, 1), four channels of 30 times the size."""
    g = _generator(seed, stream)
    x = torch.randn((M, K), generator=g, device="cuda")
    x[:, torch.randperm(K, generator=g, device="cuda")[:4]] *= 30
    return x.half()


def _quantise(x, amax, qmax):
    """(codes, fp16 scale) of Eq. (1): scale fp16(fp32(max) / qmax), codes from
    the correctly rounded fp32 quotient, rounded half to even."""
    s = (amax.double() / qmax).float().half()
    d = s.double()
    q = (x.double() / torch.where(d == 0, torch.ones_like(d), d)).float().round().clamp_(-qmax, qmax)
    return torch.where(d == 0, torch.zeros_like(q), q), s


def _base(w):
    """Base codes and scales of fp32 w [N, K], one scale per row and 128 columns."""
    N, K = w.shape
    v = w.view(N, K // BLOCK, BLOCK)
    q, s = _quantise(v, v.abs().amax(2, keepdim=True), 7)
    return q, s


def _residual(w, q, s):
    """fp32 residual w - s q, one rounding, as [N/128, 128, K/128, 128]."""
    N, K = w.shape
    r = (w.view(N, K // BLOCK, BLOCK).double() - s.double() * q.double()).float()
    return r.view(N // BLOCK, BLOCK, K // BLOCK, BLOCK)


def _csr(mask):
    rowptr = torch.zeros(mask.shape[0] + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = mask.sum(1).cumsum(0).int()
    return rowptr, mask.nonzero()[:, 1].int().contiguous()


def _mask(N, K, density, skew, seed, stream):
    """Which blocks have a residual: spread evenly, or (skew) four fifths of
    them in eight hot block rows."""
    g = _generator(seed, stream)
    NB, KB = N // BLOCK, K // BLOCK
    n = _blocks(N, K, density)
    key = torch.rand((NB, KB), generator=g, device="cuda")
    hot = torch.zeros((NB, KB), dtype=torch.bool, device="cuda")
    hot[torch.randperm(NB, generator=g, device="cuda")[:8]] = True
    n_hot = min(int(round(0.8 * n)), int(hot.sum())) if skew else 0
    mask = torch.zeros(NB * KB, dtype=torch.bool, device="cuda")
    if n_hot:
        mask[torch.where(hot, key, key + 2).view(-1).topk(n_hot, largest=False).indices] = True
    if n > n_hot:
        rest = torch.where(mask.view(NB, KB), key + 8, key + 4 * hot if skew else key)
        mask[rest.view(-1).topk(n - n_hot, largest=False).indices] = True
    return mask.view(NB, KB)


def _checkpoint(N, K, density, skew, seed, stream):
    """Codes and scales of one quantised layer: q [N, K/128, 128], s, the block
    mask, rq [n, 128, 128] and sr [n, 128, 1]."""
    w = _weight(N, K, seed, stream)
    q, s = _base(w)
    mask = _mask(N, K, density, skew, seed, stream + 1)
    r = _residual(w, q, s).permute(0, 2, 1, 3)[mask]
    rq, sr = _quantise(r, r.abs().amax(2, keepdim=True), 7)
    return q.to(torch.int8), s, mask, rq.to(torch.int8), sr


def _nibbles(q):
    b = q.view(torch.uint8) & 15
    return (b[..., 0::2] | (b[..., 1::2] << 4)).contiguous()


def _packed(N, K, density, skew, seed, stream):
    """The layer as a loader leaves it: repacked into the library's layout."""
    q, s, mask, rq, sr = _checkpoint(N, K, density, skew, seed, stream)
    rowptr, kb = _csr(mask)
    return mq.repack_weights(_nibbles(q).view(N, K // 2), s.view(N, K // BLOCK), rowptr, kb, _nibbles(rq),
                             sr.view(-1, BLOCK).contiguous())


def _step_shapes(case):
    """(layer, operator, K, N, stream of its weight) of a decode step."""
    return [(i, j, K, N, 100 + 10 * (4 * i + j)) for i in range(case["layers"])
            for j, (K, N) in enumerate(STEP_OPS)]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "prepare":
        x = _tokens(case["tokens"], case["K"], seed, 2) if case["criterion"] == "dhessian" else None
        return {"kind": kind, "w": _weight(case["N"], case["K"], seed, 10), "x": x, "criterion": case["criterion"],
                "nnzb": _blocks(case["N"], case["K"], case["density"])}
    M = case["M"]
    if kind == "step":
        calls, need = [], 1
        xs = [_tokens(M, K, seed, 2 + j) for j, (K, _) in enumerate(STEP_OPS)]
        for _, j, K, N, stream in _step_shapes(case):
            calls.append((xs[j], _packed(N, K, case["density"], case["skew"], seed, stream),
                          torch.empty((M, N), dtype=torch.float16, device="cuda")))
            need = max(need, mq.linear_workspace_bytes(M, N, K))
        workspace = torch.empty(need, dtype=torch.uint8, device="cuda")

        def step():
            for x, pw, y in calls:
                mq.linear(x, pw, out=y, workspace=workspace)

        step()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            step()
        return {"kind": kind, "graph": graph, "calls": calls, "workspace": workspace}
    K = case["K"]
    widths = [case["N"]] + ([case["N2"]] * 2 if kind == "shared" else [])
    weights = [_packed(N, K, case["density"], case["skew"], seed, 100 + 10 * i) for i, N in enumerate(widths)]
    return {"kind": kind, "x": _tokens(M, K, seed, 2), "weights": weights}


def run(state):
    kind = state["kind"]
    if kind == "linear":
        return mq.linear(state["x"], state["weights"][0])
    if kind == "step":
        state["graph"].replay()
        return [y for _, _, y in state["calls"]]
    if kind == "shared":
        xq, s_x = mq.quantize_act(state["x"])
        return [mq.fused_gemm(xq, s_x, pw) for pw in state["weights"]]
    if kind == "a8":
        xq, s_x = mq.quantize_act8(state["x"])
        return mq.fused_gemm_a8(xq, s_x, state["weights"][0])
    pw = mq.prepare_weight(state["w"], state["nnzb"], state["criterion"], state["x"])
    return {"Wq": pw.Wq, "s_w": pw.s_w, "rowptr": pw.rowptr, "kb": pw.kb, "Rq": pw.Rq, "s_r": pw.s_r,
            "score": pw.score}


# ------------------------------------------------------------ work, checks --
def _layer_work(M, N, K, density, input_bytes):
    n = _blocks(N, K, density)
    return (N * K / 2 + N * K / 64 + n * (BLOCK * 64 + 2 * BLOCK + 4) + 4 * (N // BLOCK + 1) + input_bytes
            + 2.0 * M * N, 2.0 * M * (N * K + n * BLOCK * BLOCK))


def work(case):
    kind = case["kind"]
    if kind == "prepare":
        N, K = case["N"], case["K"]
        n, T = _blocks(N, K, case["density"]), case["tokens"] if case["criterion"] == "dhessian" else 0
        return {"bytes": 4.0 * N * K + N * K / 2 + N * K / 64 + 8 * (N // BLOCK) * (K // BLOCK)
                + n * (BLOCK * 64 + 2 * BLOCK + 4) + 4 * (N // BLOCK + 1) + 2.0 * T * K,
                "flops": 6.0 * N * K + 2.0 * T * K}
    M = case["M"]
    if kind == "step":
        parts = [_layer_work(M, N, K, case["density"], 2.0 * M * K) for _, _, K, N, _ in _step_shapes(case)]
    else:
        widths = [case["N"]] + ([case["N2"]] * 2 if kind == "shared" else [])
        parts = [_layer_work(M, N, case["K"], case["density"], 2.0 * M * case["K"] if i == 0 else 0.0)
                 for i, N in enumerate(widths)]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


def tolerance(case):
    # prepare: codes, scales and the selection are fixed by the method; the
    # scores are fp64 sums of up to 2^14 terms.  Layers: the integer group sums
    # are exact and added in fp32, the result is rounded to fp16 once (2^-11 at
    # most, about 2.1e-4 in the 2-norm against 64 bits).
    if case["kind"] == "prepare":
        return {"rel": 1e-12, "differ": 0.0}
    return {"rel": 8e-4, "max": 4e-3}


def _tokens64(x, qmax):
    q, s = _quantise(x, x.abs().amax(1, keepdim=True), qmax)
    return q.double(), s.double()


def _layer64(xq, sx, N, K, density, skew, seed, stream):
    q, s, mask, rq, sr = _checkpoint(N, K, density, skew, seed, stream)
    w = (q.double() * s.double()).view(N // BLOCK, BLOCK, K // BLOCK, BLOCK).permute(0, 2, 1, 3)
    w[mask] += rq.double() * sr.double()
    return sx * (xq @ w.permute(0, 2, 1, 3).reshape(N, K).t())


def _scores64(case, seed, w, q, s):
    r = _residual(w, q, s)
    if case["criterion"] == "frob":
        return r.double().square().sum((1, 3))
    h = 2.0 / case["tokens"] * _tokens(case["tokens"], case["K"], seed, 2).double().square().sum(0)
    rq, sr = _quantise(r, r.abs().amax(3, keepdim=True), 7)
    h = h.view(1, 1, -1, BLOCK)
    e = (r.double() - sr.double() * rq.double()).square()
    return ((h * r.double().square()).sum((1, 3)) - (h * e).sum((1, 3))).clamp(min=0)


def exact(case, seed):
    kind = case["kind"]
    if kind == "prepare":
        N, K = case["N"], case["K"]
        w = _weight(N, K, seed, 10)
        q, s = _base(w)
        score = _scores64(case, seed, w, q, s)
        n = _blocks(N, K, case["density"])
        mask = torch.zeros(score.numel(), dtype=torch.bool, device="cuda")
        mask[score.view(-1).sort(descending=True, stable=True).indices[:n]] = True
        rowptr, kb = _csr(mask.view(score.shape))
        r = _residual(w, q, s).permute(0, 2, 1, 3)[mask.view(score.shape)]
        _, sr = _quantise(r, r.abs().amax(2, keepdim=True), 7)
        # (s_w is held in the library's [K/128][N] order; packed codes: none)
        return {"Wq": None, "s_w": s.double().view(N, K // BLOCK).t().reshape(N, K // BLOCK), "rowptr": rowptr,
                "kb": kb, "Rq": None, "s_r": sr.double().view(-1, BLOCK), "score": score}
    M = case["M"]
    if kind == "step":
        xs = [_tokens64(_tokens(M, K, seed, 2 + j), 7) for j, (K, _) in enumerate(STEP_OPS)]
        return [_layer64(*xs[j], N, K, case["density"], case["skew"], seed, stream)
                for _, j, K, N, stream in _step_shapes(case)]
    K = case["K"]
    xq, sx = _tokens64(_tokens(M, K, seed, 2), 127 if kind == "a8" else 7)
    widths = [case["N"]] + ([case["N2"]] * 2 if kind == "shared" else [])
    ys = [_layer64(xq, sx, N, K, case["density"], case["skew"], seed, 100 + 10 * i) for i, N in enumerate(widths)]
    return ys if kind == "shared" else ys[0]
