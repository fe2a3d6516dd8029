"""The calls whose speed counts, as a serving or encoding program makes them.

Six kinds of case, each through the public Python entry points:

* ``call``: one projection, called by itself (``pq_gemv``);
* ``layer``: the projections of a decoder layer for one decode step, recorded
  once as a launch list and replayed, as a serving loop does: q + k + v and
  gate + up grouped (``pq_gemv_batched``), o and down alone with a workspace
  (``pq_gemv_ex``), and in one case the output head;
* ``prefill``: one projection over the tokens of a prompt (``pq_gemm_ex``);
* ``subspace``: one projection with a codebook per subspace (``pq_gemv_ex``),
  from one token to a short prompt;
* ``ragged``: one projection whose sizes fit no tile, word or id group
  (``pq_gemm``);
* ``encode``: k-means encoding of a dense weight matrix (``pq_encode``).

A format is (id bits, sub-vector length d, codewords C).  Codebooks, ids and
activations follow the recipe of the repository's synthetic workloads: N(0,
0.02) codewords, uniform ids, N(0, 1) activations, all fp16; weights to encode
are N(0, 0.02).
"""

import math

import torch

import paper_2605_04084_amd as fasq

# effective 4, 2, 3 and 4 bits per weight
FORMATS = {"b8d2": (8, 2, 256), "b8d4": (8, 4, 256), "b12d4": (12, 4, 4096), "b16d4": (16, 4, 65536)}


def listed():
    return [
        # the smallest unit of work: one key projection for one token, called
        # from Python (latency of a call)
        {"name": "call_k_proj", "kind": "call", "bits": 8, "d": 2, "C": 256, "M": 1, "K": 4096, "N": 1024},
        # token-by-token decode of a Llama-3-8B layer at effective 4 bits
        {"name": "layer_b8d2_m1", "kind": "layer", "fmt": "b8d2", "M": 1, "hidden": 4096, "kv": 1024, "ffn": 14336, "head": 0},
        # the same at effective 3 bits, with the output head that ends the step
        {"name": "layer_b12d4_m1_head", "kind": "layer", "fmt": "b12d4", "M": 1, "hidden": 4096, "kv": 1024, "ffn": 14336, "head": 128256},
        # a few concurrent sequences on the Qwen3-8B layer with its 65536-entry codebooks
        {"name": "layer_b16d4_m4", "kind": "layer", "fmt": "b16d4", "M": 4, "hidden": 4096, "kv": 1024, "ffn": 12288, "head": 0},
        # a full decode batch on the effective-4-bit layer
        {"name": "layer_b8d2_m16", "kind": "layer", "fmt": "b8d2", "M": 16, "hidden": 4096, "kv": 1024, "ffn": 14336, "head": 0},
        # the paper's general layout (a codebook per subspace), one decode token
        {"name": "subspace_m1", "kind": "subspace", "bits": 8, "d": 2, "C": 256, "M": 1, "K": 4096, "N": 4096},
        # the same layer over a short prompt
        {"name": "subspace_m48", "kind": "subspace", "bits": 8, "d": 2, "C": 256, "M": 48, "K": 4096, "N": 4096},
        # a chat turn through the q projection
        {"name": "prefill_b8d2_m128", "kind": "prefill", "fmt": "b8d2", "M": 128, "K": 4096, "N": 4096},
        # a long prompt through the gate projection at effective 3 bits
        {"name": "prefill_b12d4_m2048", "kind": "prefill", "fmt": "b12d4", "M": 2048, "K": 4096, "N": 14336},
        # a page of text through the 65536-entry format
        {"name": "prefill_b16d4_m512", "kind": "prefill", "fmt": "b16d4", "M": 512, "K": 4096, "N": 4096},
        # a small odd-sized projection (an adapter or a task head) over a few tokens
        {"name": "ragged_m37", "kind": "ragged", "bits": 8, "d": 4, "C": 256, "M": 37, "K": 1516, "N": 1003},
        # offline: one attention projection into the effective-3-bit format
        {"name": "encode_b12d4", "kind": "encode", "bits": 12, "d": 4, "C": 4096, "K": 4096, "N": 4096, "iters": 4},
    ]


def _log_int(rng, lo, hi, step=1):
    """An integer multiple of ``step`` in [lo, hi], uniform over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(max(int(round(v / step)), -(-lo // step)), hi // step) * step


def draw(rng):
    kind = rng.choice(["call", "layer", "layer", "prefill", "prefill", "subspace", "ragged", "encode"])
    if kind == "call":
        bits, d, C = rng.choice(list(FORMATS.values()) + [(8, 1, 256), (8, 2, 64), (8, 8, 256)])
        return {"kind": kind, "bits": bits, "d": d, "C": C, "M": rng.choice([1, 1, 2, 3, 8]),
                "K": _log_int(rng, 512, 8192, 128), "N": _log_int(rng, 256, 8192)}
    if kind == "layer":
        fmt = rng.choice(["b8d2", "b8d2", "b12d4", "b16d4", "b8d4"])
        hidden = _log_int(rng, 1024, 4096, 128)
        return {"kind": kind, "fmt": fmt, "M": rng.choice([1, 1, 2, 4, 7, 8, 13, 16]), "hidden": hidden,
                "kv": max(128, hidden // rng.choice([1, 4, 8]) // 8 * 8),
                "ffn": _log_int(rng, 2 * hidden, int(3.5 * hidden), 128),
                "head": rng.choice([0, 0, 0, _log_int(rng, 16000, 64000)])}
    if kind == "prefill":
        fmt = rng.choice(["b8d2", "b8d4", "b12d4", "b16d4"])
        return {"kind": kind, "fmt": fmt, "M": _log_int(rng, 17, 512 if fmt == "b16d4" else 2048),
                "K": _log_int(rng, 1024, 4096, 64), "N": _log_int(rng, 1024, 4096 if fmt == "b16d4" else 14336)}
    if kind == "subspace":
        bits, d, C = rng.choice([(8, 2, 256), (8, 2, 256), (8, 4, 256), (8, 1, 64), (8, 2, 100), (12, 4, 512)])
        return {"kind": kind, "bits": bits, "d": d, "C": C, "M": rng.choice([1, 1, 3, 16, _log_int(rng, 17, 64)]),
                "K": _log_int(rng, 512, 4096, 128), "N": _log_int(rng, 256, 4096)}
    if kind == "ragged":
        bits, d, C = rng.choice([(8, 4, 256), (8, 3, 256), (8, 2, 200), (12, 4, 1000), (8, 6, 256), (16, 2, 5000)])
        return {"kind": kind, "bits": bits, "d": d, "C": C, "M": _log_int(rng, 1, 64),
                "K": _log_int(rng, 150, 2100) // d * d, "N": _log_int(rng, 100, 2100)}
    bits, d, C = rng.choice([(8, 2, 256), (8, 4, 256), (12, 4, 4096), (8, 8, 256), (8, 1, 16), (16, 4, 16384), (8, 3, 200)])
    K = _log_int(rng, 512, 4096, 8) // d * d
    iters = rng.choice([1, 2, 4])
    rows = int(80e9 / (iters + 1) / C / (K // d))  # no more distances than the listed encoding
    return {"kind": "encode", "bits": bits, "d": d, "C": C, "K": K, "N": _log_int(rng, 256, max(257, min(4096, rows))), "iters": iters}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, shape, std):
    return (torch.randn(shape, generator=g, device="cuda") * std).to(torch.float16)


def _ids(g, N, S, bits, C):
    """Packed uniform ids in [0, C): uint8 [N x R]."""
    R = (S * bits + 7) // 8
    if C == 1 << bits and S * bits % 8 == 0:  # every bit pattern is an id
        return torch.randint(0, 256, (N, R), generator=g, device="cuda", dtype=torch.uint8)
    u = torch.randint(0, C, (N, S), generator=g, device="cuda", dtype=torch.int32)
    if bits == 8:
        return u.to(torch.uint8)
    if bits == 16:
        return torch.stack([u & 255, u >> 8], 2).to(torch.uint8).reshape(N, R)
    if S % 2:
        u = torch.cat([u, torch.zeros_like(u[:, :1])], 1)
    a, b = u[:, 0::2], u[:, 1::2]
    packed = torch.stack([a & 255, (a >> 8) | ((b & 15) << 4), b >> 4], 2).to(torch.uint8).reshape(N, -1)
    return packed[:, :R].contiguous()


def _unpack(idx, S, bits):
    """The ids of packed rows, int64 [N x S]."""
    v = idx.to(torch.int64)
    if bits == 8:
        return v
    if bits == 16:
        return v[:, 0::2] | (v[:, 1::2] << 8)
    pad = -v.shape[1] % 3
    if pad:
        v = torch.cat([v, torch.zeros_like(v[:, :pad])], 1)
    t = v.reshape(v.shape[0], -1, 3)
    u = torch.stack([t[:, :, 0] | ((t[:, :, 1] & 15) << 8), (t[:, :, 1] >> 4) | (t[:, :, 2] << 4)], 2)
    return u.reshape(v.shape[0], -1)[:, :S]


def _matrix(g, N, K, bits, d, C):
    cb = _normal(g, (C, d), 0.02)
    return _ids(g, N, K // d, bits, C), cb


def _layer_shapes(case):
    """name, N, K of the layer's matrices, grouped by the activations they read."""
    h, kv, f = case["hidden"], case["kv"], case["ffn"]
    groups = [[("q", h, h), ("k", kv, h), ("v", kv, h)], [("o", h, h)], [("gate", f, h), ("up", f, h)], [("down", h, f)]]
    if case["head"]:
        groups.append([("head", case["head"], h)])
    return groups


def _layer_inputs(case, seed):
    g = _gen(seed)
    bits, d, C = FORMATS[case["fmt"]]
    groups = []
    for mats in _layer_shapes(case):
        x = _normal(g, (case["M"], mats[0][2]), 1.0)
        groups.append((x, [_matrix(g, N, K, bits, d, C) for _, N, K in mats]))
    return groups


def _plain_inputs(case, seed):
    g = _gen(seed)
    bits, d, C = FORMATS[case["fmt"]] if "fmt" in case else (case["bits"], case["d"], case["C"])
    S = case["K"] // d
    x = _normal(g, (case["M"], case["K"]), 1.0)
    cb = _normal(g, (S, C, d) if case["kind"] == "subspace" else (C, d), 0.02)
    return x, _ids(g, case["N"], S, bits, C), cb, bits, d, C


def _encode_inputs(case, seed):
    g = _gen(seed)
    N, K, d, C = case["N"], case["K"], case["d"], case["C"]
    w = _normal(g, (N, K), 0.02)
    pick = torch.randperm(N * (K // d), generator=g, device="cuda")[:C].sort().values
    return w, w.view(-1, d)[pick].contiguous()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "layer":
        groups = _layer_inputs(case, seed)
        bits, d, C = FORMATS[case["fmt"]]
        M, outs, spaces = case["M"], [], []
        lst = fasq.LaunchList()
        with lst:
            for x, mats in groups:
                ys = [torch.empty((M, idx.shape[0]), dtype=torch.float16, device="cuda") for idx, _ in mats]
                if len(mats) > 1:
                    fasq.pq_gemv_batched(x, [m[0] for m in mats], bits, d, [m[1] for m in mats], outs=ys)
                else:
                    idx, cb = mats[0]
                    need = fasq.gemv_ex_workspace_bytes(M, x.shape[1], idx.shape[0], bits, d, C, 0)
                    ws = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
                    fasq.pq_gemv_ex(x, idx, bits, d, cb, out=ys[0], workspace=ws)
                    spaces.append(ws)
                outs += ys
        return {"kind": kind, "list": lst, "outs": outs, "keep": (groups, spaces)}
    if kind == "encode":
        w, init = _encode_inputs(case, seed)
        need = fasq.encode_workspace_bytes(case["N"], case["K"], case["d"], case["C"])
        ws = torch.empty(need, dtype=torch.uint8, device="cuda")
        return {"kind": kind, "args": (w, case["d"], case["bits"], init, case["iters"]), "ws": ws}
    x, idx, cb, bits, d, C = _plain_inputs(case, seed)
    need = 0
    if kind == "prefill":
        need = fasq.gemm_ex_workspace_bytes(case["M"], case["K"], case["N"], bits, d, C)
    elif kind == "subspace":
        need = fasq.gemv_ex_workspace_bytes(case["M"], case["K"], case["N"], bits, d, C, C * d)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
    return {"kind": kind, "args": (x, idx, bits, d, cb), "ws": ws}


def run(state):
    kind = state["kind"]
    if kind == "layer":
        state["list"].run()
        return state["outs"]
    if kind == "call":
        return fasq.pq_gemv(*state["args"])
    if kind == "prefill":
        return fasq.pq_gemm_ex(*state["args"], workspace=state["ws"])
    if kind == "subspace":
        return fasq.pq_gemv_ex(*state["args"], workspace=state["ws"])
    if kind == "ragged":
        return fasq.pq_gemm(*state["args"])
    codebook, idx = fasq.pq_encode(*state["args"], workspace=state["ws"])
    return {"codebook": codebook, "idx": idx}


# ---------------------------------------------------------------------------
# What the path cannot do without
# ---------------------------------------------------------------------------

def _matmul_work(M, K, N, bits, d, cb_values):
    R = (K // d * bits + 7) // 8
    return N * R + 2 * cb_values + 2 * M * K + 2 * M * N, 2 * M * K * N


def work(case):
    kind = case["kind"]
    if kind == "layer":
        bits, d, C = FORMATS[case["fmt"]]
        bytes_, flops = 0, 0
        for mats in _layer_shapes(case):
            for i, (_, N, K) in enumerate(mats):
                b, f = _matmul_work(case["M"], K, N, bits, d, C * d)
                bytes_ += b - (2 * case["M"] * K if i else 0)  # x once per group
                flops += f
        return {"bytes": bytes_, "flops": flops}
    if kind == "encode":
        N, K, d, C = case["N"], case["K"], case["d"], case["C"]
        points = N * (K // d)
        # each input and output once; a distance per point and codeword
        # (2 d operations as a contraction) for every assignment
        return {"bytes": 2 * N * K + 4 * C * d + N * ((K // d * case["bits"] + 7) // 8),
                "flops": (case["iters"] + 1) * points * C * 2 * d}
    bits, d, C = FORMATS[case["fmt"]] if "fmt" in case else (case["bits"], case["d"], case["C"])
    books = case["K"] // d if kind == "subspace" else 1
    b, f = _matmul_work(case["M"], case["K"], case["N"], bits, d, books * C * d)
    return {"bytes": b, "flops": f}


def tolerance(case):
    # the encoder's arithmetic is defined to the bit (fp32 distances without
    # fused multiply-add, exact sums, one rounding)
    if case["kind"] == "encode":
        return "exact"
    # fp32 sums rounded once to fp16: 2.1e-4 off the 64-bit result (2-norm),
    # 4.9e-4 at most of a value or of the result's root mean square
    return {"rel": 8e-4, "max": 2e-3}


# ---------------------------------------------------------------------------
# The same results in 64 bits, by plain torch
# ---------------------------------------------------------------------------

def _exact_matmul(x, idx, bits, d, cb):
    N, (M, K) = idx.shape[0], x.shape
    S = K // d
    x64, out = x.double(), torch.empty((M, N), dtype=torch.float64, device="cuda")
    rows = max(1, (1 << 26) // K)
    for n0 in range(0, N, rows):
        u = _unpack(idx[n0:n0 + rows], S, bits)
        if cb.dim() == 3:
            w = cb[torch.arange(S, device="cuda")[None, :], u]
        else:
            w = cb[u]
        out[:, n0:n0 + rows] = x64 @ w.reshape(-1, K).double().t().contiguous()
    return out


def _exact_assign(points, cb):
    """Nearest codeword by the defined fp32 distance, lowest index on ties."""
    C, d = cb.shape
    order = torch.arange(C, device="cuda", dtype=torch.int32)
    c32, out = cb.float(), torch.empty(points.shape[0], dtype=torch.int64, device="cuda")
    block = max(1, (1 << 27) // C)
    for b0 in range(0, points.shape[0], block):
        p = points[b0:b0 + block].float()
        dist = torch.zeros((p.shape[0], C), device="cuda")
        for i in range(d):
            diff = p[:, i:i + 1] - c32[None, :, i]
            dist += diff * diff
        nearest = dist == dist.amin(1, keepdim=True)
        out[b0:b0 + block] = torch.where(nearest, order, C).amin(1).long()
    return out


def _exact_encode(case, seed):
    w, cb = _encode_inputs(case, seed)
    N, K, d, C, bits = case["N"], case["K"], case["d"], case["C"], case["bits"]
    points = w.view(-1, d)
    q = (points.double() * 2.0 ** 24).long()  # fp16 values are whole multiples of 2^-24
    for _ in range(case["iters"]):
        u = _exact_assign(points, cb)
        sums = torch.zeros((C, d), dtype=torch.int64, device="cuda").index_add_(0, u, q)
        count = torch.bincount(u, minlength=C)
        mean = sums.double() * 2.0 ** -24 / count.double().clamp(min=1)[:, None]
        cb = torch.where(count[:, None] > 0, _to_half(mean), cb)
    u = _exact_assign(points, cb).view(N, K // d).int()
    if bits == 8:
        idx = u.to(torch.uint8)
    elif bits == 16:
        idx = torch.stack([u & 255, u >> 8], 2).to(torch.uint8).reshape(N, -1)
    else:
        if u.shape[1] % 2:
            u = torch.cat([u, torch.zeros_like(u[:, :1])], 1)
        a, b = u[:, 0::2], u[:, 1::2]
        idx = torch.stack([a & 255, (a >> 8) | ((b & 15) << 4), b >> 4], 2).to(torch.uint8).reshape(N, -1)
        idx = idx[:, :(K // d * 12 + 7) // 8].contiguous()
    return {"codebook": cb, "idx": idx}


def _to_half(v):
    """fp64 to fp16 in one rounding (through numpy: torch goes by way of fp32)."""
    return torch.from_numpy(v.cpu().numpy().astype("float16")).cuda()


def exact(case, seed):
    if case["kind"] == "encode":
        return _exact_encode(case, seed)
    if case["kind"] == "layer":
        bits, d, _ = FORMATS[case["fmt"]]
        return [_exact_matmul(x, idx, bits, d, cb) for x, mats in _layer_inputs(case, seed) for idx, cb in mats]
    x, idx, cb, bits, d, _ = _plain_inputs(case, seed)
    return _exact_matmul(x, idx, bits, d, cb)
