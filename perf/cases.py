"""The workloads whose time matters for this library, as plain cases.

A case is a dict of plain values.  `kind` names the operator it calls through
the Python binding:

* "attention": O = softmax(scale Q K^T) V over [B, H, L, d] tensors through
  `attn_fwd`, or through `attn_fwd_noalloc` (`entry`), which serving loops and
  graph captures call;
* "softmax": the row softmax, plain or over stacked causal score blocks;
* "gemm": C = A B with 16-bit or fp32 inputs and an fp32 result.

`listed()` holds the named workloads of the package (inputs.py) and a few
generic ones beside them; `draw()` gives others of the same ranges.  Inputs are
N(0, 1) values made on the GPU from the seed, rounded once to the storage type,
K optionally multiplied by a constant; every output is returned whole.
"""
import math

import torch

from paper_2609_10937_amd import capi

_TORCH = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
_BYTES = {"bf16": 2, "f16": 2, "f32": 4}


def _attention(B, H, L, d, dtype="bf16", causal=False, k_scale=1.0, entry="fwd"):
    return {"kind": "attention", "B": B, "H": H, "L": L, "d": d, "dtype": dtype, "causal": causal,
            "k_scale": k_scale, "entry": entry}


def _softmax(rows, n, dtype="bf16", causal=False):
    return {"kind": "softmax", "rows": rows, "n": n, "dtype": dtype, "causal": causal}


def _gemm(M, N, K, dtype="bf16"):
    return {"kind": "gemm", "M": M, "N": N, "K": K, "dtype": dtype}


def listed():
    return [
        # One short head: the smallest call, where the launch and the host path are the time.
        dict(_attention(1, 1, 128, 64, "f16"), name="attn_tiny_f16_l128_d64"),
        # A short prompt with few heads: a few microseconds of work spread over the whole chip.
        dict(_attention(1, 8, 1024, 128), name="attn_h8_l1024_d128"),
        # The headline workload: one long head, which alone has too few query tiles for the chip.
        dict(_attention(1, 1, 16384, 128), name="attn_single_head_l16384_d128"),
        # A batched causal prefill of ordinary length, with logits that keep raising the running maximum.
        dict(_attention(2, 16, 4096, 128, causal=True, k_scale=3.0), name="attn_causal_b2h16_l4096_d128_kx3"),
        # The largest: a batched causal prefill of long sequences at full occupancy.
        dict(_attention(4, 32, 16384, 128, causal=True), name="attn_causal_b4h32_l16384_d128"),
        # Many heads of short sequences: thousands of short query tiles.
        dict(_attention(1, 1024, 512, 128), name="attn_heads1024_l512_d128"),
        # A serving call that may not allocate: odd length, small heads, f16, causal.
        dict(_attention(2, 8, 1999, 64, "f16", True, entry="noalloc"), name="attn_noalloc_causal_b2h8_l1999_d64_f16"),
        # The largest head dimension, causal, ordinary length.
        dict(_attention(1, 16, 4096, 256, causal=True), name="attn_causal_h16_l4096_d256"),
        # The scores of one head at L = 16384: memory bound.
        dict(_softmax(16384, 16384), name="softmax_16384x16384"),
        # Causal score blocks of an odd length, f16: rows without 16-byte alignment.
        dict(_softmax(4 * 2049, 2049, "f16", True), name="softmax_causal_4x2049_f16"),
        # The square product of the paper's worked example.
        dict(_gemm(4096, 4096, 4096), name="gemm_4096_bf16"),
        # fp32, the type of that example, with ragged sides.
        dict(_gemm(2999, 2500, 1500, "f32"), name="gemm_2999x2500x1500_f32"),
    ]


# A drawn case costs no more than the largest listed one: 2 B H L^2 d multiply
# and add operations of causal attention at B = 4, H = 32, L = 16384, d = 128.
_MOST_FLOPS = 2.0 * 4 * 32 * 16384.0 ** 2 * 128


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attention", "attention", "attention", "softmax", "gemm"])
    if kind == "attention":
        d = rng.choice([64, 96, 128, 128, 256])
        L = _log_int(rng, 100, 16384)
        if rng.random() < 0.4:
            L = max(128, L // 128 * 128)
        causal = rng.random() < 0.5
        B, H = rng.choice([1, 1, 2, 4]), _log_int(rng, 1, 128)
        case = _attention(B, H, L, d, rng.choice(["bf16", "f16"]), causal, rng.choice([1.0, 1.0, 3.0]))
        while work(case)["flops"] > _MOST_FLOPS:
            case["H"] = max(1, case["H"] // 2)
        # attn_fwd_noalloc takes split plans up to 32 MiB of partial results (at most 16 splits).
        if 16 * case["B"] * case["H"] * L * (2 * d + 8) <= 32 << 20 and rng.random() < 0.5:
            case["entry"] = "noalloc"
        return case
    if kind == "softmax":
        n = _log_int(rng, 128, 32768)
        if rng.random() < 0.5:
            n = max(8, n // 8 * 8)
        dtype = rng.choice(["bf16", "f16"])
        if rng.random() < 0.3 and n <= 8192:
            return _softmax(n * rng.randint(1, max(1, min(32, (1 << 26) // (n * n)))), n, dtype, True)
        return _softmax(_log_int(rng, 16, max(32, min(65536, (1 << 28) // n))), n, dtype)
    dtype = rng.choice(["bf16", "f16", "f32"])
    step, top = (4, 4096) if dtype == "f32" else (8, 8192)
    return _gemm(_log_int(rng, 16, top), step * _log_int(rng, 64 // step, top // step),
                 step * _log_int(rng, 64 // step, top // step), dtype)


def _normal(gen, shape, dtype, times=1.0):
    x = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)
    if times != 1.0:
        x *= times
    return x.to(_TORCH[dtype])


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dt = case["dtype"]
    if case["kind"] == "attention":
        shape = (case["B"], case["H"], case["L"], case["d"])
        return tuple(_normal(gen, shape, dt, m) for m in (1.0, case["k_scale"], 1.0))
    if case["kind"] == "softmax":
        return (_normal(gen, (case["rows"], case["n"]), dt, 2.0),)
    return _normal(gen, (case["M"], case["K"]), dt), _normal(gen, (case["K"], case["N"]), dt)


def _scale(d):
    return float(torch.tensor(1.0) / torch.sqrt(torch.tensor(float(d))))


def prepare(case, seed):
    """The operands and the output buffer."""
    x = _inputs(case, seed)
    if case["kind"] == "gemm":
        out = torch.empty((case["M"], case["N"]), dtype=torch.float32, device="cuda")
    else:
        out = torch.empty_like(x[0])
    return {"case": case, "in": x, "out": out,
            "scale": _scale(case["d"]) if case["kind"] == "attention" else None}


def run(state):
    case, x, out = state["case"], state["in"], state["out"]
    if case["kind"] == "attention":
        fn = capi.attn_fwd_noalloc if case["entry"] == "noalloc" else capi.attn_fwd
        fn(x[0], x[1], x[2], out, state["scale"], case["causal"])
    elif case["kind"] == "softmax":
        capi.attn_softmax(x[0], out, causal=case["causal"])
    else:
        capi.attn_gemm(x[0], x[1], out)
    return out


def work(case):
    e = _BYTES[case["dtype"]]
    if case["kind"] == "attention":
        B, H, L, d = case["B"], case["H"], case["L"], case["d"]
        pairs = L * (L + 1) / 2 if case["causal"] else L * L
        return {"bytes": 4.0 * B * H * L * d * e, "flops": 4.0 * B * H * pairs * d}
    if case["kind"] == "softmax":
        # Causal: the columns above the diagonal are written, not read.
        rows, n = case["rows"], case["n"]
        read = rows * (n + 1) / 2 if case["causal"] else rows * n
        return {"bytes": (read + rows * n) * e, "flops": 0.0}
    M, N, K = case["M"], case["N"], case["K"]
    return {"bytes": float((M * K + K * N) * e + M * N * 4), "flops": 2.0 * M * N * K}


def tolerance(case):
    """About four times the 2-norm error against exact(): the rounding of
    the 16-bit result and, for attention, of the 16-bit weights and of a split's
    partial results; for the products, fp32 sums in any order."""
    if case["kind"] == "gemm":
        return {"rel": 5e-6 if case["dtype"] == "f32" else 3e-6}
    return {"rel": 1e-2 if case["dtype"] == "bf16" else 1.2e-3}


def exact(case, seed):
    """The same outputs in 64 bits: plain torch products, one head at a time."""
    x = _inputs(case, seed)
    if case["kind"] == "gemm":
        return x[0].double() @ x[1].double()
    if case["kind"] == "softmax":
        s = x[0].double()
        if case["causal"]:
            n = case["n"]
            above = torch.ones((n, n), dtype=torch.bool, device="cuda").triu_(1)
            for b in range(case["rows"] // n):
                s[b * n:(b + 1) * n].masked_fill_(above, -math.inf)
        s -= s.amax(dim=1, keepdim=True)
        s.exp_()
        s /= s.sum(dim=1, keepdim=True)
        return s
    B, H, L, d = case["B"], case["H"], case["L"], case["d"]
    scale = _scale(d)
    out = torch.empty((B, H, L, d), dtype=torch.float64, device="cuda")
    cols = torch.arange(L, device="cuda")
    for b in range(B):
        for h in range(H):
            q, k, v = (t[b, h].double() for t in x)
            kt = k.t().contiguous()
            for r0 in range(0, L, 4096):
                r1 = min(L, r0 + 4096)
                end = r1 if case["causal"] else L
                s = q[r0:r1] @ kt[:, :end].contiguous()
                s *= scale
                if case["causal"]:
                    s.masked_fill_(cols[None, :end] > cols[r0:r1, None], -math.inf)
                s -= s.amax(dim=1, keepdim=True)
                s.exp_()
                s /= s.sum(dim=1, keepdim=True)
                out[b, h, r0:r1] = s @ v[:end]
    return out
