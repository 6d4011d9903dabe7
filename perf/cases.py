"""Performance cases of the library: calls that its users make, over the range they make them in.

Every case goes through the public entry points (``cqsa_plan`` once, in ``prepare``; then ``cqsa_forward``,
``cqsa_forward_noalloc`` and ``cqsa_backward``).  A case is a dict of plain values:

  op        "fwd" (forward), "noalloc" (the forward that allocates nothing), "bwd" (backward after a forward made
            beforehand), "fwd_bwd" (a training step's attention: forward, then backward)
  dtype     "bf16", "f16" or "f32"; B, L, H, d: the [B, L, H, d] tensors; causal
  depth     CQS depth (0: undecomposed, -1: automatic, the smallest that fits the budget)
  c         chunk count of the interest set (7, 13 or 21)
  budget_mb device budget in MB (10^6 bytes; 0: uncapped)
  host      True: all tensors in pinned host memory, tasks streamed through the device
  out16     True: O in the input dtype
"""
import math

import torch

import paper_2604_20819_amd as cq

INTEREST = {7: (0, 1, 3), 13: (0, 1, 3, 9), 21: (0, 1, 4, 14, 16)}
# task tokens over call tokens at depth 1: every token lies in l tasks (rounding up included)
INTEREST_TOKENS = {7: 3.1, 13: 4.2, 21: 5.3}
TORCH = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}


def _case(op, dtype, L, H, d, B=1, causal=False, depth=1, c=7, budget_mb=0, host=False, out16=False):
    return dict(op=op, dtype=dtype, B=B, L=L, H=H, d=d, causal=causal, depth=depth, c=c, budget_mb=budget_mb, host=host,
                out16=out16)


def listed():
    cases = {
        # the exactness check in fp32 at its size: the smallest call, where launches and latency count
        "f32_L1024_fwd": _case("fwd", "f32", 1024, 1, 64),
        # a serving loop that may not allocate: a short prompt, a few heads, a length that is no multiple of a tile
        "bf16_L3000_noalloc": _case("noalloc", "bf16", 3000, 4, 128),
        # a short causal training step, undecomposed: the launch holds few work groups
        "f16_L2048_fwd_bwd_undecomposed": _case("fwd_bwd", "f16", 2048, 8, 64, causal=True, depth=0),
        # ragged everything: odd length, batch 2, three heads, d = 96, another interest set, 16-bit O
        "bf16_L5003_d96_c13_out16": _case("fwd", "bf16", 5003, 3, 96, B=2, c=13, out16=True),
        # the paper's shape (fp16, causal, H = 8, d = 64) at the short end of its length sweep, forward and backward
        "f16_L8192_fwd_bwd": _case("fwd_bwd", "f16", 8192, 8, 64, causal=True),
        # the same shape undecomposed, as the ratio against the decomposed call needs it
        "f16_L16384_fwd_undecomposed": _case("fwd", "f16", 16384, 8, 64, causal=True, depth=0),
        # the widest head dim, forward and backward
        "bf16_L16384_d256_fwd_bwd": _case("fwd_bwd", "bf16", 16384, 8, 256),
        # one level of decomposition, uncapped: the forward and the backward of the middle-sized workload
        "bf16_L32768_fwd": _case("fwd", "bf16", 32768, 16, 128),
        "bf16_L32768_bwd": _case("bwd", "bf16", 32768, 16, 128),
        # out of core: everything in pinned host memory, the budget an eighth of the 1M-token headline's for an
        # eighth of its tokens (two levels, accumulator on the host)
        "bf16_L131072_host_500MB_fwd": _case("fwd", "bf16", 131072, 8, 128, depth=-1, budget_mb=500, host=True),
        # a long causal prefill under an 8 GB budget
        "f16_L131072_8GB_fwd": _case("fwd", "f16", 131072, 32, 128, causal=True, depth=-1, budget_mb=8000),
        # a long causal training step, batch 2, under a 16 GB budget: the largest
        "bf16_B2_L65536_16GB_fwd_bwd": _case("fwd_bwd", "bf16", 65536, 16, 128, B=2, causal=True, depth=-1, budget_mb=16000),
    }
    return [dict(name=n, **c) for n, c in cases.items()]


def _pairs(case):
    L = case["L"]
    return L * (L + 1) // 2 if case["causal"] else L * L


def _flops(case):
    per = {"fwd": 4, "noalloc": 4, "bwd": 10, "fwd_bwd": 14}[case["op"]]
    return float(per * case["d"] * case["B"] * case["H"] * _pairs(case))


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more call: short to 64K tokens, every dtype, head dim, depth and direction."""
    kind = rng.choices(("fwd", "fwd_bwd", "bwd", "noalloc", "f32", "host"), (30, 20, 15, 12, 13, 10))[0]
    d = rng.choice((32, 64, 64, 64, 96, 128, 128, 128, 160, 192, 224, 256))
    H = rng.choice((1, 2, 3, 4, 5, 8, 8, 12, 16, 16, 24, 32))
    B = rng.choice((1, 1, 1, 1, 2, 3))
    causal = rng.random() < 0.6
    dtype = rng.choice(("bf16", "bf16", "f16"))
    depth = rng.choice((0, 1, 1, 1, 1, 2))
    c = rng.choice((7, 7, 7, 7, 7, 7, 7, 13, 21)) if depth == 1 else 7
    if kind == "f32":
        return _case("fwd", "f32", _log_int(rng, 256, 4096), min(H, 8), d, B, causal, depth, c)
    if kind == "host":
        return _case("fwd", dtype, _log_int(rng, 4096, 65536), rng.choice((4, 8)), rng.choice((64, 128)), 1, causal,
                     rng.choice((1, 2)), 7, 0, True)
    if kind == "noalloc":
        # the task statistics (and, undecomposed, nothing but the plan) have to fit the fixed scratch
        tokens = {0: 0, 1: INTEREST_TOKENS[c], 2: 9}[depth] * H * B * (4 * d + 12)
        top = 16384 if tokens == 0 else max(300, min(16384, int(0.85 * (64 << 20) / tokens)))
        L = _log_int(rng, 256, top)
        return _case("noalloc", dtype, L, H, d, B, causal, depth, c)
    case = _case(kind, dtype, _log_int(rng, 256, 65536), H, d, B, causal, depth, c,
                 out16=kind == "fwd" and rng.random() < 0.25)
    # no more than a fifth of the largest listed case's products: the least favourable shapes cost five times as much each
    while _flops(case) > 4e13:
        case["L"] = int(case["L"] * 0.7)
    return case


def _inputs(case, seed, n):
    """n standard-normal [B, L, H, d] tensors on the GPU (zero mean, unit variance, as the method is evaluated on)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    shape = (case["B"], case["L"], case["H"], case["d"])
    return [torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).to(TORCH[case["dtype"]]) for _ in range(n)]


def _wants_backward(case):
    return case["op"] in ("bwd", "fwd_bwd")


def prepare(case, seed):
    host, bwd = case["host"], _wants_backward(case)
    opts = cq.make_opts(B=case["B"], dtype=case["dtype"], c=case["c"], interest=INTEREST[case["c"]], depth=case["depth"],
                        inputs_on_device=not host, acc_on_device=not host, with_backward=bwd, out16=case["out16"])
    plan = cq.cqsa_plan(case["L"], case["H"], case["d"], case["causal"], case["budget_mb"] * 10 ** 6, opts)
    ins = _inputs(case, seed, 4 if bwd else 3)
    if host:
        pinned = [torch.empty(x.shape, dtype=x.dtype, pin_memory=True) for x in ins]
        for p, x in zip(pinned, ins):
            p.copy_(x)
        ins = pinned

    def out(*shape, dtype=torch.float32):
        return torch.empty(shape, dtype=dtype, pin_memory=True) if host else torch.empty(shape, dtype=dtype, device="cuda")

    shape = (case["B"], case["L"], case["H"], case["d"])
    state = dict(op=case["op"], plan=plan, Q=ins[0], K=ins[1], V=ins[2],
                 O=out(*shape, dtype=TORCH[case["dtype"]] if case["out16"] else torch.float32),
                 LSE=out(case["B"], case["H"], case["L"]))
    if bwd:
        state.update(dO=ins[3], dQ=out(*shape), dK=out(*shape), dV=out(*shape))
    if case["op"] == "bwd":
        cq.cqsa_forward(plan, state["Q"], state["K"], state["V"], state["O"], state["LSE"])
    return state


def run(s):
    res = {}
    if s["op"] == "noalloc":
        cq.cqsa_forward_noalloc(s["plan"], s["Q"], s["K"], s["V"], s["O"], s["LSE"])
    elif s["op"] != "bwd":
        cq.cqsa_forward(s["plan"], s["Q"], s["K"], s["V"], s["O"], s["LSE"])
    if s["op"] != "bwd":
        res.update(O=s["O"], LSE=s["LSE"])
    if s["op"] in ("bwd", "fwd_bwd"):
        cq.cqsa_backward(s["plan"], s["Q"], s["K"], s["V"], s["O"], s["LSE"], s["dO"], s["dQ"], s["dK"], s["dV"])
        res.update(dQ=s["dQ"], dK=s["dK"], dV=s["dV"])
    return res


def work(case):
    """Each input read once and each output written once; 2 d operations per product of a kept pair (2 products forward,
    5 backward)."""
    elems = case["B"] * case["L"] * case["H"] * case["d"]
    rows = case["B"] * case["L"] * case["H"]
    e = 4 if case["dtype"] == "f32" else 2
    fwd = elems * (3 * e + (e if case["out16"] else 4)) + 4 * rows
    bwd = elems * (4 * e + 4 + 3 * 4) + 4 * rows
    bytes_ = {"fwd": fwd, "noalloc": fwd, "bwd": bwd, "fwd_bwd": fwd + bwd}[case["op"]]
    return {"bytes": float(bytes_), "flops": _flops(case)}


def tolerance(case):
    """Relative 2-norm; about four times the distance to the 64-bit result.  16-bit calls round P (and dS) to the input
    dtype before the second product; fp32 calls differ by the order of their sums."""
    return {"rel": {"bf16": 8e-3, "f16": 1e-3, "f32": 2e-6}[case["dtype"]]}


def exact(case, seed):
    """Dense attention in float64, one (batch, head) and a block of query rows at a time; causal blocks stop at their last
    row's key."""
    bwd = _wants_backward(case)
    B, L, H, d, causal = case["B"], case["L"], case["H"], case["d"], case["causal"]
    ins = _inputs(case, seed, 4 if bwd else 3)
    scale = 1.0 / math.sqrt(d)
    rows = max(64, min(L, (1 << 28) // L))
    O = torch.empty((B, L, H, d), dtype=torch.float64, device="cuda")
    LSE = torch.empty((B, H, L), dtype=torch.float64, device="cuda")
    G = [torch.zeros((B, L, H, d), dtype=torch.float64, device="cuda") for _ in range(3)] if bwd else []
    idx = torch.arange(L, device="cuda")
    for b in range(B):
        for h in range(H):
            q, k, v = (x[b, :, h].double().contiguous() for x in ins[:3])
            kt, vt = k.t().contiguous(), v.t().contiguous()
            do = ins[3][b, :, h].double().contiguous() if bwd else None
            for r0 in range(0, L, rows):
                r1 = min(L, r0 + rows)
                n = r1 if causal else L
                s = (q[r0:r1] * scale) @ kt[:, :n].contiguous()
                if causal:
                    s[:, r0:].masked_fill_(idx[r0:n][None, :] > idx[r0:r1][:, None], -math.inf)
                m = s.amax(dim=1, keepdim=True)
                p = s.sub_(m).exp_()
                l = p.sum(dim=1, keepdim=True)
                p.div_(l)
                o = p @ v[:n]
                O[b, r0:r1, h] = o
                LSE[b, h, r0:r1] = (m + l.log())[:, 0]
                if bwd:
                    g = do[r0:r1]
                    ds = g @ vt[:, :n].contiguous()
                    ds.sub_((g * o).sum(dim=1, keepdim=True)).mul_(p)
                    G[0][b, r0:r1, h] = ds @ k[:n] * scale
                    G[1][b, :n, h] += ds.t().contiguous() @ q[r0:r1] * scale
                    G[2][b, :n, h] += p.t().contiguous() @ g
                    del ds
                del s, p
    res = {} if case["op"] == "bwd" else dict(O=O, LSE=LSE)
    if bwd:
        res.update(dQ=G[0], dK=G[1], dV=G[2])
    return res
