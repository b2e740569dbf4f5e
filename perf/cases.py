"""Performance cases of the adapter path: what programs that train and serve FrameFT adapters call.

`listed()` are the standing cases, `draw(rng)` further ones of the same ranges.  `prepare(case, seed)`
makes what such a program holds (frames, plans, coefficients, activations and output buffers on the
GPU), `run(state)` is one pass through the package's public calls, `work(case)` the bytes and
operations the pass cannot do without, `exact(case, seed)` its results from the definitions in
float64.

Kinds of case:
  step     one adapted layer in training: forward, then backward with dX and dC.  The program keeps C
           in its own support order (a torch parameter under any optimizer), so the step converts
           the coefficients to the plan's layout and dC back.  saved: the forward keeps the
           backward-ordered copy for the backward.
  forward  inference with an unmerged adapter: the layer's output (the frozen weight's product, here
           a copy of a fixed tensor) has the adapter's term added to it (beta = 1).
  merge    W = W0 + s P_out C P_in^T into a weight buffer: loading an adapter for serving, or hot
           swapping it.
  tenants  one serving batch in which every adapter has its own support and its own number of tokens.
  stack    the same projection of several layers, one support, one batched forward and backward; the
           coefficients live in the plan's layout, the gradients are handed out in support order.
"""
import math

import numpy as np
import torch

import paper_2608_26430_amd as ff
from paper_2608_26430_amd import inputs

ALPHA = 200.0


def listed():
    def case(name, kind, n, rho_in, m, rho_out, nnz, tokens, dtype="bf16", **more):
        return dict(name=name, kind=kind, n=n, rho_in=rho_in, m=m, rho_out=rho_out, nnz=nnz, tokens=tokens,
                    dtype=dtype, **more)

    return [
        # the smallest layer, in fp32: launches and latency, nothing else
        case("linear256_f32_step", "step", 256, 16, 256, 16, 512, 64, "f32", saved=False),
        # one decoding step of a small batch through an unmerged q_proj adapter
        case("qproj_decode", "forward", 4096, 64, 4096, 64, 10_000, 16),
        # the benchmark's training step: Llama-2-7B q_proj, 8 x 512 tokens
        case("qproj_step", "step", 4096, 64, 4096, 64, 10_000, 4096, saved=True),
        # Llama-2-7B MLP projections in training (blocks 128 and 344 wide), both directions
        case("mlp_up_step", "step", 4096, 64, 11008, 64, 50_000, 4096, saved=False),
        case("mlp_down_step", "step", 11008, 64, 4096, 64, 50_000, 4096, saved=False),
        # ViT-B/16 qkv in training, 64 images x 197 tokens (narrow blocks, many tokens)
        case("vit_qkv_step", "step", 768, 64, 2304, 64, 3_000, 64 * 197, saved=False),
        # the paper's own frames (rho = 2: one DFT over the whole width)
        case("rho2_qproj_step", "step", 4096, 2, 4096, 2, 5_000, 4096, saved=False),
        case("rho2_query_step", "step", 1024, 2, 1024, 2, 1_000, 4096, saved=False),
        # Llama-70B down projection in training, the largest layer
        case("llama70b_down_step", "step", 28672, 128, 8192, 128, 200_000, 8192, saved=False),
        # an adapter merged into a bf16 q_proj weight
        case("qproj_merge", "merge", 4096, 64, 4096, 64, 10_000, 0),
        # a serving batch of sixteen users' adapters, requests of 1 to 128 tokens
        case("tenants_qproj", "tenants", 4096, 64, 4096, 64, 10_000, 128, count=16),
        # gate_proj of eight layers in training, batched, 2048 tokens each
        case("gate_stack_step", "stack", 4096, 64, 11008, 64, 10_000, 2048, count=8),
    ]


# -------------------------------------------------------------------------------------- draws

_MAX_COST = 8192 * (28672 + 8192)   # tokens x (n + m) of the largest listed step


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _side(rng, rho, cap):
    """A width rho k with k a multiple of 4 (blocks 2k of 8 to 512 wide), 256 to cap wide."""
    k = 4 * _log_int(rng, max(1, 256 // (4 * rho)), max(1, min(64, cap // (4 * rho))))
    return rho * k


def draw(rng):
    kind = rng.choice(["step"] * 6 + ["forward"] * 3 + ["merge"] * 2 + ["tenants"] * 2 + ["stack"])
    dtype = "f32" if kind in ("step", "forward", "merge") and rng.random() < 0.2 else "bf16"
    if kind in ("step", "forward") and rng.random() < 0.2:
        # rho = 2: widths 2 k with k = 16 k2 or 64 k2, k2 <= 64
        rho_in = rho_out = 2
        n = m = 128 * _log_int(rng, 8, 32)
    else:
        rho_in = rho_out = rng.choice([16, 32, 64, 64, 64, 128])
        if rng.random() < 0.3:   # attention projections: square
            n = m = _side(rng, rho_in, 8192)
        else:
            n, m = _side(rng, rho_in, 28672), _side(rng, rho_out, 28672)
        if dtype == "f32":       # the fp32 layers in use are the smaller models'
            n, m = min(n, 4096), min(m, 4096)
            n, m = n // (4 * rho_in) * (4 * rho_in), m // (4 * rho_out) * (4 * rho_out)
    while n + m > 36864:         # the widest pair of sides in use
        n, m = max(n // 2 // (4 * rho_in), 1) * 4 * rho_in, max(m // 2 // (4 * rho_out), 1) * 4 * rho_out
    nnz = min(_log_int(rng, (n + m) // 2, 6 * (n + m)), n * m // 4)
    case = dict(kind=kind, n=n, rho_in=rho_in, m=m, rho_out=rho_out, nnz=nnz, dtype=dtype)
    if kind == "step":
        case.update(tokens=min(_log_int(rng, 16, 12608), _MAX_COST // (n + m)),
                    saved=rng.random() < 0.5)
    elif kind == "forward":
        case.update(tokens=min(_log_int(rng, 1, 4096), _MAX_COST // (n + m)))
    elif kind == "merge":
        case.update(tokens=0)
    elif kind == "tenants":
        case.update(tokens=_log_int(rng, 8, 512), count=rng.randint(2, 24))
    else:
        count = rng.randint(2, 12)
        case.update(tokens=min(_log_int(rng, 128, 2048), _MAX_COST // ((n + m) * count)), count=count)
    return case


# -------------------------------------------------------------------------------------- inputs

def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _scale(case):
    return ALPHA / math.sqrt(float(case["n"]) * float(case["m"]))


def _counts(case, seed):
    """Tokens of every adapter of a tenants case: 1 to `tokens`."""
    g = inputs.rng(seed + 17)
    return [int(t) for t in g.integers(1, case["tokens"] + 1, size=case["count"])]


def _data(case, seed):
    """Supports, coefficients (support order) and tensors of every adapter, from the seed alone:
    activations and gradients N(0, 1), coefficients N(0, 0.02), a uniform support, W0 ~ N(0, 1/n)."""
    n, m, nnz, T, kind = case["n"], case["m"], case["nnz"], case["tokens"], case["kind"]
    count = case.get("count", 1)
    g = inputs.rng(seed)
    nsup = count if kind == "tenants" else 1
    sups = [inputs.support(g, m, n, nnz) for _ in range(nsup)]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed + 1)
    dt = _dtype(case)

    def randn(shape, std=1.0):
        return (torch.randn(shape, generator=gen, device="cuda") * std).to(dt)

    d = dict(sups=sups, c=[torch.randn((nnz,), generator=gen, device="cuda") * 0.02 for _ in range(count)])
    if kind == "merge":
        d["W0"] = randn((m, n), 1.0 / math.sqrt(n))
        return d
    d["X"] = [randn((T, n)) for _ in range(count)]
    if kind in ("step", "stack"):
        d["G"] = [randn((T, m)) for _ in range(count)]
    if kind == "forward":
        d["Y0"] = randn((T, m))
    return d


def prepare(case, seed):
    n, m, T, kind = case["n"], case["m"], case["tokens"], case["kind"]
    count = case.get("count", 1)
    d = _data(case, seed)
    dt = _dtype(case)
    f_in = ff.framegen(n, n // case["rho_in"], case["rho_in"])
    f_out = f_in if (m, case["rho_out"]) == (n, case["rho_in"]) else ff.framegen(m, m // case["rho_out"],
                                                                                 case["rho_out"])
    plans = [ff.plan_create(f_in, f_out, r, c, max_tokens=max(T, 1), max_batch=count if kind == "stack" else 1)
             for r, c in d["sups"]]
    plan = plans[0]
    st = dict(kind=kind, scale=_scale(case), plans=plans, plan=plan, **d)
    st["c_plan"] = [ff.coef_to_plan(plans[i % len(plans)], d["c"][i]) for i in range(count)]
    if kind == "merge":
        st["W"] = torch.empty((m, n), dtype=dt, device="cuda")
        return st
    # (rows past a tenant's tokens are never written: they stay zero)
    st["Y"] = [torch.zeros((T, m), dtype=dt, device="cuda") for _ in range(count)]
    pa = ff.binding.pointer_array
    if kind in ("step", "stack"):
        st["dX"] = [torch.empty((T, n), dtype=dt, device="cuda") for _ in range(count)]
        st["dC"] = [torch.empty((plan.coef_slots,), device="cuda") for _ in range(count)]
        st["dC_user"] = [torch.empty((case["nnz"],), device="cuda") for _ in range(count)]
    if kind == "step":
        st["save"] = plan.new_saved() if case["saved"] else None
    elif kind == "tenants":
        st["group"] = ff.plan_group(plans)
        st["tokens"] = torch.tensor(_counts(case, seed), dtype=torch.int32, device="cuda")
        st["fptr"] = (pa(st["X"], "cuda"), pa(st["c_plan"], "cuda"), pa(st["Y"], "cuda"))
    elif kind == "stack":
        st["fptr"] = (pa(st["X"], "cuda"), pa(st["c_plan"], "cuda"), pa(st["Y"], "cuda"))
        st["bptr"] = (pa(st["X"], "cuda"), pa(st["G"], "cuda"), pa(st["c_plan"], "cuda"), pa(st["dX"], "cuda"),
                      pa(st["dC"], "cuda"))
    return st


def run(st):
    kind, s, plan = st["kind"], st["scale"], st["plan"]
    if kind == "step":
        X, G, Y, dX, dC, c, save = st["X"][0], st["G"][0], st["Y"][0], st["dX"][0], st["dC"][0], st["c_plan"][0], st["save"]
        ff.coef_to_plan(plan, st["c"][0], c)
        ff.adapter_fwd(plan, X, c, s, Y=Y, save=save)
        ff.adapter_bwd(plan, X, G, c, s, dX=dX, dC=dC, saved=save)
        return Y, dX, ff.coef_to_user(plan, dC, st["dC_user"][0])
    if kind == "forward":
        Y = st["Y"][0]
        Y.copy_(st["Y0"])
        return ff.adapter_fwd(plan, st["X"][0], st["c_plan"][0], s, Y=Y, beta=1.0)
    if kind == "merge":
        st["W"].copy_(st["W0"])
        return ff.merge_delta(plan, st["c_plan"][0], s, st["W"], beta=1.0)
    if kind == "tenants":
        return ff.adapter_fwd_group(st["group"], st["X"], st["c_plan"], s, st["Y"], tokens=st["tokens"],
                                    ptrs=st["fptr"])
    ff.adapter_fwd_batched(plan, st["X"], st["c_plan"], s, st["Y"], ptrs=st["fptr"])
    ff.adapter_bwd_batched(plan, st["X"], st["G"], st["c_plan"], s, st["dX"], st["dC"], ptrs=st["bptr"])
    return st["Y"], st["dX"], [ff.coef_to_user(plan, dC, du) for dC, du in zip(st["dC"], st["dC_user"])]


# -------------------------------------------------------------------------------------- bounds

def work(case):
    n, m, nnz, kind = case["n"], case["m"], case["nnz"], case["kind"]
    esz = 2 if case["dtype"] == "bf16" else 4
    kn, km = n // case["rho_in"], m // case["rho_out"]
    # per token: a size-k complex transform of each block (5 k log2 k), rho / 2 of them per side
    fn, fm = 2.5 * n * math.log2(max(kn, 2)), 2.5 * m * math.log2(max(km, 2))
    if kind == "merge":
        return {"bytes": 2.0 * esz * n * m + 4 * nnz,       # W0 read, the merged weight written
                "flops": 2.0 * nnz * (2 * kn) * (2 * km)}
    # mean of 1 .. tokens
    rows = case["count"] * (case["tokens"] + 1) / 2 if kind == "tenants" else case["tokens"] * case.get("count", 1)
    cvals = 4.0 * nnz * case.get("count", 1)
    if kind == "tenants":
        return {"bytes": rows * esz * (n + m) + cvals, "flops": rows * (fn + fm + 2 * nnz)}
    if kind == "forward":
        return {"bytes": rows * esz * (n + 2 * m) + cvals, "flops": rows * (fn + fm + 2 * nnz)}
    return {"bytes": rows * esz * (3 * n + 2 * m) + 2 * cvals, "flops": rows * (3 * fn + 2 * fm + 6 * nnz)}


def tolerance(case):
    """About four times the error against float64, which is that of one rounding of the activations'
    type at each stage (bf16: 3.8e-3 on Y, dX and dC; fp32: 1.5e-7); a merged weight is rounded once
    (bf16: 1.7e-3)."""
    if case["dtype"] == "f32":
        return {"rel": 1e-6}
    return {"rel": 7e-3} if case["kind"] == "merge" else {"rel": 1.5e-2}


# -------------------------------------------------------------------------------------- float64

def _block(k):
    """The realified k-point unitary DFT whose columns are the frame vectors of one block:
    B[2j.., 2i..] = exp(2 pi i (i j mod k) / k) / sqrt(k) as a 2 x 2 rotation."""
    ij = np.outer(np.arange(k), np.arange(k)) % k
    ang = 2.0 * np.pi * ij / k
    B = np.empty((k, 2, k, 2))
    B[:, 0, :, 0] = B[:, 1, :, 1] = np.cos(ang)
    B[:, 1, :, 0] = np.sin(ang)
    B[:, 0, :, 1] = -B[:, 1, :, 0]
    return torch.from_numpy(B.reshape(2 * k, 2 * k) / math.sqrt(k)).cuda()


def _pos(idx, rho, k):
    """Block order (block r, frequency i, part s) of the canonical index i rho + 2 r + s."""
    i, r, s = idx // rho, idx % rho // 2, idx % 2
    return torch.from_numpy((r * 2 * k + 2 * i + s).astype(np.int64)).cuda()


def _analysis(B, x):
    """P^T x of float64 rows, transposed: coefficients (block order) x tokens."""
    W = B.shape[0]
    return (x.reshape(-1, W) @ B).reshape(x.shape).t().contiguous()


def _synthesis(B, z):
    """P z of coefficients x tokens: float64 rows."""
    W = B.shape[0]
    x = z.t().contiguous()
    return (x.reshape(-1, W) @ B.t()).reshape(x.shape)


def exact(case, seed):
    n, m, nnz, T, kind = case["n"], case["m"], case["nnz"], case["tokens"], case["kind"]
    count, s = case.get("count", 1), _scale(case)
    kn, km = n // case["rho_in"], m // case["rho_out"]
    d = _data(case, seed)
    Bn, Bm = _block(kn), _block(km)
    pos = [(_pos(r, case["rho_out"], km), _pos(c, case["rho_in"], kn)) for r, c in d["sups"]]
    if kind == "merge":
        (rows, cols), c = pos[0], d["c"][0].double()
        C = torch.zeros((m, n), dtype=torch.float64, device="cuda")
        C[rows, cols] = c
        dW = (Bm @ C.view(m // (2 * km), 2 * km, n)).view(m, n)
        del C
        dW = (dW.view(-1, 2 * kn) @ Bn.t()).view(m, n)
        return d["W0"].double() + s * dW
    step = max(1, min(T, (1 << 26) // max(nnz, n + m)))
    counts = _counts(case, seed) if kind == "tenants" else [T] * count
    Ys, dXs, dCs = [], [], []
    for i in range(count):
        rows, cols = pos[i % len(pos)]
        c = d["c"][i].double()[:, None]
        Y = torch.zeros((T, m), dtype=torch.float64, device="cuda")
        back = kind in ("step", "stack")
        dX = torch.zeros((T, n), dtype=torch.float64, device="cuda") if back else None
        dC = torch.zeros((nnz,), dtype=torch.float64, device="cuda")
        for t0 in range(0, counts[i], step):
            t1 = min(counts[i], t0 + step)
            zc = _analysis(Bn, d["X"][i][t0:t1].double())[cols]
            v = torch.zeros((m, t1 - t0), dtype=torch.float64, device="cuda").index_add_(0, rows, zc * c)
            Y[t0:t1] = s * _synthesis(Bm, v)
            if back:
                ur = _analysis(Bm, d["G"][i][t0:t1].double())[rows]
                dC += s * (ur * zc).sum(1)
                q = torch.zeros((n, t1 - t0), dtype=torch.float64, device="cuda").index_add_(0, cols, ur * c)
                dX[t0:t1] = s * _synthesis(Bn, q)
        if kind == "forward":
            Y += d["Y0"].double()
        Ys.append(Y)
        dXs.append(dX)
        dCs.append(dC)
    if kind == "step":
        return Ys[0], dXs[0], dCs[0]
    if kind == "forward":
        return Ys[0]
    return Ys if kind == "tenants" else (Ys, dXs, dCs)
