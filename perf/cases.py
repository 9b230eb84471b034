"""Cases that the framework's speed is measured on, through its public calls.

A user of this library fine-tunes a GPT-2-style model under DP-SGD: hooks hand
it activations and output gradients, and it turns them into per-example norms,
clip factors and noised clipped sums. The cases are those calls over the sizes
such a program meets: whole steps, the calls of a step one at a time, the
smallest configuration, prompts that are no multiple of any tile, logit
gradients as PyTorch lays them out (rows of V = 50257 elements) and padded,
bf16 and fp32, short and long sequences.

Shapes are those of GPT-2 and DistilGPT2 (12 and 6 blocks of width 768,
vocabulary 50257), of the paper's batches (24 prompts of at most 128 tokens)
and of the repository's benchmark. Activations are N(0, 1); output gradients
N(0, 1e-3), scaled per example as losses of different examples differ; ids
follow a Zipf law; logit gradients are softmax minus one-hot.
"""
from __future__ import annotations

import math

import torch

from paper_2609_40335_amd import dpghost as dp

GPT2_V = 50257
N_POS = 1024
CLIP, SIGMA, SEED, STEP = 1.0, 1.0, 1234, 7


# ------------------------------------------------------------------- cases
def _case(kind, dtype, B, T, blocks, d, V=0, pad=True, noised=False, bias=False, name=None):
    c = {"kind": kind, "dtype": dtype, "B": B, "T": T, "blocks": blocks, "d": d, "V": V,
         "pad": pad, "noised": noised, "bias": bias}
    return c if name is None else {"name": name, **c}


def listed():
    return [
        # The smallest call sequence: one block of width 64 with a tied head of
        # 512 ids in fp32, as in a smoke test or a unit test of a training loop.
        _case("step", "fp32", 4, 16, 1, 64, V=512, pad=False, noised=True, name="step_tiny_fp32"),
        # The benchmark's step: GPT-2 small, tied, 32 prompts of 128 tokens.
        _case("step", "bf16", 32, 128, 12, 768, V=GPT2_V, noised=True, name="step_gpt2_b32_t128"),
        # DistilGPT2, tied, at twice the batch and twice the length.
        _case("step", "bf16", 64, 256, 6, 768, V=GPT2_V, noised=True, name="step_distil_b64_t256"),
        # One layer at a time, as a hook calls the library: the norm of an MLP
        # layer, and its clipped sum in nn.Linear's [out, in] layout.
        _case("layer", "bf16", 24, 128, 1, 768, name="layer_fc_b24_t128"),
        # The paper's batch at a prompt length that is no multiple of a tile,
        # logit gradients as PyTorch lays them out; norms with the biases.
        _case("norms", "bf16", 24, 100, 12, 768, V=GPT2_V, pad=False, bias=True,
              name="norms_gpt2_b24_t100"),
        # ... and the clipped sums of the same batch (no noise: eq. 3's bracket).
        _case("sums", "bf16", 24, 100, 12, 768, V=GPT2_V, pad=False, name="sums_gpt2_b24_t100"),
        # Long ragged documents: the norms take the per-example gradients.
        _case("norms", "bf16", 6, 1000, 12, 768, V=GPT2_V, name="norms_gpt2_b6_t1000"),
        # Full-precision fine-tuning of DistilGPT2 at the paper's batch.
        _case("norms", "fp32", 24, 128, 6, 768, V=GPT2_V, pad=False, name="norms_distil_fp32"),
        _case("sums", "fp32", 24, 128, 6, 768, V=GPT2_V, pad=False, name="sums_distil_fp32"),
        # Full-length documents, GPT-2 small: per-example gradients kept in HBM
        # by the norm and summed from there.
        _case("store", "bf16", 16, 1024, 12, 768, V=GPT2_V, noised=True, name="store_gpt2_b16_t1024"),
        # The token-keyed calls on ragged documents: embedding norm with its
        # buckets, tied cross term, an untied embedding's noise and sum.
        _case("tokens", "bf16", 8, 1000, 0, 768, V=GPT2_V, noised=True, name="tokens_b8_t1000"),
        # LayerNorm gains and biases and the position table.
        _case("vectors", "bf16", 32, 128, 12, 768, noised=True, name="vectors_gpt2_b32_t128"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "layer", "norms", "norms", "sums", "sums", "store", "tokens",
                       "vectors"])
    dtype = "bf16" if kind == "store" or rng.random() < 0.7 else "fp32"
    T = _log(rng, 8, 1024)
    if rng.random() < 0.4:
        T = max(16, T // 16 * 16)
    d = _log(rng, 48, 1024)
    if rng.random() < 0.8:
        d = max(64, d // 8 * 8)
    V = GPT2_V if rng.random() < 0.4 else _log(rng, 500, GPT2_V)
    blocks = rng.choice([1, 2, 4, 6])
    pad = rng.random() < 0.5
    tokens = 8192 if dtype == "bf16" else 2048
    if kind == "store":
        T, d, pad = max(256, T // 32 * 32), max(64, d // 8 * 8), True
        tokens, blocks = 4096, min(blocks, 2)
    B = max(1, min(64, _log(rng, 2, 64), tokens // T))
    return _case(kind, dtype, B, T, blocks, d, V=0 if kind in ("layer", "vectors") else V, pad=pad,
                 noised=kind not in ("norms", "layer") and rng.random() < 0.6,
                 bias=kind == "norms" and rng.random() < 0.5)


# ------------------------------------------------------------------- shapes
def _up(x, m):
    return (x + m - 1) // m * m


def _linears(case):
    d = case["d"]
    if case["kind"] == "layer":
        return [(d, 4 * d)]
    return [(d, 3 * d), (d, d), (d, 4 * d), (4 * d, d)] * case["blocks"]


def _es(case):
    return 2 if case["dtype"] == "bf16" else 4


class _Flat:
    """Views of one fp32 buffer, each starting at a multiple of 64 elements."""

    def __init__(self, shapes, device="cuda", dtype=torch.float32):
        self.at, off = [], 0
        for s in shapes:
            self.at.append(off)
            off += _up(math.prod(s), 64)
        self.buf = torch.zeros(max(off, 1), device=device, dtype=dtype)
        self.views = [self.buf[o:o + math.prod(s)].view(*s) for o, s in zip(self.at, shapes)]


# ------------------------------------------------------------------- inputs
def _inputs(case, seed):
    """Every operand of the case on the GPU, from the seed alone."""
    g = torch.Generator(device="cuda").manual_seed(1000003 * (seed + 1) + 17)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    B, T, d, V, kind = case["B"], case["T"], case["d"], case["V"], case["kind"]
    scale = torch.exp(0.5 * torch.randn(B, 1, 1, device="cuda", generator=g))

    def normal(w, std=1.0, per_example=False):
        x = torch.randn(B, T, w, device="cuda", generator=g)
        if per_example:
            x *= scale * std
        return x.to(dt)

    s = {}
    if kind in ("step", "layer", "norms", "sums", "store"):
        s["lin"] = [(normal(a), normal(b, 1e-3, True)) for a, b in _linears(case)]
    if V:
        cdf = torch.arange(1, V + 1, device="cuda", dtype=torch.float64).pow(-1.1).cumsum(0)
        u = torch.rand(B, T, device="cuda", dtype=torch.float64, generator=g) * cdf[-1]
        s["ids"] = torch.searchsorted(cdf, u, right=True).clamp_(max=V - 1).to(torch.int32)
        s["H"] = normal(d)
        s["dE"] = normal(d, 1e-3, True)
        ldz = _up(V, 64) if case["pad"] else V
        z = torch.zeros(B, T, ldz, device="cuda", dtype=dt)
        for b in range(B):
            p = torch.softmax(torch.randn(T, V, device="cuda", generator=g), dim=1)
            p[torch.arange(T - 1, device="cuda"), s["ids"][b, 1:].long()] -= 1.0
            p[T - 1] = 0.0
            z[b, :, :V] = p / T
        s["Gz"] = z[:, :, :V]
    if kind == "vectors":
        s["ln"] = [(normal(d), normal(d, 1e-3, True)) for _ in range(2 * case["blocks"] + 1)]
        s["dE"] = normal(d, 1e-3, True)
    c = torch.rand(B, device="cuda", generator=g) * 1.2 + 0.02
    s["c"] = c.clamp_(max=1.0)   # clip factors of a batch some of whose examples are below C
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    B, T, d, V, kind = case["B"], case["T"], case["d"], case["V"], case["kind"]
    s["case"] = case
    s["n2"] = torch.zeros(B, device="cuda")
    if kind in ("step", "store", "tokens", "vectors"):
        s["c"] = torch.zeros(B, device="cuda")
        s["c_b"] = torch.zeros(B, device="cuda")
    if kind == "layer":
        A, G = s["lin"][0]
        s["out"] = torch.zeros(G.shape[2], A.shape[2], device="cuda")
    if kind in ("step", "norms", "store"):
        layers = list(s["lin"]) + ([(s["H"], s["Gz"])] if V else [])
        bias = None
        if case["bias"]:
            s["bias"] = _Flat([(B, G.shape[2]) for _, G in s["lin"]])
            bias = s["bias"].views + ([None] if V else [])
        s["norm_group"] = dp.LinearGroup(layers, bias_grads=bias)
    if kind in ("step", "sums", "store"):
        shapes = [(A.shape[2], G.shape[2]) for A, G in s["lin"]] + ([(V, d)] if V else [])
        s["grads"] = _Flat(shapes)
        s["tids"] = list(range(len(shapes)))
        if kind == "store":
            grp = s["norm_group"]
            grp.set_outputs(s["grads"].views)
            s["store"] = torch.empty(grp.store_bytes(), dtype=torch.uint8, device="cuda")
            s["tr"] = [False] * len(s["lin"]) + [True]
        else:
            layers = list(s["lin"]) + ([(s["Gz"], s["H"])] if V else [])
            s["sum_group"] = dp.LinearGroup(layers, s["grads"].views)
    if kind in ("step", "tokens"):
        s["seg"] = torch.zeros(B, T, dtype=torch.int32, device="cuda")
        s["nu"] = torch.zeros(B, dtype=torch.int32, device="cuda")
    if kind == "tokens":
        s["cross"] = torch.zeros(B, device="cuda")
        s["E"] = torch.zeros(V, d, device="cuda")
    if kind == "vectors":
        n = len(s["ln"])
        s["group"] = dp.VectorGroup([p for x, g in s["ln"] for p in ((x, g), (None, g))])
        s["outs"] = _Flat([(d,)] * (2 * n))
        s["P"] = torch.zeros(max(N_POS, T), d, device="cuda")
        s["tids"] = list(range(2 * n))
    return s


# --------------------------------------------------------------------- runs
def run(s):
    case = s["case"]
    kind, B, V = case["kind"], case["B"], case["V"]
    sigma = SIGMA if case["noised"] else 0.0
    if kind == "layer":
        A, G = s["lin"][0]
        dp.dp_ghost_norm_linear(A, G, s["n2"])
        dp.dp_clipped_grad_sum(A, G, s["c"], s["out"], transpose_out=True)
        return {"norm2": s["n2"], "grad": s["out"]}
    if kind == "norms":
        s["norm_group"].ghost_norm(s["n2"])
        return {"norm2": s["n2"], **({"bias": s["bias"].buf} if case["bias"] else {})}
    if kind == "sums":
        if case["noised"]:
            s["sum_group"].clipped_sum_noised(s["c"], s["tids"], sigma, CLIP, B, SEED, STEP)
        else:
            s["sum_group"].clipped_sum(s["c"])
        return {"grads": s["grads"].buf}
    if kind == "store":
        grp = s["norm_group"]
        grp.ghost_norm_store(s["n2"], s["store"])
        dp.dp_clip_factors(s["n2"], CLIP, s["c"])
        grp.clipped_sum_noised_store(s["c"], s["store"], s["tids"], sigma, CLIP, B, SEED, STEP,
                                     transpose_out=s["tr"])
        return {"norm2": s["n2"], "c": s["c"], "grads": s["grads"].buf}
    if kind == "step":
        s["norm_group"].ghost_norm(s["n2"])
        dp.dp_ghost_norm_embedding(s["ids"], s["dE"], V, s["n2"], accumulate=True, seg_id=s["seg"],
                                   n_unique=s["nu"])
        dp.dp_tied_cross_term(s["ids"], s["dE"], s["H"], s["Gz"], V, s["n2"], scale=2.0,
                              accumulate=True)
        dp.dp_clip_factors_scaled(s["n2"], CLIP, 1.0 / B, s["c_b"], c=s["c"])
        s["sum_group"].clipped_sum_noised(s["c"], s["tids"], sigma, CLIP, B, SEED, STEP)
        dp.dp_clipped_grad_sum(None, s["dE"], s["c_b"], s["grads"].views[-1], ids=s["ids"], V=V,
                               accumulate=True)
        return {"norm2": s["n2"], "c": s["c"], "seg": s["seg"], "nu": s["nu"],
                "grads": s["grads"].buf}
    if kind == "tokens":
        dp.dp_ghost_norm_embedding(s["ids"], s["dE"], V, s["n2"], seg_id=s["seg"],
                                   n_unique=s["nu"])
        dp.dp_tied_cross_term(s["ids"], s["dE"], s["H"], s["Gz"], V, s["cross"])
        dp.dp_clip_factors_scaled(s["n2"], CLIP, 1.0 / B, s["c_b"], c=s["c"])
        dp.dp_noise_fill(s["E"], sigma, CLIP, B, SEED, 3, STEP)
        dp.dp_clipped_grad_sum(None, s["dE"], s["c_b"], s["E"], ids=s["ids"], V=V,
                               accumulate=True)
        return {"norm2": s["n2"], "cross": s["cross"], "c": s["c"], "seg": s["seg"],
                "nu": s["nu"], "E": s["E"]}
    g = s["group"]
    g.grads_and_norm(s["n2"])
    dp.dp_ghost_norm_positional(s["dE"], s["n2"], accumulate=True)
    dp.dp_clip_factors(s["n2"], CLIP, s["c"])
    g.clipped_sum_noised(s["c"], s["outs"].views, s["tids"], sigma, CLIP, B, SEED, STEP)
    dp.dp_clipped_grad_sum_positional_noised(s["dE"], s["c"], s["P"], len(s["tids"]), sigma, CLIP,
                                             B, SEED, STEP)
    return {"norm2": s["n2"], "c": s["c"], "outs": s["outs"].buf, "P": s["P"]}


# --------------------------------------------------------------------- work
def work(case):
    B, T, d, V, kind = case["B"], case["T"], case["d"], case["V"], case["kind"]
    K, es = B * T, _es(case)
    nbytes = flops = 0.0
    layers = _linears(case) if kind not in ("tokens", "vectors") else []
    if V and kind != "tokens":
        layers = layers + [(d, V)]
    for a, b in layers:
        nbytes += K * es * (a + b)
        if kind != "sums":   # the cheaper of the Gram and the direct form
            flops += min(float(K) * (T + 1) * (a + b), 2.0 * K * a * b)
        if kind in ("sums", "step", "layer"):
            flops += 2.0 * K * a * b
        if kind == "store":
            flops += 2.0 * B * a * b
        if kind != "norms":
            nbytes += 4.0 * a * b
        if kind == "norms" and case["bias"]:
            nbytes += 4.0 * B * b
    if kind in ("step", "tokens"):
        n = d * es
        nbytes += K * n + 8.0 * K               # dE, ids, buckets
        flops += 2.0 * K * T * d + 2.0 * K * d  # the cross term's products, the sums
        if kind == "tokens":
            # H, the logit gradients at the T ids of every row, the matrix
            nbytes += K * n + float(K) * T * es + 4.0 * V * d
    if kind == "vectors":
        n = 2 * case["blocks"] + 1
        nbytes += K * d * es * (2.0 * n + 1) + 4.0 * d * (2 * n + max(N_POS, T))
        flops += 2.0 * K * d * (3 * n + 2)
    return {"bytes": nbytes + 8.0 * B, "flops": flops}


def tolerance(case):
    # Whole-number outputs (buckets) stay the same. bf16 operands multiply
    # exactly and add up in fp32; the noise is fp32. Only the clipped sum of
    # sequences that are no multiple of a tile may round c_i A to bf16.
    if case["dtype"] == "bf16" and case["kind"] in ("step", "sums", "layer") and case["T"] % 64:
        return {"rel": 5e-3, "max": 2e-2}
    return {"rel": 1e-5, "max": 1e-3}


# -------------------------------------------------------------------- exact
def _philox(blk, tid):
    """The four words of each Philox4x32-10 block (Salmon et al., SC'11)."""
    lo = 0xFFFFFFFF
    c = [blk & lo, blk >> 32, torch.full_like(blk, tid), torch.full_like(blk, STEP)]
    k0, k1 = SEED & lo, SEED >> 32
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((p1 >> 32) & lo) ^ c[1] ^ k0, p1 & lo, ((p0 >> 32) & lo) ^ c[3] ^ k1, p0 & lo]
        k0, k1 = (k0 + 0x9E3779B9) & lo, (k1 + 0xBB67AE85) & lo
    return c


def _noised(case, out, tid):
    """(out + sigma C z) / B in place, z the generator's normals in 64 bits."""
    flat, n, step = out.view(-1), out.numel(), 1 << 24
    sigma = SIGMA if case["noised"] else 0.0
    for j0 in range(0, n, step):
        m = min(step, n - j0)
        w = _philox(torch.arange(j0 // 4, j0 // 4 + (m + 3) // 4, device=out.device), tid)
        u = [(x.double() + 0.5) * 2.0 ** -32 for x in w]
        z = []
        for p in (0, 2):
            r = torch.sqrt(-2.0 * torch.log(u[p]))
            z += [r * torch.cos(2 * math.pi * u[p + 1]), r * torch.sin(2 * math.pi * u[p + 1])]
        flat[j0:j0 + m] += sigma * CLIP * torch.stack(z, 1).view(-1)[:m]
    out /= case["B"]


def exact(case, seed):
    s = _inputs(case, seed)
    B, T, d, V, kind = case["B"], case["T"], case["d"], case["V"], case["kind"]
    f64 = torch.float64

    def rows(x, w):   # [B*T, width], row k times the weight of its example
        return (x.to(f64) * w.view(B, 1, 1)).reshape(B * T, -1)

    def sum_of(A, G, w, out):
        torch.mm(rows(A, w).t(), G.to(f64).reshape(B * T, -1), out=out)

    def norm_of(A, G):
        return torch.stack([torch.mm(A[b].to(f64).t(), G[b].to(f64)).square().sum()
                            for b in range(B)])

    def embedding(b):
        g = torch.zeros(V, d, device="cuda", dtype=f64)
        return g.index_add_(0, s["ids"][b].long(), s["dE"][b].to(f64))

    def factors(n2):
        return torch.clamp(CLIP / torch.sqrt(n2), max=1.0)

    def buckets():
        seg = torch.zeros(B, T, dtype=torch.int32, device="cuda")
        nu = torch.zeros(B, dtype=torch.int32, device="cuda")
        for b in range(B):
            u, inv = torch.unique(s["ids"][b], return_inverse=True)
            seg[b], nu[b] = inv.to(torch.int32), u.numel()
        return seg, nu

    ones = torch.ones(B, device="cuda", dtype=f64)
    if kind == "layer":
        A, G = s["lin"][0]
        out = torch.zeros(G.shape[2], A.shape[2], device="cuda", dtype=f64)
        sum_of(G, A, s["c"].to(f64), out)
        return {"norm2": norm_of(A, G), "grad": out}
    lin = s.get("lin", [])
    n2 = torch.zeros(B, device="cuda", dtype=f64)
    if kind in ("step", "norms", "store"):
        for A, G in lin:
            n2 += norm_of(A, G)
        if V and kind != "step":
            n2 += norm_of(s["H"], s["Gz"])
    if kind == "norms":
        if not case["bias"]:
            return {"norm2": n2}
        bias = _Flat([(B, G.shape[2]) for _, G in lin], dtype=f64)
        for v, (_, G) in zip(bias.views, lin):
            v.copy_(G.to(f64).sum(1))
            n2 += v.square().sum(1)
        return {"norm2": n2, "bias": bias.buf}
    if kind in ("step", "sums", "store"):
        if kind == "step":
            for b in range(B):
                n2[b] += (embedding(b) + torch.mm(s["Gz"][b].to(f64).t(), s["H"][b].to(f64))
                          ).square().sum()
        c = s["c"].to(f64) if kind == "sums" else factors(n2)
        shapes = [(A.shape[2], G.shape[2]) for A, G in lin] + ([(V, d)] if V else [])
        grads = _Flat(shapes, dtype=f64)
        pairs = list(lin) + ([(s["Gz"], s["H"])] if V else [])
        for k, ((X, Y), out) in enumerate(zip(pairs, grads.views)):
            sum_of(X, Y, c, out)
            if kind == "step" and k == len(pairs) - 1:
                out.index_add_(0, s["ids"].view(-1).long(), rows(s["dE"], c))
            if kind != "sums" or case["noised"]:
                _noised(case, out, k)
        if kind == "sums":
            return {"grads": grads.buf}
        got = {"norm2": n2, "c": c, "grads": grads.buf}
        if kind == "step":
            got["seg"], got["nu"] = buckets()
        return got
    if kind == "tokens":
        cross = torch.zeros(B, device="cuda", dtype=f64)
        for b in range(B):
            n2[b] = embedding(b).square().sum()
            P = torch.mm(s["H"][b].to(f64), s["dE"][b].to(f64).t())
            cross[b] = (P * s["Gz"][b][:, s["ids"][b].long()].to(f64)).sum()
        c = factors(n2)
        E = torch.zeros(V, d, device="cuda", dtype=f64)
        E.index_add_(0, s["ids"].view(-1).long(), rows(s["dE"], c))
        _noised(case, E, 3)
        seg, nu = buckets()
        return {"norm2": n2, "cross": cross, "c": c, "seg": seg, "nu": nu, "E": E}
    outs = _Flat([(d,)] * (2 * len(s["ln"])), dtype=f64)
    per = []
    for x, g in s["ln"]:
        per += [(x.to(f64) * g.to(f64)).sum(1), g.to(f64).sum(1)]
    n2 = sum(p.square().sum(1) for p in per) + s["dE"].to(f64).square().sum((1, 2))
    c = factors(n2)
    for k, (p, v) in enumerate(zip(per, outs.views)):
        v.copy_((p * c.view(B, 1)).sum(0))
        _noised(case, v, k)
    P = torch.zeros(max(N_POS, T), d, device="cuda", dtype=f64)
    P[:T] = (s["dE"].to(f64) * c.view(B, 1, 1)).sum(0)
    _noised(case, P, len(per))
    return {"norm2": n2, "c": c, "outs": outs.buf, "P": P}
