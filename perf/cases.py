"""Timed cases of libkata: the calls a program makes through the Python binding,
over the range of sizes, types and options that are used in earnest.

    listed()            the fixed cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs on the GPU, from the seed alone
    run(state)          one pass through the public entry points
    work(case)          bytes and operations of one pass
    tolerance(case)     how far two correct implementations may differ
    exact(case, seed)   the outputs of run() in 64 bits, from the definition

Inputs follow the recipe of the seeded workloads: q and k rows of unit length,
v ~ N(0, 1) (recall-shaped cases draw their keys from a pool and present them
again with noise), rounded to bf16 where the case is bf16.
"""
import math

import torch

import paper_2607_17419_amd as kata

DEV = "cuda:0"
RELU_EPS = 1e-3
POOL, NOISE_STD = 512, 0.1  # recall-shaped keys: pool size, query noise per coordinate
PREFIX = 256                # tokens behind a decode case's state


def _case(kind, B, H, T, d, dv, C, dtype, **more):
    c = {"kind": kind, "B": B, "H": H, "T": T, "d": d, "dv": dv, "C": C, "dtype": dtype,
         "g": 1, "feature": 0, "normalize": True, "recall": False}
    c.update(more)
    return c


def listed():
    named = {
        # one token of one sequence through one layer: a chat's decode step, where the
        # launch and its tail count
        "decode_one": _case("decode", 1, 16, 1, 64, 64, 64, "bf16"),
        # a serving batch of 256 sequences: the state of 2.2 GB read and written once
        "decode_batch": _case("decode", 256, 16, 1, 64, 64, 64, "bf16"),
        # the state of four prompts of ordinary length, before decoding goes on from it
        "prefill_state": _case("prefill", 4, 16, 2000, 64, 64, 64, "bf16"),
        # a short prompt: one span per head, a few small launches
        "fwd_short": _case("fwd", 1, 16, 200, 64, 64, 64, "bf16"),
        # the paper's B = 8, H = 16 latency-table shape at T = 4096
        "fwd_mid": _case("fwd", 8, 16, 4096, 64, 64, 64, "bf16"),
        # one long sequence, the shape of the headline figure
        "fwd_long": _case("fwd", 1, 16, 131072, 64, 64, 64, "bf16"),
        # recall-shaped inputs at d = 32 with a length that fills neither chunk nor span
        "fwd_recall": _case("fwd", 4, 8, 16301, 32, 64, 128, "bf16", recall=True),
        # KATA-M2 (two feature blocks) over a medium sequence, ragged
        "fwd_m2": _case("fwd", 2, 16, 30011, 64, 64, 64, "bf16", g=2),
        # the O(T^2) form at the length where the two forms meet
        "fwd_quadratic": _case("quadratic", 1, 16, 4096, 64, 64, 64, "bf16"),
        # linear features with the normalised readout, the associative-scan table's shape
        "lin_relu": _case("lin", 1, 16, 131072, 64, 64, 128, "bf16", feature=kata.LIN_RELU),
        # one layer's training step at the paper's training shape: forward, then gradients
        "train_mid": _case("train", 8, 16, 4096, 64, 64, 64, "bf16"),
        # the same step in fp32 for a small model
        "train_f32": _case("train", 1, 8, 1000, 64, 64, 64, "f32"),
    }
    return [dict(c, name=name) for name, c in named.items()]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _sizes(rng, t_lo, t_hi, tokens, b_hi=8, h_hi=16):
    """B, H, T with T log-uniform in [t_lo, t_hi] and at most `tokens` head-tokens."""
    T = _log_int(rng, t_lo, t_hi)
    B = _log_int(rng, 1, b_hi)
    H = rng.choice([h for h in (1, 2, 4, 8, 12, 16) if h <= h_hi])
    while B * H * T > tokens and B > 1:
        B = max(1, B // 2)
    while B * H * T > tokens and H > 1:
        H = max(1, H // 2)
    return B, H, min(T, tokens)


def draw(rng):
    kind = rng.choice(("decode", "prefill", "fwd", "fwd", "m2", "quadratic", "lin", "train",
                       "train", "train_f32"))
    if kind == "decode":
        return _case(kind, _log_int(rng, 1, 256), rng.choice((4, 8, 16)), 1,
                     rng.choice((32, 64)), 64, 64, rng.choice(("bf16", "f32")))
    if kind == "prefill":
        B, H, T = _sizes(rng, 16, 8192, 131072)
        return _case(kind, B, H, T, rng.choice((32, 64)), 64, 64, rng.choice(("bf16", "f32")))
    if kind == "fwd":
        B, H, T = _sizes(rng, 16, 131072, 1 << 20)
        d = rng.choice((32, 64, 64))
        return _case(kind, B, H, T, d, 64, rng.choice((64, 128)), "bf16",
                     recall=rng.random() < 0.25)
    if kind == "m2":
        B, H, T = _sizes(rng, 16, 131072, 1 << 20)
        return _case("fwd", B, H, T, 64, 64, 64, "bf16", g=2)
    if kind == "quadratic":
        B, H, T = _sizes(rng, 16, 8192, 131072)
        return _case(kind, B, H, T, rng.choice((32, 64, 64)), 64, 64, "bf16")
    if kind == "lin":
        B, H, T = _sizes(rng, 64, 131072, 2 << 20)
        feature = rng.randrange(5)
        return _case(kind, B, H, T, 64, 64, rng.choice((64, 128)), "bf16", feature=feature,
                     normalize=feature != kata.LIN_IDENTITY)
    if kind == "train":
        B, H, T = _sizes(rng, 64, 8192, 1 << 19)
        return _case(kind, B, H, T, 64, 64, 64, "bf16")
    B, H, T = _sizes(rng, 32, 2048, 8192, b_hi=4, h_hi=8)
    return _case("train", B, H, T, rng.choice((16, 32, 64)), rng.choice((16, 32, 64)),
                 rng.choice((32, 64)), "f32")


# ---- inputs ---------------------------------------------------------------------

def _unit(x):
    return x / x.norm(dim=-1, keepdim=True).clamp_min(1e-30)


def _packed_pairs(d):
    return torch.triu_indices(d, d, device=DEV)  # row-major upper triangle


def _decode_state(gen, B, H, d, dv):
    """The packed state of a PREFIX-token prompt, fp32, a few heads at a time."""
    a, b = _packed_pairs(d)
    n = a.numel()
    S = torch.empty((B * H, n, dv), dtype=torch.float32, device=DEV)
    z = torch.empty((B * H, n), dtype=torch.float32, device=DEV)
    for h in range(0, B * H, 512):
        m = min(512, B * H - h)
        k = _unit(torch.randn((m, d, PREFIX), generator=gen, device=DEV).transpose(1, 2))
        k = k.transpose(1, 2).contiguous()
        v = torch.randn((m, PREFIX, dv), generator=gen, device=DEV)
        phi = k[:, a] * k[:, b]
        torch.bmm(phi, v, out=S[h:h + m])
        torch.sum(phi, dim=2, out=z[h:h + m])
    return S.view(B, H, n, dv), z.view(B, H, n)


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    B, H, T, d, dv = (case[x] for x in ("B", "H", "T", "d", "dv"))
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=DEV)

    s = dict(case)
    if case["recall"]:
        pool = _unit(normal(B * H, POOL, d))
        idx = torch.randint(0, POOL, (B * H, T), generator=gen, device=DEV)
        head = torch.arange(B * H, device=DEV)[:, None]
        k = pool[head, idx]
        t = torch.arange(T, device=DEV)[None, :]
        j = (torch.rand((B * H, T), generator=gen, device=DEV) * t).long()
        q = _unit(k.gather(1, j[:, :, None].expand(-1, -1, d)) + NOISE_STD * normal(B * H, T, d))
        q, k = q.view(B, H, T, d), k.view(B, H, T, d)
    else:
        q, k = _unit(normal(B, H, T, d)), _unit(normal(B, H, T, d))
    s["q"], s["k"], s["v"] = (x.to(dtype).contiguous() for x in (q, k, normal(B, H, T, dv)))
    if case["kind"] == "train":
        s["dout"] = normal(B, H, T, dv)
    if case["kind"] == "decode":
        s["q"], s["k"], s["v"] = (s[x][:, :, 0].contiguous() for x in ("q", "k", "v"))
        s["S"], s["z"] = _decode_state(gen, B, H, d, dv)
    return s


# ---- one pass -------------------------------------------------------------------

def run(s):
    kind, q, k, v, C = s["kind"], s.get("q"), s["k"], s["v"], s["C"]
    if kind == "decode":
        return kata.decode_step(s["S"], s["z"], q, k, v), s["S"], s["z"]
    if kind == "prefill":
        return kata.prefill_state(k, v)
    if kind == "quadratic":
        return kata.fwd_quadratic(q, k, v)
    if kind == "lin":
        return kata.lin_fwd_chunked(q, k, v, C, s["feature"], eps=RELU_EPS,
                                    normalize=s["normalize"])
    if kind == "fwd":
        if s["g"] > 1:
            return kata.mg_fwd_chunked(q, k, v, C, s["g"])
        return kata.fwd_chunked(q, k, v, C)
    # a training step; the bf16 forward also saves the row denominators
    if s["dtype"] == "bf16":
        out, den = kata.fwd_chunked_train(q, k, v, C)
        return (out, den) + tuple(kata.bwd_chunked(q, k, v, out, s["dout"], C, den=den))
    out = kata.fwd_chunked(q, k, v, C)
    return (out,) + tuple(kata.bwd_chunked(q, k, v, out, s["dout"], C))


# ---- what a pass cannot do without ------------------------------------------------

def work(case):
    """Each input read once and each output written once; the operations of the
    cheaper of the quadratic and the chunked-state form."""
    B, H, T, d, dv, C, g = (case[x] for x in ("B", "H", "T", "d", "dv", "C", "g"))
    kind, bh = case["kind"], B * H
    e = 2 if case["dtype"] == "bf16" else 4
    n = g * (d // g) * (d // g + 1) // 2
    rows = bh * T
    if kind == "decode":
        return {"bytes": bh * (8 * n * (dv + 1) + e * (2 * d + dv) + 4 * dv),
                "flops": bh * n * (4 * dv + 4)}
    if kind == "prefill":
        return {"bytes": e * rows * (d + dv) + 4 * bh * n * (dv + 1),
                "flops": rows * n * (2 * dv + 2)}
    io = rows * (e * (2 * d + dv) + 4 * dv)
    quad = T * (T + 1) * (d + dv)
    if kind == "lin":
        psi = kata.lin_dim(d, case["feature"])
        return {"bytes": io, "flops": bh * min(quad, T * (4 * psi * dv + C * (d + dv)))}
    chunked = T * (4 * n * dv + (C + 1) * (d + dv))
    if kind == "quadratic":
        return {"bytes": io, "flops": bh * quad}
    if kind == "fwd":
        return {"bytes": io, "flops": bh * min(quad, chunked)}
    # the backward reads q, k, v, o, do and writes dq, dk, dv
    io += rows * (e * (2 * d + dv) + 8 * dv + 4 * (2 * d + dv))
    quad += T * (T + 1) * (3 * d + 2 * dv)
    chunked += T * (10 * n * dv + (C + 1) * (3 * d + 2 * dv))
    return {"bytes": io, "flops": bh * min(quad, chunked)}


def tolerance(case):
    """About four times the measured distance from the 64-bit outputs."""
    if case["kind"] == "decode":
        return {"rel": 2e-6, "max": 1e-4}  # fp32 state, one update
    if case["kind"] == "prefill":
        return {"rel": 5e-5, "max": 1e-3}  # fp32 sums over up to 8192 tokens
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3}
    return {"rel": 1.2e-2, "max": 0.5}


# ---- the definition in 64 bits ------------------------------------------------------

def _psi(x, feature):
    if feature == kata.LIN_RELU:
        return x.clamp_min(0) + RELU_EPS
    if feature == kata.LIN_ELU:
        return torch.where(x > 0, x + 1, x.exp())
    if feature == kata.LIN_LORENTZ:
        return torch.cat((x, x.norm(dim=-1, keepdim=True)), -1)
    if feature == kata.LIN_LORENTZ_S:
        y, t = x[:, :-1], x[:, -1:]
        return torch.cat((y, y.norm(dim=-1, keepdim=True) * (1 + t * t)), -1)
    return x


def _exact_decode(case, seed):
    s = prepare(case, seed)
    a, b = _packed_pairs(case["d"])
    q, k, v = (s[x].double() for x in ("q", "k", "v"))
    S, z = s.pop("S").double(), s.pop("z").double()
    pk = k[..., a] * k[..., b]
    S += pk[..., None] * v[:, :, None, :]
    z += pk
    pq = q[..., a] * q[..., b] * torch.where(a == b, 1.0, 2.0).double()
    num = torch.matmul(pq[:, :, None, :], S)[:, :, 0]
    den = (pq * z).sum(-1, keepdim=True)
    return num / den, S, z


def _exact_prefill(case, seed):
    s = prepare(case, seed)
    B, H, d, dv = (case[x] for x in ("B", "H", "d", "dv"))
    a, b = _packed_pairs(d)
    S = torch.empty((B * H, a.numel(), dv), dtype=torch.float64, device=DEV)
    z = torch.empty((B * H, a.numel()), dtype=torch.float64, device=DEV)
    k, v = s["k"].flatten(0, 1), s["v"].flatten(0, 1)
    for h in range(B * H):
        kt = k[h].double().t().contiguous()
        phi = kt[a] * kt[b]
        S[h] = phi @ v[h].double()
        z[h] = phi.sum(1)
    return S.view(B, H, -1, dv), z.view(B, H, -1)


def exact(case, seed):
    if case["kind"] == "decode":
        return _exact_decode(case, seed)
    if case["kind"] == "prefill":
        return _exact_prefill(case, seed)
    s = prepare(case, seed)
    B, H, T, d, dv = (case[x] for x in ("B", "H", "T", "d", "dv"))
    train = case["kind"] == "train"
    q, k, v = (s[x].flatten(0, 1) for x in ("q", "k", "v"))
    out = torch.empty((B * H, T, dv), dtype=torch.float64, device=DEV)
    den = torch.empty((B * H, T), dtype=torch.float64, device=DEV)
    if train:
        dq, dk = (torch.zeros((B * H, T, d), dtype=torch.float64, device=DEV) for _ in range(2))
        dvv = torch.zeros((B * H, T, dv), dtype=torch.float64, device=DEV)
        dout = s["dout"].flatten(0, 1)
    rows = 4096
    for h in range(B * H):
        qh, kh, vh = (x[h].double() for x in (q, k, v))
        if case["kind"] == "lin":
            qh, kh = _psi(qh, case["feature"]), _psi(kh, case["feature"])
        blocks = [(x, x + d // case["g"]) for x in range(0, d, d // case["g"])]
        for r in range(0, T, rows):
            e = min(T, r + rows)
            if case["kind"] == "lin":
                w = qh[r:e] @ kh[:e].t()
            else:
                w = 0
                for x, y in blocks:
                    sc = qh[r:e, x:y] @ kh[:e, x:y].t()
                    w = w + sc * sc
            w = torch.tril(w, diagonal=r)
            D = w.sum(1) if case["normalize"] else torch.ones(e - r, dtype=torch.float64,
                                                              device=DEV)
            o = w @ vh[:e]
            o = torch.where(D[:, None] > 0, o / D[:, None], torch.zeros_like(o))
            out[h, r:e], den[h, r:e] = o, D
            if train:  # g = 1: sc holds the scores of the block
                do = dout[h, r:e].double()
                a = do / D[:, None]
                dw = torch.tril(a @ vh[:e].t() - (a * o).sum(1, keepdim=True), diagonal=r)
                dw *= 2 * sc
                dq[h, r:e] = dw @ kh[:e]
                dk[h, :e] += dw.t() @ qh[r:e]
                dvv[h, :e] += w.t() @ a
    out = out.view(B, H, T, dv)
    if not train:
        return out
    grads = tuple(x.view(B, H, T, -1) for x in (dq, dk, dvv))
    return ((out, den.view(B, H, T)) if case["dtype"] == "bf16" else (out,)) + grads
