"""The fp32 quadratic form behind the fp32 forward and backward (one feature
block): widths that do and do not fill their 16 / 32 / 64 (128, 256) classes, T
around the 32-row tiles and the eight waves' shares of the walk, fp32 and bf16
inputs, rows with a zero denominator, and the lengths where the chunk states
take over."""
import numpy as np
import pytest

from gpu_helpers import log

pytestmark = pytest.mark.gpu

U = 2.0 ** -24  # unit roundoff of fp32


@pytest.fixture(scope="module")
def kata():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_17419_amd as k
    k.lib()  # raises if libkata.so is missing: no fallback
    return k


def _inputs(dtype, B, H, T, d, dv, seed=11):
    import torch
    gen = torch.Generator().manual_seed(seed)
    tt = torch.bfloat16 if dtype == "bf16" else torch.float32
    def unit(x):
        return x / x.norm(dim=-1, keepdim=True)
    q, k = (unit(torch.randn((B, H, T, d), generator=gen)).to(tt) for _ in range(2))
    v = torch.randn((B, H, T, dv), generator=gen).to(tt)
    return q, k, v, torch.randn((B, H, T, dv), generator=gen)


def _dense(q, k, v, dout):
    """Outputs, gradients and, for each, the sums of their terms' magnitudes."""
    q, k, v, g = (x.double().numpy() for x in (q, k, v, dout))
    s = np.tril(np.matmul(q, k.swapaxes(-1, -2)))
    w = s * s
    D = w.sum(-1, keepdims=True)
    inv = np.divide(1.0, D, out=np.zeros_like(D), where=D > 0)
    o = np.matmul(w, v) * inv
    a = g * inv
    c = np.tril(np.matmul(a, v.swapaxes(-1, -2)) - (a * o).sum(-1, keepdims=True)) * s
    ab = np.abs
    cm = np.tril(np.matmul(ab(a), ab(v).swapaxes(-1, -2)) + (ab(a) * ab(o)).sum(-1, keepdims=True))
    sm = np.tril(np.matmul(ab(q), ab(k).swapaxes(-1, -2)))
    tr = lambda x: x.swapaxes(-1, -2)
    vals = (o, 2 * np.matmul(c, k), 2 * np.matmul(tr(c), q), np.matmul(tr(w), a))
    mags = (np.matmul(sm * sm, ab(v)) * inv, 2 * np.matmul(cm * sm, ab(k)),
            2 * np.matmul(tr(cm * sm), ab(q)), np.matmul(tr(sm * sm), ab(a)))
    return vals, mags


# fp32 rounding of a term: its products and the sums of d, dv or T values that
# it passes, in the scores (twice), D, a_t and the result; the sums run over
# at most T / 8 + 8 values one after the other, so (4 (d + dv) + T) roundoffs
# bound every output with room to spare, and each is far below it in practice
def _tol(T, d, dv):
    return (4 * (d + dv) + T + 16) * U


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,H,T,d,dv,C", [
    (1, 1, 1, 16, 16, 32), (1, 2, 31, 7, 5, 16), (2, 4, 33, 16, 64, 32), (1, 3, 64, 32, 16, 64),
    (1, 2, 65, 33, 30, 64), (1, 8, 256, 64, 33, 24), (1, 2, 257, 24, 40, 32), (3, 3, 300, 48, 64, 48)])
def test_forward_and_gradients(kata, dtype, B, H, T, d, dv, C):
    import torch
    log(f"case fp32 quadratic {dtype} B{B} H{H} T{T} d{d} dv{dv} C{C}")
    q, k, v, g = _inputs(dtype, B, H, T, d, dv)
    if T > 40:
        q[:, :, [3, 32, 40]] = 0  # zero denominators
    vals, mags = _dense(q, k, v, g)
    qd, kd, vd, gd = (x.cuda() for x in (q, k, v, g))
    out = kata.fwd_chunked(qd, kd, vd, C)
    exact = torch.from_numpy(vals[0].astype(np.float32)).cuda()
    got = (out,) + tuple(kata.bwd_chunked(qd, kd, vd, exact, gd, C))
    torch.cuda.synchronize()
    for name, x, ref, mag in zip(("o", "dq", "dk", "dv"), got, vals, mags):
        err = np.abs(x.double().cpu().numpy() - ref)
        worst = (err / np.maximum(mag, 1e-30)).max()
        log(f"  {name}: worst error {worst / U:.1f} roundoffs of the magnitude sum")
        assert np.all(err <= _tol(T, d, dv) * mag + 1e-30), name
    if T > 40:
        assert not got[0][:, :, [3, 32, 40]].any() and not got[1][:, :, [3, 32, 40]].any()


@pytest.mark.parametrize("dv", [66, 128, 130, 256])
def test_wide_values(kata, dv):
    import torch
    log(f"case fp32 quadratic forward B1 H2 T100 d64 dv{dv}")
    q, k, v, g = _inputs("f32", 1, 2, 100, 64, dv)
    vals, mags = _dense(q, k, v, g)
    out = kata.fwd_chunked(q.cuda(), k.cuda(), v.cuda(), 64)
    torch.cuda.synchronize()
    assert np.all(np.abs(out.double().cpu().numpy() - vals[0]) <= _tol(100, 64, dv) * mags[0] + 1e-30)


@pytest.mark.parametrize("d,dv,T", [(7, 5, 4096), (16, 16, 8192)])
def test_against_chunk_states(kata, d, dv, T):
    """T + 40 tokens run through the chunk states, T in the quadratic form: the
    same first T outputs; and the gradients of a cotangent that is zero past T,
    given the same forward output, are the same too."""
    import torch
    log(f"case fp32 quadratic against chunk states B1 H2 T{T} d{d} dv{dv}")
    q, k, v, g = (x.cuda() for x in _inputs("f32", 1, 2, T + 40, d, dv))
    g[:, :, T:] = 0
    cut = lambda x: x[:, :, :T].contiguous()
    long = kata.fwd_chunked(q, k, v, 32)
    short = kata.fwd_chunked(cut(q), cut(k), cut(v), 32)
    assert float((long[:, :, :T] - short).abs().max()) <= 2e-5 * float(long.abs().max())
    a = kata.bwd_chunked(q, k, v, long, g, 32)
    b = kata.bwd_chunked(cut(q), cut(k), cut(v), cut(long), cut(g), 32)
    torch.cuda.synchronize()
    for name, x, y in zip(("dq", "dk", "dv"), a, b):
        assert float((cut(x) - y).norm() / y.norm()) <= 2e-5, name
        assert not x[:, :, T:].any() or name == "dq"


def test_more_tokens_than_one_launch_holds(kata):
    """65535 heads of 2100 tokens: the pair tiles would need 2^32 threads or more
    in one launch, so the chunk states form these gradients; the first and the
    last heads equal the same heads by themselves (quadratic form)."""
    import torch
    BH, T, d, dv = 65535, 2100, 7, 5
    assert BH * -(-T // 128) * 8 * 512 >= 1 << 32
    log(f"case fp32 gradients B{BH} H1 T{T} d{d} dv{dv}")
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, k, v, g = (torch.randn((BH, 1, T, w), generator=gen, device="cuda") for w in (d, d, dv, dv))
    g[:, :, :32] = 0  # rows whose few weights may nearly vanish
    out = kata.fwd_chunked(q, k, v, 32)
    grads = kata.bwd_chunked(q, k, v, out, g, 32)
    torch.cuda.synchronize()
    for part in (slice(0, 2), slice(BH - 2, BH)):
        cut = [x[part].contiguous() for x in (q, k, v, out, g)]
        alone = kata.bwd_chunked(*cut, 32)
        for name, x, y in zip(("dq", "dk", "dv"), grads, alone):
            assert float((x[part] - y).norm() / y.norm()) <= 2e-5, name


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,dv", [(16, 16), (64, 64), (7, 5), (33, 30), (64, 200)])
def test_reads_stay_inside_a_head(kata, dtype, d, dv):
    """A head between two whose every value is NaN: rows past its T (or before its
    first) that were read from them would show, even with weight zero.  T below
    and above the 16 and 28 rows that a tile's later loads lie past its first."""
    import torch
    for T in (1, 5, 10, 20, 27, 28, 33, 45):
        log(f"case fp32 quadratic between NaN heads {dtype} T{T} d{d} dv{dv}")
        ins = _inputs(dtype, 1, 1, T, d, dv)
        alone = [x.cuda() for x in ins]
        three = [torch.full((1, 3) + x.shape[2:], float("nan"), dtype=x.dtype, device="cuda")
                 for x in ins]
        for x, y in zip(three, alone):
            x[:, 1:2] = y
        ref = kata.fwd_chunked(*alone[:3], 32)
        got = kata.fwd_chunked(*three[:3], 32)
        torch.cuda.synchronize()
        assert torch.isfinite(ref).all() and torch.equal(got[:, 1:2], ref), (T, "o")
        if dv > 64:
            continue  # the gradients of wide values are not formed quadratically
        out = torch.full_like(three[3], float("nan"))
        out[:, 1:2] = ref
        refs = kata.bwd_chunked(*alone[:3], ref, alone[3], 32)
        gots = kata.bwd_chunked(*three[:3], out, three[3], 32)
        torch.cuda.synchronize()
        for name, x, y in zip(("dq", "dk", "dv"), gots, refs):
            assert torch.isfinite(y).all() and torch.equal(x[:, 1:2], y), (T, name)


def _causal(q, k, v, g, o=None):
    """Outputs and gradients (of the given o, or their own), each a sum over its own
    pairs i <= t alone, with the sums of the terms' magnitudes: one head, float64."""
    q, k, v, g = (x[0, 0].double().numpy() for x in (q, k, v, g))
    T = len(q)
    S = [[q[t] @ k[i] for i in range(t + 1)] for t in range(T)]
    D = np.array([sum(s * s for s in S[t]) for t in range(T)])
    inv = np.array([1.0 / x if x > 0 else 0.0 for x in D])
    own, om = np.zeros_like(v), np.zeros_like(v)
    for t in range(T):
        for i in range(t + 1):
            own[t] += S[t][i] ** 2 * v[i] * inv[t] if D[t] > 0 else 0.0
            om[t] += (np.abs(q[t]) @ np.abs(k[i])) ** 2 * np.abs(v[i]) * inv[t]
    o = own if o is None else o[0, 0].double().numpy()
    vals = [own] + [np.zeros_like(x) for x in (q, k, v)]
    mags = [om] + [np.zeros_like(x) for x in (q, k, v)]
    ab = np.abs
    for t in range(T):
        a = g[t] * inv[t]
        b = -(g[t] @ o[t]) * inv[t]
        for i in range(t + 1):
            c = a @ v[i] + b
            cm = ab(a) @ ab(v[i]) + ab(g[t]) @ ab(o[t]) * inv[t]
            sm = ab(q[t]) @ ab(k[i])
            vals[1][t] += 2 * c * S[t][i] * k[i]
            vals[2][i] += 2 * c * S[t][i] * q[t]
            vals[3][i] += S[t][i] ** 2 * a
            mags[1][t] += 2 * cm * sm * ab(k[i])
            mags[2][i] += 2 * cm * sm * ab(q[t])
            mags[3][i] += sm * sm * ab(a)
    return vals, mags


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("d,dv", [(16, 16), (64, 64), (33, 30), (24, 200)])
def test_non_finite_values_stay_causal(kata, dtype, bad, d, dv):
    """One non-finite entry of v, k, q or dout: the outputs that its pairs belong to
    are not finite, and every other output is right.  Row 5 is among the rows with
    fp64 scores, 20 in the first tile, 50 in the second of three."""
    import torch
    T = 70
    for t0 in (5, 20, 50):
        clean = _inputs(dtype, 1, 1, T, d, dv, seed=t0)
        with np.errstate(all="ignore"):
            o = torch.from_numpy(_causal(*clean)[0][0].astype(np.float32))[None, None]
        for which, name in enumerate(("q", "k", "v", "dout")):
            if dv > 64 and name not in ("k", "v"):
                continue
            log(f"case fp32 quadratic {dtype} d{d} dv{dv}: {bad} in {name} at row {t0}")
            ins = [x.clone() for x in clean]
            ins[which][0, 0, t0, 1] = bad
            with np.errstate(all="ignore"):
                vals, mags = _causal(*ins, o=o)
            qd, kd, vd, gd, od = (x.cuda() for x in (*ins, o))
            got = [kata.fwd_chunked(qd, kd, vd, 32)]
            if dtype == "bf16" and d == dv == 64:  # the bf16 matrix-core forward
                got = [torch.from_numpy(vals[0])[None, None]]
            if dv <= 64:
                got += kata.bwd_chunked(qd, kd, vd, od, gd, 32)
            torch.cuda.synchronize()
            for what, x, ref, mag in zip(("o", "dq", "dk", "dv"), got, vals, mags):
                x = x[0, 0].double().cpu().numpy()
                fin = np.isfinite(ref)
                assert np.array_equal(np.isfinite(x), fin), (name, t0, what)
                assert fin[:t0 if name in ("k", "v") and what in ("o", "dq") else 0].all()
                # a finite output without a finite bound is the zero of D_t = NaN
                mag = np.where(np.isfinite(mag), mag, 0.0)[fin]
                assert np.all(np.abs(x[fin] - ref[fin]) <= _tol(T, d, dv) * mag + 1e-30), (
                    name, t0, what)


@pytest.mark.parametrize("B,H,T,d,dv", [(1, 8, 1500, 8, 8), (8, 8, 1500, 8, 8), (1, 2, 1500, 1, 1),
                                        (64, 8, 1100, 1, 1), (8, 8, 2048, 8, 64), (1, 2, 2048, 8, 64)])
def test_either_side_of_the_rule(kata, B, H, T, d, dv):
    """Few and many heads of narrow widths, which the rule sends to the pair tiles and
    to the chunk states: outputs and gradients of the first and the last head."""
    import torch
    log(f"case fp32 rule B{B} H{H} T{T} d{d} dv{dv}")
    q, k, v, g = _inputs("f32", B, H, T, d, dv)
    g[:, :, :32] = 0  # rows whose few weights may nearly vanish
    ends = ((0, 0), (B - 1, H - 1))
    pick = lambda x, e: x[e[0], e[1]][None, None]
    refs = [_dense(*(pick(x, e) for x in (q, k, v, g))) for e in ends]
    out = kata.fwd_chunked(*(x.cuda() for x in (q, k, v)), 64)
    given = out.clone()
    for e, (vals, _) in zip(ends, refs):
        given[e] = torch.from_numpy(vals[0][0, 0].astype(np.float32)).cuda()
    grads = kata.bwd_chunked(*(x.cuda() for x in (q, k, v)), given, g.cuda(), 64)
    torch.cuda.synchronize()
    for e, (vals, mags) in zip(ends, refs):
        for name, x, ref, mag in zip(("o", "dq", "dk", "dv"), (out, *grads), vals, mags):
            # the chunk states sum over the n features what the pairs sum over d
            err = np.abs(pick(x, e).double().cpu().numpy() - ref)[:, :, 32:]
            tol = _tol(T, d, dv) + 4 * (d * (d + 1) // 2) * U
            assert np.all(err <= tol * mag[:, :, 32:] + 1e-30), (e, name)
