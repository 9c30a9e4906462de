"""The matrix-core chunk-state kernel behind kata_prefill_state, at the edges of
its tiles: widths that do and do not split into 16-byte pieces, every value
width class (up to 32, 64, 128, 256 columns), few and many tiles (one wave or
four per tile), token counts around the staged block, and the overflow route."""
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


def _pairs(d, g):
    m = d // g
    a, b = np.triu_indices(m)
    return (np.concatenate([a + i * m for i in range(g)]),
            np.concatenate([b + i * m for i in range(g)]))


def _inputs(dtype, H, T, d, dv, seed):
    import torch
    gen = torch.Generator().manual_seed(seed)
    tt = torch.bfloat16 if dtype == "bf16" else torch.float32
    return (torch.randn((1, H, T, d), generator=gen).to(tt),
            torch.randn((1, H, T, dv), generator=gen).to(tt))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("H,T,d,dv,g", [
    (1, 1, 64, 64, 1), (2, 63, 64, 64, 1), (2, 65, 64, 64, 2), (3, 128, 32, 32, 1),
    (2, 100, 7, 5, 1), (2, 129, 24, 40, 3), (1, 70, 64, 256, 1), (1, 64, 40, 129, 1),
    (8, 65, 64, 64, 1), (40, 33, 33, 66, 1)])
def test_state_edges(kata, dtype, H, T, d, dv, g):
    import torch
    log(f"case state {dtype} H{H} T{T} d{d} dv{dv} g{g}")
    k, v = _inputs(dtype, H, T, d, dv, 7)
    S, z = kata.mg_prefill_state(k.cuda(), v.cuda(), g)
    torch.cuda.synchronize()
    a, b = _pairs(d, g)
    k64, v64 = k.double().numpy()[0], v.double().numpy()[0]
    phi = k64[:, :, a] * k64[:, :, b]
    # fp32 products and sums in any order: each of the T terms passes at most
    # T + 1 additions and two product roundings
    tol = (T + 3) * U
    for got, ref, mag in (
            (S, np.einsum("htf,htj->hfj", phi, v64),
             np.einsum("htf,htj->hfj", np.abs(phi), np.abs(v64))),
            (z, phi.sum(1), np.abs(phi).sum(1))):
        err = np.abs(got.cpu().numpy()[0].astype(np.float64) - ref)
        assert np.all(err <= tol * mag + 1e-37), (err / np.maximum(mag, 1e-30)).max()


def test_state_overflow_matches_fp32(kata):
    """A product k_a k_b past fp32's range gives the infinities (and no NaN)
    that fp32 arithmetic gives, and leaves the other features alone."""
    import torch
    k, v = _inputs("bf16", 2, 70, 64, 64, 8)
    k[0, 1, 5, 3] = 3e25
    S, z = kata.prefill_state(k.cuda(), v.cuda())
    torch.cuda.synchronize()
    a, b = _pairs(64, 1)
    kf, vf = k.float()[0], v.float()[0]
    ref = torch.matmul((kf[:, :, a] * kf[:, :, b]).transpose(1, 2).contiguous(), vf)
    got = S.cpu()[0]
    assert int(torch.isinf(ref).sum()) == 64
    assert torch.equal(torch.isinf(got), torch.isinf(ref))
    assert not torch.isnan(got).any() and torch.isinf(z.cpu()[0, 1]).sum() == 1
    fin = torch.isfinite(ref)
    assert torch.allclose(got[fin], ref[fin], rtol=1e-4, atol=1e-4)


@pytest.mark.parametrize("B,H,d,dv,g", [
    (1, 1, 64, 64, 1), (1, 3, 1, 4, 1), (2, 2, 33, 32, 1), (1, 5, 24, 128, 3), (1, 2, 64, 256, 2),
    (3, 1, 40, 8, 5), (1, 2, 48, 24, 1), (1, 2, 7, 5, 1), (6, 16, 64, 64, 1), (18, 16, 64, 64, 1),
    (24, 1, 64, 256, 1),  # large heads past the caches
    # small heads: 512 and more than 512 of them, 1280 and more for eight columns
    (64, 8, 8, 16, 1), (513, 1, 8, 16, 2), (160, 8, 16, 8, 1), (1281, 1, 16, 8, 1)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_decode_step_forms(kata, dtype, B, H, d, dv, g):
    """Few heads, many heads and value widths with and without a wide form: two
    steps against fp64.  Each S, z entry takes one product and one addition, each
    output sums n entries twice rounded; (n / 32 + 64) roundoffs of the magnitude
    sums bound the order of any of the kernels' sums."""
    import torch
    log(f"case decode {dtype} B{B} H{H} d{d} dv{dv} g{g}")
    gen = torch.Generator(device="cuda").manual_seed(3)
    tt = torch.bfloat16 if dtype == "bf16" else torch.float32
    a, b = (torch.from_numpy(x).cuda() for x in _pairs(d, g))
    n = a.numel()
    S = torch.randn((B, H, n, dv), generator=gen, device="cuda")
    z = torch.rand((B, H, n), generator=gen, device="cuda") + 4.0 * (a == b)
    S64, z64 = S.double(), z.double()
    for _ in range(2):
        q, k = (torch.randn((B, H, d), generator=gen, device="cuda").to(tt) for _ in range(2))
        v = torch.randn((B, H, dv), generator=gen, device="cuda").to(tt)
        out = kata.mg_decode_step(S, z, q, k, v, g)
        q6, k6, v6 = q.double(), k.double(), v.double()
        pk = k6[..., a] * k6[..., b]
        S64 += pk[..., None] * v6[:, :, None, :]
        z64 += pk
        assert float((S.double() - S64).abs().max()) <= 8 * U * float(S64.abs().max())
        assert float((z.double() - z64).abs().max()) <= 8 * U * float(z64.abs().max())
        pq = q6[..., a] * q6[..., b] * torch.where(a == b, 1.0, 2.0)
        den = (pq * z64).sum(-1, keepdim=True)
        num = (pq[..., None] * S64).sum(2)
        ref = torch.where(den > 0, num / den, torch.zeros_like(num))
        tol = (n / 32 + 64) * U
        bound = tol * ((pq.abs()[..., None] * S64.abs()).sum(2) / den.abs() + ref.abs() *
                       (pq.abs() * z64.abs()).sum(-1, keepdim=True) / den.abs())
        sure = den.abs() > 1e-3 * (pq.abs() * z64.abs()).sum(-1, keepdim=True)
        assert bool((((out.double() - ref).abs() <= bound + 1e-30) | ~sure).all())


@pytest.mark.parametrize("d,dv", [(64, 64), (32, 64), (24, 16), (5, 4)])
def test_decode_infinite_state_entry(kata, d, dv):
    """An infinity in the state's last row (which threads past the last row load
    again) reaches its own output column as an infinity, and no other column."""
    import torch
    log(f"case decode, infinity in the last state row: B1 H2 d{d} dv{dv}")
    gen = torch.Generator(device="cuda").manual_seed(4)
    n = d * (d + 1) // 2
    S = torch.randn((1, 2, n, dv), generator=gen, device="cuda")
    z = torch.rand((1, 2, n), generator=gen, device="cuda") + 1.0
    q, k = (torch.rand((1, 2, d), generator=gen, device="cuda") + 0.1 for _ in range(2))
    v = torch.randn((1, 2, dv), generator=gen, device="cuda")
    clean = kata.decode_step(S.clone(), z.clone(), q, k, v)
    S[0, 1, n - 1, 2] = float("inf")
    out = kata.decode_step(S, z, q, k, v)  # all weights and z positive
    torch.cuda.synchronize()
    assert float(out[0, 1, 2]) == float("inf")
    clean[0, 1, 2] = float("inf")
    assert torch.equal(out, clean)


def test_decode_of_more_heads_than_a_wide_launch_holds(kata):
    """2^22 + 8 small heads: 1024 threads each would be 2^32 or more in one launch.
    The first and the last heads equal the same heads by themselves."""
    import torch
    BH, d, dv = (1 << 22) + 8, 1, 4
    log(f"case decode B{BH} H1 d{d} dv{dv}")
    gen = torch.Generator(device="cuda").manual_seed(6)
    S = torch.randn((BH, 1, 1, dv), generator=gen, device="cuda")
    z = torch.rand((BH, 1, 1), generator=gen, device="cuda")
    q, k = (torch.randn((BH, 1, d), generator=gen, device="cuda") for _ in range(2))
    v = torch.randn((BH, 1, dv), generator=gen, device="cuda")
    ends = (slice(0, 3), slice(BH - 3, BH))
    alone = []
    for part in ends:
        S1, z1 = S[part].clone(), z[part].clone()
        out = kata.decode_step(S1, z1, *(x[part].clone() for x in (q, k, v)))
        alone.append((out, S1, z1))
    out = kata.decode_step(S, z, q, k, v)
    torch.cuda.synchronize()
    for part, refs in zip(ends, alone):
        for x, y in zip((out, S, z), refs):  # one product and one sum, or their quotient
            assert torch.allclose(x[part], y, rtol=8 * U, atol=0)


@pytest.mark.parametrize("H,T,d,dv,g", [(2, 200, 64, 64, 1), (16, 130, 64, 64, 2), (2, 100, 7, 5, 1),
                                        (1, 100, 64, 256, 1)])
@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_state_non_finite_inputs(kata, H, T, d, dv, g, bad, dtype):
    """One non-finite entry of v or k gives the infinities and NaN of fp32
    arithmetic in its own state entries, and the sums elsewhere (one wave and four
    per tile, both staging forms)."""
    import torch
    a, b = (torch.from_numpy(x) for x in _pairs(d, g))
    for name in ("v", "k"):
        log(f"case state {dtype} {bad} in {name}: H{H} T{T} d{d} dv{dv} g{g}")
        k, v = _inputs(dtype, H, T, d, dv, 9)
        (v if name == "v" else k)[0, H - 1, 70, 3] = bad
        S, z = kata.mg_prefill_state(k.cuda(), v.cuda(), g)
        torch.cuda.synchronize()
        phi = (k.double()[..., a] * k.double()[..., b])[0]
        vd = v.double()[0]
        ref = torch.zeros((H, a.numel(), dv), dtype=torch.float64)
        mag = torch.zeros_like(ref)
        for t in range(T):  # not a product of matrices: its order is the library's
            term = phi[:, t, :, None] * vd[:, t, None, :]
            ref += term
            mag += term.abs()
        for got, r, m in ((S.cpu()[0].double(), ref, mag),
                          (z.cpu()[0].double(), phi.sum(1), phi.abs().sum(1))):
            fin = torch.isfinite(r)
            assert torch.equal(torch.isnan(got), torch.isnan(r))
            assert torch.equal(got[torch.isinf(r)], r[torch.isinf(r)])
            assert bool(((got - r).abs()[fin] <= (T + 3) * U * m[fin] + 1e-37).all())
