"""The quadratic-form gradients of bf16 inputs (d = dv = C = 64, g = 1) at the
edges of their tiles and of their dispatch: T around the 32-row tiles and the
128-row workgroups, head counts that are and are not multiples of eight (two
orders of the workgroups), saved and recomputed denominators, zero
denominators, and the length where the chunk states take over.

Tolerance: the products of the gradients carry at most two factors rounded to
bf16 (unit roundoff 2^-9 to nearest), so a term is off by less than 2^-7 of
itself; 2e-2 per head leaves the terms of either sign room to cancel."""
import numpy as np
import pytest

import workloads
from gpu_helpers import log, to_device

pytestmark = pytest.mark.gpu

REL = 2e-2


@pytest.fixture(scope="module")
def kata():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_17419_amd as k
    k.lib()  # raises if libkata.so is missing: no fallback
    return k


def _inputs(B, H, T, seed=5):
    inp = workloads.make_inputs("mid_bf16", B=B, H=H, T=T)
    dout = np.random.default_rng(seed).standard_normal(inp["v"].shape).astype(np.float32)
    return inp, dout


def _close(got, ref, what):
    for name, a, b in zip(("dq", "dk", "dv"), got, ref):
        a = a.double().cpu().numpy().reshape(-1, b.shape[2] * b.shape[3])
        b = np.asarray(b, dtype=np.float64).reshape(a.shape)
        rel = (np.linalg.norm(a - b, axis=1) / np.maximum(np.linalg.norm(b, axis=1), 1e-30)).max()
        log(f"  {what} {name}: {rel:.2e}")
        assert np.isfinite(a).all() and rel <= REL, (what, name, rel)


@pytest.mark.parametrize("B,H,T", [(1, 1, 2), (1, 3, 32), (2, 4, 33), (1, 2, 127), (1, 8, 128),
                                   (1, 5, 129), (2, 8, 544), (1, 3, 641), (5, 8, 160)])
def test_quadratic_gradients_at_tile_edges(kata, orc, B, H, T):
    import torch
    log(f"case quadratic gradients B{B} H{H} T{T}")
    inp, dout = _inputs(B, H, T)
    q, k, v = (to_device(inp[n], "bf16") for n in ("q_dev", "k_dev", "v_dev"))
    # the exact forward output and denominators
    out = torch.from_numpy(orc.fwd(inp["q"], inp["k"], inp["v"]).astype(np.float32)).cuda()
    s = np.einsum("bhtx,bhix->bhti", inp["q"].astype(np.float64), inp["k"].astype(np.float64))
    den = torch.from_numpy(np.tril(s * s).sum(-1).astype(np.float32)).cuda()
    d_out = torch.from_numpy(dout).cuda()
    ref = orc.bwd_mg(inp["q"], inp["k"], inp["v"], dout, 1)
    _close(kata.bwd_chunked(q, k, v, out, d_out, 64, den=den), ref, "saved den")
    _close(kata.bwd_chunked(q, k, v, out, d_out, 64), ref, "own den")


def test_zero_denominator_rows_pass_no_gradient(kata, orc):
    import torch
    log("case quadratic gradients, zero denominators B1 H2 T200")
    inp, dout = _inputs(1, 2, 200)
    q, k, v = (to_device(inp[n], "bf16") for n in ("q_dev", "k_dev", "v_dev"))
    q[0, 1, [0, 31, 32, 150, 199]] = 0
    qz = q.float().cpu().numpy()
    out = torch.from_numpy(orc.fwd(qz, inp["k"], inp["v"]).astype(np.float32)).cuda()
    got = kata.bwd_chunked(q, k, v, out, torch.from_numpy(dout).cuda(), 64)
    _close(got, orc.bwd_mg(qz, inp["k"], inp["v"], dout, 1), "zero rows")
    assert not got[0][0, 1, [0, 31, 32, 150, 199]].any()


@pytest.mark.parametrize("T", [8192, 4100])
def test_quadratic_against_chunk_states(kata, T):
    """Eight heads of these lengths take the quadratic form, one head alone the
    chunk states: the same gradients from the same forward."""
    import torch
    log(f"case quadratic against chunk states B1 H8 T{T}")
    inp, dout = _inputs(1, 8, T)
    q, k, v = (to_device(inp[n], "bf16") for n in ("q_dev", "k_dev", "v_dev"))
    out, den = kata.fwd_chunked_train(q, k, v, 64)
    d_out = torch.from_numpy(dout).cuda()
    got = kata.bwd_chunked(q, k, v, out, d_out, 64, den=den)
    for h in (0, 5):
        one = kata.bwd_chunked(*(x[:, h:h + 1].contiguous() for x in (q, k, v, out, d_out)), 64,
                               den=den[:, h:h + 1].contiguous())
        _close([g[:, h:h + 1] for g in got], [x.cpu().numpy() for x in one], f"head {h}")
