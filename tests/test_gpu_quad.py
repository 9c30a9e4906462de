"""The bf16 quadratic form at the edges of its tiles and of its dispatch: T
around the 32-row tiles, the two-tile stages and the 128- and 256-query
workgroups; one wave or two per query tile; head counts that are and are not
multiples of eight; and the default forward on both sides of the length where
the span pipeline takes over."""
import numpy as np
import pytest

import workloads
from gpu_helpers import assert_bf16_close, log, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kata():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_17419_amd as k
    k.lib()  # raises if libkata.so is missing: no fallback
    return k


def _qkv(inp):
    return tuple(to_device(inp[n], "bf16") for n in ("q_dev", "k_dev", "v_dev"))


@pytest.mark.parametrize("name,g", [("mid_bf16", 1), ("mid_bf16", 2), ("recall_bf16", 1)])
@pytest.mark.parametrize("B,H,T", [(1, 1, 1), (1, 3, 63), (1, 8, 64), (1, 2, 65), (2, 4, 129),
                                   (1, 5, 255), (1, 16, 257), (3, 1, 513), (2, 8, 672)])
def test_tile_edges(kata, orc, name, g, B, H, T):
    log(f"case quadratic {name} g{g} B{B} H{H} T{T}")
    inp = workloads.make_inputs(name, B=B, H=H, T=T)
    got = kata.mg_fwd_quadratic(*_qkv(inp), g).cpu().numpy()
    ref = orc.fwd_mg(inp["q"], inp["k"], inp["v"], g) if g > 1 else orc.fwd(inp["q"], inp["k"],
                                                                           inp["v"])
    assert_bf16_close(got, ref, f"T{T}")


@pytest.mark.parametrize("B,H,T", [(8, 16, 1100), (1, 8, 4200), (33, 8, 550)])
def test_one_and_two_waves_per_tile(kata, orc, B, H, T):
    """Workgroup counts on both sides of the rule, three heads against the oracle
    (the last head and those at the ends of the XCD groups)."""
    log(f"case quadratic B{B} H{H} T{T} d64")
    inp = workloads.make_inputs("mid_bf16", B=B, H=H, T=T)
    got = kata.fwd_quadratic(*_qkv(inp)).cpu().numpy().reshape(B * H, T, 64)
    for bh in (0, 7, B * H - 1):
        sel = lambda x: x.reshape(B * H, T, x.shape[-1])[bh][None, None]
        assert_bf16_close(got[bh][None, None],
                          orc.fwd(sel(inp["q"]), sel(inp["k"]), sel(inp["v"])), f"head {bh}")


@pytest.mark.parametrize("name,g,B,H,T", [("mid_bf16", 1, 1, 2, 6144), ("mid_bf16", 2, 1, 17, 3584),
                                          ("mid_bf16", 2, 1, 2, 5632),
                                          ("mid_bf16", 1, 1, 129, 5632),
                                          ("recall_bf16", 1, 1, 17, 3072),
                                          ("recall_bf16", 1, 1, 2, 4608)])
def test_default_forward_either_side_of_the_rule(kata, name, g, B, H, T):
    """T tokens run quadratically, T + 33 through span states; the first T outputs
    are the same up to bf16 rounding, and so are an explicit span's."""
    import torch
    log(f"case default forward {name} g{g} B{B} H{H} T{T} and T + 33")
    inp = workloads.make_inputs(name, B=B, H=H, T=T + 33)
    q, k, v = _qkv(inp)
    cut = lambda x: x[:, :, :T].contiguous()
    short = kata.mg_fwd_chunked(cut(q), cut(k), cut(v), 128, g)
    quad = kata.mg_fwd_quadratic(cut(q), cut(k), cut(v), g)
    assert torch.equal(short, quad)
    for other in (kata.mg_fwd_chunked(q, k, v, 128, g)[:, :, :T],
                  kata.mg_fwd_chunked(cut(q), cut(k), cut(v), 128, g, span_chunks=8)):
        rel = ((other - short).norm(dim=-1) / short.norm(dim=-1)).max()
        assert float(rel) <= 2e-2, float(rel)
