"""Bias of the fused attention from a window of diagonals (all that lies beyond the last bucket's first distance clamped to
its edge, the causal mask in it) and, where that would be long, from the slice of every diagonal a workgroup can touch."""
from dataclasses import replace

import pytest

import synth_inputs as SI
from oracle import t5_oracle as O
from parity_util import block_floors, check_bf16, make_case, rel_err, run_block_gpu

pytestmark = pytest.mark.gpu

BASE = SI.BlockConfig("bias_window", 2, 620, 64, 128, 2, 64, 128, attn_scale=0.125)


# 620 positions: nearly every sub-tile beyond the window, a few, or (4096) the slice, for windows of up to 592 values; with 256
# and 64 channels dq has the slice and the others the window
@pytest.mark.parametrize("max_distance", [20, 128, 256, 4096])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d_kv", [64, 128])
def test_window_and_slice(d_kv, causal, max_distance):
    import paper_2203_17189_amd as P
    cfg = replace(BASE, causal=causal, d_kv=d_kv, attn_scale=d_kv ** -0.5, max_distance=max_distance,
                  name=f"bias_window_{d_kv}_{int(causal)}_{max_distance}")
    want = P.PATH_MFMA_ATTN_FWD | P.PATH_MFMA_ATTN_BWD
    assert P.t5_block_kernel_path(cfg) & want == want
    w, x, dy = make_case(cfg)
    y, saved = O.block_fwd(cfg, x, w)
    dx, g = O.block_bwd(cfg, dy, w, saved)
    gy, gdx, gg = run_block_gpu(cfg, w, x, dy)
    errs = {"y": rel_err(gy, y), "dx": rel_err(gdx, dx), **{n: rel_err(gg[n], g[n]) for n in g}}
    check_bf16(cfg.name, errs, block_floors(cfg, w, x, dy, (y, dx, g)))


def test_slice_of_a_long_causal_sequence():
    """More positions than leave room for a third stage of dk/dv beside their slice: 80 tokens behind 7600 with no gradient of
    their own change nothing before them."""
    import torch
    import paper_2203_17189_amd as P
    from parity_util import upload_case
    cfg = replace(BASE, batch=1, seq=7680, d_model=64, n_heads=1, d_ff=64, causal=True, max_distance=1024, name="bias_slice_long")
    w, x, dy = make_case(cfg)
    grads = []
    for seq in (7600, 7680):
        cut = replace(cfg, seq=seq)
        dw, dx_in, ddy = upload_case(cut, w, x[:, :seq], dy[:, :seq])
        ddy[:, 7600:] = 0
        _, stash = P.t5_block_fwd(cut, dx_in, dw)
        dx, g = P.t5_block_bwd(cut, ddy, dx_in, dw, stash)
        assert not dx[:, 7600:].any()
        grads.append(dict(g, dx=dx[:, :7600].float()))
    for n in grads[0]:  # the same roundings, but for sums in another order that fall on the other side of one: 2^-8 here and there
        a, b = grads[0][n].double(), grads[1][n].double()
        assert (a - b).norm() <= 2e-3 * a.norm(), n
