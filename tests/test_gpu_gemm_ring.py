"""128x128 tiles of the bf16 GEMM with three stages of A and two of B: every remainder of the loop's six-tile rounds, and the
gated-GELU backward, which always takes them, with as few k-tiles as a layer can have."""
import pytest

import synth_inputs as SI
from oracle import t5_oracle as O
from parity_util import block_floors, check_bf16, make_case, rel_err, run_block_gpu
from test_gpu_gemm_tiles import _check_gemm, _tile

pytestmark = pytest.mark.gpu


# last tiles of 8 rows and 8 columns.  5000 rows: 360 tiles, two stages but for the first; 6024: 432, the ring
@pytest.mark.parametrize("M", [5000, 6024])
@pytest.mark.parametrize("nk", range(16, 22))
def test_every_loop_remainder(nk, M):
    assert _tile(M, 1032, 64 * nk) == "128x128, two per unit"
    _check_gemm(M, 1032, 64 * nk, True)


# 6400 x 1024, 400 tiles: the gradient behind the feed-forward is a sum of two products over d_ff, that behind the attention of
# three over 384; the runs' ends fall on every tile of the loop's rounds of six, and A's cursor passes them a tile before B's
@pytest.mark.parametrize("d_ff", [576, 640, 704, 768, 832, 896])
def test_several_runs_of_k(d_ff):
    assert _tile(6400, 1024, 2 * d_ff) == _tile(6400, 1024, 3 * 384) == "128x128, two per unit"
    cfg = SI.BlockConfig(f"gemm_ring_runs_{d_ff}", 67, 64, 100, 1024, 6, 64, d_ff, attn_scale=0.125)
    w, x, dy = make_case(cfg)
    y, saved = O.block_fwd(cfg, x, w)
    dx, g = O.block_bwd(cfg, dy, w, saved)
    gy, gdx, gg = run_block_gpu(cfg, w, x, dy)
    errs = {"y": rel_err(gy, y), "dx": rel_err(gdx, dx), **{n: rel_err(gg[n], g[n]) for n in g}}
    check_bf16(cfg.name, errs, block_floors(cfg, w, x, dy, (y, dx, g)))


# 4224 x 1024: 264 tiles, more than one per compute unit; 3968: 248, and four stages of 64
@pytest.mark.parametrize("seq", [66, 62])
@pytest.mark.parametrize("d_model", [64, 128, 192])   # one, two and three k-tiles
def test_gated_gelu_backward_few_k_tiles(d_model, seq):
    cfg = SI.BlockConfig(f"gemm_ring_{d_model}", 64, 64, seq, d_model, 1, 64, 1024, attn_scale=0.125)
    w, x, dy = make_case(cfg)
    y, saved = O.block_fwd(cfg, x, w)
    dx, g = O.block_bwd(cfg, dy, w, saved)
    gy, gdx, gg = run_block_gpu(cfg, w, x, dy)
    errs = {"y": rel_err(gy, y), "dx": rel_err(gdx, dx), **{n: rel_err(gg[n], g[n]) for n in g}}
    check_bf16(cfg.name, errs, block_floors(cfg, w, x, dy, (y, dx, g)))


@pytest.mark.parametrize("nk", [*range(1, 7), *range(12, 17)])
def test_one_tile_per_unit_every_loop_remainder(nk):
    """Four stages, of 32 and from 12 k-tiles of 64 on of those: as many k-tiles as there are stages, fewer, more; last tiles of
    64 rows and 8 columns."""
    assert _tile(3648, 776, 64 * nk) == "128x128"
    _check_gemm(3648, 776, 64 * nk, True)


@pytest.mark.parametrize("d_ff", [1024, 1088, 2048, 2112])  # stages of 32, and from above 1024 on of 64
def test_stored_weights_one_tile_per_unit(d_ff):
    """2100 x 1024 outputs, 136 tiles, over d_ff: the forward products that read weights as they are stored."""
    cfg = SI.BlockConfig(f"gemm_stored_{d_ff}", 65, 30, 70, 1024, 16, 64, d_ff, attn_scale=0.125)
    w, x, dy = make_case(cfg)
    y, saved = O.block_fwd(cfg, x, w)
    dx, g = O.block_bwd(cfg, dy, w, saved)
    gy, gdx, gg = run_block_gpu(cfg, w, x, dy)
    errs = {"y": rel_err(gy, y), "dx": rel_err(gdx, dx), **{n: rel_err(gg[n], g[n]) for n in g}}
    check_bf16(cfg.name, errs, block_floors(cfg, w, x, dy, (y, dx, g)))
