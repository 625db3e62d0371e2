"""Backward of the fused attention where the last tile of 64 queries is not full: the queries past the end must add
nothing to dk and dv, whether the kernel masks them or seeds their scores with an infinity."""
from dataclasses import replace

import pytest

import synth_inputs as SI
from oracle import t5_oracle as O
from parity_util import block_floors, check_bf16, make_case, rel_err, run_block_gpu

pytestmark = pytest.mark.gpu

BASE = SI.BlockConfig("attention_tails", 62, 2, 65, 128, 2, 64, 256, attn_scale=0.125)


@pytest.mark.parametrize("seq", [63, 65, 127, 193])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d_kv", [64, 128])
def test_ragged_last_query_tile(d_kv, causal, seq):
    import paper_2203_17189_amd as P
    cfg = replace(BASE, seq=seq, causal=causal, d_kv=d_kv, attn_scale=d_kv ** -0.5,
                  name=f"attention_tails_{d_kv}_{int(causal)}_{seq}")
    want = P.PATH_MFMA_ATTN_FWD | P.PATH_MFMA_ATTN_BWD
    assert P.t5_block_kernel_path(cfg) & want == want
    w, x, dy = make_case(cfg)
    y, saved = O.block_fwd(cfg, x, w)
    dx, g = O.block_bwd(cfg, dy, w, saved)
    gy, gdx, gg = run_block_gpu(cfg, w, x, dy)
    errs = {"y": rel_err(gy, y), "dx": rel_err(gdx, dx), **{n: rel_err(gg[n], g[n]) for n in g}}
    check_bf16(cfg.name, errs, block_floors(cfg, w, x, dy, (y, dx, g)))


@pytest.mark.parametrize("batch", [3, 66])   # 24 and 528 workgroups: the two forms of the bias-free dk/dv kernel
@pytest.mark.parametrize("seq", [33, 64])
def test_cross_attention_forms(batch, seq):
    import paper_2203_17189_amd as P
    from parity_util import decoder_floors, make_decoder_case, run_decoder_block_gpu
    cfg = replace(BASE, batch=batch, seq=seq, causal=True, enc_seq=500, name=f"cross_forms_{batch}_{seq}")
    assert P.t5_block_kernel_path(cfg) & P.PATH_MFMA_ATTN_BWD
    w, x, enc, dy = make_decoder_case(cfg)
    y, saved = O.decoder_block_fwd(cfg, x, enc, w)
    dx, denc, g = O.decoder_block_bwd(cfg, dy, w, saved)
    gy, gdx, gdenc, gg = run_decoder_block_gpu(cfg, w, x, enc, dy)
    errs = {"y": rel_err(gy, y), "dx": rel_err(gdx, dx), "denc": rel_err(gdenc, denc),
            **{n: rel_err(gg[n], g[n]) for n in g}}
    check_bf16(cfg.name, errs, decoder_floors(cfg, w, x, enc, dy, (y, dx, denc, g)))


def test_long_causal_sequence():
    """5100 positions: the bias slice in LDS no longer leaves room for three workgroups on a compute unit."""
    cfg = replace(BASE, batch=1, seq=5100, causal=True, d_model=64, n_heads=1, d_ff=64, name="attention_tails_long")
    w, x, dy = make_case(cfg)
    y, saved = O.block_fwd(cfg, x, w)
    dx, g = O.block_bwd(cfg, dy, w, saved)
    gy, gdx, gg = run_block_gpu(cfg, w, x, dy)
    errs = {"y": rel_err(gy, y), "dx": rel_err(gdx, dx), **{n: rel_err(gg[n], g[n]) for n in g}}
    check_bf16(cfg.name, errs, block_floors(cfg, w, x, dy, (y, dx, g)))
