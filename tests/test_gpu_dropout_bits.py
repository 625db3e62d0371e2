"""Dropout of the attention probabilities: the forward leaves its keep decisions as bits, a word per query, 64-key tile and lane
half, and the backward reads them.  Lengths at which words, tiles and workgroups are only partly used."""
from dataclasses import replace

import pytest

import synth_inputs as SI
from oracle import t5_oracle as O
from parity_util import (block_floors, check_bf16, decoder_floors, make_case, make_decoder_case, rel_err, run_block_gpu,
                         run_decoder_block_gpu)

pytestmark = pytest.mark.gpu

BASE = SI.BlockConfig("dropout_bits", 63, 3, 64, 128, 2, 64, 128, attn_scale=0.125, dropout_rate=0.2, dropout_seed=0x1234567890AB)


@pytest.mark.parametrize("seq", [33, 64, 97, 129, 190])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d_kv", [64, 128])
def test_self_attention(d_kv, causal, seq):
    import paper_2203_17189_amd as P
    cfg = replace(BASE, seq=seq, causal=causal, d_kv=d_kv, attn_scale=d_kv ** -0.5,
                  name=f"dropout_bits_{d_kv}_{int(causal)}_{seq}")
    assert P.t5_block_kernel_path(cfg) & P.PATH_MFMA_ATTN_BWD
    w, x, dy = make_case(cfg)
    y, saved = O.block_fwd(cfg, x, w)
    dx, g = O.block_bwd(cfg, dy, w, saved)
    gy, gdx, gg = run_block_gpu(cfg, w, x, dy)
    errs = {"y": rel_err(gy, y), "dx": rel_err(gdx, dx), **{n: rel_err(gg[n], g[n]) for n in g}}
    check_bf16(cfg.name, errs, block_floors(cfg, w, x, dy, (y, dx, g)))


@pytest.mark.parametrize("max_distance", [128, 4096])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d_kv", [64, 128])
def test_beside_either_form_of_the_bias(d_kv, causal, max_distance):
    """620 positions, ten key tiles to a row of words: the bias from the window of diagonals, or (4096) from the slice, which
    lies behind the keep words in LDS."""
    import paper_2203_17189_amd as P
    cfg = replace(BASE, batch=2, seq=620, causal=causal, d_kv=d_kv, attn_scale=d_kv ** -0.5, max_distance=max_distance,
                  name=f"dropout_bits_bias_{d_kv}_{int(causal)}_{max_distance}")
    assert P.t5_block_kernel_path(cfg) & P.PATH_MFMA_ATTN_BWD
    w, x, dy = make_case(cfg)
    y, saved = O.block_fwd(cfg, x, w)
    dx, g = O.block_bwd(cfg, dy, w, saved)
    gy, gdx, gg = run_block_gpu(cfg, w, x, dy)
    errs = {"y": rel_err(gy, y), "dx": rel_err(gdx, dx), **{n: rel_err(gg[n], g[n]) for n in g}}
    check_bf16(cfg.name, errs, block_floors(cfg, w, x, dy, (y, dx, g)))


@pytest.mark.parametrize("seq,enc_seq", [(33, 100), (129, 35), (64, 129)])
def test_cross_attention(seq, enc_seq):
    import paper_2203_17189_amd as P
    cfg = replace(BASE, seq=seq, causal=True, enc_seq=enc_seq, name=f"dropout_bits_cross_{seq}_{enc_seq}")
    assert P.t5_block_kernel_path(cfg) & P.PATH_MFMA_CROSS_ATTN
    w, x, enc, dy = make_decoder_case(cfg)
    y, saved = O.decoder_block_fwd(cfg, x, enc, w)
    dx, denc, g = O.decoder_block_bwd(cfg, dy, w, saved)
    gy, gdx, gdenc, gg = run_decoder_block_gpu(cfg, w, x, enc, dy)
    errs = {"y": rel_err(gy, y), "dx": rel_err(gdx, dx), "denc": rel_err(gdenc, denc),
            **{n: rel_err(gg[n], g[n]) for n in g}}
    check_bf16(cfg.name, errs, decoder_floors(cfg, w, x, enc, dy, (y, dx, denc, g)))
