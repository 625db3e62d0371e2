"""The tile families of the bf16 GEMM at the sizes where the choice between them turns, and every remainder of the
256x256 loop's six-tile rounds; dropout copies; weights that do not start on 16 bytes."""
from dataclasses import replace

import pytest
import torch

import synth_inputs as SI
from parity_util import make_case, upload_case

pytestmark = pytest.mark.gpu


def _check_gemm(M, N, K, kc):
    import paper_2203_17189_amd as P
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + 3 * N + 7 * K)
    a = torch.randn((M, K) if kc else (K, M), generator=gen, device="cuda").bfloat16()
    b = torch.randn((N, K) if kc else (K, N), generator=gen, device="cuda").bfloat16()
    c = P.t5_gemm_bf16(a, b, kc, kc)
    ad, bd = a.double(), b.double()
    ref = ad @ bd.t().contiguous() if kc else ad.t().contiguous() @ bd
    # exact products, float32 sums of K terms of unit variance: error of a random walk of K roundings, well below 2e-5 sqrt(K)
    assert float((c.double() - ref).abs().max()) <= 2e-5 * K ** 0.5 * 4, (M, N, K)


@pytest.mark.parametrize("nk", list(range(1, 8)) + [12, 13])
def test_256_tiles_every_loop_remainder(nk):
    _check_gemm(8192, 2048, 64 * nk, True)


@pytest.mark.parametrize("M,N,K", [(1332, 768, 768),      # 64x64, one round
                                   (1020, 1032, 128),     # 64x64, 272 tiles: 128x64
                                   (3648, 768, 192),      # 128x128, one per unit
                                   (5000, 1024, 256),     # 128x128, two per unit
                                   (8991, 776, 320),      # the same, ragged
                                   (8200, 2040, 192)])    # 256x256, ragged
def test_tile_families_k_contiguous(M, N, K):
    _check_gemm(M, N, K, True)


@pytest.mark.parametrize("M,N,K", [(768, 768, 8960), (2048, 768, 14592), (1024, 512, 32768), (4096, 2048, 4096), (8, 8, 64)])
def test_split_plans_m_contiguous(M, N, K):
    _check_gemm(M, N, K, False)


def test_weights_off_16_bytes():
    """The weight pack reads such weights element by element; the forward is bit for bit that of aligned ones."""
    import paper_2203_17189_amd as P
    cfg = SI.BlockConfig("off16", 80, 2, 64, 128, 2, 64, 160, attn_scale=0.125)
    w, x, dy = make_case(cfg)
    dw, dx, _ = upload_case(cfg, w, x, dy)
    want, _ = P.t5_block_fwd(cfg, dx, dw)
    off = {}
    for k, v in dw.items():
        buf = torch.empty(v.numel() + 2, dtype=v.dtype, device="cuda")
        buf[2:] = v.flatten()
        off[k] = buf[2:].view(v.shape)
        assert off[k].data_ptr() % 16 != 0
    got, _ = P.t5_block_fwd(cfg, dx, dict(dw, **{k: off[k] for k in ("wq", "wk", "wv", "wo", "wi0", "wi1", "wo_ff")}))
    assert torch.equal(got, want)


@pytest.mark.parametrize("d_model", [128, 72])
def test_masked_gradient_copy(d_model):
    """dWo_ff of a layer is a^T (dy o M): with one token it is the outer product, zero exactly where the mask is."""
    import paper_2203_17189_amd as P
    cfg = SI.BlockConfig("maskcopy", 81, 1, 1, d_model, 2, 8, 64, dtype="f32", dropout_rate=0.25, dropout_seed=99)
    w, x, dy = make_case(cfg)
    dw, dx, ddy = upload_case(cfg, w, x, dy)
    _, stash = P.t5_block_fwd(cfg, dx, dw)
    _, g = P.t5_block_bwd(cfg, ddy, dx, dw, stash)
    keep = P.t5_dropout_keep(99, 4, 0.25, 1, d_model).bool()[0]
    cols = (g["wo_ff"] != 0).any(0)
    assert torch.equal(cols, keep)
