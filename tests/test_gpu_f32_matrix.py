"""float32 block on the float32 matrix kernels, at the sizes where they change: the three GEMM tiles (by number of
output tiles), k-slices of the weight gradients, ragged edges and unaligned rows (element loads), fused and unfused
gated GELU, one or two attention wavefronts, heads of 5 to 136 channels (the last on the general kernels), causal and
dropout masks, one to many encoder positions."""
from dataclasses import replace

import numpy as np
import pytest

import synth_inputs as SI
from oracle import t5_oracle as O
from parity_util import TOL_F32, make_case, make_decoder_case, rel_err, run_block_gpu, run_decoder_block_gpu

pytestmark = pytest.mark.gpu

C = SI.BlockConfig("f32_matrix", 70, 2, 32, 64, 4, 16, 256, dtype="f32", attn_scale=0.25)
CASES = [replace(C, batch=1, seq=1),                                                      # one token
         replace(C, batch=1, seq=31, d_model=65, n_heads=3, d_kv=5, d_ff=33),              # nothing aligned
         replace(C, batch=2, seq=33, d_model=68, n_heads=2, d_kv=36, d_ff=100, causal=True),
         replace(C, batch=9, seq=65, d_model=96, n_heads=2, d_kv=64, d_ff=160, causal=True, dropout_rate=0.125,
                 dropout_seed=77),                                                         # k-slices (585 tokens)
         replace(C, batch=3, seq=200, d_model=64, n_heads=1, d_kv=128, d_ff=96, mlp="geglu_erf"),
         replace(C, batch=2, seq=70, d_model=60, n_heads=3, d_kv=50, d_ff=64, causal=True),  # 64-channel tiles, element loads
         replace(C, batch=2, seq=40, d_model=60, n_heads=1, d_kv=66, d_ff=64, dropout_rate=0.25, dropout_seed=5),  # 128
         replace(C, batch=2, seq=20, d_model=60, n_heads=1, d_kv=33, d_ff=64),             # one wavefront, element loads
         replace(C, batch=75, seq=130, d_model=64, n_heads=2, d_kv=16, d_ff=64, causal=True),  # dq: 450 workgroups, four wavefronts
         replace(C, batch=2, seq=40, d_model=64, n_heads=1, d_kv=136, d_ff=64),            # general attention kernels
         replace(C, batch=21, seq=129, d_model=520, n_heads=4, d_kv=32, d_ff=1056, mlp="relu"),   # 128 x 128 tiles
         replace(C, batch=13, seq=100, d_model=256, n_heads=4, d_kv=64, d_ff=512, deterministic=True)]


# Few tiles: one to three batches of 32 k for four or eight wavefronts, batches that run over a segment's end, k not a
# multiple of 4, 8 or 32, columns from several matrices, results narrower than a tile
SMALL_CASES = [replace(C, batch=1, seq=33, d_model=36, n_heads=1, d_kv=20, d_ff=68, num_buckets=32),
               replace(C, batch=3, seq=43, d_model=132, n_heads=3, d_kv=12, d_ff=164, mlp="geglu_erf", dropout_rate=0.25, dropout_seed=9),
               replace(C, batch=1, seq=97, d_model=260, n_heads=2, d_kv=64, d_ff=1060, causal=True),
               replace(C, batch=2, seq=40, d_model=96, n_heads=3, d_kv=32, d_ff=36, mlp="relu", dropout_rate=0.125, dropout_seed=4)]


# Products with operands in three bf16 parts: 64 x 64 and 128 x 128 tiles, k not a multiple of their k-tiles, several
# segments, columns from several matrices, sliced and whole weight gradients (540 and 400 tokens)
SPLIT_CASES = [replace(C, batch=32, seq=130, d_model=132, n_heads=3, d_kv=20, d_ff=260),
               replace(C, batch=32, seq=130, d_model=388, n_heads=5, d_kv=52, d_ff=772, causal=True),
               replace(C, batch=4, seq=135, d_model=772, n_heads=12, d_kv=64, d_ff=1028, mlp="relu"),
               replace(C, batch=4, seq=100, d_model=516, n_heads=8, d_kv=64, d_ff=1540, dropout_rate=0.125, dropout_seed=3)]


def _check(pairs):
    for name, got, want in pairs:
        if name in ("wq", "wk") and not np.any(np.abs(want) > 1e-12):  # one key: no gradient through the softmax
            assert np.abs(got).max() < 1e-5
            continue
        assert rel_err(got, want)[0] <= TOL_F32[0], (name, rel_err(got, want))


@pytest.mark.parametrize("cfg", CASES + SMALL_CASES + SPLIT_CASES, ids=lambda c: f"{c.batch}x{c.seq}_d{c.d_model}_k{c.d_kv}_f{c.d_ff}")
def test_block_f32_matrix(cfg):
    if cfg.dropout_rate:
        cfg = replace(cfg, dropout_rate=float(np.float32(cfg.dropout_rate)))
    w, x, dy = make_case(cfg)
    y, saved = O.block_fwd(cfg, x, w)
    dx, g = O.block_bwd(cfg, dy, w, saved)
    if cfg.seq == 1:
        g = {k: v for k, v in g.items() if k not in ("rel_table",)}
    gy, gdx, gg = run_block_gpu(cfg, w, x, dy)
    _check([("y", gy, y), ("dx", gdx, dx)] + [(n, gg[n], g[n]) for n in g])


@pytest.mark.parametrize("seq,enc_seq", [(1, 2), (33, 32), (32, 97), (130, 31)])
def test_decoder_f32_matrix(seq, enc_seq):
    cfg = replace(C, batch=2, seq=seq, enc_seq=enc_seq, causal=seq > 1, d_model=72, d_kv=24, name="f32_matrix_dec")
    w, x, enc, dy = make_decoder_case(cfg)
    y, saved = O.decoder_block_fwd(cfg, x, enc, w)
    dx, denc, g = O.decoder_block_bwd(cfg, dy, w, saved)
    if seq == 1:
        g = {k: v for k, v in g.items() if k not in ("rel_table",)}
    gy, gdx, gdenc, gg = run_decoder_block_gpu(cfg, w, x, enc, dy)
    _check([("y", gy, y), ("dx", gdx, dx), ("denc", gdenc, denc)] + [(n, gg[n], g[n]) for n in g])


@pytest.mark.parametrize("seq,d_kv", [(20, 16), (50, 16), (100, 64), (140, 128)])
def test_causal_rows_before_a_nan_token(seq, d_kv):
    """A token that is not finite changes no row before it (float32, causal), also inside its own tile of keys."""
    import torch
    import paper_2203_17189_amd as P
    from parity_util import upload_case
    cfg = replace(C, batch=1, seq=seq, d_kv=d_kv, causal=True, name="f32_nan")
    w, x, dy = make_case(cfg)
    dw, dx, _ = upload_case(cfg, w, x, dy)
    y0, _ = P.t5_block_fwd(cfg, dx, dw)
    bad = seq - 7
    dx2 = dx.clone().view(seq, -1)
    dx2[bad] = float("nan")
    y1, _ = P.t5_block_fwd(cfg, dx2.view_as(dx), dw)
    y0, y1 = y0.view(seq, -1), y1.view(seq, -1)
    # the plain multiply-adds of that tile differ from the matrix unit's by float32 rounding
    assert rel_err(y1[:bad].cpu().numpy().astype(np.float64), y0[:bad].cpu().numpy().astype(np.float64))[0] <= TOL_F32[0]
    assert torch.isnan(y1[bad:]).any(dim=1).all()


FAR = {"-inf": -np.inf, "lowest": np.finfo(np.float32).min}


@pytest.mark.parametrize("value", sorted(FAR))
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("seq,d_kv", [(200, 16), (130, 64), (70, 18)])
def test_local_attention_by_the_bias_table(seq, d_kv, causal, value):
    """Far buckets of -inf, or of the lowest float32 (which times log2 e is -inf): whole key tiles without a visible key,
    before (causal) or around the tiles that have some."""
    cfg = replace(C, batch=2, seq=seq, d_kv=d_kv, causal=causal, attn_scale=d_kv ** -0.5, name="f32_local")
    w, x, dy = make_case(cfg)
    w = dict(w, rel_table=w["rel_table"].copy())
    near = 20 if causal else 12  # buckets of distances below about 25 (causal) and 12
    side = 32 if causal else 16
    far = np.arange(32) % side >= near
    w["rel_table"][far] = FAR[value]
    y, saved = O.block_fwd(cfg, x, w)
    dx, g = O.block_bwd(cfg, dy, w, saved)
    gy, gdx, gg = run_block_gpu(cfg, w, x, dy)
    assert np.all(gg["rel_table"][far] == 0)
    _check([("y", gy, y), ("dx", gdx, dx)] + [(n, gg[n], g[n]) for n in g])


def test_every_bucket_at_the_lowest_value():
    """Scores that all round to the same number: uniform attention, as the maximum of the whole row gives it."""
    cfg = replace(C, batch=1, seq=40, name="f32_lowest")
    w, x, dy = make_case(cfg)
    w = dict(w, rel_table=np.full_like(w["rel_table"], FAR["lowest"]))
    y, _ = O.block_fwd(cfg, x, w)
    import paper_2203_17189_amd as P
    from parity_util import to_np, upload_case
    dw, dx, _ = upload_case(cfg, w, x, dy)
    _check([("y", to_np(P.t5_block_fwd(cfg, dx, dw)[0]), y)])


@pytest.mark.parametrize("seq,d_kv", [(20, 16), (50, 16), (100, 64), (140, 128), (45, 18)])
def test_causal_gradients_after_a_nan_gradient(seq, d_kv):
    """An output gradient that is not finite reaches the keys its query sees, none after it, also inside its own tile of
    queries: dx of the later rows is that of the clean gradient (float32, causal)."""
    import torch
    import paper_2203_17189_amd as P
    from parity_util import upload_case
    cfg = replace(C, batch=1, seq=seq, d_kv=d_kv, causal=True, name="f32_nan_grad")
    w, x, dy = make_case(cfg)
    dw, dx, ddy = upload_case(cfg, w, x, dy)
    _, stash = P.t5_block_fwd(cfg, dx, dw)
    g0, _ = P.t5_block_bwd(cfg, ddy, dx, dw, stash)
    bad = seq - 12
    ddy = ddy.clone().view(seq, -1)
    ddy[bad] = float("nan")
    g1, _ = P.t5_block_bwd(cfg, ddy.view_as(dx), dx, dw, stash)
    g0, g1 = g0.view(seq, -1), g1.view(seq, -1)
    assert torch.isnan(g1[:bad + 1]).any(dim=1).all()
    # the plain multiply-adds of that tile differ from the matrix unit's by float32 rounding
    assert rel_err(g1[bad + 1:].cpu().numpy().astype(np.float64),
                   g0[bad + 1:].cpu().numpy().astype(np.float64))[0] <= TOL_F32[0]


@pytest.mark.parametrize("value", [np.inf, 3.4e38, -np.inf])
@pytest.mark.parametrize("d", [132, 772])
def test_split_products_of_an_infinite_weight(d, value):
    """One weight that is infinite, or rounds to infinity in bf16: its column of y as float32 products give it (0 times
    infinity is not a number), the others untouched."""
    import paper_2203_17189_amd as P
    from parity_util import to_np, upload_case
    cfg = replace(C, batch=32, seq=130, d_model=d, n_heads=3, d_kv=20, d_ff=260, mlp="relu", name="f32_inf")
    w, x, dy = make_case(cfg)
    dw, dx, _ = upload_case(cfg, w, x, dy)
    y0 = to_np(P.t5_block_fwd(cfg, dx, dw)[0]).reshape(-1, d)
    dw["wo_ff"] = dw["wo_ff"].clone()
    dw["wo_ff"][7, 5] = value
    y1, _ = P.t5_block_fwd(cfg, dx, dw)
    y1 = to_np(y1).reshape(-1, d)
    _, saved = O.block_fwd(cfg, x, w)
    a = np.float32(saved["a"].reshape(-1, 260)[:, 7])
    sure = np.abs(a) > 1e-6  # (elsewhere the device's own sum may have the other sign)
    with np.errstate(all="ignore"):
        want = a * np.float32(value)
    far = np.isinf(want) & sure
    assert far.sum() > 100 and np.all(y1[far, 5] == want[far])
    if np.isinf(value):
        assert np.all(np.isnan(y1[~sure & (a == 0), 5]) | np.isinf(y1[~sure & (a == 0), 5]))
    else:
        near = np.isfinite(want) & sure
        # an error of the activations is one of their scale, not of each value: relative to the column's RMS as everywhere
        assert rel_err(y1[near, 5], np.float64(want[near]))[0] <= TOL_F32[0]
    keep = np.arange(d) != 5
    assert rel_err(y1[:, keep], y0[:, keep])[0] <= TOL_F32[0]
