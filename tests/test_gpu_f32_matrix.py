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


# 64 x 64 tiles by the dozen, short of 128: 32 x 64 tiles and eight wavefronts for one to three k-contiguous segments that are not a
# multiple of their k-tiles, 32 x 32 ones for the others; a last row tile of 9, a last column tile of 4
STAGED_CASES = [replace(C, batch=3, seq=131, d_model=772, n_heads=3, d_kv=20, d_ff=100),
                replace(C, batch=1, seq=361, d_model=836, n_heads=5, d_kv=52, d_ff=68, mlp="relu", causal=True)]


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


@pytest.mark.parametrize("cfg", CASES + SMALL_CASES + STAGED_CASES + SPLIT_CASES, ids=lambda c: f"{c.batch}x{c.seq}_d{c.d_model}_k{c.d_kv}_f{c.d_ff}")
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


# As SPLIT_CASES, at lengths that put several sequences into every tile of rows: 64 x 64 and 128 x 128 tiles, one and several segments
# and matrices side by side, weight gradients whole and in slices that start inside k
MIXED_CASES = [replace(C, batch=208, seq=20, d_model=132, n_heads=3, d_kv=20, d_ff=260, mlp="relu", name="f32_mixed"),
               replace(C, batch=208, seq=20, d_model=388, n_heads=6, d_kv=52, d_ff=772, causal=True, name="f32_mixed"),
               replace(C, batch=20, seq=20, d_model=516, n_heads=9, d_kv=64, d_ff=1536, name="f32_mixed")]
MIXED_IDS = ["64x64", "128x128_slices", "64x64_whole"]
# 2-norm error of a tensor against 64 bits: 2e-7 to 1.4e-6 over this file's cases with ordinary values
TOL_NORM = 2e-6


def _norm_err(got, want):
    return float(np.linalg.norm(got - want) / np.linalg.norm(want))


@pytest.mark.parametrize("power", [-100, -118])
@pytest.mark.parametrize("cfg", MIXED_CASES, ids=MIXED_IDS)
def test_small_gradients_beside_ordinary_ones(cfg, power):
    """Sequences whose output gradient is 2^-118 of the others' keep every bit that float32 has: their dx is the scaled dx
    of the ordinary gradient (all of it normal numbers)."""
    w, x, dy = make_case(cfg)
    _, saved = O.block_fwd(cfg, x, w)
    dx, _ = O.block_bwd(cfg, dy, w, saved)
    small = np.arange(cfg.batch) % 3 == 1
    scale = np.where(small, 2.0 ** power, 1.0)[:, None, None]
    shape = (cfg.batch, cfg.seq, cfg.d_model)
    _, gdx, _ = run_block_gpu(cfg, w, x, dy.reshape(shape) * scale)
    gdx = gdx.reshape(shape) / scale
    for rows in (small, ~small):
        assert _norm_err(gdx[rows], dx.reshape(shape)[rows]) <= TOL_NORM


@pytest.mark.parametrize("cfg", MIXED_CASES, ids=MIXED_IDS)
def test_weights_of_mixed_magnitude(cfg):
    """Channels of q, v and hidden units times 2^114 or 2^-114, undone by k, wo and wo_ff: y and dx are those of the plain
    weights, every gradient that of its weight over the factor.  (Split products form results with operands from 2^112 or sums from
    2^96 on again: in every kind of product of a layer, beside results that they do not.)"""
    w, x, dy = make_case(cfg)
    y, saved = O.block_fwd(cfg, x, w)
    dx, g = O.block_bwd(cfg, dy, w, saved)

    def factors(n):
        return np.ldexp(1.0, np.array([0, -114, 114])[np.arange(n) // 5 % 3])
    fi, ff = factors(cfg.n_heads * cfg.d_kv), factors(cfg.d_ff)
    gate = "wi0" if cfg.mlp == "relu" else "wi1"
    by = {"wq": fi, "wk": 1 / fi, "wv": fi, "wo": 1 / fi[:, None], gate: ff, "wo_ff": 1 / ff[:, None]}
    gy, gdx, gg = run_block_gpu(cfg, {k: v * by.get(k, 1.0) for k, v in w.items()}, x, dy)
    for name, got, want in [("y", gy, y), ("dx", gdx, dx)] + [(n, gg[n] * by.get(n, 1.0), g[n]) for n in g]:
        assert _norm_err(got.reshape(want.shape), want) <= TOL_NORM, (name, _norm_err(got.reshape(want.shape), want))


@pytest.mark.parametrize("cfg", MIXED_CASES, ids=MIXED_IDS)
@pytest.mark.parametrize("where", ["x", "dy"])
def test_other_sequences_keep_their_bits(cfg, where):
    """A token, or an output gradient, that is not finite: y and dx of the other sequences are the same bits as without it."""
    import torch
    import paper_2203_17189_amd as P
    from parity_util import upload_case
    w, x, dy = make_case(cfg)
    dw, dx, ddy = upload_case(cfg, w, x, dy)
    bad = cfg.batch // 2 + 1
    out = []
    for value in (0.5, float("nan"), float("inf")):
        (dx if where == "x" else ddy).view(cfg.batch, cfg.seq, -1)[bad, 11, 7] = value
        y, stash = P.t5_block_fwd(cfg, dx, dw)
        gx, g = P.t5_block_bwd(cfg, ddy, dx, dw, stash)
        out.append((y.view(cfg.batch, cfg.seq, -1).clone(), gx.view(cfg.batch, cfg.seq, -1).clone(), g["wo_ff"].clone()))
    keep = torch.arange(cfg.batch, device="cuda") != bad
    for y, gx, gw in out[1:]:
        assert torch.equal(y[keep], out[0][0][keep]) and torch.equal(gx[keep], out[0][1][keep])
        assert not torch.isfinite(gx[bad]).all()
        if where == "dy":  # dWo_ff = a^T dy: one column (of a late k-slice), its other columns the same bits
            cols = torch.arange(cfg.d_model, device="cuda") != 7
            assert torch.equal(gw[:, cols], out[0][2][:, cols]) and not torch.isfinite(gw[:, 7]).any()


def test_gradient_of_one_token_is_its_rounded_products():
    """A sum with one term: dWo_ff[f] = a_f dy, every element within a rounding of it as float32 products are."""
    import torch
    import paper_2203_17189_amd as P
    from parity_util import upload_case
    cfg = MIXED_CASES[2]
    w, x, dy = make_case(cfg)
    dw, dx, ddy = upload_case(cfg, w, x, dy)
    ddy.view(-1, cfg.d_model)[torch.arange(cfg.batch * cfg.seq, device="cuda") != 123] = 0.0
    _, stash = P.t5_block_fwd(cfg, dx, dw)
    _, g = P.t5_block_bwd(cfg, ddy, dx, dw, stash)
    ratio = g["wo_ff"].double() / ddy.view(-1, cfg.d_model)[123].double()  # a_f (1 + rounding)
    lo, hi = ratio.abs().min(1).values, ratio.abs().max(1).values
    # 2^-24 for the rounded sum of the parts' products; seven roundings of the small ones, 2^-7 of it in all; what the
    # product of the two last parts adds, 2^-34
    bound = 2.0 ** -24 * (1 + 7 * 2.0 ** -7 + 2.0 ** -10)
    some = hi > 1e-30
    assert some.sum() > 1000 and float(((hi - lo) / lo)[some].max()) <= 2 * bound * (1 + 1e-6)


def test_small_products_add_no_more_than_16_terms_in_a_row():
    """64 equal tokens of which the first has an output gradient of 1 and the others just under half a rounding of that: what
    stands in one run of sums with the first is lost, the rest is not."""
    import torch
    import paper_2203_17189_amd as P
    from parity_util import upload_case
    cfg = replace(C, batch=2, seq=32, mlp="relu", name="f32_runs")
    w, x, dy = make_case(cfg)
    w = dict(w, rel_table=np.zeros_like(w["rel_table"]))
    x = np.broadcast_to(x.reshape(64, -1)[:1], (64, cfg.d_model)).reshape(x.shape)
    tiny = np.float32(2.0 ** -25 * 0.999)
    dy = np.full_like(dy, tiny)
    dy.reshape(64, -1)[0] = 1.0
    dw, dx, ddy = upload_case(cfg, w, x, dy)
    _, stash = P.t5_block_fwd(cfg, dx, dw)
    g = P.t5_block_bwd(cfg, ddy, dx, dw, stash)[1]["wo_ff"].double()
    ddy.zero_()
    ddy.view(64, -1)[0] = 1.0
    a = P.t5_block_bwd(cfg, ddy, dx, dw, stash)[1]["wo_ff"].double()  # one term each: the activation itself
    assert (a > 0).any()
    want = a * (1.0 + 63 * float(tiny))
    # 15 terms beside the first; the sums of accumulators and wavefronts, and of the terms that are kept, in four roundings
    assert float((g - want).abs().max() / want.abs().max()) <= 15 * 2.0 ** -25 + 4 * 2.0 ** -24
    assert torch.equal(g == 0, a == 0)
