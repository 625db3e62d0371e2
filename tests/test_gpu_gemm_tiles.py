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


def _tile(M, N, K, resid=False):
    """The tile that a plain store, or one with residual, of these sizes gets (rounds over the 256 compute units, as
    launch_layout counts them)."""
    def tiles(bm, bn):
        return -(-M // bm) * -(-N // bn)
    t128 = tiles(128, 128)
    if t128 <= 256:
        return "64x64" if tiles(64, 64) <= 256 else "128x64" if tiles(128, 64) <= 256 else "128x128"
    rem = t128 % 512
    w = ((0.49 if K <= 768 else 0.56 if K < 1024 else 0.52 if K == 1024 else 0.555 if K <= 2048 else 0.61) if resid
         else (0.40 if N % 256 else 0.53) if K < 640 else 0.62)
    c128 = w * (t128 // 512 + (1.0 if rem > 256 or (rem and (K > 3072 or (K >= 1024 and t128 <= 1024))) else 0.65 if rem else 0.0))
    c128_192 = 0.62 * -(-t128 // 512) if K > 1024 else c128
    c256 = -(-tiles(256, 256) // 256)
    if N % 192 == 0 and 0.88 * -(-tiles(256, 192) // 256) < min(c256, c128_192):
        return "256x192"
    if resid and K <= 512 and tiles(256, 256) >= 192:
        return "256x128"
    return "256x256" if c256 <= c128 else "128x128, two per unit"


@pytest.mark.parametrize("M,N,K,tile", [(1332, 768, 768, "64x64"),
                                        (1020, 1000, 128, "64x64"),
                                        (1020, 1032, 128, "128x64"),
                                        (3648, 768, 192, "128x128"),
                                        (5000, 1024, 256, "128x128, two per unit"),
                                        (8991, 776, 320, "128x128, two per unit"),
                                        (8200, 2040, 192, "128x128, two per unit"),
                                        (8190, 2040, 192, "128x128, two per unit"),
                                        (8190, 2048, 192, "256x256"),       # clamped rows of the first operand
                                        (8190, 2040, 704, "256x256"),       # ... of both
                                        (8185, 2041, 832, "256x256"),
                                        (8192, 2048, 64, "256x256")])
def test_tile_families_k_contiguous(M, N, K, tile):
    assert _tile(M, N, K) == tile
    _check_gemm(M, N, K, True)


# from K = 1024 on: a last round that is not full behind four full ones, and behind one; the first K that counts it as full; 256x192
# against three rounds
@pytest.mark.parametrize("M,N,K,tile", [(16777, 2048, 1024, "128x128, two per unit"), (18432, 2040, 3072, "128x128, two per unit"),
                                        (16777, 2048, 3136, "256x256"), (8190, 1032, 1024, "256x256"),
                                        (22001, 768, 1024, "128x128, two per unit"), (22001, 768, 1088, "256x192")])
def test_tiles_of_several_rounds(M, N, K, tile):
    assert _tile(M, N, K) == tile
    _check_gemm(M, N, K, True)


def _wgrad_plan(M, N, K, ngr=1):
    """Tile and k-slices that wgrad_plan gives a weight gradient (ngr of them in one launch)."""
    def tiles(b):
        return -(-M // b) * -(-N // b) * ngr
    nk, best = K // 64, None
    for sp in range(1, 33):
        if sp > 1 and nk // sp < 8:
            break
        w256, w128 = tiles(256) * sp, tiles(128) * sp
        r256, rem = -(-w256 // 256), w128 % 512
        k256 = 1.45 * r256 * nk / sp
        atomics = (0.145 if ngr == 1 and r256 >= 4 else 0.193) * w256 if sp > 1 else 8.0
        c256 = k256 + 5.0 + (max(17.4 * (r256 - 1), atomics - k256 * (r256 - 1) / r256) if ngr > 1 else atomics)
        rounds = w128 // 512 * 1.75 + ((1.65 if ngr == 1 and sp > 1 and rem <= 480 else 1.75) if rem > 256 else 1.0 if rem else 0.0)
        c128 = (0.62 if ngr > 1 and w128 > 512 else 0.58) * rounds * nk / sp + (0.048 * w128 if sp > 1 else 0.0) + 3.0
        for cost, tile in ((c128, 128), (c256, 256)):
            if best is None or cost < best[0]:
                best = (cost, tile, sp)
    return best[1:]


@pytest.mark.parametrize("M,N,K,tile,slices", [(768, 768, 8960, 128, 7), (2048, 768, 14592, 128, 5), (1024, 512, 32768, 128, 8),
                                               (4096, 2048, 4096, 128, 1), (8, 8, 64, 128, 1), (768, 2304, 20480, 128, 4),
                                               (2048, 768, 65536, 256, 10), (768, 4096, 13312, 256, 5),
                                               (2056, 760, 65536, 256, 9),   # last tiles of 8 rows and 248 columns
                                               (5120, 2048, 4416, 256, 1), (5112, 2056, 8960, 256, 1), (2048, 10240, 16384, 256, 3)])
def test_split_plans_m_contiguous(M, N, K, tile, slices):
    assert _wgrad_plan(M, N, K) == (tile, slices)
    _check_gemm(M, N, K, False)


@pytest.mark.parametrize("batch,seq,slices", [(11, 407, 1), (41, 409, 3)])
def test_weight_gradients_over_a_ragged_number_of_tokens(batch, seq, slices):
    """256x256 tiles, sliced and whole, over tokens that are not a multiple of the k-tile: the ungated layer's products
    from the hidden activations that the layer itself has, in float64."""
    import paper_2203_17189_amd as P
    d, f, tokens = 2048, 5120, batch * seq
    assert tokens % 64 and _wgrad_plan(d, f, tokens) == _wgrad_plan(f, d, tokens) == (256, slices)
    cfg = SI.BlockConfig("ragged_wgrad", 98, batch, seq, d, 4, 64, f, attn_scale=0.125, mlp="relu")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    w = _layer_weights(cfg, gen)
    w["wo"].zero_()  # the attention sublayer adds nothing: the feed-forward's input is x's norm
    x, dy = [torch.randn((batch, seq, d), generator=gen, device="cuda").bfloat16() for _ in range(2)]
    _, stash = P.t5_block_fwd(cfg, x, w)
    _, g = P.t5_block_bwd(cfg, dy, x, w, stash)
    xd = x.view(tokens, d).double()
    n = (xd * torch.rsqrt(xd.square().mean(1, keepdim=True) + 1e-6) * w["ln2_scale"].double()).bfloat16().double()
    u = n @ w["wi0"].double()
    a = u.clamp(min=0).bfloat16().double()
    du = ((dy.view(tokens, d).double() @ w["wo_ff"].double().t().contiguous()) * (a > 0)).bfloat16().double()
    want = {"wo_ff": a.t().contiguous() @ dy.view(tokens, d).double(), "wi0": n.t().contiguous() @ du}
    for k, v in want.items():
        # single bf16 roundings of a, du and n that fall the other way, units that are zero on one side only
        assert float((g[k].double() - v).norm() / v.norm()) <= 2e-3, k


def test_grouped_weight_gradients_on_256x256_tiles():
    """Twelve layers in grouped launches (256x256 tiles in two slices and 128x128 whole) against one launch a layer (remat), whose
    activations are the same bits: float32 sums in another order."""
    import paper_2203_17189_amd as P
    from types import SimpleNamespace
    blk = SI.BlockConfig("grouped", 99, 8, 512, 768, 12, 64, 2048, attn_scale=0.125, causal=True)
    tokens, layers, vocab = 4096, 12, 512
    assert [_wgrad_plan(*mn, tokens, layers) for mn in ((2048, 768), (768, 4096), (768, 768), (768, 2304))] == \
        [(256, 2), (256, 2), (128, 1), (256, 2)]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(12)
    ws = [_layer_weights(blk, gen) for _ in range(layers)]
    rnd = lambda *n: torch.randn(n, generator=gen, device="cuda").bfloat16()  # noqa: E731
    w = dict(embedding=rnd(vocab, 768), rel_table=ws[0]["rel_table"], final_scale=rnd(768), logits_w=rnd(768, vocab) * 0.05,
             layers=[{k: v for k, v in lw.items() if k != "rel_table"} for lw in ws])
    tok, tgt = [torch.randint(0, vocab, (8, 512), generator=gen, device="cuda", dtype=torch.int32) for _ in range(2)]
    out = []
    for remat in (0, 1):
        c = SimpleNamespace(block=blk, n_layers=layers, vocab=vocab, tied_logits=0, remat=remat, z_loss=0.0)
        out.append(P.t5_stack_loss_and_grad(c, tok, tgt, w)[1]["layers"])
    for a, b in zip(*out):
        for k in ("wq", "wk", "wv", "wo", "wi0", "wi1", "wo_ff"):
            assert float((a[k] - b[k]).norm() / b[k].norm()) <= 2e-6, k


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


@pytest.mark.parametrize("dtype,d_model", [("f32", 128), ("f32", 72), ("f32", 70),      # pieces of 4 elements; one by one
                                           ("bf16", 128), ("bf16", 72), ("bf16", 76)])  # pieces of 8; one by one
def test_masked_gradient_copy(dtype, d_model):
    """dWo_ff of a layer is a^T (dy o M): with one token the outer product of the hidden row and the masked, rescaled
    gradient, whose elements are those that the general generator keeps."""
    import paper_2203_17189_amd as P
    cfg = SI.BlockConfig("maskcopy", 81, 1, 1, d_model, 2, 8, 64, dtype=dtype, dropout_rate=0.25, dropout_seed=99)
    w, x, dy = make_case(cfg)
    dw, dx, ddy = upload_case(cfg, w, x, dy)
    _, stash = P.t5_block_fwd(cfg, dx, dw)
    _, g = P.t5_block_bwd(cfg, ddy, dx, dw, stash)
    keep = P.t5_dropout_keep(99, 4, 0.25, 1, d_model).bool()[0]
    assert torch.equal((g["wo_ff"] != 0).any(0), keep)
    masked = torch.where(keep, ddy.flatten().float() * torch.tensor(4 / 3, device="cuda"), 0.0).to(ddy.dtype).double()
    ref = int(masked.abs().argmax())
    a = g["wo_ff"].double()[:, ref:ref + 1] / masked[ref]
    # one product per element, in float32: two roundings of 2^-24 each, in the element and in a
    assert float((g["wo_ff"].double() - a * masked).abs().max()) <= 4 * 2.0 ** -24 * float((a * masked).abs().max())


@pytest.mark.parametrize("full,ragged,seq", [(292, 291, 64), (96, 95, 64), (8, 7, 64)])  # 256x256, 128x128, small tiles
@pytest.mark.parametrize("mlp,rate", [("geglu_tanh", 0.0), ("geglu_tanh", 0.125), ("relu", 0.0)])
def test_rows_do_not_depend_on_the_last_tile(full, ragged, seq, mlp, rate):
    """y and dx of a batch are, bit for bit, those of the same sequences in a larger batch that fills its last tile of rows."""
    import paper_2203_17189_amd as P
    cfg = SI.BlockConfig("last_rows", 82, full, seq, 512, 6, 64, 1024, attn_scale=0.125, mlp=mlp, dropout_rate=rate,
                         dropout_seed=5)
    w, x, dy = make_case(cfg)
    out = []
    for b in (full, ragged):
        c = replace(cfg, batch=b)
        dw, tx, tdy = upload_case(c, w, x[:b], dy[:b])
        y, stash = P.t5_block_fwd(c, tx, dw)
        dx, _ = P.t5_block_bwd(c, tdy, tx, dw, stash)
        out.append((y.view(b, seq, -1)[:ragged].clone(), dx.view(b, seq, -1)[:ragged].clone()))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("nk", [10, 11, 12, 13, 14, 15])
def test_256x192_tiles_every_loop_remainder(nk):
    assert _tile(14500, 768, 64 * nk) == "256x192"
    _check_gemm(14500, 768, 64 * nk, True)  # 57 x 3 tiles of 256x256 in one round, 57 x 4 of 256x192 too; a last row tile of 164


def test_256x192_tiles_with_residual():
    """A layer of 114 sequences (256x192 tiles in every product of 768 columns: both with residual, the gradients of both
    norms' outputs) against its two halves (128x128 tiles): the same sums in another order, so what differs are single bf16 roundings:
    the bar of a result against the exact one."""
    import numpy as np
    import paper_2203_17189_amd as P
    from parity_util import STATED_BF16, rel_err
    cfg = SI.BlockConfig("tiles_192", 95, 114, 128, 768, 16, 64, 1024, attn_scale=0.125)
    for k, resid in ((1024, True), (2048, False), (3072, False)):
        assert _tile(114 * 128, 768, k, resid) == "256x192" and _tile(57 * 128, 768, k, resid) == "128x128, two per unit"
    w, x, dy = make_case(replace(cfg, batch=2))
    dw, dx, ddy = upload_case(replace(cfg, batch=2), w, x, dy)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    dx, ddy = [torch.randn((114, 128, 768), generator=gen, device="cuda").bfloat16() for _ in range(2)]

    def run(c, x, dy):
        y, stash = P.t5_block_fwd(c, x, dw)
        g, _ = P.t5_block_bwd(c, dy, x, dw, stash)
        return [v.float().cpu().numpy().astype(np.float64) for v in (y, g)]
    whole = run(cfg, dx, ddy)
    halves = [run(replace(cfg, batch=57), dx[b:b + 57].contiguous(), ddy[b:b + 57].contiguous()) for b in (0, 57)]
    for i in range(2):
        e = rel_err(whole[i], np.concatenate([h[i] for h in halves]))
        assert e[0] <= STATED_BF16[0] and e[1] <= STATED_BF16[1], e


@pytest.mark.parametrize("mlp", ["geglu_tanh", "relu"])
def test_256x192_rows_do_not_depend_on_the_last_tile(mlp):
    """y and dx of 255 sequences (14535 rows: 199 in the last row tile) are, bit for bit, those of the same sequences among 256
    (57 full row tiles)."""
    import paper_2203_17189_amd as P
    cfg = SI.BlockConfig("last_rows_192", 94, 256, 57, 768, 16, 64, 1024, attn_scale=0.125, mlp=mlp)
    for b in (255, 256):
        assert _tile(b * 57, 768, 1024, True) == _tile(b * 57, 768, 3072) == "256x192"
    gen = torch.Generator(device="cuda")
    gen.manual_seed(6)
    dw = _layer_weights(cfg, gen)
    x, dy = [torch.randn((256, 57, 768), generator=gen, device="cuda").bfloat16() for _ in range(2)]
    out = []
    for b in (256, 255):
        c = replace(cfg, batch=b)
        y, stash = P.t5_block_fwd(c, x[:b].contiguous(), dw)
        dx, _ = P.t5_block_bwd(c, dy[:b].contiguous(), x[:b].contiguous(), dw, stash)
        out.append((y[:255].clone(), dx[:255].clone()))
    assert torch.isfinite(out[1][0].float()).all()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("d,heads,dk,f,batch,seq,enc,mlp", [(128, 2, 64, 192, 1, 40, 0, "geglu_tanh"),   # 64x64 tiles
                                                            (512, 6, 64, 1024, 3, 333, 0, "geglu_erf"),
                                                            (768, 12, 64, 2048, 4, 333, 0, "geglu_tanh"),  # 128x64, 128x128
                                                            (768, 12, 64, 2048, 13, 200, 77, "geglu_tanh"),
                                                            (1024, 3, 128, 2880, 9, 250, 0, "relu"),       # two per unit
                                                            (1088, 5, 64, 2816, 1, 300, 130, "relu")])
def test_stored_and_packed_weights_give_the_same_layer(d, heads, dk, f, batch, seq, enc, mlp):
    """Few tokens read the weights as they are stored; a weight that does not start on 16 bytes sends the layer back to the
    packed copies.  Every sum runs over k in the same order: the same bits."""
    import paper_2203_17189_amd as P
    cfg = SI.BlockConfig("direct", 96, batch, seq, d, heads, dk, f, attn_scale=0.125, mlp=mlp, enc_seq=enc, causal=enc > 0)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d + f)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda").bfloat16()  # noqa: E731
    i = heads * dk
    shapes = dict(ln1_scale=(d,), wq=(d, i), wk=(d, i), wv=(d, i), wo=(i, d), rel_table=(32, heads), ln2_scale=(d,),
                  wi0=(d, f), wi1=(d, f), wo_ff=(f, d))
    if mlp == "relu":
        del shapes["wi1"]
    if enc:
        shapes.update(lnx_scale=(d,), xq=(d, i), xk=(d, i), xv=(d, i), xo=(i, d))
    w = {k: rnd(*s) * (1.0 if len(s) == 1 else s[0] ** -0.5) for k, s in shapes.items()}
    x = rnd(batch, seq, d)
    e = rnd(batch, enc, d) if enc else None
    off = torch.empty(w["wo"].numel() + 4, device="cuda", dtype=torch.bfloat16)[4:].view_as(w["wo"]).copy_(w["wo"])
    assert off.data_ptr() % 16 == 8
    for n in range(2):
        ww = dict(w, wo=off) if n else w
        y = P.t5_decoder_block_fwd(cfg, x, e, ww)[0] if enc else P.t5_block_fwd(cfg, x, ww)[0]
        if n == 0:
            y0 = y.clone()
    assert torch.isfinite(y0.float()).all() and torch.equal(y0, y)


def _layer_weights(cfg, gen):
    """Weights of a layer (with cross-attention where cfg.enc_seq > 0) in bf16, fan-in scaled."""
    d, i, f = cfg.d_model, cfg.n_heads * cfg.d_kv, cfg.d_ff
    shapes = dict(ln1_scale=(d,), wq=(d, i), wk=(d, i), wv=(d, i), wo=(i, d), rel_table=(32, cfg.n_heads), ln2_scale=(d,),
                  wi0=(d, f), wi1=(d, f), wo_ff=(f, d))
    if cfg.mlp == "relu":
        del shapes["wi1"]
    if cfg.enc_seq:
        shapes.update(lnx_scale=(d,), xq=(d, i), xk=(d, i), xv=(d, i), xo=(i, d))
    rnd = lambda *n: torch.randn(n, generator=gen, device="cuda").bfloat16()  # noqa: E731
    return {k: rnd(*n) * (1.0 if len(n) == 1 else n[0] ** -0.5) for k, n in shapes.items()}


# (the decoder layers: the encoder's side sliced and the decoder's whole, and the other way round)
@pytest.mark.parametrize("d,f,batch,seq,enc,mlp,det", [(768, 2048, 1, 40, 0, "geglu_tanh", False), (768, 2048, 4, 128, 0, "geglu_tanh", False),
                                                       (512, 1024, 9, 333, 0, "geglu_tanh", False), (2048, 2560, 2, 150, 0, "geglu_tanh", False),
                                                       (768, 2048, 40, 333, 0, "geglu_tanh", False),
                                                       (512, 1024, 9, 333, 0, "relu", False), (768, 2048, 4, 128, 0, "relu", False),
                                                       (512, 1024, 4, 50, 1100, "geglu_tanh", False), (512, 1024, 4, 1100, 50, "relu", False),
                                                       (512, 1024, 9, 333, 0, "geglu_tanh", True), (512, 1024, 4, 50, 1100, "relu", True),
                                                       (512, 1024, 4, 1100, 50, "geglu_tanh", True)])
def test_weight_gradients_overwrite_what_the_buffers_hold(d, f, batch, seq, enc, mlp, det):
    """Gradients that one slice stores whole are not cleared first, sliced ones are: either way nothing of what the buffers
    held is left, and with accumulate it stays.  (float32 atomics: sums in another order, 1e-6 of the largest value.)"""
    import paper_2203_17189_amd as P
    from paper_2203_17189_amd import binding as B
    cfg = SI.BlockConfig("overwrite", 97, batch, seq, d, 4, 64, f, attn_scale=0.125, enc_seq=enc, causal=enc > 0, mlp=mlp,
                         deterministic=det)
    if enc:  # dXk | dXv against dXq and dXo
        assert (_wgrad_plan(d, 512, batch * enc)[1] > 1) == (enc > seq) and (_wgrad_plan(d, 256, batch * seq)[1] > 1) == (seq > enc)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(batch)
    dw = _layer_weights(cfg, gen)
    dx, ddy = [torch.randn((batch, seq, d), generator=gen, device="cuda").bfloat16() for _ in range(2)]
    e = torch.randn((batch, enc, d), generator=gen, device="cuda").bfloat16() if enc else None
    stash = P.t5_decoder_block_fwd(cfg, dx, e, dw)[1] if enc else P.t5_block_fwd(cfg, dx, dw)[1]
    out = []
    for fill, acc in ((0.0, False), (float("nan"), False), (3.0, True)):
        g = B.alloc_decoder_grads(cfg, dw) if enc else B.alloc_grads(cfg, dw)
        for v in g.values():
            v.fill_(fill)
        if enc:
            P.t5_decoder_block_bwd(cfg, ddy, dx, e, dw, stash, grads=g, accumulate=acc)
        else:
            P.t5_block_bwd(cfg, ddy, dx, dw, stash, grads=g, accumulate=acc)
        out.append(g)
    for k, v in out[0].items():
        assert torch.isfinite(v).all(), k
        tol = 4e-6 * float(v.abs().max()) + 4e-6
        assert float((out[1][k] - v).abs().max()) <= tol, k
        assert float((out[2][k] - 3.0 - v).abs().max()) <= tol + 4e-6, k  # (one rounding at 3 more)
