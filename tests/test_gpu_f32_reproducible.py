"""float32 gradients are bit-identical from run to run, in the default mode and in the reproducible one, where the k-slices
of the weight gradients (512 tokens and more) are summed: all but the bias-table gradient, and in the default mode the
embedding gradient of a stack, which meet in float32 atomics."""
from dataclasses import replace

import pytest
import torch

import synth_inputs as SI
from oracle import t5_oracle as O
from parity_util import TOL_F32, make_case, make_decoder_case, rel_err, to_dev, to_np

pytestmark = pytest.mark.gpu

C = SI.BlockConfig("f32_repro", 71, 5, 250, 128, 2, 32, 256, dtype="f32", attn_scale=0.2)


def _same(a, b, skip=("rel_table",)):
    for k in a:
        assert k in skip or torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("deterministic", [False, True])
@pytest.mark.parametrize("shape", [dict(), dict(mlp="relu", d_ff=96), dict(batch=16, d_model=512, n_heads=6, d_kv=64, d_ff=1024),
                                   dict(batch=32, d_model=768, n_heads=12, d_kv=64, d_ff=512)],  # 128x128 tiles, sliced
                         ids=["small", "relu", "d512", "d768"])
def test_block(shape, deterministic):
    import paper_2203_17189_amd as P
    cfg = replace(C, deterministic=deterministic, **shape)
    w, x, dy = make_case(cfg)
    dw = {k: to_dev(v, "f32") for k, v in w.items()}
    tx, tdy = to_dev(x, "f32"), to_dev(dy, "f32")
    _, stash = P.t5_block_fwd(cfg, tx, dw)
    dx1, g1 = P.t5_block_bwd(cfg, tdy, tx, dw, stash)
    acc = {k: v.clone() for k, v in g1.items()}
    for _ in range(3):
        dx2, g2 = P.t5_block_bwd(cfg, tdy, tx, dw, stash)
        assert torch.equal(dx1, dx2)
        _same(g1, g2)
    P.t5_block_bwd(cfg, tdy, tx, dw, stash, grads=acc, accumulate=True)
    for k in ("wq", "wo", "wi0", "wo_ff"):
        assert rel_err(to_np(acc[k]), 2 * to_np(g1[k]))[0] <= TOL_F32[0], k
    if cfg.tokens <= 2000:
        _, saved = O.block_fwd(cfg, x, w)
        _, g = O.block_bwd(cfg, dy, w, saved)
        for k in g:
            assert rel_err(to_np(g1[k]), g[k])[0] <= TOL_F32[0], k


@pytest.mark.parametrize("deterministic", [False, True])
def test_decoder_layer(deterministic):
    import paper_2203_17189_amd as P
    cfg = replace(C, causal=True, enc_seq=130, deterministic=deterministic, name="f32_repro_dec")
    w, x, enc, dy = make_decoder_case(cfg)
    dw = {k: to_dev(v, "f32") for k, v in w.items()}
    tx, te, tdy = to_dev(x, "f32"), to_dev(enc, "f32"), to_dev(dy, "f32")
    _, stash = P.t5_decoder_block_fwd(cfg, tx, te, dw)
    dx1, denc1, g1 = P.t5_decoder_block_bwd(cfg, tdy, tx, te, dw, stash)
    for _ in range(3):
        dx2, denc2, g2 = P.t5_decoder_block_bwd(cfg, tdy, tx, te, dw, stash)
        assert torch.equal(dx1, dx2) and torch.equal(denc1, denc2)
        _same(g1, g2)


@pytest.mark.parametrize("deterministic", [False, True])
@pytest.mark.parametrize("tied", [False, True], ids=["untied", "tied"])
def test_stack(tied, deterministic):
    import test_gpu_parity_stack as TS
    blk = replace(C, batch=4, causal=True, deterministic=deterministic)
    sc = SI.StackConfig("f32_repro_stack", blk, n_layers=2, vocab=192, tied_logits=tied)
    w, tokens, targets = TS._case(sc)
    _, g1 = TS._run(sc, w, tokens, targets)
    skip = ("rel_table", "layers") + (() if deterministic else ("embedding",))
    for _ in range(3):
        _, g2 = TS._run(sc, w, tokens, targets)
        _same(g1, g2, skip)
        for a, b in zip(g1["layers"], g2["layers"]):
            _same(a, b)


def test_side_stream():
    """The slices are added up on the stream that the weight gradients run on."""
    import paper_2203_17189_amd as P
    w, x, dy = make_case(C)
    dw = {k: to_dev(v, "f32") for k, v in w.items()}
    tx, tdy = to_dev(x, "f32"), to_dev(dy, "f32")
    _, stash = P.t5_block_fwd(C, tx, dw)
    _, g1 = P.t5_block_bwd(C, tdy, tx, dw, stash)
    P.t5_wgrad_overlap_enable(True)
    try:
        for _ in range(3):
            _, g2 = P.t5_block_bwd(C, tdy, tx, dw, stash)
            torch.cuda.synchronize()
            _same(g1, g2)
    finally:
        P.t5_wgrad_overlap_enable(False)


def _buffers(P, cfg, dw, tx, guard):
    from paper_2203_17189_amd import binding as B
    n = P.t5_decoder_block_workspace_bytes(cfg) if cfg.enc_seq else P.t5_block_workspace_bytes(cfg)
    ws = torch.full((n + guard,), 0xA5, dtype=torch.uint8, device="cuda")
    return n, ws, (B.alloc_decoder_grads if cfg.enc_seq else B.alloc_grads)(cfg, dw), torch.empty_like(tx)


@pytest.mark.parametrize("enc_seq", [0, 130])
@pytest.mark.parametrize("d_model,d_ff", [(128, 256), (126, 250), (132, 66)])  # sliced; not aligned: whole; some of each
def test_slices_stay_inside_the_workspace(enc_seq, d_model, d_ff):
    import paper_2203_17189_amd as P
    cfg = replace(C, d_model=d_model, d_ff=d_ff, causal=bool(enc_seq), enc_seq=enc_seq, name="f32_guard")
    w, x, enc, dy = make_decoder_case(cfg) if enc_seq else (*make_case(cfg)[:2], None, make_case(cfg)[2])
    dw = {k: to_dev(v, "f32") for k, v in w.items()}
    tx, tdy = to_dev(x, "f32"), to_dev(dy, "f32")
    n, ws, grads, dx = _buffers(P, cfg, dw, tx, 8 << 20)
    if enc_seq:
        te = to_dev(enc, "f32")
        _, stash = P.t5_decoder_block_fwd(cfg, tx, te, dw)
        P.t5_decoder_block_bwd(cfg, tdy, tx, te, dw, stash, dx=dx, grads=grads, workspace=ws[:n])
    else:
        _, stash = P.t5_block_fwd(cfg, tx, dw)
        P.t5_block_bwd(cfg, tdy, tx, dw, stash, dx=dx, grads=grads, workspace=ws[:n])
    assert bool((ws[n:] == 0xA5).all())


def test_captured_step():
    """The step recorded into a graph gives the eager bits on every replay, with other inputs and eager work between."""
    import paper_2203_17189_amd as P
    w, x, dy = make_case(C)
    dw = {k: to_dev(v, "f32") for k, v in w.items()}
    tx, tdy = to_dev(x, "f32"), to_dev(dy, "f32")
    y, stash = P.t5_block_fwd(C, tx, dw)
    sets = [_buffers(P, C, dw, tx, 0) for _ in range(2)]

    def step(n, ws, grads, dx):
        P.t5_block_fwd(C, tx, dw, y=y, stash=stash)
        P.t5_block_bwd(C, tdy, tx, dw, stash, dx=dx, grads=grads, workspace=ws)

    fwd_ws = torch.empty(P.t5_block_workspace_bytes(C), dtype=torch.uint8, device="cuda")

    def captured(n, ws, grads, dx):
        P.t5_block_fwd(C, tx, dw, y=y, stash=stash, workspace=fwd_ws)
        P.t5_block_bwd(C, tdy, tx, dw, stash, dx=dx, grads=grads, workspace=ws)

    captured(*sets[0])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        captured(*sets[0])
    for rep in range(4):
        _, x2, dy2 = make_case(C, seed_offset=rep + 1)
        tx.copy_(to_dev(x2, "f32"))
        tdy.copy_(to_dev(dy2, "f32"))
        g.replay()
        step(*sets[1])
        torch.cuda.synchronize()
        assert torch.equal(sets[0][3], sets[1][3]), rep
        _same(sets[1][2], sets[0][2])
