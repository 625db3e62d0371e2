"""Weight gradients over a number of tokens that is not a multiple of the k-tile: the last, zero-filled k-tile of the
m-contiguous GEMM, alone (fewer tokens than one tile), after whole tiles, on the last of several k-slices, in the
two-pass reproducible reduction and in grouped launches."""
from dataclasses import replace

import pytest

import synth_inputs as SI
from oracle import t5_oracle as O
from parity_util import block_floors, check_bf16, make_case, rel_err, run_block_gpu

pytestmark = pytest.mark.gpu

BASE = SI.BlockConfig("ragged_tokens", 60, 1, 33, 128, 2, 64, 256, attn_scale=0.125)


@pytest.mark.parametrize("batch,seq", [(1, 33), (1, 63), (1, 65), (3, 43), (5, 205), (7, 331)])
@pytest.mark.parametrize("deterministic", [False, True])
def test_block_ragged_tokens(batch, seq, deterministic):
    cfg = replace(BASE, batch=batch, seq=seq, deterministic=deterministic, name=f"ragged_tokens_{batch}x{seq}")
    w, x, dy = make_case(cfg)
    y, saved = O.block_fwd(cfg, x, w)
    dx, g = O.block_bwd(cfg, dy, w, saved)
    gy, gdx, gg = run_block_gpu(cfg, w, x, dy)
    errs = {"y": rel_err(gy, y), "dx": rel_err(gdx, dx), **{n: rel_err(gg[n], g[n]) for n in g}}
    check_bf16(cfg.name, errs, block_floors(cfg, w, x, dy, (y, dx, g)))


def test_stack_ragged_tokens_grouped():
    """Two layers with grouped weight gradients over 5 x 37 tokens against the same layers launched one by one
    (reproducible mode): two float32 summation orders of the same products."""
    import torch
    import paper_2203_17189_amd as P
    from parity_util import to_dev, to_np
    sc = SI.StackConfig("ragged_stack", SI.BlockConfig("ragged_stack", 61, 5, 37, 128, 2, 64, 256, causal=True,
                                                       attn_scale=0.125), 2, 192)
    w = SI.make_stack_weights(sc)
    dw = {k: [{n: to_dev(v, "bf16") for n, v in lw.items()} for lw in t] if k == "layers" else to_dev(t, "bf16")
          for k, t in w.items()}
    tok, tgt = (torch.from_numpy(a).cuda() for a in SI.make_tokens(sc))
    out = []
    for det in (False, True):
        s = replace(sc, block=replace(sc.block, deterministic=det))
        _, g = P.t5_stack_loss_and_grad(s, tok, tgt, dw)
        torch.cuda.synchronize()
        out.append(g)
    for l in range(2):
        for n, a in out[0]["layers"][l].items():
            # K = 185 products of float32-accumulated bf16 pairs: reordering moves a sum by a few ulps of its largest term
            assert rel_err(to_np(a), to_np(out[1]["layers"][l][n]))[0] <= 2e-5, (l, n)


@pytest.mark.parametrize("batch,seq", [(3, 43), (7, 331)])
@pytest.mark.parametrize("deterministic", [False, True])
def test_backward_stays_inside_its_workspace(batch, seq, deterministic):
    """Bytes behind the workspace keep their values."""
    import torch
    import paper_2203_17189_amd as P
    from parity_util import upload_case
    cfg = replace(BASE, batch=batch, seq=seq, deterministic=deterministic, name="ragged_guard")
    dw, dx, ddy = upload_case(cfg, *make_case(cfg))
    _, stash = P.t5_block_fwd(cfg, dx, dw)
    n = P.t5_block_workspace_bytes(cfg)
    buf = torch.full((n + (4 << 20),), 0xA5, dtype=torch.uint8, device="cuda")
    P.t5_block_bwd(cfg, ddy, dx, dw, stash, workspace=buf[:n])
    assert bool((buf[n:] == 0xA5).all())


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_norm_backward_does_not_depend_on_when_the_residual_is_read(dtype):
    """1025 to 2048 columns: from 12289 rows on the backward of the norms requests the residual's row early.  dx of 12304 rows
    is that of the same sequences in two smaller batches (bf16: bit for bit, the general-shape kernels form a row's products
    by themselves; float32 products go by the number of rows), and the scale gradients are the sums of theirs."""
    import torch
    import paper_2203_17189_amd as P
    cfg = SI.BlockConfig("norm_rows", 93, 769, 16, 1032, 1, 8, 24, dtype=dtype, attn_scale=0.25)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(8)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rnd = lambda *n: torch.randn(n, generator=gen, device="cuda")  # noqa: E731
    d, i, f = 1032, 8, 24
    w = dict(ln1_scale=1 + 0.1 * rnd(d), wq=rnd(d, i) / 90, wk=rnd(d, i) / 32, wv=rnd(d, i) / 32, wo=rnd(i, d) / 3, rel_table=rnd(32, 1),
             ln2_scale=1 + 0.1 * rnd(d), wi0=rnd(d, f) / 32, wi1=rnd(d, f) / 32, wo_ff=rnd(f, d) / 5)
    w = {k: v.to(dt) for k, v in w.items()}
    x, dy = [rnd(769, 16, d).to(dt) for _ in range(2)]

    def run(a, b):
        from dataclasses import replace
        c = replace(cfg, batch=b - a)
        xs, dys = x[a:b].contiguous(), dy[a:b].contiguous()
        _, stash = P.t5_block_fwd(c, xs, w)
        dx, g = P.t5_block_bwd(c, dys, xs, w, stash)
        return dx, g["ln1_scale"].double(), g["ln2_scale"].double()
    whole, parts = run(0, 769), [run(0, 400), run(400, 769)]
    assert torch.isfinite(whole[0].float()).all()
    both = torch.cat([p[0] for p in parts])
    assert torch.equal(whole[0], both) or dtype == "f32" and float((whole[0] - both).norm() / both.norm()) <= 2e-6
    for k in (1, 2):
        want = parts[0][k] + parts[1][k]
        # float32 sums of 12304 rows in another order
        assert float((whole[k] - want).abs().max()) <= 1e-5 * float(want.abs().max()) + 1e-6
