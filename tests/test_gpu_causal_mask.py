"""The causal mask of the bf16 attention is a choice, not a sum: whatever the product of a query and a later key comes to, it takes
no part, in the forward and in the gradients."""
from dataclasses import replace

import pytest
import torch

import synth_inputs as SI
from parity_util import make_case, upload_case

pytestmark = pytest.mark.gpu

BASE = SI.BlockConfig("causal_mask", 66, 1, 200, 128, 2, 64, 128, causal=True, attn_scale=1.0)
SPLIT = 83  # queries before it have one large channel, keys from it on


def _case(cfg, key):
    """The layer's inputs: channel 5 of a head's queries is about 4e19 before SPLIT and 0 after it, the same channel of
    its keys 0 before SPLIT and about `key` after it."""
    w, x, dy = make_case(cfg)
    x = x.copy().reshape(cfg.seq, cfg.d_model)
    x[:SPLIT, 0], x[SPLIT:, 0], x[:SPLIT, 1], x[SPLIT:, 1] = 3.0, 0.0, 0.0, 3.0
    w = {k: v.copy() for k, v in w.items()}
    w["ln1_scale"][:] = 1.0
    w["wq"][:, 5] = w["wk"][:, 5] = 0.0
    w["wq"][0, 5], w["wk"][1, 5] = 1.5e19, key / 3
    return upload_case(cfg, w, x.reshape(1, cfg.seq, cfg.d_model), dy * 0.01)


# max_distance 128: the bias from a window of diagonals, 4096: from a slice
@pytest.mark.parametrize("max_distance", [128, 4096])
@pytest.mark.parametrize("dropout", [0.0, 0.2])
@pytest.mark.parametrize("d_kv", [64, 128])
def test_masked_products_that_overflow(d_kv, dropout, max_distance):
    """Finite queries and keys whose product is infinite only where it is masked: the same output, and the same gradients of
    the values and the keys, as where those products are zero."""
    import paper_2203_17189_amd as P
    cfg = replace(BASE, d_kv=d_kv, dropout_rate=dropout, dropout_seed=77, max_distance=max_distance)
    assert P.t5_block_kernel_path(cfg) & P.PATH_MFMA_ATTN_BWD
    out = []
    for key in (0.0, 6e19):
        w, x, dy = _case(cfg, key)
        y, stash = P.t5_block_fwd(cfg, x, w)
        dx, g = P.t5_block_bwd(cfg, dy, x, w, stash)
        assert all(torch.isfinite(t).all() for t in (y, dx, *g.values())), key
        out.append((y, g))
    assert torch.equal(out[0][0], out[1][0])
    for n in ("wk", "wv", "wo", "wi0", "wi1", "wo_ff"):  # (the same sums, their slices perhaps in another order)
        a, b = out[0][1][n], out[1][1][n]
        assert ((a - b).abs() <= 1e-5 * a.abs().amax(0) * cfg.seq ** 0.5).all(), n


@pytest.mark.parametrize("d_kv", [64, 128])
def test_rows_before_a_key_that_is_not_finite(d_kv):
    """An infinite key changes no row before it, also inside its own tile of keys."""
    import paper_2203_17189_amd as P
    cfg = replace(BASE, d_kv=d_kv)
    rows = []
    for key in (0.0, 9e38):
        w, x, _ = _case(cfg, key)
        rows.append(P.t5_block_fwd(cfg, x, w)[0].view(cfg.seq, -1)[:SPLIT])
    assert torch.isfinite(rows[1]).all() and torch.equal(rows[0], rows[1])
