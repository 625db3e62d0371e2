"""Local attention by the bias table (bf16): far buckets of -inf or of the lowest bf16 number, so that whole key tiles have
no visible key, before the tiles that have some (causal) or around them."""
from dataclasses import replace

import numpy as np
import pytest

import synth_inputs as SI
from oracle import t5_oracle as O
from parity_util import block_floors, check_bf16, make_case, rel_err, run_block_gpu

pytestmark = pytest.mark.gpu

BASE = SI.BlockConfig("local_attention", 63, 2, 300, 128, 2, 64, 256, attn_scale=0.125)
FAR = {"-inf": -np.inf, "lowest": -float(np.array([0x7F7F0000], np.uint32).view(np.float32)[0])}


@pytest.mark.parametrize("value", sorted(FAR))
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d_kv", [64, 128])
def test_far_buckets_masked(d_kv, causal, value):
    import paper_2203_17189_amd as P
    cfg = replace(BASE, d_kv=d_kv, causal=causal, attn_scale=d_kv ** -0.5, name=f"local_{d_kv}_{int(causal)}_{value}")
    want = P.PATH_MFMA_ATTN_FWD | P.PATH_MFMA_ATTN_BWD
    assert P.t5_block_kernel_path(cfg) & want == want
    w, x, dy = make_case(cfg)
    w = dict(w, rel_table=w["rel_table"].copy())
    far = np.arange(32) % (32 if causal else 16) >= (20 if causal else 12)
    w["rel_table"][far] = FAR[value]
    y, saved = O.block_fwd(cfg, x, w)
    dx, g = O.block_bwd(cfg, dy, w, saved)
    gy, gdx, gg = run_block_gpu(cfg, w, x, dy)
    assert np.all(gg["rel_table"][far] == 0)
    errs = {"y": rel_err(gy, y), "dx": rel_err(gdx, dx), **{n: rel_err(gg[n], g[n]) for n in g}}
    check_bf16(cfg.name, errs, block_floors(cfg, w, x, dy, (y, dx, g)))
