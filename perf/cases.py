"""Timed cases of the library: what a training or scoring program calls, through the public entry points.

Kinds of case
  block      t5_block_fwd + t5_block_bwd: one encoder or decoder-only layer of a training step
  score      t5_block_fwd alone: the same layer in evaluation
  decoder    t5_decoder_block_fwd + t5_decoder_block_bwd: a decoder layer with cross-attention
  lm         t5_stack_loss_and_grad: a whole decoder-only model, loss and every gradient
  encdec     t5_encdec_loss_and_grad: the encoder-decoder pair, loss and every gradient
  adafactor  adafactor_step_multi over the ten tensors of a layer

Widths and lengths are those of this repository's own workloads (d_model 64, 512, 768, 2048) and one generic
width between them; batches and sequence lengths of the drawn cases run over the whole range, odd ones among them.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import torch

import paper_2203_17189_amd as P
from paper_2203_17189_amd import binding as B

DEV = "cuda"
BUCKETS, MAX_DISTANCE, EPS, Z_LOSS = 32, 128, 1e-6, 1e-4
MASK32 = 0xFFFFFFFF

# d_model, heads, d_kv, d_ff
TINY = (64, 4, 16, 256)
SMALL = (512, 6, 64, 1024)
BASE = (768, 12, 64, 2048)
MIDDLE = (1024, 16, 64, 2816)
XL = (2048, 32, 64, 5120)
GPT = (2048, 16, 128, 5120)
XL_SHARE = (2048, 4, 64, 640)  # one of eight tensor-parallel shares of XL

MOST_FLOPS = 1.0e13  # of a drawn case


def _case(name, kind, width, batch, seq, **more):
    c = dict(name=name, kind=kind, d_model=width[0], heads=width[1], d_kv=width[2], d_ff=width[3], batch=batch, seq=seq,
             enc_seq=0, causal=False, dtype="bf16", mlp="geglu_tanh", dropout=0.0, deterministic=False, layers=1,
             vocab=0, tied=False, remat=False)
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: a toy model being debugged, or a unit test's training step; launches and host time
        _case("tiny_f32", "block", TINY, 2, 32, dtype="f32"),
        # float32 training of a small layer (the dtype in which a recipe is first made to work), lengths not padded
        _case("small_f32_ragged", "block", SMALL, 16, 250, dtype="f32"),
        # scoring a handful of sequences of whatever length they have: latency of one forward layer
        _case("base_score", "score", BASE, 4, 333),
        # pre-training layers at the widths of the T5.1.1 sizes: the ordinary training step
        _case("small_train", "block", SMALL, 64, 512),
        # the last, short batch of an epoch, or one that is packed to its longest sequence: no size is a round number
        _case("base_train_ragged", "block", BASE, 27, 333),
        # fine-tuning: dropout at every site
        _case("base_finetune", "block", BASE, 128, 512, dropout=0.1),
        # decoder-only layer with long rows and 128-wide heads
        _case("gpt_causal_train", "block", GPT, 16, 2048, causal=True),
        # the largest layer
        _case("xl_train", "block", XL, 32, 1024),
        # decoder layer of the encoder-decoder model, 114 target positions over 512 inputs (the pre-training lengths)
        _case("decoder_train", "decoder", BASE, 128, 114, enc_seq=512, causal=True),
        # whole models, one step's loss and gradients
        _case("lm_base_step", "lm", BASE, 32, 512, causal=True, layers=12, vocab=32128),
        _case("encdec_base_step", "encdec", BASE, 32, 114, enc_seq=512, causal=True, layers=12, vocab=32128),
        # the optimizer over the largest layer's tensors
        _case("adafactor_xl", "adafactor", XL, 1, 1),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    for _ in range(10000):
        kind = rng.choice(["block"] * 8 + ["score"] * 3 + ["decoder"] * 4 + ["lm", "encdec", "adafactor"])
        more = dict(mlp=rng.choice(["geglu_tanh"] * 4 + ["relu", "geglu_erf"]))
        if kind in ("block", "score", "decoder") and rng.random() < 0.25:
            # float32: the small widths, up to the listed case's size
            width = rng.choice([TINY, SMALL, SMALL, BASE])
            more["dtype"] = "f32"
            tokens, seq = log_int(64, 4000), log_int(17, 512)
        else:
            width = rng.choice([SMALL, BASE, MIDDLE, XL, GPT, XL_SHARE])
            tokens, seq = log_int(128, 32768), log_int(32, 2048)
        if kind in ("lm", "encdec"):
            width = rng.choice([SMALL, BASE])
            tokens, seq = log_int(512, 8192), log_int(64, 600)
            more.update(layers=rng.randint(2, 6), vocab=rng.choice([32128, 8064]), tied=rng.random() < 0.4,
                        remat=rng.random() < 0.3)
        if kind in ("block", "score", "lm"):
            more["causal"] = kind == "lm" or rng.random() < 0.5
        if kind in ("decoder", "encdec"):
            more.update(causal=True, enc_seq=log_int(32, 1024))
        if kind != "adafactor" and kind != "score":
            more["dropout"] = 0.1 if rng.random() < 0.25 else 0.0
            more["deterministic"] = rng.random() < 0.1
        if kind == "adafactor":
            tokens = seq = 1
        c = _case("", kind, width, max(1, round(tokens / seq)), seq, **more)
        del c["name"]
        if c["batch"] * c["seq"] <= 32768 and c["batch"] * c["enc_seq"] <= 65536 and work(c)["flops"] <= MOST_FLOPS:
            return c
    raise RuntimeError("no case")


# ------------------------------------------------------------------ configurations and inputs
def _block_cfg(c, seq=None, causal=None, enc_seq=None):
    return SimpleNamespace(batch=c["batch"], seq=seq or c["seq"], d_model=c["d_model"], n_heads=c["heads"], d_kv=c["d_kv"],
                           d_ff=c["d_ff"], causal=c["causal"] if causal is None else causal, dtype=c["dtype"],
                           num_buckets=BUCKETS, max_distance=MAX_DISTANCE, rms_eps=EPS, attn_scale=1.0, mlp=c["mlp"],
                           dropout_rate=c["dropout"], dropout_seed=0x5EED5EED5EED, deterministic=c["deterministic"],
                           enc_seq=c["enc_seq"] if enc_seq is None else enc_seq)


def _shapes(c, cross):
    """{name: (shape, spread, centre)} of a layer's weights: fan-in initialisation, the scale of the logits folded into
    the query projections, norm scales and bias tables as they stand some way into training."""
    d, i, f = c["d_model"], c["heads"] * c["d_kv"], c["d_ff"]
    s = {"ln1_scale": ((d,), 0.1, 1.0), "wq": ((d, i), (d * c["d_kv"]) ** -0.5, 0.0), "wk": ((d, i), d ** -0.5, 0.0),
         "wv": ((d, i), d ** -0.5, 0.0), "wo": ((i, d), i ** -0.5, 0.0), "rel_table": ((BUCKETS, c["heads"]), 0.1, 0.0),
         "ln2_scale": ((d,), 0.1, 1.0), "wi0": ((d, f), d ** -0.5, 0.0), "wi1": ((d, f), d ** -0.5, 0.0),
         "wo_ff": ((f, d), f ** -0.5, 0.0)}
    if c["mlp"] == "relu":
        del s["wi1"]
    if cross:
        s.update(lnx_scale=((d,), 0.1, 1.0), xq=((d, i), (d * c["d_kv"]) ** -0.5, 0.0), xk=((d, i), d ** -0.5, 0.0),
                 xv=((d, i), d ** -0.5, 0.0), xo=((i, d), i ** -0.5, 0.0))
    return s


def _dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _inputs(c, seed):
    """Weights, activations and tokens of a case, from the seed alone."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    dt = _dtype(c)

    def normal(shape, spread=1.0, centre=0.0, dtype=dt):
        return (torch.randn(shape, generator=gen, device=DEV) * spread + centre).to(dtype)

    def layer(cross, table=True):
        return {n: normal(*s) for n, s in _shapes(c, cross).items() if table or n != "rel_table"}

    def stacked(cross):
        """A model's layers, each kind of weight one array over the layers."""
        return {n: torch.stack([normal(*s) for _ in range(c["layers"])]) for n, s in _shapes(c, cross).items()
                if n != "rel_table"}

    def tokens(n, seq):
        # rank-frequency law of natural text
        p = 1.0 / (torch.arange(c["vocab"], device=DEV, dtype=torch.float32) + 10.0)
        perm = torch.randperm(c["vocab"], generator=gen, device=DEV)
        return perm[torch.multinomial(p, n * seq, replacement=True, generator=gen)].to(torch.int32).view(n, seq)

    b, s, d, kind = c["batch"], c["seq"], c["d_model"], c["kind"]
    if kind == "adafactor":
        t = {}
        for n, (shape, spread, centre) in _shapes(c, False).items():
            r, k = shape if len(shape) == 2 else (1, shape[0])
            fact = len(shape) == 2 and n != "rel_table"
            rows = 0.5 + torch.rand(r, 1, generator=gen, device=DEV)
            cols = 0.5 + torch.rand(1, k, generator=gen, device=DEV)
            t[n] = dict(param=normal(shape, spread, centre, torch.float32), factored=fact,
                        grad=(normal((r, k), 1e-2, 0.0, torch.float32) * rows * cols).view(shape),
                        v_row=1e-4 * rows.flatten() ** 2 if fact else None, v_col=1e-4 * cols.flatten() ** 2 if fact else None,
                        v_full=None if fact else 1e-4 * (rows * cols) ** 2)
        return t
    if kind in ("block", "score", "decoder"):
        i = dict(w=layer(kind == "decoder"), x=normal((b, s, d)))
        if kind != "score":
            i["dy"] = normal((b, s, d))
        if kind == "decoder":
            i["enc"] = normal((b, c["enc_seq"], d))
        return i
    ends = dict(embedding=normal((c["vocab"], d)))
    if not c["tied"]:
        ends["logits_w"] = normal((d, c["vocab"]), d ** -0.5)
    table = lambda: normal((BUCKETS, c["heads"]), 0.1)  # noqa: E731
    scale = lambda: normal((d,), 0.1, 1.0)  # noqa: E731
    i = dict(tokens=tokens(b, s), targets=tokens(b, s))
    i["targets"][torch.rand(b, s, generator=gen, device=DEV) < 0.1] = -1  # padding
    if kind == "lm":
        i["w"] = dict(ends, rel_table=table(), final_scale=scale(), layers=stacked(False))
    else:
        i["enc_tokens"] = tokens(b, c["enc_seq"])
        i["w"] = dict(ends, enc_rel_table=table(), enc_final_scale=scale(), dec_rel_table=table(), dec_final_scale=scale(),
                      enc_layers=stacked(False), dec_layers=stacked(True))
    return i


def _per_layer(stack):
    n = len(next(iter(stack.values())))
    return [{k: v[l] for k, v in stack.items()} for l in range(n)]


def prepare(case, seed):
    c, kind = case, case["kind"]
    i = _inputs(c, seed)
    bytes_ = lambda n: torch.empty(max(int(n), 256), dtype=torch.uint8, device=DEV)  # noqa: E731
    if kind == "adafactor":
        tensors = [dict(t, bf16_copy_out=torch.empty_like(t["param"], dtype=torch.bfloat16)) for t in i.values()]
        return dict(kind=kind, tensors=tensors, step=100, ws=bytes_(P.adafactor_multi_workspace_bytes(tensors)))
    if kind in ("block", "score", "decoder"):
        cfg = _block_cfg(c)
        st = dict(i, kind=kind, cfg=cfg, y=torch.empty_like(i["x"]))
        if kind == "decoder":
            st.update(stash=bytes_(P.t5_decoder_block_stash_bytes(cfg)), ws=bytes_(P.t5_decoder_block_workspace_bytes(cfg)),
                      dx=torch.empty_like(i["x"]), denc=torch.empty_like(i["enc"]), grads=B.alloc_decoder_grads(cfg, i["w"]))
        else:
            st.update(stash=bytes_(P.t5_block_stash_bytes(cfg)), ws=bytes_(P.t5_block_workspace_bytes(cfg)))
            if kind == "block":
                st.update(dx=torch.empty_like(i["x"]), grads=B.alloc_grads(cfg, i["w"]))
        return st
    zeros = lambda w: {k: zeros(v) if isinstance(v, dict) else torch.zeros(v.shape, device=DEV) for k, v in w.items()}  # noqa: E731
    grads = zeros(i["w"])  # float32, each kind of weight one array over the layers
    split = lambda w: {k: _per_layer(v) if isinstance(v, dict) else v for k, v in w.items()}  # noqa: E731
    st = dict(kind=kind, tokens=i["tokens"], targets=i["targets"], w=split(i["w"]), grads=split(grads), out=grads,
              loss=torch.zeros(1, device=DEV))
    if kind == "lm":
        st["cfg"] = SimpleNamespace(block=_block_cfg(c), n_layers=c["layers"], vocab=c["vocab"], tied_logits=c["tied"],
                                    remat=c["remat"], z_loss=Z_LOSS)
        st["ws"] = bytes_(P.t5_stack_workspace_bytes(st["cfg"]))
    else:
        st["enc_tokens"] = i["enc_tokens"]
        st["cfg"] = SimpleNamespace(enc_block=_block_cfg(c, seq=c["enc_seq"], causal=False, enc_seq=0), dec_block=_block_cfg(c),
                                    n_enc_layers=c["layers"], n_dec_layers=c["layers"], vocab=c["vocab"],
                                    tied_logits=c["tied"], remat=c["remat"], z_loss=Z_LOSS)
        st["ws"] = bytes_(P.t5_encdec_workspace_bytes(st["cfg"]))
    return st


def run(st):
    kind = st["kind"]
    if kind == "adafactor":
        st["step"] += 1
        P.adafactor_step_multi(st["tensors"], step=st["step"], lr=1e-2, workspace=st["ws"])
        return [{k: t[k] for k in ("param", "v_row", "v_col", "v_full", "bf16_copy_out")} for t in st["tensors"]]
    if kind == "lm":
        P.t5_stack_loss_and_grad(st["cfg"], st["tokens"], st["targets"], st["w"], grads=st["grads"], workspace=st["ws"],
                                 loss=st["loss"])
        return dict(st["out"], loss=st["loss"])
    if kind == "encdec":
        P.t5_encdec_loss_and_grad(st["cfg"], st["enc_tokens"], st["tokens"], st["targets"], st["w"], grads=st["grads"],
                                  workspace=st["ws"], loss=st["loss"])
        return dict(st["out"], loss=st["loss"])
    cfg = st["cfg"]
    if kind == "decoder":
        P.t5_decoder_block_fwd(cfg, st["x"], st["enc"], st["w"], y=st["y"], stash=st["stash"], workspace=st["ws"])
        P.t5_decoder_block_bwd(cfg, st["dy"], st["x"], st["enc"], st["w"], st["stash"], dx=st["dx"], denc=st["denc"],
                               grads=st["grads"], workspace=st["ws"])
        return dict(y=st["y"], dx=st["dx"], denc=st["denc"], **st["grads"])
    P.t5_block_fwd(cfg, st["x"], st["w"], y=st["y"], stash=st["stash"], workspace=st["ws"])
    if kind == "score":
        return dict(y=st["y"])
    P.t5_block_bwd(cfg, st["dy"], st["x"], st["w"], st["stash"], dx=st["dx"], grads=st["grads"], workspace=st["ws"])
    return dict(y=st["y"], dx=st["dx"], **st["grads"])


def work(case):
    c, kind = case, case["kind"]
    es = 2 if c["dtype"] == "bf16" else 4
    d, i, f = c["d_model"], c["heads"] * c["d_kv"], c["d_ff"]

    def params(cross):
        return sum(math.prod(s[0]) for s in _shapes(c, cross).values())

    def fwd(tokens, seq, causal, enc_seq=0, batch=c["batch"]):
        """FLOPs of one layer's forward: 2 M N K of each product, the half of the scores that a causal mask leaves."""
        n = tokens * (8 * d * i + 4 * seq * i * (0.5 if causal else 1.0) + (4 if c["mlp"] == "relu" else 6) * d * f)
        if enc_seq:
            n += tokens * (4 * d * i + 4 * enc_seq * i) + batch * enc_seq * 4 * d * i
        return n

    if kind == "adafactor":
        # gradient and parameter read, parameter and its bf16 copy written; a dozen operations an element
        return {"bytes": 14 * params(False), "flops": 12 * params(False)}
    t, te = c["batch"] * c["seq"], c["batch"] * c["enc_seq"]
    n = fwd(t, c["seq"], c["causal"], c["enc_seq"])
    if kind == "score":
        return {"bytes": es * (2 * t * d + params(False)), "flops": n}
    if kind in ("block", "decoder"):
        p = params(kind == "decoder")
        # x, dy read and y, dx written (and the encoder output and its gradient); weights read, float32 gradients written
        return {"bytes": es * (4 * t * d + 2 * te * d + p) + 4 * p, "flops": 3 * n}
    p = c["layers"] * params(kind == "encdec") + (1 if c["tied"] else 2) * c["vocab"] * d
    if kind == "encdec":
        p += c["layers"] * params(False)
        n += fwd(te, c["enc_seq"], False)
    return {"bytes": (es + 4) * p, "flops": 3 * (c["layers"] * n + 2 * t * d * c["vocab"])}


def tolerance(case):
    if case["kind"] == "adafactor":
        return {"rel": 1e-5, "max": 1e-2}  # the bf16 copies: one rounding may fall the other way
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3}  # 64-bit comparison: up to 2e-6
    if case["kind"] in ("lm", "encdec"):
        return {"rel": 0.03, "max": 0.9}  # roundings of every layer travel through the others
    return {"rel": 0.015, "max": 0.3}  # 64-bit comparison: up to 7e-3


# ------------------------------------------------------------------ the same in 64 bits, plain torch
def _mix(x):
    """32-bit finaliser of the dropout generator, on int64 tensors or whole numbers."""
    x = x ^ (x >> 16)
    x = (x * 0x7FEB352D) & MASK32
    x = x ^ (x >> 15)
    x = (x * 0x846CA68B) & MASK32
    return x ^ (x >> 16)


def _keep(rate, seed, site, row0, rows, cols):
    """Multipliers [rows, cols] of a dropout site from its row row0 on: 1 / (1 - rate) where kept, else 0."""
    rate32 = float(torch.tensor(rate, dtype=torch.float32))
    k0 = _mix((seed & MASK32) ^ ((site * 0x9E3779B9) & MASK32))
    row = torch.arange(row0, row0 + rows, device=DEV, dtype=torch.int64)
    k1 = _mix(row ^ k0 ^ (seed >> 32))
    m = torch.empty(rows, cols, dtype=torch.float64, device=DEV)
    col = torch.arange(cols, device=DEV, dtype=torch.int64)
    per = max(1, (1 << 26) // cols)
    for r in range(0, rows, per):
        m[r:r + per] = (_mix(k1[r:r + per, None] ^ col) >= int(rate32 * 2.0 ** 32)).double()
    return m / (1.0 - rate32)


def _bias(table, s, causal):
    rel = torch.arange(s, device=DEV)[None, :] - torch.arange(s, device=DEV)[:, None]  # key - query
    n_side = BUCKETS if causal else BUCKETS // 2
    base = torch.zeros_like(rel) if causal else (rel > 0) * n_side
    n = (-rel).clamp(min=0) if causal else rel.abs()
    e = n_side // 2
    far = e + (torch.log(n.clamp(min=1).double() / e) / math.log(MAX_DISTANCE / e) * (n_side - e) + 1e-9).floor().long()
    return table[base + torch.where(n < e, n, far.clamp(max=n_side - 1))].permute(2, 0, 1)  # [heads, s, s]


def _norm(x, scale):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + EPS) * scale


class _Layer:
    """One layer on sequences b0 .. of the batch, in 64 bits; `seed`: its dropout seed."""

    def __init__(self, c, seq, causal, seed, b0):
        self.c, self.s, self.causal, self.seed, self.b0 = c, seq, causal, seed, b0

    def drop(self, x, site):
        if not self.c["dropout"]:
            return x
        rows = x.shape[0] * self.s
        return x * _keep(self.c["dropout"], self.seed, site, self.b0 * self.s, rows, x.shape[-1]).view(x.shape)

    def attend(self, xq, xkv, wq, wk, wv, wo, bias, site):
        h, k = self.c["heads"], self.c["d_kv"]
        heads = lambda x, w: (x @ w).unflatten(-1, (h, k)).transpose(1, 2).contiguous()  # noqa: E731
        q, kk, v = heads(xq, wq), heads(xkv, wk), heads(xkv, wv)
        a = q @ kk.transpose(2, 3).contiguous()
        if bias is not None:
            a = a + bias
            if self.causal:
                a = a.masked_fill(torch.ones(self.s, self.s, dtype=torch.bool, device=DEV).triu(1), -math.inf)
        p = torch.softmax(a, -1)
        if self.c["dropout"]:
            n = p.shape[0] * h * self.s
            p = p * _keep(self.c["dropout"], self.seed, site, self.b0 * h * self.s, n, p.shape[-1]).view(p.shape)
        return (p @ v).transpose(1, 2).flatten(2) @ wo

    def __call__(self, x, w, bias, enc=None):
        n = _norm(x, w["ln1_scale"])
        x = x + self.drop(self.attend(n, n, w["wq"], w["wk"], w["wv"], w["wo"], bias, 1), 2)
        if enc is not None:
            n = _norm(x, w["lnx_scale"])
            x = x + self.drop(self.attend(n, enc, w["xq"], w["xk"], w["xv"], w["xo"], None, 5), 6)
        n = _norm(x, w["ln2_scale"])
        u = n @ w["wi0"]
        if self.c["mlp"] == "relu":
            a = u.clamp(min=0)
        else:
            approx = "tanh" if self.c["mlp"] == "geglu_tanh" else "none"
            a = torch.nn.functional.gelu(u, approximate=approx) * (n @ w["wi1"])
        return x + self.drop(self.drop(a, 3) @ w["wo_ff"], 4)


def _leaf(w):
    if isinstance(w, dict):
        return {k: _leaf(v) for k, v in w.items()}
    return w.double().requires_grad_()


def _grad(w):
    return {k: _grad(v) if isinstance(v, dict) else v.grad for k, v in w.items()}


def _sequences(c, most_bytes=6e9):
    """Sequences of the batch that are worked on at a time."""
    widest = max(c["seq"], c["enc_seq"])
    one = 8 * widest * (6 * c["heads"] * widest + 8 * c["d_ff"] + 20 * c["d_model"] + 4 * c["vocab"])
    return max(1, min(c["batch"], int(most_bytes / one / max(1, c["layers"]))))


def _exact_model(c, i):
    w = _leaf(i["w"])
    seed, drop, per = 0x5EED5EED5EED, c["dropout"], _sequences(c, 4e10)
    counted = int(((i["targets"] >= 0) & (i["targets"] < c["vocab"])).sum())
    total = torch.zeros(1, dtype=torch.float64, device=DEV)
    layer_seed = lambda l: (seed + (l + 1) * 0x9E3779B97F4A7C15) & (2 ** 64 - 1)  # noqa: E731
    for b in range(0, c["batch"], per):
        end = lambda seq: _Layer(c, seq, True, seed, b)  # noqa: E731
        enc, first, names = None, 0, ("rel_table", "layers", "final_scale", 7, 8)
        if c["kind"] == "encdec":
            x = end(c["enc_seq"]).drop(w["embedding"][i["enc_tokens"][b:b + per].long()], 7)
            bias = _bias(w["enc_rel_table"], c["enc_seq"], False)
            for l, lw in enumerate(_per_layer(w["enc_layers"])):
                x = _Layer(c, c["enc_seq"], False, layer_seed(l), b)(x, lw, bias)
            enc = end(c["enc_seq"]).drop(_norm(x, w["enc_final_scale"]), 8)
            first, names = c["layers"], ("dec_rel_table", "dec_layers", "dec_final_scale", 9, 10)
        x = end(c["seq"]).drop(w["embedding"][i["tokens"][b:b + per].long()], names[3])
        bias = _bias(w[names[0]], c["seq"], True)
        for l, lw in enumerate(_per_layer(w[names[1]])):
            x = _Layer(c, c["seq"], True, layer_seed(first + l), b)(x, lw, bias, enc)
        nf = end(c["seq"]).drop(_norm(x, w[names[2]]), names[4])
        logits = nf @ w["embedding"].t() * c["d_model"] ** -0.5 if c["tied"] else nf @ w["logits_w"]
        lse = torch.logsumexp(logits, -1)
        t = i["targets"][b:b + per].long()
        got = logits.gather(-1, t.clamp(min=0)[..., None])[..., 0]
        loss = torch.where(t >= 0, lse - got + Z_LOSS * lse.square(), 0.0).sum() / counted
        loss.backward()
        total += loss.detach()
    return dict(_grad(w), loss=total)


def exact(case, seed):
    c, kind = case, case["kind"]
    i = _inputs(c, seed)
    if kind == "adafactor":
        out, beta = [], 1.0 - 101.0 ** -0.8
        for t in i.values():
            p, g = t["param"].double(), t["grad"].double()
            p2, g2 = (p, g) if p.dim() == 2 else (p[None], g[None])
            q = g2.square() + 1e-30
            if t["factored"]:
                vr = beta * t["v_row"].double() + (1 - beta) * q.mean(1)
                vc = beta * t["v_col"].double() + (1 - beta) * q.mean(0)
                v, state = vr[:, None] * vc[None] / vr.mean(), dict(v_row=vr, v_col=vc, v_full=None)
            else:
                v = beta * t["v_full"].double() + (1 - beta) * q
                state = dict(v_row=None, v_col=None, v_full=v)
            u = g2 * torch.rsqrt(v)
            u = u / u.square().mean().sqrt().clamp(min=1.0)
            new = (p2 - 1e-2 * p2.square().mean().sqrt().clamp(min=1e-3) * u).view(p.shape)
            out.append(dict(state, param=new, bf16_copy_out=new))
        return out
    if kind in ("lm", "encdec"):
        return _exact_model(c, i)
    grads = kind != "score"
    w = _leaf(i["w"])
    ys, dxs, dencs, per = [], [], [], _sequences(c)
    with torch.set_grad_enabled(grads):
        for b in range(0, c["batch"], per):
            x = i["x"][b:b + per].double().requires_grad_(grads)
            enc = i["enc"][b:b + per].double().requires_grad_() if kind == "decoder" else None
            y = _Layer(c, c["seq"], c["causal"], 0x5EED5EED5EED, b)(x, w, _bias(w["rel_table"], c["seq"], c["causal"]), enc)
            ys.append(y.detach())
            if grads:
                (y * i["dy"][b:b + per].double()).sum().backward()
                dxs.append(x.grad)
                if enc is not None:
                    dencs.append(enc.grad)
    out = dict(y=torch.cat(ys))
    if grads:
        out.update(_grad(w), dx=torch.cat(dxs))
    if dencs:
        out["denc"] = torch.cat(dencs)
    return out
