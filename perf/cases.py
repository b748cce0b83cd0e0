"""The work that programs give this framework, as cases to be timed and compared.

A case is one call (or the calls of one step) through the public entry points:

  edges   the step around the model: select -> embed -> unmask
  layers  decoder layers over the compacted rows (`ssm_denoise_step`)
  head    final norm, LM head and row statistics (`ssm_denoise_step` of a model without layers)
  attn    attention alone (`ssm_attention`)
  whole   a denoising step through `Decoder.step`, with its logits

Shapes are those of the repository's own configurations: the 8B shape with 32
heads, the 7B shape with grouped-query heads, and the small float32 model.
"""
import math
from types import SimpleNamespace

import torch

from paper_2608_23167_amd import _lib as L
from paper_2608_23167_amd import api
from paper_2608_23167_amd.decoder import Decoder
from paper_2608_23167_amd.model import DeviceKVCache, DeviceModel

DEV = "cuda"

SHAPES = {
    "llada8b": dict(d_model=4096, n_heads=32, n_kv_heads=32, head_dim=128, ffn_dim=12288,
                    vocab=126464, dtype="bf16"),
    "dream7b": dict(d_model=3584, n_heads=28, n_kv_heads=4, head_dim=128, ffn_dim=18944,
                    vocab=152064, dtype="bf16"),
    "tiny": dict(d_model=128, n_heads=4, n_kv_heads=4, head_dim=32, ffn_dim=512, vocab=512,
                 dtype="f32"),
}
# The head of a `layers` case: the call always ends in a head, and a small one
# over four layers keeps the layers the measured part (the full head has cases of its own).
LAYERS_VOCAB = 2048
TOPK, ALPHA = 5, 0.4


def listed():
    return [
        # Every call of a step but the model, for a batch of 8 long prompts at the first step of a
        # block: 4336 rows a sequence, most of them plain embeddings, 176 of them soft ones.
        dict(name="edges_start_b8", kind="edges", model="llada8b", batch=8, prompt=4096, gen=4160,
             block=64, block_idx=0, prefix=True, local=128, middle=32, tail=16, n_per_step=8),
        # The smallest whole step: the float32 model, 108 rows, launches and latency only.
        dict(name="whole_f32_108", kind="whole", model="tiny", layers=2, batch=1, prompt=32,
             gen=128, block=32, block_idx=1, cache=False, local=32, middle=8, tail=4),
        # The flagship call: one cached decoding step of the 8B model, 120 rows, every layer.
        dict(name="whole_llada_120", kind="whole", model="llada8b", layers=32, batch=1, prompt=256,
             gen=256, block=32, block_idx=3, cache=True, local=64, middle=16, tail=8),
        # The same cached step in middle layers alone: what 31 of 32 steps of a short generation do.
        dict(name="layers_decode_120", kind="layers", model="llada8b", layers=4, act="one", batch=1,
             cached=352, prefix=0, block=32, suffix=88, ragged=False),
        # A cached step of a long generation: 240 rows over 1776 keys.
        dict(name="layers_decode_240", kind="layers", model="llada8b", layers=4, act="one", batch=1,
             cached=1536, prefix=0, block=64, suffix=176, ragged=False),
        # A small served batch whose prompts differ in length.
        dict(name="layers_decode_b4_ragged", kind="layers", model="llada8b", layers=4, act="one",
             batch=4, cached=320, prefix=0, block=32, suffix=87, ragged=True),
        # A large served batch: 32 sequences, 3840 rows in one cached step.
        dict(name="layers_decode_b32", kind="layers", model="llada8b", layers=4, act="one",
             batch=32, cached=352, prefix=0, block=32, suffix=88, ragged=False),
        # The first step of a block of a short generation in the leading layers, which keep the
        # projection inputs as a pair.
        dict(name="layers_start_376_pair", kind="layers", model="llada8b", layers=4, act="pair",
             batch=1, cached=0, prefix=256, block=32, suffix=88, ragged=False),
        # The first step of a block in the middle of a long generation.
        dict(name="layers_start_1776", kind="layers", model="llada8b", layers=4, act="one", batch=1,
             cached=0, prefix=1536, block=64, suffix=176, ragged=False),
        # A step without the prefix cache on the grouped-query model, at an odd row count.
        dict(name="layers_dream_1127", kind="layers", model="dream7b", layers=4, act="one", batch=1,
             cached=0, prefix=992, block=32, suffix=103, ragged=False),
        # The head of the flagship step.
        dict(name="head_120", kind="head", model="llada8b", rows=120),
        # Attention alone: the cached step of a batch of 8 over a 4096-token prefix.
        dict(name="attn_b8_240x4336", kind="attn", dtype="bf16", batch=8, heads=32, kv_heads=32,
             q=240, keys=4336),
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["edges", "layers", "layers", "layers", "layers", "layers", "head", "attn",
                       "attn", "whole"])
    if kind == "edges":
        block = rng.choice([16, 32, 64])
        blocks = _log(rng, 4, 32)
        return dict(kind="edges", model=rng.choice(["llada8b", "dream7b", "tiny"]),
                    batch=_log(rng, 1, 8), prompt=_log(rng, 16, 4096), gen=block * blocks,
                    block=block, block_idx=rng.randrange(0, blocks - 1),
                    prefix=rng.random() < 0.5, local=rng.randrange(0, 2 * block + 1),
                    middle=rng.randrange(0, 33), tail=rng.randrange(1, 17), n_per_step=_log(rng, 1, 8))
    if kind == "layers":
        model = rng.choice(["llada8b", "llada8b", "dream7b"])
        block, suffix = rng.choice([16, 32, 64]), rng.randrange(20, 200)
        act = rng.choice(["one", "one", "pair"])
        if rng.random() < 0.6:      # cached step, one sequence or a batch
            batch = _log(rng, 1, min(16, 3300 // ((block + suffix) * (2 if act == "pair" else 1))))
            return dict(kind="layers", model=model, layers=4, act=act, batch=batch,
                        cached=_log(rng, 100, 2500 if batch < 5 else 600), prefix=0, block=block,
                        suffix=suffix, ragged=batch > 1 and rng.random() < 0.5)
        return dict(kind="layers", model=model, layers=4, act=act, batch=1, cached=0,
                    prefix=_log(rng, 100, 1300 if act == "pair" else 2000), block=block, suffix=suffix, ragged=False)
    if kind == "head":
        return dict(kind="head", model=rng.choice(["llada8b", "dream7b"]), rows=_log(rng, 16, 480))
    if kind == "attn":
        kv = rng.choice([4, 8, 32])
        q = _log(rng, 16, 1500)
        batch = _log(rng, 1, max(1, min(8, 3000 // q)))
        return dict(kind="attn", dtype=rng.choice(["bf16", "f16"]), batch=batch,
                    heads=rng.choice([28, 32]) if kv == 4 else 32, kv_heads=kv, q=q,
                    keys=_log(rng, 64, min(6000, 10_000_000 // (batch * q))))
    block = rng.choice([16, 32])
    blocks = rng.randrange(3, 9)
    return dict(kind="whole", model="tiny", layers=2, batch=rng.choice([1, 1, 2]),
                prompt=_log(rng, 8, 200), gen=block * blocks, block=block,
                block_idx=rng.randrange(0, blocks - 1), cache=rng.random() < 0.5,
                local=rng.randrange(8, 40), middle=rng.randrange(0, 17), tail=rng.randrange(1, 9))


# ---- inputs -----------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) & 0x7FFFFFFF)
    return g


def _shape(model, layers, vocab=None):
    s = dict(SHAPES[model])
    if vocab:
        s["vocab"] = vocab
    return SimpleNamespace(n_layers=layers, mask_id=s["vocab"] - 1, rope_base=10000.0, rms_eps=1e-5,
                           **s)


def _normal(g, size, std, dtype, mean=0.0):
    return torch.empty(size, dtype=dtype, device=DEV).normal_(mean, std, generator=g)


def _weights(shape, g, tok_emb=True):
    """Random-init weights: N(0, 0.02) matrices, norm gains around one."""
    dt = torch.float32 if shape.dtype == "f32" else torch.bfloat16
    d, hd, F = shape.d_model, shape.head_dim, shape.ffn_dim
    H, Hk, V = shape.n_heads, shape.n_kv_heads, shape.vocab

    def W(r, c):
        return _normal(g, (r, c), 0.02, dt)

    def norm():
        return _normal(g, (d,), 0.1, dt, 1.0)

    layers = []
    for _ in range(shape.n_layers):
        lw = SimpleNamespace(attn_norm=norm(), wq=W(H * hd, d), wk=W(Hk * hd, d), wv=W(Hk * hd, d),
                             wo=W(d, H * hd), ffn_norm=norm(), w_gate=W(F, d), w_up=W(F, d),
                             w_down=W(d, F))
        lw.tensors = lambda lw=lw: [lw.attn_norm, lw.wq, lw.wk, lw.wv, lw.wo, lw.ffn_norm,
                                    lw.w_gate, lw.w_up, lw.w_down]
        layers.append(lw)
    lm_head = W(V, d)
    return SimpleNamespace(tok_emb=W(V, d) if tok_emb else lm_head, final_norm=norm(),
                           lm_head=lm_head, layers=layers)


def _positions(case):
    """Row positions of a step: prefix, block, then the kept suffix tokens spread over the rest."""
    P = case["cached"] + case["prefix"]
    head = torch.arange(case["cached"], P + case["block"], dtype=torch.int32)
    tail = P + case["block"] + 3 * torch.arange(case["suffix"], dtype=torch.int32)
    return torch.cat([head, tail])


def _pads(case):
    if not case["ragged"]:
        return None
    return [(case["cached"] // 2) * s // (case["batch"] - 1) for s in range(case["batch"])]


def _layers_inputs(case, seed):
    shape = _shape(case["model"], case["layers"], LAYERS_VOCAB)
    g = _gen(seed)
    w = _weights(shape, g, tok_emb=False)
    rows = case["prefix"] + case["block"] + case["suffix"]
    # the residual stream: embeddings before the leading layers, which keep the
    # pair; a few units per element in the middle of the stack
    x = _normal(g, (case["batch"], rows, shape.d_model), 0.02 if case["act"] == "pair" else 4.0,
                torch.float32)
    cap = case["cached"] + rows
    size = (shape.n_layers, case["batch"], shape.n_kv_heads, cap, shape.head_dim)
    k, v = _normal(g, size, 1.0, torch.float16), _normal(g, size, 1.0, torch.float16)
    return shape, w, rows, x, k, v


def _edges_inputs(case, seed):
    shape = _shape(case["model"], 0)
    g = _gen(seed)
    B, V, Lt = case["batch"], shape.vocab, case["prompt"] + case["gen"]
    dt = torch.float32 if shape.dtype == "f32" else torch.bfloat16
    P = case["prompt"] + case["block_idx"] * case["block"]

    def ids(*size):
        return torch.randint(0, V - 1, size, generator=g, device=DEV, dtype=torch.int32)

    def weights(*size):      # descending, summing to one
        u = torch.rand(size, generator=g, device=DEV).sort(dim=-1, descending=True).values
        return (u / u.sum(-1, keepdim=True)).contiguous()

    i = SimpleNamespace(shape=shape, emb=_normal(g, (V, shape.d_model), 0.02, dt), P=P)
    i.tokens0 = ids(B, Lt)
    i.tokens0[:, P:] = shape.mask_id
    half = torch.rand((B, case["block"]), generator=g, device=DEV) < 0.5
    blk = i.tokens0[:, P:P + case["block"]]
    blk[half] = ids(B, case["block"])[half]
    i.pred_ids, i.pred_w = ids(B, Lt, TOPK), weights(B, Lt, TOPK)
    i.pred_step = torch.where(torch.rand((B, Lt), generator=g, device=DEV) < 0.8, 6, -1).to(torch.int32)
    p = _params(case)
    i.n_rows, _, i.first_out = api.ssm_select_count(p)
    i.n_out = i.n_rows - i.first_out
    i.topk_ids, i.topk_w = ids(B, i.n_out, TOPK), weights(B, i.n_out, TOPK)
    i.argmax = i.topk_ids[:, :, 0].contiguous()
    i.conf = torch.rand((B, i.n_out), generator=g, device=DEV)
    return i


def _params(case):
    return api.select_params(case["prompt"], case["gen"], case["block"], case["block_idx"],
                             case["local"], case["middle"], 0, case["tail"], case["prefix"])


def _whole_inputs(case, seed):
    shape = _shape(case["model"], case["layers"])
    g = _gen(seed)
    w = _weights(shape, g)
    B, Lt, V = case["batch"], case["prompt"] + case["gen"], shape.vocab
    P = case["prompt"] + case["block_idx"] * case["block"]

    def ids(*size):
        return torch.randint(0, V - 1, size, generator=g, device=DEV, dtype=torch.int32)

    tokens = ids(B, Lt)
    tokens[:, P + case["block"] // 2:] = shape.mask_id
    pred_ids = ids(B, Lt, TOPK)
    u = torch.rand((B, Lt, TOPK), generator=g, device=DEV).sort(dim=-1, descending=True).values
    pred_w = u / u.sum(-1, keepdim=True)
    pred_step = torch.where(torch.rand((B, Lt), generator=g, device=DEV) < 0.8, 6, -1).to(torch.int32)
    dt = torch.float32 if shape.dtype == "f32" else torch.float16
    kv_seed = int(torch.randint(0, 1 << 30, (1,), generator=g, device=DEV).item())
    return shape, w, tokens, pred_ids, pred_w, pred_step, P, dt, kv_seed


def _whole_kv(shape, case, P, dt, kv_seed):
    g = _gen(kv_seed)
    size = (shape.n_layers, case["batch"], shape.n_kv_heads, P, shape.head_dim)
    return _normal(g, size, 1.0, dt), _normal(g, size, 1.0, dt)


def _attn_inputs(case, seed):
    g = _gen(seed)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float16
    q = _normal(g, (case["batch"], case["heads"], case["q"], 128), 1.0, dt)
    k = _normal(g, (case["batch"], case["kv_heads"], case["keys"], 128), 1.0, dt)
    v = _normal(g, (case["batch"], case["kv_heads"], case["keys"], 128), 1.0, dt)
    return q, k, v


def _head_inputs(case, seed):
    shape = _shape(case["model"], 0)
    g = _gen(seed)
    w = _weights(shape, g, tok_emb=False)
    return shape, w, _normal(g, (1, case["rows"], shape.d_model), 4.0, torch.float32)


def _outputs(B, n, k=TOPK):
    return (torch.zeros((B, n), dtype=torch.int32, device=DEV), torch.zeros((B, n), device=DEV),
            torch.zeros((B, n, k), dtype=torch.int32, device=DEV),
            torch.zeros((B, n, k), device=DEV))


# ---- state ------------------------------------------------------------------
def prepare(case, seed):
    s = SimpleNamespace(case=case, kind=case["kind"])
    if s.kind == "edges":
        s.i = _edges_inputs(case, seed)
        i, B = s.i, case["batch"]
        s.model = DeviceModel(i.shape, SimpleNamespace(
            tok_emb=i.emb, final_norm=i.emb[0].contiguous(), lm_head=i.emb, layers=[]))
        s.params = _params(case)
        s.tokens = torch.empty_like(i.tokens0)
        s.pos = torch.zeros(i.n_rows, dtype=torch.int32, device=DEV)
        s.tok_c = torch.zeros((B, i.n_rows), dtype=torch.int32, device=DEV)
        s.region = torch.zeros(i.n_rows, dtype=torch.int8, device=DEV)
        s.x = torch.zeros((B, i.n_rows, i.shape.d_model), device=DEV)
        # the prediction state of the step before, and the one that this step writes
        s.next_ids, s.next_w, s.next_step = i.pred_ids.clone(), i.pred_w.clone(), i.pred_step.clone()
        s.selected = torch.zeros(B * case["block"], dtype=torch.uint8, device=DEV)
        s.left = torch.zeros(B, dtype=torch.int32, device=DEV)
    elif s.kind == "layers":
        shape, w, s.rows, s.x, k, v = _layers_inputs(case, seed)
        s.model = DeviceModel(shape, w, pair_layers=case["layers"] if case["act"] == "pair" else 0)
        s.cache = DeviceKVCache(shape, case["batch"], case["cached"] + s.rows)
        s.cache.k.copy_(k)
        s.cache.v.copy_(v)
        s.pos = _positions(case).to(DEV)
        s.pads = _pads(case)
        s.mode = L.SSM_CACHE_READ if case["cached"] else L.SSM_CACHE_WRITE
        s.out = _outputs(case["batch"], s.rows - case["prefix"])
        s.hidden = torch.zeros_like(s.x)
        s.ws = torch.zeros(api.ssm_workspace_size(s.model, case["batch"], s.rows),
                           dtype=torch.uint8, device=DEV)
    elif s.kind == "head":
        shape, w, s.x = _head_inputs(case, seed)
        s.model = DeviceModel(shape, w)
        s.rows = case["rows"]
        s.cache = DeviceKVCache(_shape(case["model"], 1), 1, s.rows)
        s.pos = torch.arange(s.rows, dtype=torch.int32, device=DEV)
        s.out = _outputs(1, s.rows)
        s.ws = torch.zeros(api.ssm_workspace_size(s.model, 1, s.rows), dtype=torch.uint8, device=DEV)
    elif s.kind == "attn":
        s.q, s.k, s.v = _attn_inputs(case, seed)
        s.out = torch.zeros((case["batch"], case["q"], case["heads"] * 128), device=DEV)
        s.ws = torch.zeros(api.ssm_attention_workspace_size(case["batch"], case["heads"], case["q"]) or 1,
                           dtype=torch.uint8, device=DEV)
    else:
        shape, w, tokens, pred_ids, pred_w, pred_step, P, dt, kv_seed = _whole_inputs(case, seed)
        wl = SimpleNamespace(model=shape, batch=case["batch"], prompt_len=case["prompt"],
                             gen_len=case["gen"], total_len=case["prompt"] + case["gen"],
                             block_size=case["block"], n_blocks=case["gen"] // case["block"],
                             local_budget=case["local"], middle_budget=case["middle"],
                             tail_budget=case["tail"], middle_mode=0, tail_mode=0,
                             cache=case["cache"], topk=TOPK, alpha=ALPHA)
        s.dec = Decoder(wl, DeviceModel(shape, w))
        s.dec.tokens.copy_(tokens)
        s.dec.pred_ids.copy_(pred_ids)
        s.dec.pred_w.copy_(pred_w)
        s.dec.pred_step.copy_(pred_step)
        if case["cache"]:
            k, v = _whole_kv(shape, case, P, dt, kv_seed)
            s.dec.cache.k[:, :, :, :P] = k
            s.dec.cache.v[:, :, :, :P] = v
        # the rows of this step, as the decoder will count them
        n_rows, _, s.first = api.ssm_select_count(s.dec.params(case["block_idx"], not case["cache"]))
        s.n_out = n_rows - s.first
        s.logits = torch.zeros((case["batch"], s.n_out, shape.vocab), device=DEV)
    return s


def run(s):
    c = s.case
    if s.kind == "edges":
        i = s.i
        s.tokens.copy_(i.tokens0)
        n_rows, _, first = api.ssm_select_suffix(s.params, s.tokens, s.pos, s.tok_c, s.region)
        api.ssm_embed_suffix(s.model, s.tok_c, s.pos, s.region, n_rows, i.pred_ids, i.pred_w,
                             i.pred_step, 6, TOPK, ALPHA, s.x)
        api.ssm_unmask(s.tokens, i.P, c["block"], i.shape.mask_id, L.SSM_UNMASK_TOPN,
                       c["n_per_step"], 0.9, i.argmax, i.conf, i.topk_ids, i.topk_w, TOPK,
                       n_rows - first, s.pos[first:], 7, s.next_ids, s.next_w, s.next_step,
                       s.selected, s.left)
        return {"pos": s.pos, "tok": s.tok_c, "region": s.region, "x": s.x, "tokens": s.tokens,
                "ids": s.next_ids, "w": s.next_w, "step": s.next_step, "selected": s.selected,
                "left": s.left}
    if s.kind == "layers":
        argmax, conf, ids, w = s.out
        api.ssm_denoise_step(s.model, s.cache, s.mode, c["cached"], s.pos, s.rows, s.x, c["prefix"],
                             TOPK, argmax, conf, ids, w, s.ws, hidden=s.hidden, pad=s.pads)
        # this step's keys and values, in the cache's slots
        n = c["cached"]
        return {"hidden": s.hidden, "conf": conf, "k": s.cache.k[:, :, :, n:n + s.rows],
                "v": s.cache.v[:, :, :, n:n + s.rows]}
    if s.kind == "head":
        argmax, conf, ids, w = s.out
        api.ssm_denoise_step(s.model, s.cache, L.SSM_CACHE_OFF, 0, s.pos, s.rows, s.x, 0, TOPK,
                             argmax, conf, ids, w, s.ws)
        return {"argmax": argmax, "conf": conf, "ids": ids, "w": w}
    if s.kind == "attn":
        api.ssm_attention(s.q, s.k, s.v, c["keys"], s.out, s.ws)
        return s.out
    s.dec.step_idx = 7
    s.dec.step(c["block_idx"], not c["cache"], logits=s.logits, unmask=False)
    n = c["batch"] * s.n_out
    return {"logits": s.logits, "conf": s.dec.conf[:n], "w": s.dec.topk_w[:n * TOPK]}


# ---- what a pass cannot do without ------------------------------------------
def _layer_params(sh):
    return (sh.d_model * (sh.n_heads + 2 * sh.n_kv_heads) * sh.head_dim
            + sh.d_model * sh.n_heads * sh.head_dim + 3 * sh.d_model * sh.ffn_dim)


def _model_work(sh, B, rows, keys, n_out, layers, es):
    """Weights once, the residual stream in and out, keys and values read and written."""
    M = B * rows
    p = _layer_params(sh) * layers
    kv = 2 * B * keys * sh.n_kv_heads * sh.head_dim * layers * (4 if es == 4 else 2)
    return {"bytes": (p + sh.vocab * sh.d_model) * es + 8 * M * sh.d_model + kv,
            "flops": 2 * M * p + 4 * M * keys * sh.n_heads * sh.head_dim * layers
            + 2 * B * n_out * sh.vocab * sh.d_model}


def work(case):
    kind = case["kind"]
    if kind == "attn":
        B, H, q, n = case["batch"], case["heads"], case["q"], case["keys"]
        return {"bytes": 2 * B * 128 * (H * q + 2 * case["kv_heads"] * n) + 4 * B * q * H * 128,
                "flops": 4 * B * H * q * n * 128}
    sh = _shape(case["model"], 0, LAYERS_VOCAB if kind == "layers" else None)
    es = 4 if sh.dtype == "f32" else 2
    if kind == "edges":
        n_rows, n_suffix, first = api.ssm_select_count(_params(case))
        B, d = case["batch"], sh.d_model
        # every row's embedding written; a table row read per token, TOPK of them per soft row
        table = (n_rows - n_suffix) + n_suffix * 0.8 * TOPK
        return {"bytes": B * (n_rows * (4 * d + 8) + table * d * es
                              + n_suffix * TOPK * 8 * 3), "flops": 2 * B * n_suffix * TOPK * d}
    if kind == "head":
        return _model_work(sh, 1, case["rows"], 0, case["rows"], 0, es)
    if kind == "layers":
        rows = case["prefix"] + case["block"] + case["suffix"]
        return _model_work(sh, case["batch"], rows, case["cached"] + rows,
                           rows - case["prefix"], case["layers"], es)
    P = case["prompt"] + case["block_idx"] * case["block"]
    n_rows, _, first = api.ssm_select_count(_params(dict(case, prefix=not case["cache"])))
    w = _model_work(sh, case["batch"], n_rows, n_rows + (P if case["cache"] else 0),
                    n_rows - first, case["layers"], es)
    w["bytes"] += 4 * case["batch"] * (n_rows - first) * sh.vocab      # the logits
    return w


def tolerance(case):
    kind = case["kind"]
    if kind == "edges":        # float32 sums of a handful of terms
        return {"rel": 1e-6, "max": 1e-5}
    if case.get("model") == "tiny":   # float32 throughout
        return {"rel": 2e-5, "max": 2e-4}
    if kind == "attn":         # probabilities of 8 (bf16) or 11 (f16) bits
        return {"rel": 8e-3 if case["dtype"] == "bf16" else 2e-3}
    if kind == "head":         # one bf16 rounding of the normalised row; ties of the top k
        return {"rel": 8e-3, "differ": 0.01}
    if kind == "layers":       # a few roundings to bf16 and f16 in each of four layers
        return {"rel": 1.2e-2}
    return {"rel": 0.03}       # the same in 32 layers: 1e-2 against 64 bits


# ---- the same in 64 bits ----------------------------------------------------
def _norm64(x, g, eps):
    return x / torch.sqrt(x.square().mean(-1, keepdim=True) + eps) * g.double()


def _rope64(x, pos, base):
    """x [heads, n, dh] at positions pos [n]."""
    half = x.shape[-1] // 2
    f = base ** (-2.0 * torch.arange(half, dtype=torch.float64, device=DEV) / x.shape[-1])
    a = pos.double()[:, None] * f
    c, s = a.cos(), a.sin()
    x1, x2 = x[..., :half], x[..., half:]
    return torch.cat([x1 * c - x2 * s, x2 * c + x1 * s], -1)


def _attn64(q, k, v):
    """q [H, n, dh], k and v [Hkv, keys, dh] -> [n, H * dh], a head at a time."""
    H, g = q.shape[0], q.shape[0] // k.shape[0]
    out = []
    for h in range(H):
        p = torch.softmax(q[h] @ k[h // g].T.contiguous() / math.sqrt(q.shape[-1]), -1)
        out.append(p @ v[h // g])
    return torch.cat(out, -1)


def _model64(sh, w, x, pos, pads, kp, vp):
    """Layers over x [B, n, d]; kp, vp: each layer's cached prefix [layers, B, Hkv, P, dh] or None."""
    x = x.double()
    B, n, _ = x.shape
    H, Hk, dh = sh.n_heads, sh.n_kv_heads, sh.head_dim
    ks, vs = [], []
    for l, lw in enumerate(w.layers):
        wq, wk, wv, wo = (t.double() for t in (lw.wq, lw.wk, lw.wv, lw.wo))
        wg, wu, wd = (t.double() for t in (lw.w_gate, lw.w_up, lw.w_down))
        y, kl, vl = torch.empty_like(x), [], []
        for b in range(B):
            pad = pads[b] if pads else 0
            h = _norm64(x[b], lw.attn_norm, sh.rms_eps)
            heads = lambda t, m: t.view(n, m, dh).transpose(0, 1).contiguous()  # noqa: E731
            q = _rope64(heads(h @ wq.T, H), pos - pad, sh.rope_base)
            k = _rope64(heads(h @ wk.T, Hk), pos - pad, sh.rope_base)
            v = heads(h @ wv.T, Hk)
            kl.append(k)
            vl.append(v)
            if kp is not None:
                k = torch.cat([kp[l, b, :, pad:].double(), k], 1)
                v = torch.cat([vp[l, b, :, pad:].double(), v], 1)
            r = x[b] + _attn64(q, k, v) @ wo.T
            h = _norm64(r, lw.ffn_norm, sh.rms_eps)
            y[b] = r + (torch.nn.functional.silu(h @ wg.T) * (h @ wu.T)) @ wd.T
        x = y
        ks.append(torch.stack(kl))
        vs.append(torch.stack(vl))
    return x, ks, vs


def _stats64(sh, w, x):
    """Head and row statistics over x [B, n, d]."""
    h = _norm64(x, w.final_norm, sh.rms_eps)
    logits = torch.cat([h @ w.lm_head[i:i + 8192].double().T for i in range(0, sh.vocab, 8192)], -1)
    z = logits.clone()
    z[..., sh.mask_id] = -math.inf
    top = z.topk(TOPK, -1)
    conf = torch.exp(top.values[..., 0] - torch.logsumexp(z, -1))
    return logits, top.indices.int(), conf, torch.softmax(top.values, -1)


def _embed64(emb, mask_id, tokens, pos, soft_from, pred_ids, pred_w, pred_step, prev):
    """Rows of every sequence: table rows, and soft embeddings from row `soft_from` on."""
    p = pos.long()
    x = emb[tokens[:, p].long()].double()
    soft = torch.zeros_like(x)
    for i in range(TOPK):
        soft += pred_w[:, p, i, None].double() * emb[pred_ids[:, p, i].long()].double()
    mixed = (1 - ALPHA) * emb[mask_id].double() + ALPHA * soft
    use = pred_step[:, p] == prev
    use[:, :soft_from] = False
    return torch.where(use[..., None], mixed, x)


def _select64(case, prefix):
    """Positions of the kept rows: prefix, block, local, strided middle, spread tail."""
    b, s_end = case["block"], case["prompt"] + case["gen"]
    P = case["prompt"] + case["block_idx"] * b
    s0 = P + b
    local = list(range(s0, min(s0 + case["local"], s_end)))
    lo = s0 + len(local)
    tail_lo = max(lo, s_end - b)
    n, t = tail_lo - lo, s_end - tail_lo
    m, k = min(case["middle"], n), min(case["tail"], t)
    middle = [lo + i * n // m for i in range(m)]
    tail = [tail_lo + (i * (t - 1) // (k - 1) if k > 1 else t - 1) for i in range(k)]
    head = list(range(0 if prefix else P, P + b))
    return head + local + middle + tail, len(head)


def exact(case, seed):
    kind = case["kind"]
    if kind == "attn":
        q, k, v = _attn_inputs(case, seed)
        return torch.stack([_attn64(a.double(), b.double(), c.double()) for a, b, c in zip(q, k, v)])
    if kind == "layers":
        sh, w, rows, x, k, v = _layers_inputs(case, seed)
        n = case["cached"]
        x, ks, vs = _model64(sh, w, x, _positions(case).to(DEV), _pads(case),
                             k[:, :, :, :n] if n else None, v[:, :, :, :n] if n else None)
        conf = _stats64(sh, w, x[:, case["prefix"]:])[2]
        return {"hidden": x, "conf": conf, "k": torch.stack(ks), "v": torch.stack(vs)}
    if kind == "head":
        sh, w, x = _head_inputs(case, seed)
        _, ids, conf, tw = _stats64(sh, w, x.double())
        return {"argmax": ids[..., 0].contiguous(), "conf": conf, "ids": ids, "w": tw}
    if kind == "edges":
        i = _edges_inputs(case, seed)
        pos, head = _select64(case, case["prefix"])
        at = torch.tensor(pos, dtype=torch.int32, device=DEV)
        x = _embed64(i.emb, i.shape.mask_id, i.tokens0, at, head, i.pred_ids, i.pred_w, i.pred_step, 6)
        # the state that the unmasking writes is whole numbers and copies
        return {"pos": at, "tok": i.tokens0[:, at.long()], "region": None, "x": x, "tokens": None,
                "ids": None, "w": None, "step": None, "selected": None, "left": None}
    sh, w, tokens, pred_ids, pred_w, pred_step, P, dt, kv_seed = _whole_inputs(case, seed)
    pos, head = _select64(case, not case["cache"])
    at = torch.tensor(pos, dtype=torch.int32, device=DEV)
    x = _embed64(w.tok_emb, sh.mask_id, tokens, at, head, pred_ids, pred_w, pred_step, 6)
    k = v = None
    if case["cache"]:
        k, v = _whole_kv(sh, case, P, dt, kv_seed)
    x, _, _ = _model64(sh, w, x, at, None, k, v)
    logits, _, conf, tw = _stats64(sh, w, x[:, head - case["block"]:])
    return {"logits": logits, "conf": conf.reshape(-1), "w": tw.reshape(-1)}
