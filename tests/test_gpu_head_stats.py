"""Row statistics of the LM head against the logits of the same call: ids in
order (larger logit, then lower id), confidence and renormalised weights, at the
edges of the row tiles, for vocabularies that do and do not divide into the
column tiles, with ties within and across the 64-column segments, on every
kernel that the head may take (test_projection_plan.py asks for it).
"""
import dataclasses

import pytest
import torch

from synthetic import LLADA_8B, TINY, make_weights, seeded_normal

pytestmark = pytest.mark.gpu


def _head(base, rows, vocab, k, mask_id, pair):
    """(logits, argmax, conf, ids, weights) of a model without layers; `pair`: the
    head multiplies both parts of the bfloat16 pair."""
    from paper_2608_23167_amd import _lib as L
    from paper_2608_23167_amd import api
    from paper_2608_23167_amd.model import DeviceKVCache, DeviceModel
    dims = dict(d_model=512, n_heads=4, n_kv_heads=4, ffn_dim=512) if base is LLADA_8B else {}
    shape = dataclasses.replace(base, name="head", n_layers=0, vocab=vocab, mask_id=mask_id, **dims)
    w = make_weights(shape, seed=5, device="cuda", norm_jitter=0.1, logit_scale=20.0)
    n = vocab // 3
    w.lm_head[n:2 * n] = w.lm_head[:n].clone()          # every one of these logits twice
    w.lm_head[2 * n:2 * n + 9] = 0                       # and nine zeros
    x = seeded_normal((1, rows, shape.d_model), 6, "head.x", device="cuda")
    x[0, 0] = 0                                          # a row of equal logits
    m = DeviceModel(shape, w, act_mode=L.SSM_ACT_BF16X2 if pair else L.SSM_ACT_BF16)
    cache = DeviceKVCache(dataclasses.replace(shape, n_layers=1), 1, rows)
    out = (torch.zeros(rows, dtype=torch.int32, device="cuda"), torch.zeros(rows, device="cuda"),
           torch.zeros(rows * k, dtype=torch.int32, device="cuda"), torch.zeros(rows * k, device="cuda"))
    logits = torch.zeros(rows * vocab, device="cuda")
    ws = torch.zeros(api.ssm_workspace_size(m, 1, rows), dtype=torch.uint8, device="cuda")
    pos = torch.arange(rows, dtype=torch.int32, device="cuda")
    api.ssm_denoise_step(m, cache, L.SSM_CACHE_OFF, 0, pos, rows, x, 0, k, *out, ws, logits=logits)
    torch.cuda.synchronize()
    quiet = tuple(torch.zeros_like(t) for t in out)      # without the logits stored
    api.ssm_denoise_step(m, cache, L.SSM_CACHE_OFF, 0, pos, rows, x, 0, k, *quiet, ws)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(out, quiet))
    return (logits.view(rows, vocab).double().cpu(), out[0].cpu(), out[1].cpu(),
            out[2].view(rows, k).cpu(), out[3].view(rows, k).cpu())


# (base, rows, vocabulary, k, mask id, pair): the last rows of a 256-row tile, its
# second 128 rows and a second tile, with one part of the operand and with two
HEADS = [
    (LLADA_8B, 1, 128, 8, 127, False), (LLADA_8B, 63, 384, 5, 0, False),
    (LLADA_8B, 128, 1024, 8, 1000, False), (LLADA_8B, 129, 1024, 8, 64, False),
    (LLADA_8B, 129, 640, 1, 639, False), (LLADA_8B, 257, 2048, 5, 2047, False),
    (LLADA_8B, 300, 20480, 8, 700, False), (LLADA_8B, 120, 40960, 8, 40959, False),
    (LLADA_8B, 129, 40960, 8, 40959, False), (LLADA_8B, 240, 40960, 5, 27000, False),
    (LLADA_8B, 257, 32768, 8, 32767, False), (LLADA_8B, 300, 32768, 5, 0, False),
    (LLADA_8B, 120, 1024, 8, 1000, True), (LLADA_8B, 300, 20480, 8, 700, True),
    (LLADA_8B, 300, 32768, 8, 32767, True),
    (TINY, 33, 32, 8, 31, False), (TINY, 100, 4096, 5, 77, False)]


@pytest.mark.parametrize("base,rows,vocab,k,mask_id,pair", HEADS)
def test_statistics_follow_the_logits(base, rows, vocab, k, mask_id, pair):
    """Ids are exact.  The sum of up to 4e4 float32 exponentials, in parts, is
    off by a few hundred roundings at most: 5e-5."""
    logits, argmax, conf, ids, w = _head(base, rows, vocab, k, mask_id, pair)
    z = logits.clone()
    z[:, mask_id] = -float("inf")
    order = torch.sort(z, dim=1, descending=True, stable=True)
    assert torch.equal(ids.long(), order.indices[:, :k])
    assert torch.equal(argmax.long(), order.indices[:, 0])
    ref = torch.exp(order.values[:, 0] - torch.logsumexp(z, 1))
    assert float((conf.double() / ref - 1).abs().max()) < 5e-5
    ref_w = torch.softmax(order.values[:, :k], 1)
    assert float((w.double() - ref_w).abs().max()) < 5e-5


@pytest.mark.parametrize("base,vocab", [(TINY, 512), (LLADA_8B, 1024)])
def test_infinite_logits(base, vocab):
    """A row whose best logit is +inf has no finite confidence (exp(inf - inf));
    logits of -inf count for nothing.  An infinite weight gives both: rows whose
    operand is positive there get +inf, the others -inf."""
    from paper_2608_23167_amd import _lib as L
    from paper_2608_23167_amd import api
    from paper_2608_23167_amd.model import DeviceKVCache, DeviceModel
    rows, k, mask_id = 40, 5, vocab - 1
    dims = dict(d_model=512, n_heads=4, n_kv_heads=4, ffn_dim=512) if base is LLADA_8B else {}
    shape = dataclasses.replace(base, name="head", n_layers=0, vocab=vocab, mask_id=mask_id, **dims)
    w = make_weights(shape, seed=5, device="cuda", norm_jitter=0.1, logit_scale=20.0)
    w.lm_head[77, 3] = float("inf")
    x = seeded_normal((1, rows, shape.d_model), 6, "head.inf", device="cuda")
    m = DeviceModel(shape, w)
    cache = DeviceKVCache(dataclasses.replace(shape, n_layers=1), 1, rows)
    argmax, conf = torch.zeros(rows, dtype=torch.int32, device="cuda"), torch.zeros(rows, device="cuda")
    ids, tw = torch.zeros(rows * k, dtype=torch.int32, device="cuda"), torch.zeros(rows * k, device="cuda")
    logits = torch.zeros(rows * vocab, device="cuda")
    ws = torch.zeros(api.ssm_workspace_size(m, 1, rows), dtype=torch.uint8, device="cuda")
    pos = torch.arange(rows, dtype=torch.int32, device="cuda")
    api.ssm_denoise_step(m, cache, L.SSM_CACHE_OFF, 0, pos, rows, x, 0, k, argmax, conf, ids, tw, ws,
                         logits=logits)
    torch.cuda.synchronize()
    z = logits.view(rows, vocab).double().cpu()
    z[:, mask_id] = -float("inf")
    up = x[0, :, 3].cpu() > 0
    assert 0 < int(up.sum()) < rows and torch.equal(z[:, 77] == float("inf"), up)
    assert torch.equal(argmax.cpu().long(), z.argmax(1))
    assert torch.isnan(conf.cpu()[up]).all()
    ref = torch.softmax(z[~up], 1).amax(1)
    assert float((conf.cpu()[~up].double() / ref - 1).abs().max()) < 5e-5
