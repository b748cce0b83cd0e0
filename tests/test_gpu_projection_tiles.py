"""The projection kernels at the edges of their tiles: one decoder layer over
row counts just above and below whole row tiles, at widths that make the
launcher choose each tile shape and split-K factor (test_projection_plan.py
asks it), against the oracle's layer in float64.
"""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from oracle.model import layer_forward
from synthetic import LLADA_8B, TINY, make_weights, seeded_normal

pytestmark = pytest.mark.gpu

# widths: query-key-value columns divisible by 192 and 256 / by 128 only; feed
# forward 2F divisible by 192 and 256
WIDE = dict(d_model=1024, n_heads=8, n_kv_heads=8, ffn_dim=3072)
GROUPED = dict(d_model=768, n_heads=6, n_kv_heads=2, ffn_dim=6144)
# the widths of the 7B shape, where launches of up to 256 rows take gemm_pp_kernel
WIDTHS_7B = dict(d_model=3584, n_heads=28, n_kv_heads=4, ffn_dim=18944)


def _dims(d, kv, ffn):
    return dict(d_model=d, n_heads=d // 128, n_kv_heads=kv, ffn_dim=ffn)


# (widths, rows, pair): row tiles, the small-row launches and, on widths that
# are quick to check, every split-K factor of gemm_pp_kernel
CASES = [
    (WIDE, 256, False), (WIDE, 257, False), (WIDE, 385, True), (WIDE, 511, False),
    (WIDE, 513, True), (WIDE, 1025, False), (WIDE, 1776, False), (WIDE, 1776, True),
    (GROUPED, 300, False), (GROUPED, 513, False), (GROUPED, 1025, True), (GROUPED, 1281, False),
    (WIDTHS_7B, 1, False), (WIDTHS_7B, 16, False), (WIDTHS_7B, 120, False),
    (WIDTHS_7B, 240, False), (WIDTHS_7B, 256, False),
    (WIDTHS_7B, 16, True), (WIDTHS_7B, 120, True), (WIDTHS_7B, 300, True),
    (_dims(256, 1, 1280), 1, False), (_dims(256, 1, 1280), 1, True), (_dims(256, 1, 8448), 257, True),
    (_dims(512, 1, 256), 513, True), (_dims(768, 1, 256), 513, True), (_dims(1024, 1, 256), 513, False),
    (_dims(1024, 1, 2304), 256, False), (_dims(1280, 1, 768), 200, False),
    (_dims(1280, 1, 4864), 1, True), (_dims(1536, 1, 256), 513, False), (_dims(1536, 1, 7424), 1, True),
    (_dims(1792, 14, 256), 1, False), (_dims(1792, 1, 2816), 1, False), (_dims(1792, 1, 3840), 1, True),
    (_dims(2048, 1, 2816), 257, False), (_dims(2048, 1, 5376), 257, True),
    (_dims(2560, 1, 1280), 200, False), (_dims(2560, 1, 5376), 1025, True)]


# float32 models: K columns that leave a rest of 32, 64 or 96 to whole trips of
# 128, each head dimension, grouped heads
F32 = [dict(d_model=96, n_heads=3, n_kv_heads=1, head_dim=32, ffn_dim=160),
       dict(d_model=320, n_heads=5, n_kv_heads=5, head_dim=64, ffn_dim=1056),
       dict(d_model=256, n_heads=2, n_kv_heads=1, head_dim=128, ffn_dim=512)]


def _shape(dims, base=LLADA_8B):
    import dataclasses
    return dataclasses.replace(base, name="tiles", n_layers=1, vocab=512, mask_id=511, **dims)


def _view(t):
    """The same values 8 bytes into a larger buffer."""
    n = 8 // t.element_size()
    v = torch.empty(t.numel() + n, dtype=t.dtype, device=t.device)[n:].view(t.shape)
    return v.copy_(t)


def _layer(shape, rows, pair, first_out, views=False):
    """(x, GPU hidden, GPU keys, oracle hidden, oracle keys) of one layer; with
    `views`, all its weights lie at addresses that 16 does not divide."""
    from paper_2608_23167_amd import _lib as L
    from paper_2608_23167_amd import api
    from paper_2608_23167_amd.model import DeviceKVCache, DeviceModel
    w = make_weights(shape, seed=3, device="cuda", norm_jitter=0.1)
    if views:
        for holder in (w, w.layers[0]):
            for name, t in vars(holder).items():
                if torch.is_tensor(t):
                    setattr(holder, name, _view(t))
        assert all(t.data_ptr() % 16 for t in w.layers[0].tensors())
    m = DeviceModel(shape, w, pair_layers=1 if pair else 0)
    x = seeded_normal((1, rows, shape.d_model), 4, "tiles.x", device="cuda")
    pos = torch.arange(rows, dtype=torch.int32, device="cuda")
    cache = DeviceKVCache(shape, 1, rows + 3)
    n_out, k = rows - first_out, 5
    argmax = torch.zeros(n_out, dtype=torch.int32, device="cuda")
    conf = torch.zeros(n_out, device="cuda")
    ids = torch.zeros(n_out * k, dtype=torch.int32, device="cuda")
    tw = torch.zeros(n_out * k, device="cuda")
    hidden = torch.full_like(x, float("nan"))
    ws = torch.zeros(api.ssm_workspace_size(m, 1, rows), dtype=torch.uint8, device="cuda")
    api.ssm_denoise_step(m, cache, L.SSM_CACHE_WRITE, 0, pos, rows, x, first_out, k, argmax, conf,
                         ids, tw, ws, hidden=hidden)
    torch.cuda.synchronize()
    names = ("attn_norm", "wq", "wk", "wv", "wo", "ffn_norm", "w_gate", "w_up", "w_down")
    lw = SimpleNamespace(**{n: getattr(w.layers[0], n).double().cpu().numpy() for n in names})
    xs = x[0].double().cpu().numpy()
    ref = layer_forward(xs, np.arange(rows), lw, shape)
    keys = cache.k[0, 0, :, :rows].transpose(0, 1).double().cpu().numpy()
    return xs, hidden[0].double().cpu().numpy(), keys, ref.x, ref.k


def _worst(a, b):
    """Largest relative error of a row."""
    a, b = a.reshape(len(a), -1), b.reshape(len(b), -1)
    return float(np.max(np.linalg.norm(a - b, axis=1) / np.linalg.norm(b, axis=1)))


def _check(shape, rows, pair, **kw):
    x, hidden, keys, ref, ref_k = _layer(shape, rows, pair, max(rows - 40, 0), **kw)
    assert np.isfinite(hidden).all()
    e, ek = _worst(hidden - x, ref - x), _worst(keys, ref_k)
    print(f"rows {rows} pair {pair}: branch {e:.2e}, keys {ek:.2e}")
    assert e < (3e-3 if pair else 1e-2)
    assert ek < (1e-3 if pair else 5e-3)


@pytest.mark.parametrize("dims,rows,pair", CASES)
def test_layer_at_tile_edges(dims, rows, pair):
    """Per row, because an error at a tile edge touches a few rows only.  Bounds:
    a one-pass projection rounds its input to bfloat16 (2^-9 of each element at
    most, 0.17% in the mean), and a row passes at most four of them and the
    float16 attention operands in a chain: 1e-2 of the branch (hidden - x),
    which has no share of the exact residual; with the pair the float16
    operands alone remain: 3e-3.  Keys pass one projection: 5e-3."""
    _check(_shape(dims), rows, pair)


@pytest.mark.parametrize("rows,pair", [(40, False), (300, False), (513, True)])
def test_weights_that_are_views(rows, pair):
    """Weights 8 bytes into a larger buffer, at row counts where aligned ones go
    straight into LDS 16 bytes at a time: the bounds of test_layer_at_tile_edges."""
    _check(_shape(WIDE), rows, pair, views=True)


@pytest.mark.parametrize("dims", F32)
@pytest.mark.parametrize("rows", [1, 4, 33, 65, 700])
def test_float32_layer_at_tile_edges(dims, rows):
    """float32 throughout: a chain of sums of at most 1100 terms, each rounding
    6e-8, stays within 1e-5 of the branch; the residual stream itself rounds
    twice, 2^-24 of |hidden| each (1.2e-7), which counts where the branch is
    small against it.  700 keys split the attention."""
    shape = _shape(dims, TINY)
    x, hidden, keys, ref, ref_k = _layer(shape, rows, False, 0)
    err = np.linalg.norm(hidden - ref, axis=1)
    bound = 1e-5 * np.linalg.norm(ref - x, axis=1) + 1.2e-7 * np.linalg.norm(ref, axis=1)
    ek = _worst(keys, ref_k)
    print(f"rows {rows} d {shape.d_model}: error over bound {np.max(err / bound):.2f}, keys {ek:.2e}")
    assert np.all(err < bound) and ek < 1e-5


@pytest.mark.parametrize("d", [128, 1024])
def test_float32_sums_in_short_chains(d):
    """Error of the float32 head's logits, whose operand is exact here (rows of
    +1 and -1 have a mean square of one, eps vanishes beside it, and the gains
    are float32): nothing but the sums of d products rounds.  A chain of n
    fused multiply-adds of random terms is off by 0.31 sqrt(n) 2^-24 of the
    result (rms: each step rounds a partial sum of growing size by up to half a
    unit in the last place).  Sums of 32 products, added up, give
    0.31 sqrt(32 + d / 32) 2^-24; the bound is 1.25 times that.  One chain of d
    products would give 3.5 (d = 128), four chains of a quarter 4.7 (d = 1024)."""
    import dataclasses
    from paper_2608_23167_amd import _lib as L
    from paper_2608_23167_amd import api
    from paper_2608_23167_amd.model import DeviceKVCache, DeviceModel
    rows, vocab = 108, 512
    shape = dataclasses.replace(TINY, name="chains", n_layers=0, d_model=d, n_heads=d // 32,
                                n_kv_heads=d // 32, vocab=vocab, mask_id=vocab - 1, rms_eps=1e-30)
    w = make_weights(shape, seed=7, device="cuda", norm_jitter=0.1)
    g = torch.Generator(device="cuda").manual_seed(8)
    x = torch.randint(0, 2, (1, rows, d), generator=g, device="cuda").float() * 2 - 1
    m = DeviceModel(shape, w)
    cache = DeviceKVCache(dataclasses.replace(shape, n_layers=1), 1, rows)
    out = (torch.zeros(rows, dtype=torch.int32, device="cuda"), torch.zeros(rows, device="cuda"),
           torch.zeros(rows, dtype=torch.int32, device="cuda"), torch.zeros(rows, device="cuda"))
    logits = torch.zeros(rows * vocab, device="cuda")
    ws = torch.zeros(api.ssm_workspace_size(m, 1, rows), dtype=torch.uint8, device="cuda")
    pos = torch.arange(rows, dtype=torch.int32, device="cuda")
    api.ssm_denoise_step(m, cache, L.SSM_CACHE_OFF, 0, pos, rows, x, 0, 1, *out, ws, logits=logits)
    torch.cuda.synchronize()
    ref = (x[0].double() * w.final_norm.double()).cpu() @ w.lm_head.double().cpu().T
    err = float((logits.view(rows, vocab).double().cpu() - ref).norm() / ref.norm()) * 2 ** 24
    print(f"d {d}: rms error {err:.2f} x 2^-24")
    assert err < 1.25 * 0.31 * (32 + d / 32) ** 0.5
