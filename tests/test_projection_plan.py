"""Which kernel a projection of a bfloat16 model is launched on.  The choice is
made on the host from sizes and addresses alone, so these tests need no GPU;
they ask the debug library, which exports it."""
import ctypes as C
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
KINDS = ("qkv", "o", "gate_up", "down", "lm")
# (d_model, heads, key-value heads, feed-forward width, vocabulary)
LLADA = (4096, 32, 32, 12288, 126464)
DREAM = (3584, 28, 4, 18944, 152064)
GQA_8 = (4096, 32, 8, 14336, 65536)
SMALL = (1024, 8, 8, 3072, 1024)


def plan(kind, rows, dims, pair=False, weights=0):
    """(1 for gemm_pp_kernel or 0 for gemm_bf16_kernel, tile rows, columns, K splits)."""
    lib = C.CDLL(os.path.join(ROOT, "paper_2608_23167_amd", "libssm_debug.so"))
    fn = lib.ssm_debug_gemm_plan
    fn.argtypes = [C.c_char_p] + [C.c_int32] * 7 + [C.c_uint64, C.POINTER(C.c_int32)]
    out = (C.c_int32 * 4)()
    assert fn(kind.encode(), rows, *dims, int(pair), weights, out) == 0
    return tuple(out)


TILES = {(256, 256), (256, 192), (256, 128), (128, 256), (128, 192)}


@pytest.mark.parametrize("pair", [False, True])
def test_gpu_cases_reach_every_launch(pair):
    """The layers that the GPU compares with the oracle take every tile shape of
    gemm_pp_kernel, its splits 1 to 8, and gemm_bf16_kernel."""
    from test_gpu_projection_tiles import CASES
    seen = set()
    for dims, rows, p in CASES:
        if p == pair:
            args = (dims["d_model"], dims["n_heads"], dims["n_kv_heads"], dims["ffn_dim"], 512)
            seen |= {plan(kind, rows, args, pair) for kind in KINDS[:4]}
    assert {s[1:3] for s in seen if s[0]} == TILES
    assert {s[3] for s in seen if s[0]} == set(range(1, 9))
    assert any(not s[0] for s in seen)


def test_gpu_cases_reach_every_head_launch():
    from test_gpu_head_stats import HEADS
    seen = {(pair, *plan("lm", rows, (512, 4, 4, 512, vocab), pair)[:3])
            for base, rows, vocab, _, _, pair in HEADS if base.dtype == "bf16"}
    assert seen == {(p, *t) for p in (False, True) for t in ((0, 128, 128), (1, 256, 256), (1, 128, 256))}


@pytest.mark.parametrize("dims", [LLADA, DREAM, GQA_8, SMALL])
def test_unaligned_weights_go_through_registers(dims):
    for kind in KINDS:
        for rows in (1, 120, 240, 300, 513, 1776):
            for pair in (False, True):
                for weights in (2, 4, 8, 24):
                    assert plan(kind, rows, dims, pair, weights)[0] == 0, (kind, rows, pair, weights)


@pytest.mark.parametrize("dims,kind,rows", [
    (DREAM, "gate_up", range(385, 512)),      # 231 us on gemm_bf16_kernel, 282 on the other, at 440 rows
    (DREAM, "down", range(257, 512)),         # 122, 132
    (LLADA, "qkv", range(257, 512)),          # 94, 100 at 376 rows
    (LLADA, "o", range(257, 512)),            # 42, 47 at 440 rows
    (GQA_8, "qkv", range(257, 512)),          # 45, 63
    (SMALL, "gate_up", range(257, 512)),      # 17, 29
])
def test_pair_keeps_the_faster_kernel(dims, kind, rows):
    """With the pair, a fixed row count is no line between the kernels: these are
    slower on gemm_pp_kernel up to 511 rows, at whole and at ragged row tiles."""
    assert not any(plan(kind, r, dims, True)[0] for r in rows)


def test_gemm_pp_kernel_where_it_is_faster():
    assert all(plan("gate_up", r, LLADA, True)[0] for r in range(385, 2000, 7))
    assert all(plan("qkv", r, DREAM, True)[0] for r in range(257, 385))
    for dims in (LLADA, DREAM):
        for kind in ("qkv", "o", "gate_up", "down"):
            assert all(plan(kind, r, dims)[0] for r in range(257, 400)), kind
            assert all(plan(kind, r, dims, pair)[0] for r in range(512, 2000, 7) for pair in (0, 1))
    # one pass of a small model: too few tiles below 512 rows
    assert not any(plan("gate_up", r, SMALL)[0] for r in range(257, 512))
