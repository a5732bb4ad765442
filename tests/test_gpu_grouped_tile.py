"""Prefill with the heads of a kv group interleaved row by row: row tiles that begin inside a
position, end exactly at the last row, or hold fewer rows than a wavefront.  With splits given, on the
128-row kernel; with the state handed on, at most of these sizes on the kernel with 32 query rows per workgroup
(the 128-row kernel with states: test_gpu_tile_state.py)."""
import pytest
import torch

from oracle import attention as oa
from paper_2505_14201_amd import flashd, synthetic
from tests.gpu_util import check, run_flashd
from tests.test_gpu_state import check_state, run_chunks

pytestmark = pytest.mark.gpu
TILE = flashd.VARIANT_TILE
DT = {"f16": torch.float16, "bf16": torch.bfloat16}

# (Hq, Hkv, Lq, Lk): rows per kv head
SHAPES = [(3, 1, 11, 40),        # 33: one past the decode kernel
          (4, 1, 32, 200),       # 128: one full row tile
          (6, 2, 43, 43),        # 129: the last tile holds one row
          (5, 1, 77, 300),       # 385, tiles begin inside a position
          (16, 2, 100, 90),      # 800, rows that see no key
          (4, 1, 120, 960),      # no row tile saved: interleaved up to 8 keys per position,
          (4, 1, 120, 961)]      # one head after the other beyond (causal)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f16", 64)])
@pytest.mark.parametrize("causal", [False, True])
def test_interleaved_heads(shape, dtype, d, causal):
    Hq, Hkv, Lq, Lk = shape
    w = synthetic.small("t", 2, Hq, Hkv, Lq, Lk, d, dtype, causal, seed=9500 + Lq + Lk)
    q, k, v, _ = synthetic.make_qkv(w)
    ref = oa.attn(q, k, v, causal, w.scale)
    for splits in (1, 2):
        check(run_flashd(q, k, v, causal, w.scale, TILE, splits), ref, DT[dtype], f"splits={splits}")


@pytest.mark.parametrize("shape", SHAPES)
def test_interleaved_heads_with_state(shape):
    Hq, Hkv, Lq, Lk = shape
    w = synthetic.small("t", 1, Hq, Hkv, Lq, Lk, 128, "bf16", True, seed=9600 + Lq + Lk)
    q, k, v, _ = synthetic.make_qkv(w)
    o, st = run_chunks(q, k, v, True, w.scale, (Lk // 3,), in_place=True)
    check(o, oa.attn(q, k, v, True, w.scale), torch.bfloat16)
    check_state(st, oa.attn_state(q, k, v, True, w.scale), 128, torch.bfloat16, "state")
