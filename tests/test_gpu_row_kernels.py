"""The prefill kernels whose wavefronts share out the keys of a row tile (32 and 64 query rows per
workgroup), which the automatic choice takes for calls too small for the 128-row kernel: edges of row
tiles, key blocks and splits, rows without keys, fp8, states in place, negative and zero scales."""
import numpy as np
import pytest
import torch

from oracle import attention as oa
from paper_2505_14201_amd import flashd, synthetic
from tests.gpu_util import check, run_flashd
from tests.test_gpu_kv8 import run_and_ref
from tests.test_gpu_state import check_state, run_chunks

pytestmark = pytest.mark.gpu
DT = {"f16": torch.float16, "bf16": torch.bfloat16}

# (B, Hq, Hkv, Lq, Lk)
SHORT = [(1, 1, 1, 33, 129),         # one row and one key past a tile and four blocks
         (1, 4, 2, 32, 160),         # full tiles, five blocks
         (2, 6, 2, 43, 191),         # tiles begin inside a position; the last block lacks a key
         (1, 3, 1, 85, 545),
         (1, 2, 2, 200, 180),        # causal: rows that see no key
         (1, 2, 1, 40, 3001)]        # few rows and many keys: key splits
# which kernel these take depends on d, the mask and states: 64 rows, 32 or 128
TILE64 = [(2, 32, 8, 300, 300),      # 19 row tiles of 64 rows per kv head, the last of 48 rows
          (4, 16, 16, 193, 193),     # one row and one key past three tiles
          (3, 32, 8, 157, 129),      # causal: rows that see no key
          (5, 16, 16, 500, 530)]
# 64 rows with and without a mask
TILE64_ALL = {64: [(3, 32, 8, 300, 385),       # 19 row tiles per kv head, the last of 48 rows
                   (4, 16, 16, 500, 385)],     # causal: rows that see no key
              128: [(5, 16, 16, 129, 129),     # one row and one key past two tiles
                    (5, 16, 16, 150, 129)]}
# and under a mask in two chunks
TILE64_STATES = {64: [TILE64[1], *TILE64_ALL[64]], 128: [TILE64[1], TILE64_ALL[128][1]]}


@pytest.mark.parametrize("shape", SHORT + TILE64)
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f16", 128), ("f16", 64)])
@pytest.mark.parametrize("causal", [False, True])
def test_output(shape, dtype, d, causal):
    w = synthetic.small("t", *shape, d, dtype, causal, seed=4100 + shape[3] + shape[4])
    q, k, v, _ = synthetic.make_qkv(w)
    got = run_flashd(q, k, v, causal, w.scale, use_ex=False)
    check(got, oa.attn(q, k, v, causal, w.scale), DT[dtype], str(shape))
    again = run_flashd(q, k, v, causal, w.scale)
    assert torch.equal(got.view(torch.int16), again.view(torch.int16))


@pytest.mark.parametrize("shape,d", [(s, d) for d in TILE64_ALL for s in TILE64_ALL[d]])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("causal", [False, True])
def test_output_of_64_rows(shape, d, dtype, causal):
    w = synthetic.small("t", *shape, d, dtype, causal, seed=4150 + shape[3] + shape[4])
    q, k, v, _ = synthetic.make_qkv(w)
    check(run_flashd(q, k, v, causal, w.scale, use_ex=False), oa.attn(q, k, v, causal, w.scale), DT[dtype], str(shape))


@pytest.mark.parametrize("shape", [SHORT[2], SHORT[4], TILE64[1], TILE64[2]])
@pytest.mark.parametrize("scale", [-0.09, 0.0])
def test_scales_below_and_at_zero(shape, scale):
    w = synthetic.small("t", *shape, 128, "bf16", True, seed=4200 + shape[3])
    q, k, v, _ = synthetic.make_qkv(w)
    check(run_flashd(q, k, v, True, scale, use_ex=False), oa.attn(q, k, v, True, scale), torch.bfloat16)


@pytest.mark.parametrize("shape", [(1, 2, 2, 85, 545), (4, 16, 16, 193, 193), (5, 16, 16, 300, 530)])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f16", 64)])
def test_scores_of_several_hundred(shape, dtype, d):
    w = synthetic.small("t", *shape, d, dtype, True, seed=4300 + shape[3], qk_std=4.0, plant_frac=0.05)
    q, k, v, _ = synthetic.make_qkv(w)
    check(run_flashd(q, k, v, True, w.scale, use_ex=False), oa.attn(q, k, v, True, w.scale), DT[dtype])


@pytest.mark.parametrize("shape", [SHORT[2], SHORT[4], TILE64[0], TILE64[2]])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f16", 64)])
@pytest.mark.parametrize("in_place", [False, True])
def test_states(shape, dtype, d, in_place):
    """Chunks of keys, the first of which some rows do not see and the last of which some see
    nothing of."""
    w = synthetic.small("t", *shape, d, dtype, True, seed=4400 + shape[3])
    q, k, v, _ = synthetic.make_qkv(w)
    o, st = run_chunks(q, k, v, True, w.scale, (shape[4] // 2 + 1,), in_place=in_place)
    check(o, oa.attn(q, k, v, True, w.scale), DT[dtype])
    check_state(st, oa.attn_state(q, k, v, True, w.scale), d, DT[dtype], "state")


@pytest.mark.parametrize("shape,d", [(s, d) for d in TILE64_STATES for s in TILE64_STATES[d]])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("in_place", [False, True])
def test_states_of_64_rows(shape, d, dtype, in_place):
    w = synthetic.small("t", *shape, d, dtype, True, seed=4450 + shape[3])
    q, k, v, _ = synthetic.make_qkv(w)
    o, st = run_chunks(q, k, v, True, w.scale, (shape[4] // 2 + 1,), in_place=in_place)
    check(o, oa.attn(q, k, v, True, w.scale), DT[dtype])
    check_state(st, oa.attn_state(q, k, v, True, w.scale), d, DT[dtype], "state")


@pytest.mark.parametrize("shape", SHORT)
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f16", 64)])
def test_fp8_keys_and_values(shape, dtype, d):
    w = synthetic.small("t", *shape, d, dtype, True, seed=4500 + shape[3])
    got, ref = run_and_ref(w, 2.0 ** -5, 0.03)
    check(got, ref, DT[dtype], str(shape))


@pytest.mark.parametrize("shape", [(1, 4, 2, 64, 160), (4, 16, 16, 192, 192)])
def test_infinite_values_behind_the_mask(shape):
    """A wavefront that meets a row only with hidden keys holds 0 * V of them: NaN where that V is
    infinite, and left out of the fold.  Rows that share a 32-key block with the infinite value
    are not looked at (as in the other kernels, a weight of zero does not silence it there)."""
    B, Hq, Hkv, Lq, Lk = shape
    w = synthetic.small("t", *shape, 128, "bf16", True, seed=4600)
    q, k, v, _ = synthetic.make_qkv(w)
    bad = v.clone()
    bad[:, :, Lk - 1] = float("inf")
    got = run_flashd(q, k, bad, True, w.scale, use_ex=False)
    ref = oa.attn(q, k, v, True, w.scale)
    rows = slice(0, Lq - 32)                     # none of them sees a key of the last block
    assert bool(torch.isfinite(got[:, :, rows].float()).all())
    assert np.abs(got[:, :, rows].double().numpy() - ref[:, :, rows]).max() <= 2e-2


# one and two key tiles; the last takes 64 rows per workgroup
FEW_KEYS = [(1, 2, 1, 33, 1), (2, 4, 2, 40, 64), (1, 2, 2, 150, 65), (3, 8, 8, 130, 128), (2, 16, 16, 300, 127)]


@pytest.mark.parametrize("shape", FEW_KEYS)
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f16", 128), ("f16", 64)])
@pytest.mark.parametrize("causal", [False, True])
def test_at_most_two_key_tiles(shape, dtype, d, causal):
    w = synthetic.small("t", *shape, d, dtype, causal, seed=4700 + shape[3] + shape[4])
    q, k, v, _ = synthetic.make_qkv(w)
    check(run_flashd(q, k, v, causal, w.scale, use_ex=False), oa.attn(q, k, v, causal, w.scale), DT[dtype])
    got, ref = run_and_ref(w, 2.0 ** -5, 0.03)
    check(got, ref, DT[dtype], "fp8")
    if shape[4] > 1:
        o, st = run_chunks(q, k, v, causal, w.scale, (shape[4] // 2 + 1,), in_place=True)
        check(o, oa.attn(q, k, v, causal, w.scale), DT[dtype])
        check_state(st, oa.attn_state(q, k, v, causal, w.scale), d, DT[dtype], "state")
