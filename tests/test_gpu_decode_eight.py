"""Decode calls of up to 16 rows per kv head that the automatic choice leaves whole and runs on 8
wavefronts per workgroup: the shortest such contexts (some wavefronts have one block, or none that a
row sees), ragged and long ones, fp8, large scores with and without the skipped V fetch."""
import pytest
import torch

from oracle import attention as oa
from paper_2505_14201_amd import flashd, synthetic
from tests.gpu_util import check, run_flashd
from tests.test_gpu_kv8 import run_and_ref
from tests.test_gpu_skipv import run_both

pytestmark = pytest.mark.gpu
DT = {"f16": torch.float16, "bf16": torch.bfloat16}

# (B, Hq, Hkv, Lq, Lk, d)
SHAPES = [(1, 8, 2, 1, 257, 64),        # nine blocks, the last of one key
          (2, 4, 4, 16, 261, 64),       # causal: eleven rows see nothing of the last block
          (3, 32, 2, 1, 1055, 64),
          (16, 16, 16, 3, 700, 64)]     # as many workgroups as compute units
ON_FP8 = SHAPES + [(16, 32, 8, 4, 801, 128), (12, 16, 16, 1, 1100, 128)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("causal", [False, True])
def test_output(shape, dtype, causal):
    B, Hq, Hkv, Lq, Lk, d = shape
    assert flashd.auto_splits(B, Hq, Hkv, Lq, Lk, d, 2) == 1
    w = synthetic.small("t", *shape, dtype, causal, seed=4700 + Lk + Lq)
    q, k, v, _ = synthetic.make_qkv(w)
    got = run_flashd(q, k, v, causal, w.scale, use_ex=False)
    check(got, oa.attn(q, k, v, causal, w.scale), DT[dtype], str(shape))


@pytest.mark.parametrize("shape", ON_FP8)
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_fp8_keys_and_values(shape, dtype):
    w = synthetic.small("t", *shape, dtype, True, seed=4800 + shape[4])
    got, ref = run_and_ref(w, 2.0 ** -5, 0.03)
    check(got, ref, DT[dtype], str(shape))


@pytest.mark.parametrize("shape", SHAPES)
def test_scores_of_several_hundred(shape):
    w = synthetic.small("t", *shape, "bf16", True, seed=4900 + shape[4], qk_std=4.0,
                        plant_frac=0.05 if shape[1] == shape[2] else 0.0)
    q, k, v, _ = synthetic.make_qkv(w)
    check(run_flashd(q, k, v, True, w.scale, use_ex=False), oa.attn(q, k, v, True, w.scale),
          torch.bfloat16)


@pytest.mark.parametrize("shape", SHAPES)
def test_skipped_fetch_has_the_same_bits_where_nothing_is_skipped(shape):
    w = synthetic.small("t", *shape, "bf16", True, seed=5000 + shape[4])
    q, k, v, base, skip, visited, skipped = run_both(w, 0)
    assert skipped == 0 and visited > 0
    assert torch.equal(base.view(torch.int16), skip.view(torch.int16))
    check(skip, oa.attn(q, k, v, True, w.scale), torch.bfloat16)
