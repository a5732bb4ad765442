"""The merge of key splits: split counts on both sides of its instances (2, 4, 8, 16 and the
four-wavefront form), row counts that leave its last workgroup part empty, splits whose keys are all
hidden, and the partial states that the 128-row kernel hands it, at row tiles with missing rows."""
import pytest
import torch

from oracle import attention as oa
from paper_2505_14201_amd import flashd, synthetic
from tests.gpu_util import check, run_flashd

pytestmark = pytest.mark.gpu
DT = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}

# (B, Hq, Hkv, Lq, Lk, causal)
SHAPES = [(1, 1, 1, 1, 70, False),
          (1, 3, 1, 3, 700, True),                                # 9 rows
          (2, 2, 1, 133, 400, True)]                              # 266 rows a head group


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f16", 64), ("f32", 64), ("f32", 128)])
def test_split_counts(shape, dtype, d):
    B, Hq, Hkv, Lq, Lk, causal = shape
    w = synthetic.small("t", B, Hq, Hkv, Lq, Lk, d, dtype, causal, seed=9900 + Lq)
    q, k, v, _ = synthetic.make_qkv(w)
    ref = oa.attn(q, k, v, causal, w.scale)
    for splits in (1, 2, 3, 4, 5, 8, 9, 16, 17, 64):
        check(run_flashd(q, k, v, causal, w.scale, flashd.VARIANT_AUTO, splits), ref, DT[dtype],
              f"splits={splits}")
