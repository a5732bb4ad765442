"""Keys whose scores are -inf weigh nothing, in every tile-form kernel: rows that meet nothing else at first are
still empty after their first tiles, and what follows must reach them wherever its scores lie."""
import numpy as np
import pytest
import torch

from oracle import attention as oa
from paper_2505_14201_amd import flashd
from tests.gpu_util import check, run_flashd
from tests.test_gpu_state import run_chunks

pytestmark = pytest.mark.gpu
DT = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
AUTO, TILE, WIDE = flashd.VARIANT_AUTO, flashd.VARIANT_TILE, flashd.VARIANT_TILE_256
BLEND, ONLINE = flashd.VARIANT_TILE_BLEND, flashd.VARIANT_ONLINE_SOFTMAX


def inputs(B, Hq, Hkv, Lq, Lk, d, dtype, first, later, rows):
    """q, k, v for the GPU and k for the oracle.  Keys 0 .. first - 1 score -inf for all rows (an infinity in K), or
    for every third position ("some", bf16: the product of two elements of 1e30)."""
    torch.manual_seed(29 + first)
    q = torch.zeros(B, Hq, Lq, d)
    q[..., 0] = 1.0
    q[..., 1:] = 0.1 * torch.randn(B, Hq, Lq, d - 1)
    k = 0.1 * torch.randn(B, Hkv, Lk, d)
    v = torch.randn(B, Hkv, Lk, d)
    hidden = torch.zeros(Lk, dtype=torch.bool)
    hidden[:first] = True
    if later == "ordinary, then high":
        k[:, :, (first + Lk) // 2:, 0] = 300.0
    elif later == "far below zero":
        k[..., 0] = -200.0
    else:
        k[:, :, first:first + 40, 0] = -200.0
        hidden[first + 40:first + 120] = True
    hidden[Lk - 5:] = False
    big = 6.0e4 if dtype == "f16" else 1.0e30
    q[..., 5] = 0.0
    q[:, :, ::3 if rows == "some" else 1, 5] = big
    k[..., 5] = 0.0
    k[:, :, hidden, 5] = -big
    q, k, v = (t.to(DT[dtype]) for t in (q, k, v))
    kg = k.clone()
    if rows == "all":
        kg[:, :, hidden, 5] = float("-inf")
    return q, kg, v, k


CASES = [   # variant, splits, (B, Hq, Hkv, Lq, Lk)
    (AUTO, 0, (1, 8, 2, 1, 300)), (AUTO, 0, (1, 8, 2, 2, 1300)),               # decode
    (TILE, 1, (2, 8, 2, 5, 400)), (TILE, 3, (1, 24, 1, 1, 700)),               # 17 to 32 rows per kv head
    (AUTO, 0, (1, 1, 1, 33, 260)), (AUTO, 0, (1, 2, 1, 40, 3001)),             # 32 rows per workgroup
    (AUTO, 0, (4, 16, 16, 193, 260)), (AUTO, 0, (5, 16, 16, 500, 530)),        # 64
    (TILE, 1, (1, 2, 2, 300, 700)), (TILE, 2, (1, 4, 2, 70, 700)),             # 128
    (WIDE, 1, (1, 2, 2, 300, 700)),
    (BLEND, 1, (1, 2, 2, 300, 700)), (ONLINE, 1, (1, 2, 2, 300, 700)), (ONLINE, 1, (1, 8, 2, 1, 300)),
]
LATER = ["ordinary, then high", "far below zero", "low, -inf, ordinary"]


@pytest.mark.parametrize("variant,splits,shape", CASES)
@pytest.mark.parametrize("dtype,d,rows", [("bf16", 128, "some"), ("bf16", 64, "all"), ("f16", 128, "all")])
@pytest.mark.parametrize("later", LATER)
@pytest.mark.parametrize("first", [70, 130])
def test_rows_whose_first_keys_weigh_nothing(variant, splits, shape, dtype, d, rows, later, first):
    q, kg, v, k = inputs(*shape, d, dtype, first, later, rows)
    got = run_flashd(q, kg, v, False, 1.0, variant, splits)
    check(got, oa.attn(q, k, v, False, 1.0), DT[dtype], later)


@pytest.mark.parametrize("shape", [(1, 2, 2, 300, 700), (1, 1, 1, 33, 260), (4, 16, 16, 193, 260), (1, 8, 2, 1, 300)])
@pytest.mark.parametrize("dtype,d,rows", [("bf16", 128, "all"), ("bf16", 64, "some"), ("f16", 64, "all")])
@pytest.mark.parametrize("later", LATER)
@pytest.mark.parametrize("cut", [66, 160])
def test_states(shape, dtype, d, rows, later, cut):
    """In two calls, the first of which meets nothing but such keys, or some others too."""
    q, kg, v, k = inputs(*shape, d, dtype, 130, later, rows)
    o, st = run_chunks(q, kg, v, False, 1.0, (cut,), in_place=True)
    check(o, oa.attn(q, k, v, False, 1.0), DT[dtype], later)
    # (a recurrence over the finite stand-ins for -inf would lose s - ln w beside 1e60)
    g = shape[1] // shape[2]
    score = q.double() @ k.double().repeat_interleave(g, 1).transpose(-1, -2)
    lam = torch.logsumexp(score, -1).numpy()
    got = st.double().numpy()
    assert np.abs(got[..., d] - got[..., d + 1] - lam).max() <= 2e-4 + 1e-5 * np.abs(lam).max()
