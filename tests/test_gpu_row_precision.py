"""Precision of the prefill kernels whose wavefronts share out the keys of a row (32 and 64 query rows
per workgroup), beyond the tolerance that 16-bit outputs need: the state handed out is in fp32."""
import numpy as np
import pytest
import torch

from oracle import attention as oa
from paper_2505_14201_amd import flashd

pytestmark = pytest.mark.gpu


def qkv(B, H, Lq, Lk, d, dtype, std, seed):
    gen = torch.Generator().manual_seed(seed)
    return [(torch.randn(B, H, n, d, generator=gen) * std).to(dtype) for n in (Lq, Lk, Lk)]


# 32 rows per workgroup, the keys of a row on four wavefronts; 64 rows, on two
SHAPES = [(1, 4, 64, 500), (2, 2, 130, 128), (4, 16, 193, 193)]


def cuts(Lk, chunks):
    c = [0, Lk] if chunks == 1 else [0, 64 if Lk < 256 else 128, Lk]
    return list(zip(c, c[1:]))


@pytest.mark.parametrize("B,H,Lq,Lk", SHAPES)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("chunks", [1, 2])
def test_wavefronts_are_weighed_by_unrounded_sums(B, H, Lq, Lk, d, chunks):
    """V is 1 on the keys of every other 32-key block, which other wavefronts take than the rest,
    and 0 there: rounded coefficients cancel within a wavefront, and the state's o is a ratio of
    unrounded sums.  Weighed by the rounded ones it is up to 2^-9 of itself off."""
    q, k, _ = qkv(B, H, Lq, Lk, d, torch.bfloat16, 2.0, 8100 + Lk)
    v = torch.zeros_like(k)
    v[:, :, torch.arange(Lk) // 32 % 2 == 1] = 1.0
    ref = oa.attn_state(q, k, v, False, d ** -0.5)
    st = None
    for a, b in cuts(Lk, chunks):
        out = torch.empty(B, H, Lq, d + 2, device="cuda")
        flashd.attn_fwd_state(q.cuda(), k[:, :, a:b].contiguous().cuda(), v[:, :, a:b].contiguous().cuda(), False,
                              d ** -0.5, state_in=st, state_out=out)
        st = out
    torch.cuda.synchronize()
    err = np.abs(st[..., :d].cpu().double().numpy() - ref[..., :d]).max()
    # scores up to some 30 (44 in log2 units, an fp32 spacing of 2^-18) on either side of the
    # ratio, exponentials and sums a few units of 2^-24
    assert err <= 2.0 ** -17, err


MASKED = [(1, 4, 64, 128), (2, 3, 40, 100), (2, 16, 300, 127)]


@pytest.mark.parametrize("B,H,Lq,Lk", MASKED)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("scale", [0.1, -0.1])
def test_a_mask_that_hides_nothing_from_a_row_changes_no_bit_of_it(B, H, Lq, Lk, dtype, d, scale):
    """The last row sees every key with and without a mask, on 32-key blocks that are masked for the rows
    before it and on ones that are not; scores of up to some hundred."""
    q, k, v = qkv(B, H, Lq, Lk, d, dtype, 4.0, 8200 + Lk)
    got = []
    for causal in (False, True):
        st = torch.empty(B, H, Lq, d + 2, device="cuda")
        flashd.attn_fwd_state(q.cuda(), k.cuda(), v.cuda(), causal, scale, state_out=st)
        torch.cuda.synchronize()
        got.append(st[:, :, -1].cpu())
    assert torch.isfinite(got[0]).all()
    assert torch.equal(*got)
