"""The 128-row kernel behind the entry points that do not take a number of splits: chunks of keys with the
state handed on, and K and V in fp8 (widened first), at sizes where the automatic choice leaves the call to that
kernel (test_row_plan.py holds it to that).  The oracle looks at the heads of two kv heads."""
import numpy as np
import pytest
import torch

from oracle import attention as oa
from paper_2505_14201_amd import flashd
from tests.gpu_util import Guarded, check
from tests.test_gpu_state import check_state

pytestmark = pytest.mark.gpu
DT = {"f16": torch.float16, "bf16": torch.bfloat16}

# (B, Hq, Hkv, Lq, Lk, cuts, shift): under a mask the first rows see no key, some see a part, the last all
CHUNKS = [(2, 16, 16, 2077, 333, (130,), -1500),          # the last row tile holds 29 rows
          (2, 32, 8, 1031, 500, (65, 320), -400)]         # heads of a kv group interleaved
FP8 = [(2, 16, 16, 2077, 200), (2, 32, 8, 1031, 77)]


def inputs(B, Hq, Hkv, Lq, Lk, d, dtype, std, seed):
    gen = torch.Generator().manual_seed(seed)
    q, k, v = (torch.randn(B, h, n, d, generator=gen) for h, n in ((Hq, Lq), (Hkv, Lk), (Hkv, Lk)))
    return (q * std).to(dtype), (k * std).to(dtype), v.to(dtype)


def of_kv_head(x, b, h, g=1):
    return x[b:b + 1, h * g:(h + 1) * g].contiguous()


@pytest.mark.parametrize("case", CHUNKS)
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f16", 128), ("f16", 64)])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("in_place,std", [(True, 1.0), (False, 4.0), (True, 4.0)])
def test_chunks_with_the_state_handed_on(case, dtype, d, causal, in_place, std):
    B, Hq, Hkv, Lq, Lk, cuts, shift = case
    q, k, v = inputs(B, Hq, Hkv, Lq, Lk, d, DT[dtype], std, 8300 + Lk + d)
    qg = q.cuda()
    guards = [Guarded(q.numel() * 2)]
    o = guards[0].view(q.dtype, q.shape)
    st, k0 = None, 0
    for k1 in (*cuts, Lk):
        out, before = st, st if st is None else st.clone()
        if st is None or not in_place:
            guards.append(Guarded(B * Hq * Lq * (d + 2) * 4))
            out = guards[-1].view(torch.float32, (B, Hq, Lq, d + 2))
        flashd.attn_fwd_state(qg, k[:, :, k0:k1].contiguous().cuda(), v[:, :, k0:k1].contiguous().cuda(), causal,
                              d ** -0.5, o=o, state_in=st, state_out=out, causal_shift=shift - k0)
        st, k0 = out, k1
    # a last chunk that hands out no state has the same output
    alone = torch.full_like(o, float("nan"))
    a = cuts[-1]
    flashd.attn_fwd_state(qg, k[:, :, a:].contiguous().cuda(), v[:, :, a:].contiguous().cuda(), causal, d ** -0.5,
                          o=alone, state_in=before, causal_shift=shift - a)
    torch.cuda.synchronize()
    assert all(x.intact() for x in guards)
    assert torch.equal(alone, o)
    o, st, g = o.cpu(), st.cpu(), Hq // Hkv
    for b, h in ((0, 0), (B - 1, Hkv - 1)):
        ref = oa.attn_state(of_kv_head(q, b, h, g), of_kv_head(k, b, h), of_kv_head(v, b, h), causal, d ** -0.5,
                            shift=shift)
        check(of_kv_head(o, b, h, g), ref[..., :d], DT[dtype], f"o of kv head {b}, {h}")
        check_state(of_kv_head(st, b, h, g), ref, d, DT[dtype], f"state of kv head {b}, {h}")


@pytest.mark.parametrize("shape", FP8)
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f16", 64)])
@pytest.mark.parametrize("causal", [False, True])
def test_fp8_widened_first(shape, dtype, d, causal):
    B, Hq, Hkv, Lq, Lk = shape
    q, k, v = inputs(B, Hq, Hkv, Lq, Lk, d, DT[dtype], 1.0, 8400 + Lk)
    kscale, vscale = 0.03, 0.045
    k8, v8 = (k.float() / kscale).to(torch.float8_e4m3fn), (v.float() / vscale).to(torch.float8_e4m3fn)
    guard = Guarded(q.numel() * 2)
    o = guard.view(q.dtype, q.shape)
    flashd.attn_fwd_kv8(q.cuda(), k8.cuda(), v8.cuda(), o, causal, d ** -0.5, kscale, vscale)
    torch.cuda.synchronize()
    assert guard.intact()
    scale = float(np.float32(d ** -0.5) * np.float32(kscale))
    g = Hq // Hkv
    for b, h in ((0, 0), (B - 1, Hkv - 1)):
        ref = oa.attn(of_kv_head(q, b, h, g), of_kv_head(k8.float(), b, h), of_kv_head(v8.float(), b, h), causal,
                      scale) * float(np.float32(vscale))
        check(of_kv_head(o.cpu(), b, h, g), ref, DT[dtype], f"kv head {b}, {h}")
