"""Rows that see no key of a call of flashd_attn_fwd_state on the 128-row kernel: the state goes out as
it came in, in the form s = Lam, ln w = 0, in place or not, and the output is its value."""
import pytest
import torch

from paper_2505_14201_amd import flashd
from tests.gpu_util import Guarded

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("seen", [0, 300])
def test_rows_without_a_new_key(d, in_place, seen):
    """seen: the last so many rows see keys of the call (of values 0.5), the others none."""
    B, H, Lq, Lk = 2, 16, 2200, 320
    gen = torch.Generator().manual_seed(71 + d + seen)
    q = torch.randn(B, H, Lq, d, generator=gen).to(torch.bfloat16).cuda()
    k = torch.randn(B, H, Lk, d, generator=gen).to(torch.bfloat16).cuda()
    v = torch.full_like(k, 0.5)
    guards = [Guarded(B * H * Lq * (d + 2) * 4) for _ in range(1 if in_place else 2)]
    st = guards[0].view(torch.float32, (B, H, Lq, d + 2))
    st.copy_(torch.randn(B, H, Lq, d + 2, generator=gen))
    st[:, :, ::2, d + 1] = 0.0                      # every other state with ln w = 0 already
    st[:, :, 7, d] = float("-inf")                  # one that holds no key
    st[:, :, 7, :d] = 0.0
    st[:, :, 7, d + 1] = 0.0
    before = st.clone()
    out = st if in_place else guards[1].view(torch.float32, (B, H, Lq, d + 2))
    o = torch.empty_like(q)
    flashd.attn_fwd_state(q, k, v, True, d ** -0.5, o=o, state_in=st, state_out=out,
                          causal_shift=-(Lq - seen))
    torch.cuda.synchronize()
    assert all(g.intact() for g in guards)
    rows = slice(0, Lq - seen)
    assert torch.equal(out[:, :, rows, :d], before[:, :, rows, :d])
    assert torch.equal(o[:, :, rows], before[:, :, rows, :d].to(torch.bfloat16))
    assert bool((out[:, :, rows, d + 1] == 0).all())
    lam = before[:, :, rows, d] - before[:, :, rows, d + 1]
    got = out[:, :, rows, d]
    # through log2 units and back: a few units in the last place of |Lam| <= 8
    assert torch.equal(torch.isinf(got), torch.isinf(lam))
    fin = torch.isfinite(lam)
    assert float((got[fin] - lam[fin]).abs().max()) <= 8 * 2.0 ** -22
    if seen:
        # the new keys' run has the value 0.5: between it and the old value, and never outside
        new, old = out[:, :, Lq - seen:, :d], before[:, :, Lq - seen:, :d]
        lo, hi = old.clamp(max=0.5), old.clamp(min=0.5)
        assert bool((new >= lo - 1e-2).all()) and bool((new <= hi + 1e-2).all())
        assert not torch.equal(new, old)


# (B, H, Lq, Lk, d, type): the kernels with 128, 64 and 32 query rows per workgroup, fp32, decode
EMPTY = [(2, 16, 2200, 320, 64, torch.bfloat16), (2, 16, 2200, 320, 128, torch.float16),
         (4, 16, 193, 97, 64, torch.bfloat16), (1, 4, 64, 160, 128, torch.bfloat16),
         (1, 2, 40, 50, 64, torch.float32), (1, 4, 3, 300, 128, torch.bfloat16)]


@pytest.mark.parametrize("B,H,Lq,Lk,d,dtype", EMPTY)
@pytest.mark.parametrize("in_place", [False, True])
def test_empty_states_go_out_as_zeros(B, H, Lq, Lk, d, dtype, in_place):
    """A state that holds no key says so by s = -inf alone, its o may be anything: a row without keys
    of the call has zeros in the output and in the state handed out."""
    gen = torch.Generator().manual_seed(72 + Lq)
    q, k, v = (torch.randn(B, H, n, d, generator=gen).to(dtype).cuda() for n in (Lq, Lk, Lk))
    st = torch.full((B, H, Lq, d + 2), float("nan"), device="cuda")
    st[..., d], st[..., d + 1] = float("-inf"), 0.0
    out = st if in_place else torch.full_like(st, float("nan"))
    o = torch.full_like(q, float("nan"))
    seen = Lq // 3                                  # rows that see a key, behind those that do not
    flashd.attn_fwd_state(q, k, v, True, d ** -0.5, o=o, state_in=st, state_out=out, causal_shift=-(Lq - seen))
    torch.cuda.synchronize()
    assert torch.isfinite(o).all() and torch.isfinite(out[..., :d]).all()
    rows = slice(0, Lq - seen)
    assert torch.count_nonzero(o[:, :, rows]) == 0 and torch.count_nonzero(out[:, :, rows, :d]) == 0
    assert torch.isneginf(out[:, :, rows, d] - out[:, :, rows, d + 1]).all()
    assert torch.isfinite(out[:, :, Lq - seen:]).all() and bool((o[:, :, Lq - seen:] != 0).any(-1).all())
