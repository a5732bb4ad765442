"""The decode kernel with 16-column score tiles: row counts around its 16 columns, key counts
around its 32-key blocks and the turns of its four wavefronts, splits with ranges that end inside
a block or lie past the last key, and what the skip, the fp8 cache and the state add to that."""
import numpy as np
import pytest
import torch

from oracle import attention as oa
from paper_2505_14201_amd import flashd, synthetic
from tests.gpu_util import check, run_flashd
from tests.test_gpu_state import check_state, run_chunks

pytestmark = pytest.mark.gpu
TILE, AUTO = flashd.VARIANT_TILE, flashd.VARIANT_AUTO
DT = {"f16": torch.float16, "bf16": torch.bfloat16}

# (B, Hq, Hkv, Lq, Lk, causal)
SHAPES = [(1, 1, 1, 1, 1, False),
          (2, 2, 1, 1, 31, False), (1, 2, 2, 1, 32, False), (1, 4, 2, 1, 33, False),
          (1, 15, 1, 1, 127, False), (1, 16, 1, 1, 129, False),    # 15 and 16 rows
          (2, 4, 1, 4, 70, True),                                 # 16 rows, causal positions
          (1, 5, 1, 3, 2, True),                                  # rows that see no key
          (1, 17, 1, 1, 129, False)]                              # 17: the wider kernel


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f16", 64), ("f16", 128), ("bf16", 64)])
def test_edges(shape, dtype, d):
    B, Hq, Hkv, Lq, Lk, causal = shape
    w = synthetic.small("t", B, Hq, Hkv, Lq, Lk, d, dtype, causal, seed=9700 + Hq * 5 + Lk)
    q, k, v, _ = synthetic.make_qkv(w)
    ref = oa.attn(q, k, v, causal, w.scale)
    for splits in (1, 2, 5):
        if splits <= Lk:
            check(run_flashd(q, k, v, causal, w.scale, TILE, splits), ref, DT[dtype], f"splits={splits}")
            check(run_flashd(q, k, v, causal, w.scale, AUTO, splits), ref, DT[dtype], f"auto {splits}")
    check(run_flashd(q, k, v, causal, -w.scale, TILE, 1), oa.attn(q, k, v, causal, -w.scale), DT[dtype],
          "negative scale")


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_moving_references(dtype):
    """Keys that grow along the range: every block lies above the reference, by more than the
    storage type of the coefficients holds."""
    w = synthetic.small("t", 1, 8, 2, 1, 900, 128, dtype, False, seed=9800, qk_std=4.0)
    q, k, v, _ = synthetic.make_qkv(w)
    k = (k.float() * torch.linspace(0.05, 4.0, 900).view(1, 1, -1, 1)).to(k.dtype)
    ref = oa.attn(q, k, v, False, w.scale)
    for variant in (TILE, AUTO):
        for splits in (1, 3):
            check(run_flashd(q, k, v, False, w.scale, variant, splits), ref, DT[dtype])


@pytest.mark.parametrize("Lq,Lk", [(2, 33), (2, 65), (2, 97), (3, 2)])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("d", [64, 128])
def test_wavefronts_without_a_key_of_the_row(Lq, Lk, bad, d):
    """The last key is infinite or NaN in one column and stands in a block of which the first
    position sees nothing: that position's rows keep their values (zeros where it sees no key at
    all), the last position's rows, which see it, do not."""
    w = synthetic.small("t", 1, 4, 1, Lq, Lk, d, "bf16", True, seed=9840 + Lk)
    q, k, v, _ = synthetic.make_qkv(w)
    ref = np.ascontiguousarray(oa.attn(q, k, v, True, w.scale)[:, :, :1])
    v[0, 0, Lk - 1, 5] = bad
    for variant in (TILE, AUTO):
        for splits in (1, 2):
            got = run_flashd(q, k, v, True, w.scale, variant, splits)
            check(got[:, :, :1], ref, torch.bfloat16, f"variant {variant} splits {splits}")
            if Lk < Lq:
                assert torch.count_nonzero(got[:, :, 0]) == 0
            assert not torch.isfinite(got[:, :, Lq - 1, 5]).any()


@pytest.mark.parametrize("hidden", [range(0, 64), range(40, 200),
                                    [j for j in range(300) if j // 32 % 4 == 1]])
@pytest.mark.parametrize("splits", [1, 2])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f16", 64)])
def test_keys_of_score_minus_infinity(hidden, splits, dtype, d):
    """Keys whose scores are -inf weigh nothing, also where a wavefront meets them first or meets
    no others (the last range: all blocks of wavefront 1)."""
    w = synthetic.small("t", 1, 8, 2, 1, 300, d, dtype, False, seed=9850)
    q, k, v, _ = synthetic.make_qkv(w)
    q[..., 5] = q[..., 5].abs() + 0.1
    left = [j for j in range(300) if j not in set(hidden)]
    ref = oa.attn(q, k[:, :, left].contiguous(), v[:, :, left].contiguous(), False, w.scale)
    k[:, :, list(hidden), 5] = float("-inf")
    for variant in (TILE, AUTO):
        check(run_flashd(q, k, v, False, w.scale, variant, splits), ref, DT[dtype], f"variant {variant}")


def test_state_of_a_decode_step():
    w = synthetic.small("t", 2, 8, 2, 2, 333, 128, "bf16", True, seed=9810)
    q, k, v, _ = synthetic.make_qkv(w)
    o, st = run_chunks(q, k, v, True, w.scale, (40, 200), in_place=True)
    check(o, oa.attn(q, k, v, True, w.scale), torch.bfloat16)
    check_state(st, oa.attn_state(q, k, v, True, w.scale), 128, torch.bfloat16, "state")


# K through LDS, K direct from 512 workgroups on; the last in 2 splits of its own accord
@pytest.mark.parametrize("B,Hkv,Lq,Lk", [(1, 2, 1, 70), (64, 8, 1, 65), (64, 8, 4, 67), (33, 8, 1, 2050)])
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f16", 64), ("f16", 128)])
def test_fp8_cache(B, Hkv, Lq, Lk, dtype, d):
    w = synthetic.small("t", B, 4 * Hkv, Hkv, Lq, Lk, d, dtype, Lq > 1, seed=9820)
    gen = torch.Generator(device="cuda").manual_seed(9820 + Lk)
    q = torch.randn(B, 4 * Hkv, Lq, d, device="cuda", generator=gen).to(DT[dtype])
    k8, v8 = ((torch.randn(B, Hkv, Lk, d, device="cuda", generator=gen) * 32).to(torch.float8_e4m3fn)
              for _ in "kv")
    o = torch.full_like(q, float("nan"))
    flashd.attn_fwd_kv8(q, k8, v8, o, w.causal, w.scale, 1 / 32, 1 / 32)
    assert torch.isfinite(o.float()).all()
    sc = float(np.float32(w.scale) * np.float32(1 / 32))
    for b in sorted({0, B // 2, B - 1}):
        ref = oa.attn(q[b:b + 1].cpu(), k8[b:b + 1].cpu().float(), v8[b:b + 1].cpu().float(), w.causal, sc) / 32
        check(o[b:b + 1].cpu(), ref, DT[dtype], f"b={b}")


@pytest.mark.parametrize("splits", [8, 9, 16, 17, 64])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64)])
def test_merge_of_many_splits(splits, dtype, d):
    """Up to 16 splits d / 4 lanes fold a row, from 17 on four wavefronts share it."""
    w = synthetic.small("t", 1, 4, 2, 3, 140, d, dtype, True, seed=9830)
    q, k, v, _ = synthetic.make_qkv(w)
    t = torch.float32 if dtype == "f32" else DT[dtype]
    check(run_flashd(q, k, v, True, w.scale, AUTO, splits), oa.attn(q, k, v, True, w.scale), t)
