"""GPU parity of variant TILE_256, the 256-row prefill kernel (one wavefront per SIMD, matrix
and vector work interleaved by hand, operands and accumulators in fixed registers), against
the oracle, and against TILE where the call is one it cannot serve.

The shapes cover what the kernel distinguishes: row tiles with many interior blocks (the fused
steps), the first block and the diagonal blocks of a causal mask (plain steps), wavefronts that
stop early under the mask, a ragged key tail, both storage types, scores that grow (references
move: a block's coefficients are formed again, and the steps after it look at the top scores first), rows that
stay empty and a negative scale (plain steps only)."""
import numpy as np
import pytest
import torch

from oracle import attention as oa
from paper_2505_14201_amd import flashd, synthetic
from tests.gpu_util import check, run_flashd

pytestmark = pytest.mark.gpu
DT = {"f16": torch.float16, "bf16": torch.bfloat16}
WIDE = flashd.VARIANT_TILE_256


def sampled(got, q, k, v, w, n_rows, seed, what, scale=None):
    rows = synthetic.sample_rows(w, n_rows, seed=seed)
    ref = oa.attn(q, k, v, w.causal, w.scale if scale is None else scale, "definition", rows)
    idx = torch.from_numpy(rows.astype(np.int64))
    sel = got[idx[:, 0], idx[:, 1], idx[:, 2], :]
    assert torch.isfinite(got).all(), what + ": non-finite output"
    check(sel, ref, DT[w.dtype], what)


#   (B, Hq, Hkv, Lq, Lk)
SHAPES = [
    (1, 2, 2, 256, 256),       # one row tile, four key tiles
    (1, 4, 2, 512, 1024),      # GQA, Lk > Lq: the causal diagonal sits in the middle of the keys
    (2, 2, 1, 768, 700),       # ragged key tail; causal rows that see few keys
    (1, 3, 3, 1024, 1000),
    (1, 1, 1, 256, 4160),      # long rows of keys: 65 tiles, the copy ring wraps many times
    (1, 2, 2, 300, 500),       # rows past the end of the last row tile: one wavefront's block, then whole wavefronts
    (2, 3, 1, 513, 1100),      # one row in the last row tile
    (1, 2, 2, 40, 2048),       # less than one wavefront of rows
]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_wide_kernel_against_the_oracle(shape, causal, dtype):
    B, Hq, Hkv, Lq, Lk = shape
    w = synthetic.small("wide", B, Hq, Hkv, Lq, Lk, 128, dtype, causal, seed=9300 + Lq + Lk)
    q, k, v, _ = synthetic.make_qkv(w)
    got = run_flashd(q, k, v, causal, w.scale, WIDE, 1)
    sampled(got, q, k, v, w, 768, 31, f"{shape} causal={causal} {dtype}")
    if causal and Lq > Lk:
        assert torch.count_nonzero(got[:, :, :Lq - Lk]) == 0, "rows without keys must be zeros"


@pytest.mark.parametrize("dtype,qk_std", [("bf16", 6.0), ("f16", 3.0), ("f16", 6.0)])
@pytest.mark.parametrize("causal", [False, True])
def test_wide_kernel_with_large_and_growing_scores(dtype, qk_std, causal):
    """Large scores: references move often (f16 above all: a coefficient may be at most 2^13),
    so many blocks are formed again and wavefronts go from looking first to not and back."""
    w = synthetic.small("wide big", 1, 2, 2, 512, 2048, 128, dtype, causal, seed=9400,
                        qk_std=qk_std, plant_frac=0.05)
    q, k, v, _ = synthetic.make_qkv(w)
    got = run_flashd(q, k, v, causal, w.scale, WIDE, 1)
    sampled(got, q, k, v, w, 512, 32, f"{dtype} std={qk_std} causal={causal}")


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_wide_kernel_staircase_of_scores(dtype):
    """Keys whose scores rise step by step along the key axis: every few blocks some row's
    reference has to move, in the middle of a run of fused steps."""
    torch.manual_seed(5)
    Lq, Lk, d = 256, 2048, 128
    q = torch.zeros(1, 1, Lq, d)
    q[..., 0] = 1.0
    q[..., 1:] = 0.05 * torch.randn(Lq, d - 1)
    k = 0.05 * torch.randn(1, 1, Lk, d)
    k[0, 0, :, 0] = torch.arange(Lk) // 96 * 9.0          # steps of 9 nats every 96 keys
    v = torch.randn(1, 1, Lk, d)
    q, k, v = (t.to(DT[dtype]) for t in (q, k, v))
    got = run_flashd(q, k, v, False, 1.0, WIDE, 1)
    ref = oa.attn(q, k, v, False, 1.0)
    check(got, ref, DT[dtype], f"staircase {dtype}")


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("level", [-40.0, -4.0, 30.0])
def test_wide_kernel_first_block_far_from_zero(dtype, causal, level):
    """The first block of a row tile takes a fused step with zero standing in for the rows'
    reference; scores that all lie far below zero (the coefficients would vanish), a little
    below (the sum falls short of the least that is trusted) or far above (they would overflow)
    must have it formed again, and rows that see only a key or two must come out right either way."""
    torch.manual_seed(17)
    Lq, Lk, d = 512, 768, 128
    q = torch.zeros(1, 2, Lq, d)
    q[..., 0] = 1.0
    q[..., 1:] = 0.1 * torch.randn(2, Lq, d - 1)
    k = 0.1 * torch.randn(1, 2, Lk, d)
    k[..., 0] = level + 0.5 * torch.randn(2, Lk)
    v = torch.randn(1, 2, Lk, d)
    q, k, v = (t.to(DT[dtype]) for t in (q, k, v))
    got = run_flashd(q, k, v, causal, 1.0, WIDE, 1)
    ref = oa.attn(q, k, v, causal, 1.0)
    check(got, ref, DT[dtype], f"first block at {level} {dtype} causal={causal}")


@pytest.mark.parametrize("scale", [-0.09, 0.0])
def test_wide_kernel_negative_and_zero_scale(scale):
    w = synthetic.small("wide scale", 1, 2, 2, 256, 600, 128, "bf16", True, seed=9500)
    q, k, v, _ = synthetic.make_qkv(w)
    got = run_flashd(q, k, v, True, scale, WIDE, 1)
    sampled(got, q, k, v, w, 256, 33, f"scale={scale}", scale=scale)


@pytest.mark.parametrize("shape,dtype,d,splits", [
    ((1, 2, 2, 256, 512), "bf16", 64, 1),      # d = 64
    ((1, 2, 2, 256, 4096), "f16", 128, 2),     # split keys
])
def test_calls_the_wide_kernel_cannot_serve_run_as_tile(shape, dtype, d, splits):
    B, Hq, Hkv, Lq, Lk = shape
    w = synthetic.small("wide fallback", B, Hq, Hkv, Lq, Lk, d, dtype, True, seed=9600 + Lq)
    q, k, v, _ = synthetic.make_qkv(w)
    a = run_flashd(q, k, v, True, w.scale, WIDE, splits)
    b = run_flashd(q, k, v, True, w.scale, flashd.VARIANT_TILE, splits)
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))


def test_wide_kernel_is_bitwise_reproducible_and_agrees_with_tile():
    w = synthetic.small("wide repro", 2, 4, 4, 512, 1536, 128, "bf16", True, seed=9700)
    q, k, v, _ = synthetic.make_qkv(w)
    a = run_flashd(q, k, v, True, w.scale, WIDE, 1)
    b = run_flashd(q, k, v, True, w.scale, WIDE, 1)
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    t = run_flashd(q, k, v, True, w.scale, flashd.VARIANT_TILE, 1)
    # two roundings of the same row to bf16: a unit in the last place of the larger one apart
    assert (a.float() - t.float()).abs().max() <= 2.0 ** -7 * max(1.0, float(t.float().abs().max()))


def test_the_automatic_choice_takes_the_wide_kernel_where_it_says_so():
    """A shape flashd_auto_variant reports as TILE_256 (a workgroup per compute unit, 2048 keys,
    no mask): flashd_attn_fwd must return the 256-row kernel's bits, and they must agree with
    the oracle; short causal rows stay with the 128-row kernel."""
    w = synthetic.small("wide auto", 1, 64, 8, 1024, 2048, 128, "bf16", False, seed=9800)
    assert flashd.auto_variant(w.B, w.Hq, w.Hkv, w.Lq, w.Lk, w.d, flashd.BF16, False) == WIDE
    q, k, v, _ = synthetic.make_qkv(w)
    auto = run_flashd(q, k, v, False, w.scale, use_ex=False)
    wide = run_flashd(q, k, v, False, w.scale, WIDE, 1)
    assert torch.equal(auto.view(torch.int16), wide.view(torch.int16))
    sampled(auto, q, k, v, w, 1024, 37, "automatic choice, 256-row kernel")
    # under a causal mask: short queries late in a longer context (rows see 1792 keys on average)
    w = synthetic.small("wide auto causal", 8, 32, 8, 512, 2048, 128, "f16", True, seed=9802)
    assert flashd.auto_variant(w.B, w.Hq, w.Hkv, w.Lq, w.Lk, w.d, flashd.F16, True) == WIDE
    q, k, v, _ = synthetic.make_qkv(w)
    auto = run_flashd(q, k, v, True, w.scale, use_ex=False)
    wide = run_flashd(q, k, v, True, w.scale, WIDE, 1)
    assert torch.equal(auto.view(torch.int16), wide.view(torch.int16))
    sampled(auto, q, k, v, w, 1024, 38, "automatic choice under a causal mask, 256-row kernel")
    w = synthetic.small("wide auto no", 1, 8, 8, 1024, 1024, 128, "bf16", True, seed=9801)
    assert flashd.auto_variant(w.B, w.Hq, w.Hkv, w.Lq, w.Lk, w.d, flashd.BF16, True) == flashd.VARIANT_TILE
    q, k, v, _ = synthetic.make_qkv(w)
    auto = run_flashd(q, k, v, True, w.scale, use_ex=False)
    tile = run_flashd(q, k, v, True, w.scale, flashd.VARIANT_TILE, 0)
    assert torch.equal(auto.view(torch.int16), tile.view(torch.int16))


# (variant, B, Hq, Hkv, Lq, Lk, d), whether row tiles run in pairs; test_row_plan.py asks the rule itself.  The compute
# units run 256 workgroups of the 256-row kernel at once, 512 of the 128-row one at d = 128 and 768 at d = 64.
HAND_OUT = [
    (WIDE, 2, 32, 32, 2200, 2200, 128, False),         # 320 pairs: 1.25 rounds
    (WIDE, 4, 32, 32, 1024, 1100, 128, True),          # 256 pairs
    (WIDE, 8, 32, 32, 700, 720, 128, True),            # 3 row tiles, the middle one by itself, ragged: 512
    (flashd.VARIANT_TILE, 2, 32, 32, 2200, 2200, 128, False),   # 576 pairs
    (flashd.VARIANT_TILE, 3, 12, 4, 4010, 4020, 128, False),    # heads of a group as one, 564 pairs
    (flashd.VARIANT_TILE, 3, 32, 32, 2200, 2250, 64, False),    # 864 pairs
    (flashd.VARIANT_TILE, 8, 32, 32, 520, 520, 64, False),      # 768 pairs, but not two rounds of row tiles
    (flashd.VARIANT_TILE, 16, 32, 32, 300, 320, 128, True),     # 3 row tiles, ragged: 1024 pairs
    (flashd.VARIANT_TILE, 32, 32, 8, 220, 230, 128, True),      # heads of a group as one, 7 row tiles: 1024
    (flashd.VARIANT_TILE, 24, 32, 32, 300, 310, 64, True),      # 3 row tiles: 1536
    (flashd.VARIANT_TILE, 8, 32, 32, 600, 610, 64, False),      # 5 row tiles: 768 pairs, 1280 row tiles
    (flashd.VARIANT_TILE, 16, 32, 32, 560, 570, 64, True),      # 5 row tiles: 1536
]


@pytest.mark.parametrize("variant,B,Hq,Hkv,Lq,Lk,d,pairs", HAND_OUT)
def test_row_tiles_in_pairs_or_one_by_one(variant, B, Hq, Hkv, Lq, Lk, d, pairs):
    """Both ways of handing out the row tiles of a causal call (rows_in_pairs), through both prefill
    kernels: every row tile, wherever it runs (the output starts as NaN)."""
    w = synthetic.small("pairs", B, Hq, Hkv, Lq, Lk, d, "bf16", True, seed=9800 + B)
    q, k, v, _ = synthetic.make_qkv(w)
    got = run_flashd(q, k, v, True, w.scale, variant, 1)
    sampled(got, q, k, v, w, 512, 39, f"B={B} Hq={Hq} Lq={Lq} d={d}")


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("kind", ["low first block", "staircase", "planted"])
def test_small_values_of_v(kind, causal):
    """V of 2^-120 where references move: a weight far below 1 on the keys that matter would take the
    products out of the range of fp32."""
    torch.manual_seed(23)
    if kind == "planted":
        w = synthetic.small("small v", 1, 2, 2, 512, 1024, 128, "bf16", causal, seed=9900, qk_std=6.0,
                            plant_frac=0.05)
        q, k, v, _ = synthetic.make_qkv(w)
        scale = w.scale
    else:
        Lq, Lk, d = 512, 1024, 128
        q = torch.zeros(1, 2, Lq, d)
        q[..., 0] = 1.0
        q[..., 1:] = 0.1 * torch.randn(2, Lq, d - 1)
        k = 0.1 * torch.randn(1, 2, Lk, d)
        k[..., 0] = -4.0 if kind == "low first block" else torch.arange(Lk) // 96 * 12.0
        v = torch.randn(1, 2, Lk, d)
        q, k, v = (t.to(torch.bfloat16) for t in (q, k, v))
        scale = 1.0
    ref = oa.attn(q, k, v, causal, scale)
    got = run_flashd(q, k, (v.float() * 2.0 ** -120).to(torch.bfloat16), causal, scale, WIDE, 1)
    check(got.double() * 2.0 ** 120, ref, torch.bfloat16, kind)


@pytest.mark.parametrize("dtype,rows", [("bf16", "all"), ("bf16", "some"), ("f16", "all")])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("later", ["ordinary, then high", "far below zero", "low, -inf, ordinary"])
@pytest.mark.parametrize("first", [32, 70])
def test_wide_kernel_rows_whose_first_keys_weigh_nothing(first, later, rows, causal, dtype):
    """Rows whose scores in the first block are all -inf are still empty where the others of their
    wavefront are not; what follows must reach them, wherever their references then lie."""
    torch.manual_seed(29)
    Lq, Lk, d = 512, 1400, 128
    q = torch.zeros(1, 2, Lq, d)
    q[..., 0] = 1.0
    q[..., 1:] = 0.1 * torch.randn(2, Lq, d - 1)
    k = 0.1 * torch.randn(1, 2, Lk, d)
    v = torch.randn(1, 2, Lk, d)
    hidden = torch.zeros(Lk, dtype=torch.bool)
    hidden[:first] = True
    if later.startswith("ordinary"):
        k[..., 700:, 0] = 300.0
    elif later.startswith("far"):
        k[..., 0] = -200.0
    else:
        k[..., first:200, 0] = -200.0
        hidden[200:400] = True
    # hidden: from the rows with a large element in column 5 (bf16: the product of two of 1e30 is infinite)
    big = 6.0e4 if dtype == "f16" else 1.0e30
    q[..., 5] = 0.0
    q[:, :, ::3 if rows == "some" else 1, 5] = big
    k[..., 5] = 0.0
    k[:, :, hidden, 5] = -big
    q, k, v = (t.to(DT[dtype]) for t in (q, k, v))
    ref = oa.attn(q, k, v, causal, 1.0)
    if dtype == "f16":
        k[:, :, hidden, 5] = float("-inf")
    got = run_flashd(q, k, v, causal, 1.0, WIDE, 1)
    check(got, ref, DT[dtype], f"{later} {rows}")


def jumps(at, Lq, Lk, dtype, seed, height=60.0):
    """Scores that rise by `height` nats at every key of `at`, for every third row only from the second
    jump on, and for the rows 64 to 127 (one wavefront's) not at all."""
    torch.manual_seed(seed)
    d = 128
    q = torch.zeros(1, 2, Lq, d)
    q[..., 0] = 1.0
    q[..., 1] = 1.0
    q[:, :, ::3, 1] = 0.0
    q[:, :, 64:128, :2] = 0.0
    q[..., 2:] = 0.1 * torch.randn(2, Lq, d - 2)
    k = 0.1 * torch.randn(1, 2, Lk, d)
    k[..., :2] = 0.0
    for i, j in enumerate(at):
        k[:, :, j:, 1 if i == 0 else 0] += height
    v = torch.randn(1, 2, Lk, d)
    return tuple(t.to(DT[dtype]) for t in (q, k, v))


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("at", [
    (704, 3520),            # both in the first block of a period; 32 periods of 64 keys in which the steps look
                            # first lie between them, and 12 in which they do not
    (740, 3570),            # both in the second
    (704, 740, 3570),       # in both blocks of a period's neighbours, then after the hand-over
    (704, 736, 768, 800),   # every block
    (704, 2750, 2784, 4830),   # in the last period that looks first, in the first that does not
])
def test_wide_kernel_between_looking_first_and_not(at, causal, dtype):
    """After a reference has moved a wavefront's steps look at the top scores first, for 32 periods; then
    they no longer do, until the next time."""
    q, k, v = jumps(at, 512, 5600, dtype, 31)
    got = run_flashd(q, k, v, causal, 1.0, WIDE, 1)
    check(got, oa.attn(q, k, v, causal, 1.0), DT[dtype], f"{at} causal={causal}")


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("at", [(700,), (700, 735, 3000)])
def test_wide_kernel_a_row_that_is_no_number(at, dtype):
    """A row of NaN makes every block of its wavefront one to be formed again; its neighbours come out right."""
    q, k, v = jumps(at, 256, 3600, dtype, 37)
    ref = oa.attn(q, k, v, False, 1.0)
    q[:, :, 5] = float("nan")
    got = run_flashd(q, k, v, False, 1.0, WIDE, 1)
    assert torch.isnan(got[:, :, 5]).all()
    keep = [i for i in range(256) if i != 5]
    check(got[:, :, keep], np.ascontiguousarray(ref[:, :, keep]), DT[dtype], f"{at}")


@pytest.mark.parametrize("dtype,height", [("f16", 8.66), ("f16", 9.4), ("f16", 6.5), ("f16", 7.1), ("bf16", 37.0),
                                          ("bf16", 41.0)])
@pytest.mark.parametrize("causal", [False, True])
def test_wide_kernel_scores_that_settle_near_the_limits(dtype, height, causal):
    """Scores that stay just below and just above what a step trusts and what moves a reference (fp16 10
    and 14 powers of two above it, bf16 54 and 60)."""
    q, k, v = jumps((100,), 512, 1500, dtype, 41, height)
    got = run_flashd(q, k, v, causal, 1.0, WIDE, 1)
    check(got, oa.attn(q, k, v, causal, 1.0), DT[dtype], f"height={height}")
