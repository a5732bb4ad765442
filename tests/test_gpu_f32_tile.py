"""The fp32 tile kernel (what the automatic choice runs for fp32) at the edges of its row tiles
(16 rows, heads of a kv group interleaved), its 16-key blocks and its wavefronts' turns (64
keys).  Tolerance: that of the fp32 path (gpu_util.F32_REL)."""
import numpy as np
import pytest
import torch

from oracle import attention as oa
from paper_2505_14201_amd import flashd, synthetic
from tests.gpu_util import check, run_flashd
from tests.test_gpu_state import check_state, run_chunks

pytestmark = pytest.mark.gpu
AUTO, PER_KEY = flashd.VARIANT_AUTO, flashd.VARIANT_PER_KEY


@pytest.mark.parametrize("B,Hq,Hkv,Lq,Lk", [
    (1, 1, 1, 1, 1), (1, 1, 1, 15, 17), (2, 2, 2, 16, 16), (1, 3, 3, 17, 63),
    (1, 6, 2, 5, 65),         # 15 interleaved rows
    (2, 8, 2, 4, 64),         # exactly one row tile of 4 heads
    (1, 10, 2, 7, 129),       # 35 rows, 5 heads: tiles begin in the middle of a position
    (8, 1, 1, 33, 80),        # 8 units: dealt over the XCDs
    (1, 4, 4, 40, 9),         # rows that see no key
])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("splits", [1, 3])
def test_edges(B, Hq, Hkv, Lq, Lk, causal, splits):
    if splits > Lk:
        pytest.skip("more splits than keys")
    for d in (64, 128):
        w = synthetic.small("t", B, Hq, Hkv, Lq, Lk, d, "f32", causal, seed=9100 + Lq * 7 + Lk + d)
        q, k, v, _ = synthetic.make_qkv(w)
        got = run_flashd(q, k, v, causal, w.scale, AUTO, splits)
        check(got, oa.attn(q, k, v, causal, w.scale), torch.float32, f"d={d}")


@pytest.mark.parametrize("std,scale", [(4.0, None), (30.0, None), (4.0, -0.5), (1.0, 0.0)])
def test_moving_references(std, scale):
    """Scores that keep climbing past the reference, fall below it for good, or are all alike."""
    w = synthetic.small("t", 1, 4, 2, 50, 700, 64, "f32", True, seed=9300, qk_std=std)
    q, k, v, _ = synthetic.make_qkv(w)
    k = k * torch.linspace(0.1, 1.0, 700).view(1, 1, -1, 1)
    scale = w.scale if scale is None else scale
    check(run_flashd(q, k, v, True, scale, AUTO, 1), oa.attn(q, k, v, True, scale), torch.float32)


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_hidden_values_do_not_reach_a_row(bad):
    """A value that is infinite or NaN stays out of the rows its key is hidden from, as in the
    per-key kernel, and reaches every row that sees it."""
    w = synthetic.small("t", 1, 2, 1, 40, 40, 64, "f32", True, seed=9400)
    q, k, v, _ = synthetic.make_qkv(w)
    v[0, 0, 37, 5] = bad
    got = run_flashd(q, k, v, True, w.scale, AUTO, 1)
    lit = run_flashd(q, k, v, True, w.scale, PER_KEY, 1)
    assert torch.isfinite(got[:, :, :37]).all()
    assert not torch.isfinite(got[:, :, 37:, 5]).any()
    assert torch.equal(torch.isfinite(got), torch.isfinite(lit))
    clean = v.clone()
    clean[0, 0, 37, 5] = 0.0
    ref = oa.attn(q, k, clean, True, w.scale)
    check(got[:, :, :37], np.ascontiguousarray(ref[:, :, :37]), torch.float32)


@pytest.mark.parametrize("hidden", [range(0, 64), range(40, 200),
                                    [j for j in range(300) if j // 16 % 4 == 1]])
@pytest.mark.parametrize("splits", [1, 2])
def test_keys_of_score_minus_infinity(hidden, splits):
    """Keys whose scores are -inf weigh nothing, also where a wavefront meets them first or meets
    no others (the last range: all blocks of wavefront 1)."""
    for d in (64, 128):
        w = synthetic.small("t", 1, 4, 2, 9, 300, d, "f32", False, seed=9450)
        q, k, v, _ = synthetic.make_qkv(w)
        q[..., 5] = q[..., 5].abs() + 0.1
        left = [j for j in range(300) if j not in set(hidden)]
        ref = oa.attn(q, k[:, :, left].contiguous(), v[:, :, left].contiguous(), False, w.scale)
        k[:, :, list(hidden), 5] = float("-inf")
        check(run_flashd(q, k, v, False, w.scale, AUTO, splits), ref, torch.float32, f"d={d}")


@pytest.mark.parametrize("sign", [False, True])
@pytest.mark.parametrize("splits", [1, 3])
def test_large_values(splits, sign):
    """Values up to 1e38 on hundreds of keys: sums of unnormalised weights overflow, the output
    does not.  The second kv head holds ordinary values."""
    for d in (64, 128):
        w = synthetic.small("t", 1, 4, 2, 30, 700, d, "f32", True, seed=9500 + d)
        q, k, v, _ = synthetic.make_qkv(w)
        big = 2e37 * (1.0 + v[:, :1].abs().clamp(max=4.0))
        v[:, :1] = torch.where(v[:, :1] < 0, -big, big) if sign else big
        got = run_flashd(q, k, v, True, w.scale, AUTO, splits)
        ref = oa.attn(q, k, v, True, w.scale)
        for h in range(4):
            check(got[:, h:h + 1], np.ascontiguousarray(ref[:, h:h + 1]), torch.float32, f"d={d} h={h}")


@pytest.mark.parametrize("Lk", [319, 321, 383, 385, 705, 770, 1100])
@pytest.mark.parametrize("d", [64, 128])
def test_sums_that_join_in_fp64(Lk, d):
    """A wavefront's sums join those in fp64 after every 6 blocks (384 keys of a row): key counts
    around that, values of mean 1, references that move in between, and the state."""
    w = synthetic.small("t", 1, 4, 2, 21, Lk, d, "f32", True, seed=9600 + Lk, qk_std=2.0)
    q, k, v, _ = synthetic.make_qkv(w)
    k = k * torch.linspace(0.1, 2.0, Lk).view(1, 1, -1, 1)
    v = v + 1.0
    for splits in (1, 2):
        check(run_flashd(q, k, v, True, w.scale, AUTO, splits), oa.attn(q, k, v, True, w.scale),
              torch.float32, f"splits={splits}")
    o, st = run_chunks(q, k, v, True, w.scale, (Lk // 2,), in_place=True)
    check(o, oa.attn(q, k, v, True, w.scale), torch.float32)
    check_state(st, oa.attn_state(q, k, v, True, w.scale), d, torch.float32, "state")


def test_long_sums_lose_nothing():
    """300000 keys of equal score, in one range: sums in fp32 would round the same way at every key
    (2e-4 of the result).  The weights are all 1, so what is left is the rounding of chains of 6
    blocks (96 additions of 2^-24 each, at most 6e-6) and of the output."""
    q = torch.zeros(1, 1, 16, 64)
    gen = torch.Generator().manual_seed(9650)
    k = torch.randn(1, 1, 300000, 64, generator=gen)
    v = 0.7 + 7e-4 * torch.randn(1, 1, 300000, 64, generator=gen)
    got = run_flashd(q, k, v, False, 0.125, AUTO, 1)
    ref = v.double().mean(2, keepdim=True)
    err = ((got.double() - ref).abs() / ref.abs()).max().item()
    assert err <= 6.5e-6, err


@pytest.mark.parametrize("kind", ["normal", "far apart", "zero keys", "large", "small", "positive", "huge scores",
                                  "infinite key"])
@pytest.mark.parametrize("B,H,Lq,Lk,d", [
    (1, 1, 20, 128, 128), (1, 1, 17, 129, 128), (1, 2, 100, 700, 128),     # fp64 up to 128 keys, sliced beyond
    (2, 12, 170, 160, 64), (2, 12, 170, 161, 64), (2, 12, 176, 333, 64),   # sliced from 161 keys on
])
@pytest.mark.parametrize("causal", [False, True])
def test_sliced_scores(kind, B, H, Lq, Lk, d, causal):
    """Scores from fp16 slices of Q and K, and the blocks that go through fp64 beside them: keys whose
    sizes lie far apart within a block, exponents beyond the sliced range, an infinite key.  On both
    sides of the rule that chooses them."""
    w = synthetic.small("t", B, H, H, Lq, Lk, d, "f32", causal, seed=9700 + Lk + Lq)
    q, k, v, _ = synthetic.make_qkv(w)
    scale = w.scale
    if kind == "far apart":
        k = k * torch.pow(2.0, -(torch.arange(Lk) * 7 % 23).float()).view(1, 1, -1, 1)
        q[:, :, ::3] *= 2.0 ** -40
    elif kind == "zero keys":
        k[:, :, 5::7] = 0.0
        q[:, :, 4::9] = 0.0
    elif kind in ("large", "small"):
        # exponents of Q or of K beyond those that are sliced; the other and the scale undo them
        e = 110 if kind == "large" else -110
        eq, ek = (e, -e // 5) if causal else (-e // 5, e)
        q, k, scale = q * 2.0 ** eq, k * 2.0 ** ek, scale * 2.0 ** -(eq + ek)
    elif kind == "positive":
        q, k = 1.0 + q.abs().clamp(max=0.99), 1.0 + k.abs().clamp(max=0.99)
    elif kind == "huge scores":
        q, k = q * 8.0, k * 8.0
    ref_k, ref_v = k, v
    if kind == "infinite key":
        if causal:
            pytest.skip("the keys left out below would move the mask")
        q[..., 3] = q[..., 3].abs() + 0.5
        left = [j for j in range(Lk) if j % 37 != 11]
        ref_k, ref_v = k[:, :, left].contiguous(), v[:, :, left].contiguous()
        k[:, :, 11::37, 3] = float("-inf")
    check(run_flashd(q, k, v, causal, scale, AUTO, 0), oa.attn(q, ref_k, ref_v, causal, scale), torch.float32, kind)


@pytest.mark.parametrize("e", [5, 8, 12, 16, 20, 24, 30, 60])
@pytest.mark.parametrize("kind", ["K column, Q zero", "K column, Q small", "Q column, K zero", "Q column, K small",
                                  "one key", "crossed"])
@pytest.mark.parametrize("B,H,Lq,Lk,d", [(2, 12, 176, 333, 64), (1, 2, 100, 700, 128)])
def test_large_elements(kind, e, B, H, Lq, Lk, d):
    """Elements of 2^e in rows that otherwise hold ordinary ones, with little or nothing on the other
    side, so that the scores are ordinary too: what the slices of such a row keep of its other elements
    is not enough."""
    w = synthetic.small("t", B, H, H, Lq, Lk, d, "f32", True, seed=9900 + e)
    q, k, v, _ = synthetic.make_qkv(w)
    big, small = 2.0 ** e, 2.0 ** -e
    if kind.startswith("K"):
        k[..., 5] *= big
        q[..., 5] *= 0.0 if kind.endswith("zero") else small
    elif kind.startswith("Q"):
        q[..., 5] *= big
        k[..., 5] *= 0.0 if kind.endswith("zero") else small
    elif kind == "one key":
        k[:, :, Lk // 3, 7] = big
        q[..., 7] *= small
    else:
        q[..., 3] *= big
        k[..., 3] *= small
        k[..., 9] *= big
        q[..., 9] *= small
    same_as_fp64_scores(q, k, v, True, w.scale)


@pytest.mark.parametrize("kind", ["std 4", "std 30", "std 1000", "near ties", "large scale", "offset"])
@pytest.mark.parametrize("B,H,Lq,Lk,d", [(2, 12, 176, 333, 64), (1, 2, 100, 700, 128)])
def test_large_scores(kind, B, H, Lq, Lk, d):
    """Scores far from zero, and keys that differ by little at scores of ten thousand and more; the
    bound is that of ordinary scores."""
    w = synthetic.small("t", B, H, H, Lq, Lk, d, "f32", True, seed=9950 + d)
    q, k, v, _ = synthetic.make_qkv(w)
    scale = w.scale
    if kind.startswith("std"):
        q, k = q * float(kind[4:]), k * float(kind[4:])
    elif kind == "near ties":
        q = q * 64.0
        k = k[:, :, :1] * 64.0 + k * 2.0 ** -6
    elif kind == "large scale":
        scale = 40.0
    else:
        k[..., 11] += 1024.0
    same_as_fp64_scores(q, k, v, True, scale)


def same_as_fp64_scores(q, k, v, causal, scale):
    """Scores in fp64, weights and short sums in fp32: 2e-7 of the output, 2-norm, on ordinary inputs, and
    less where few keys weigh.  The bound is twice that."""
    got = run_flashd(q, k, v, causal, scale, AUTO, 0)
    ref = oa.attn(q, k, v, causal, scale)
    check(got, ref, torch.float32)
    err = np.linalg.norm(got.double().numpy() - ref) / np.linalg.norm(ref)
    assert err <= 4e-7, err
