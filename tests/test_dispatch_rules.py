"""What the automatic choice answers at the edges of its rules (host-only)."""
import pytest

from paper_2505_14201_amd import flashd

T, W = flashd.VARIANT_TILE, flashd.VARIANT_TILE_256


@pytest.mark.parametrize("B,Hq,Hkv,Lq,Lk,causal,want", [
    # 256-row tiles that are mostly padding go to the 128-row kernel: 4 heads of 16 rows are
    # half of one 128-row tile there and four 256-row tiles otherwise
    (64, 32, 8, 16, 8192, True, T),
    (64, 32, 8, 16, 8192, False, T),
    (32, 32, 32, 128, 4096, False, T),       # 256 rows against 128
    (32, 32, 32, 129, 4096, False, W),       # 256 against 256
    (32, 32, 32, 384, 4096, True, W),        # 512 against 384: the line itself
    (32, 32, 8, 300, 4096, True, T),         # 4 x 512 against 10 x 128
    (32, 32, 8, 256, 4096, True, W),
])
def test_padded_256_row_tiles(B, Hq, Hkv, Lq, Lk, causal, want):
    assert flashd.auto_variant(B, Hq, Hkv, Lq, Lk, 128, flashd.BF16, causal) == want


@pytest.mark.parametrize("B,Hq,Hkv,Lq,Lk,causal,want", [
    # the estimate: a last round of 256-row tiles that is nearly empty goes to the 128-row kernel
    (3, 8, 8, 2642, 2642, False, T), (3, 8, 8, 4096, 4096, False, W), (8, 8, 8, 2048, 2048, False, W),
    (11, 8, 1, 2176, 2176, False, T),
    # under a causal mask row tiles even out one by one
    (2, 12, 12, 5568, 5568, True, W), (1, 32, 8, 4599, 10897, True, W), (1, 16, 2, 10240, 10240, True, W),
])
def test_rounds_of_256_row_tiles(B, Hq, Hkv, Lq, Lk, causal, want):
    assert flashd.auto_variant(B, Hq, Hkv, Lq, Lk, 128, flashd.BF16, causal) == want


@pytest.mark.parametrize("B,Hq,Hkv,Lq,Lk,d,want", [
    (1, 32, 8, 1, 640, 128, 1), (1, 32, 8, 1, 641, 128, 5),     # 20 and 21 blocks of 32 keys
    (1, 32, 8, 1, 1280, 64, 1),
    (6, 32, 8, 1, 4000, 128, 4),             # 48 units: one workgroup on 192 compute units
    (20, 32, 8, 1, 4000, 128, 1),            # 160 units stay whole
    (16, 32, 8, 1, 1500, 128, 1), (16, 32, 8, 1, 8000, 128, 2),
    (40, 32, 8, 1, 4000, 128, 2), (48, 32, 8, 1, 4000, 128, 1),
    (1, 32, 8, 1, 131072, 128, 24),
    (1, 32, 1, 1, 256, 128, 1), (1, 32, 1, 1, 512, 128, 8),     # 32 rows: the wider kernel
    (1, 32, 1, 1, 511, 128, 1), (3, 24, 1, 1, 300, 128, 1),     # below 512 keys: no scratch memory
])
def test_decode_splits(B, Hq, Hkv, Lq, Lk, d, want):
    assert flashd.auto_splits(B, Hq, Hkv, Lq, Lk, d, flashd.BF16) == want


@pytest.mark.parametrize("units,rows,Lk,d,want", [
    (96, 4, 8000, 128, 2), (97, 4, 8000, 128, 2), (127, 4, 8000, 128, 2), (128, 4, 8000, 128, 2),
    (129, 4, 8000, 128, 1), (97, 4, 2016, 128, 1), (97, 4, 2017, 128, 2),
    (160, 4, 8000, 64, 3), (171, 4, 8000, 64, 1), (256, 4, 8000, 64, 1), (257, 4, 8000, 64, 2),
    (341, 4, 8000, 64, 2), (342, 4, 8000, 64, 1),
    # 17 to 32 rows, d = 64: two workgroups per compute unit; d = 128: one
    (64, 32, 20000, 64, 8), (128, 32, 1500, 64, 4), (256, 32, 20000, 64, 2), (257, 32, 20000, 64, 1),
    (64, 17, 20000, 128, 4), (128, 32, 20000, 128, 2), (170, 32, 20000, 128, 3), (171, 32, 20000, 128, 1),
    (511, 32, 20000, 64, 1), (512, 4, 20000, 128, 1),
    # 9 to 12 splits only of long ranges
    (24, 4, 10208, 64, 8), (24, 4, 10209, 64, 10),
])
def test_decode_splits_by_what_a_workgroup_streams(units, rows, Lk, d, want):
    assert flashd.auto_splits(units, rows, 1, 1, Lk, d, flashd.BF16) == want


@pytest.mark.parametrize("dtype", [flashd.BF16, flashd.F32])
@pytest.mark.parametrize("Hq,Hkv,Lq", [(32, 8, 1), (8, 1, 4), (32, 1, 1), (4, 4, 1), (12, 12, 3), (8, 2, 40)])
@pytest.mark.parametrize("d", [64, 128])
def test_scratch_memory_never_falls_with_more_keys(Hq, Hkv, Lq, d, dtype):
    """Scratch taken at the longest context serves every shorter one, and a problem that needs
    none has no shorter one that does."""
    lengths = sorted({int(1.1 ** i) + 1 for i in range(145)} | {511, 512, 2047 * 32, 2047 * 32 + 1})
    for B in (1, 2, 3, 4, 5, 8, 13, 16, 33, 64):
        at = [flashd.workspace_bytes(B, Hq, Hkv, Lq, Lk, d, dtype) for Lk in lengths]
        assert at == sorted(at), B
        for Lk, have in zip(lengths, at):
            sp = flashd.auto_splits(B, Hq, Hkv, Lq, Lk, d, dtype)
            assert have >= flashd.workspace_bytes(B, Hq, Hkv, Lq, Lk, d, dtype, splits=sp)
            assert (have == 0) == (sp == 1)
