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
