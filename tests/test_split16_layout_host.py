"""Host check of the N = 2^16 column launch's layouts (csrc/ntt.hip): slot16, the
LDS slot of a tile of 4 columns x 256 rows, is a bijection with 32 distinct
8-byte banks per half-wave in both layouts, and the row passes' tile order
(mid_row) covers a limb, with each row of a tile where the column launch's second
layout reads it.  The formulas are restated from the kernel source, which the
test reads to make sure of them."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def slot16(e):
    return e ^ (((e >> 6) & 7) << 2)


def layout_a(lane, i):  # rows lane / 4 + 16 i
    return lane + 64 * i


def layout_b(lane, i):  # rows 16 (lane / 4) + i
    return 64 * (lane >> 2) + 4 * i + (lane & 3)


def test_slot16_is_a_conflict_free_bijection():
    assert sorted(slot16(e) for e in range(1024)) == list(range(1024))
    for f in (layout_a, layout_b):
        assert sorted(f(lane, i) for lane in range(64) for i in range(16)) == list(range(1024))
        for i in range(16):
            for t0 in (0, 32):
                assert len({slot16(f(lane, i)) % 32 for lane in range(t0, t0 + 32)}) == 32, (f, i)


def mid(b, s):  # row b, column s of a tiled limb
    return (s >> 2) * 1024 + (b & 15) * 64 + (b >> 4) * 4 + (s & 3)


def test_tile_order():
    assert sorted(mid(b, s) for b in range(256) for s in range(256)) == list(range(65536))
    for lane in range(64):
        for i in range(16):
            e = layout_b(lane, i)  # row e / 4, column e % 4 of the tile, at 64 i + lane
            assert mid(e >> 2, e & 3) == 64 * i + lane
    for step in (32, 64):  # columns s + step k of a row are step 256 words apart
        assert all(mid(b, s + step) - mid(b, s) == 256 * step for b in (0, 37, 255) for s in range(256 - step))


def test_pass_row_covers_the_rows():
    for tw in (4, 8, 16):
        g = 16 // tw
        rows = [16 * ((tile % g) * tw + blk) + tile // g for tile in range(256 // tw) for blk in range(tw)]
        assert sorted(rows) == list(range(256))


def test_formulas_match_the_kernel_source():
    src = re.sub(r"\s+", " ", open(os.path.join(ROOT, "paper_2507_04775_amd", "csrc", "ntt.hip")).read())
    assert "return e ^ (((e >> 6) & 7) << 2); }" in src
    assert "(s >> 2) * 1024 + (b & 15) * 64 + (b >> 4) * 4 + (s & 3) : b * 256 + s);" in src
    assert "ip.ext + off + (s >> 2) * 1024 + (b & 15) * 64 + (b >> 4) * 4 + (s & 3);" in src
    assert "a.tiled ? 16 * ((tile % G) * TW + blk) + tile / G : tile * TW + blk;" in src
    assert "b = 16 * (blockIdx.x % groups * kIpRows + w) + blockIdx.x / groups;" in src
    assert src.count("L[slot16(64 * s + 4 * i + col)]") == 2 and src.count("L[slot16(lane + 64 * i)]") == 2
