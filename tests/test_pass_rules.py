"""The dispatch and tile rules of the GEMM passes, on the host: every kernel gets
only widths that its tiles divide, over all sizes that the entry points accept;
the 192-row kernel's tiles cover every group; and the routes of the shapes that
lines of the rules were drawn by."""

import random

import pytest

from tests import _rules as R


def sizes(seed, n):
    rng = random.Random(seed)
    for _ in range(n):
        yield (max(1, int(2 ** rng.uniform(0, 17))), rng.choice((1, 1, 2, 8, 16, 20, 64, 96, 512)),
               64 * rng.randint(1, 130), 128 * rng.randint(1, 64), rng.choice((256, 304, 64)))


@pytest.mark.parametrize("gateup", [True, False])
def test_pass_kernels_take_their_widths(gateup):
    for rows, G, ffn, d, cus in sizes(1, 20000):
        K, n = (d, ffn) if gateup else (ffn, d)
        assert R.pass_kind(gateup, rows, G, ffn, d, dtype="f32", cus=cus) == R.R64
        kind = R.pass_kind(gateup, rows, G, ffn, d, likely=random.Random(rows).randint(1, rows), cus=cus)
        if kind == R.R64:
            assert n % (32 if gateup else 64) == 0 and K % 64 == 0
        elif kind == R.STREAM:
            assert rows <= min(64 * G, 4096) and n % 64 == 0 and K % 64 == 0
        elif kind == R.RING:
            assert n % (128 if gateup else 256) == 0 and K % 64 == 0
        elif kind == R.RING128:
            assert not gateup and n % 128 == 0 and K % 64 == 0
        elif kind == R.STAGED:
            assert n % (64 if gateup else 128) == 0 and K % 64 == 0
        elif kind == R.SKINNY:
            assert not gateup and G == 1 and rows <= 64 and K % 512 == 0 and n % 32 == 0
        else:
            assert kind == R.R192 and n % (128 if gateup else 256) == 0 and K % 64 == 0 and K >= 256
        if ffn % 128 == 0 and d % 256 == 0:
            kind = R.pass_kind_fp8(gateup, rows, G, ffn, d, cus=cus)
            assert kind == R.RING or (kind == R.R192 and K >= 512)


def test_dense_kernels_take_their_widths():
    for m, _, kdim, n, cus in sizes(2, 20000):
        kind = R.dense_kind(m, n, kdim, cus=cus)
        assert kind in (R.R64, R.RING128) or (n % 256 == 0 and (kind == R.RING or kind == R.R192 and kdim >= 256))
        assert R.dense_kind(m, n - 64 or 64, kdim, dtype="f32", cus=cus) == R.R64


@pytest.mark.parametrize("unit", [32, 64])
@pytest.mark.parametrize("hmax", [128, 160, 192])
def test_tall_tiles_cover_a_group(hmax, unit):
    """Equal heights cover a group: no tile is empty or taller than allowed."""
    if hmax % unit:
        return
    for rows in list(range(1, 3000)) + [59999, 60000]:
        t = -(-rows // hmax)
        h = R.tall_rows(rows, t, unit)
        assert h % unit == 0 and h <= hmax and (t - 1) * h < rows <= t * h


def test_tall_order_visits_every_tile_in_bands():
    for tiles in list(range(1, 40)) + [63, 64, 65]:
        for nn in (1, 3, 11):
            at = R.tall_order(tiles, nn)
            assert sorted(at) == [(m, n) for m in range(tiles) for n in range(nn)]
            # a band of at most 8 m-tiles is finished before the next begins
            for i in range(0, tiles * nn, 8 * nn):
                assert len({m for m, _ in at[i:i + nn]}) <= 8


# the height whose rounds of tiles over the CUs are shortest
@pytest.mark.parametrize("counts,n_cols,gateup,fp8,want", [
    ([180] * 12 + [200] * 4, 3840, False, False, 160),
    ([370] * 8 + [100], 2048, True, False, 160),
    ([300] * 8 + [50], 2048, True, False, 128),   # 17 m-tiles of 192 make 272 tiles, two rounds
    ([300] * 8 + [50], 2048, True, True, 128),
    ([300] * 8, 2048, True, False, 192),          # 256 tiles, one round
    ([150] * 32, 2048, True, False, 192),
    ([384] * 64, 1408, True, False, 192)])
def test_tall_height_of_a_pass(counts, n_cols, gateup, fp8, want):
    assert R.tall_height(counts, n_cols, gateup, fp8) == want


# one dense group on both sides of each line, named by (rows, d, F)
@pytest.mark.parametrize("gateup,rows,d,F,kind", [
    (True, 700, 2048, 2816, R.R64), (True, 1000, 2048, 2816, R.RING),      # 484 and 704 tiles of 64 rows
    (False, 640, 5120, 384, R.R64), (False, 1000, 5120, 384, R.RING),
    (False, 1, 7168, 2048, R.SKINNY), (False, 33, 7168, 2048, R.R64),
    (False, 8, 5120, 8192, R.SKINNY), (False, 50, 1024, 512, R.SKINNY),
    (True, 1, 3072, 1536, R.STREAM), (True, 33, 3072, 1536, R.R64),
    (True, 1, 2048, 2816, R.R64), (True, 64, 7168, 2048, R.STREAM), (True, 64, 5120, 8192, R.R64),
    (False, 1, 2048, 2816, R.STREAM),
    (False, 4096, 3072, 1536, R.RING), (True, 4096, 3072, 1536, R.RING),   # 384 tiles, 128 rows high
    (True, 1000, 5120, 8192, R.RING), (True, 2048, 5120, 8192, R.R192),
    (True, 1400, 5120, 8192, R.R192)])
def test_dense_group_routes(gateup, rows, d, F, kind):
    assert R.pass_kind(gateup, rows, 1, F, d) == kind


@pytest.mark.parametrize("m,n,k,kind", [
    (640, 5120, 640, R.R64), (800, 5120, 640, R.RING), (1300, 5120, 640, R.RING),
    (1300, 5120, 384, R.RING), (1700, 5120, 640, R.R192), (2400, 2048, 2048, R.RING),
    (1300, 4096, 3072, R.RING), (4096, 3072, 3072, R.RING), (1700, 1152, 1024, R.R64), (2000, 1152, 1024, R.RING128)])
def test_dense_linear_routes(m, n, k, kind):
    assert R.dense_kind(m, n, k) == kind


# columns that the 256-wide tiles do not divide, of this pass or of the other:
# (rows, groups, d, F), gate/up and down
@pytest.mark.parametrize("rows,G,d,F,gu,dn", [
    (24 * 108, 24, 1408, 960, R.STAGED, R.R64), (64 * 300, 64, 1664, 2496, R.STAGED, R.RING128),
    (16 * 180, 16, 640, 1472, R.STAGED, R.R64), (64 * 4, 64, 1664, 2496, R.R64, R.R64),
    (64 * 130, 64, 2944, 1408, R.R192, R.RING128), (64 * 90, 64, 2944, 1408, R.RING, R.RING128),
    (2743, 24, 2304, 1088, R.R64, R.RING128), (40 * 2, 40, 896, 1024, R.R64, R.R64),
    (64 * 130, 64, 2048, 960, R.STAGED, R.R192), (16 * 48, 16, 2048, 960, R.STREAM, R.STREAM),
    (333, 1, 1408, 704, R.R64, R.R64), (3000, 1, 1664, 2496, R.STAGED, R.STAGED),
    (700, 1, 4480, 1536, R.R64, R.RING128), (3000, 1, 4480, 1536, R.R192, R.RING128)])
def test_odd_width_routes(rows, G, d, F, gu, dn):
    assert (R.pass_kind(True, rows, G, F, d), R.pass_kind(False, rows, G, F, d)) == (gu, dn)


@pytest.mark.parametrize("per,G,d,F,gu,dn", [
    (12, 64, 2048, 1408, R.R64, R.RING), (40, 64, 2048, 1408, R.R64, R.RING), (41, 64, 2048, 1408, R.RING, R.RING),
    (24, 60, 2560, 1408, R.RING, R.RING), (24, 128, 512, 384, R.R64, R.R64), (36, 128, 512, 384, R.R64, R.RING),
    (4, 24, 1280, 2560, R.R64, R.RING), (24, 24, 1280, 2560, R.R64, R.R64), (16, 32, 7168, 2048, R.RING, R.RING),
    (12, 32, 1024, 4096, R.R64, R.RING)])
def test_short_group_routes(per, G, d, F, gu, dn):
    assert (R.pass_kind(True, per * G, G, F, d), R.pass_kind(False, per * G, G, F, d)) == (gu, dn)
