"""The dispatch rules of the GEMM passes, on the host: every kernel gets only
widths that its tiles divide, over all sizes that the entry points accept."""

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
        else:
            assert kind == R.R192 and n % (128 if gateup else 256) == 0 and K % 64 == 0 and K >= 256
        if ffn % 128 == 0 and d % 256 == 0:
            kind = R.pass_kind_fp8(gateup, rows, G, ffn, d, cus=cus)
            assert kind == R.RING or (kind == R.R192 and K >= 512)


def test_dense_kernels_take_their_widths():
    for m, _, kdim, n, cus in sizes(2, 20000):
        kind = R.dense_kind(m, n, kdim, cus=cus)
        assert kind in (R.R64, R.RING) or (kind == R.R192 and n % 256 == 0 and kdim >= 256)
        assert R.dense_kind(m, n - 64 or 64, kdim, dtype="f32", cus=cus) == R.R64
