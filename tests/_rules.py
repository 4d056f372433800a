"""The rules of csrc/pass_rules.hpp and csrc/tall_tiles.hpp, built with the
host compiler."""

import ctypes
import functools
import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2511_11505_amd", "csrc")
R64, STREAM, RING, R192, SKINNY, STAGED, RING128 = range(7)
CUS = 256   # of gfx950


@functools.lru_cache(maxsize=None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "rules.so")
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, "-o", so,
                        os.path.join(HERE, "pass_rules_shim.cpp")], check=True)
        lib = ctypes.CDLL(so)
    i, q = ctypes.c_int, ctypes.c_longlong
    lib.rule_pass.argtypes = [i, i, q, q, i, i, i, i]
    lib.rule_pass_fp8.argtypes = [i, q, i, i, i, i]
    lib.rule_dense.argtypes = [i] * 5
    lib.rule_height.argtypes = [q, i, i, i, i]
    lib.tall_height.argtypes = [i] * 6
    lib.tall_rows.argtypes = [i] * 3
    return lib


def pass_kind(gateup, rows, G, ffn, d, dtype="bf16", likely=None, cus=CUS):
    return _lib().rule_pass(int(dtype == "bf16"), int(gateup), rows, rows if likely is None else likely,
                            G, ffn, d, cus)


def pass_kind_fp8(gateup, rows, G, ffn, d, cus=CUS):
    return _lib().rule_pass_fp8(int(gateup), rows, G, ffn, d, cus)


def dense_kind(m, n, kdim, dtype="bf16", cus=CUS):
    return _lib().rule_dense(int(dtype == "bf16"), m, n, kdim, cus)


def tall_height(counts, n_cols, gateup, fp8=False, cus=CUS):
    """Largest tile height of a pass of n_cols output columns over groups of
    `counts` rows: the host's choice, or the 192-row kernel's."""
    nn = n_cols // (128 if gateup else 256)
    h = _lib().rule_height(sum(counts), len(counts), nn, cus, 64 if fp8 else 32)
    if h:
        return h
    t = [0 if fp8 and h == 160 else sum(-(-n // h) for n in counts) for h in (192, 160, 128)]
    wgs = min(-(-(-(-sum(counts) // 128) + len(counts)) * nn // 8), -(-cus // 8)) * 8
    return _lib().tall_height(sum(counts), *t, nn, wgs)


def tall_rows(rows, tiles, unit):
    return _lib().tall_rows(rows, tiles, unit)


def tall_order(tiles, nn):
    a = (ctypes.c_int * (tiles * nn))()
    b = (ctypes.c_int * (tiles * nn))()
    _lib().tall_order(tiles, nn, a, b)
    return list(zip(a, b))
