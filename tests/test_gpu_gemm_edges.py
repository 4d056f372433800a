"""GPU parity of the grouped FFN and the dense linear at the edges of their
tiles and dispatch rules: row counts around fragment and tile heights, empty
groups, widths that leave a part tile, gathered and in-order rows; element by
element against the oracle.  fp32 results differ from the 64-bit oracle by
sums of at most 2048 rounded products (about sqrt(2048) 2^-24 = 3e-6 of the
rms); bf16 ones by the rounding of H and of the output."""

import numpy as np
import pytest
import torch

import oracle
from paper_2511_11505_amd import _lib as L
from paper_2511_11505_amd.block import fragment_ordered_fp8
from tests import _rules as R
from tests._util import TOL, f64, rel_err
from workloads import CONFIGS

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]
DEV = "cuda"
TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}


def ffn_case(dtype, counts, d, F, gather, seed=0):
    """Inputs of a grouped FFN: (X, rows or None, goff, wgu, wd, n_src)."""
    counts = np.array(counts)
    G, M = len(counts), int(counts.sum())
    goff = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    gen = torch.Generator(device=DEV).manual_seed(seed + d + 3 * F + G)
    n_src = M + 5
    X = torch.randn((n_src, d), generator=gen, device=DEV).to(TORCH[dtype])
    wgu = (0.05 * torch.randn((G, 2 * F, d), generator=gen, device=DEV)).to(TORCH[dtype])
    wd = (0.05 * torch.randn((G, d, F), generator=gen, device=DEV)).to(TORCH[dtype])
    rows = torch.randperm(n_src, generator=gen, device=DEV)[:M].to(torch.int32) if gather else None
    return X, rows, goff, wgu, wd, n_src


def check_ffn(dtype, X, rows, goff, wgu, wd, out):
    G, M = len(goff) - 1, int(goff[-1])
    rr = rows.cpu().numpy() if rows is not None else np.arange(M)
    Xn, outn = f64(X), f64(out)
    for gi in range(G):
        sel = rr[goff[gi]:goff[gi + 1]]
        if len(sel):
            want = oracle.swiglu(Xn[sel], f64(wgu[gi]), f64(wd[gi]))
            assert rel_err(outn[sel], want) <= TOL[dtype], f"group {gi} of {len(sel)} rows"
    assert np.all(np.isnan(outn[np.setdiff1d(np.arange(X.shape[0]), rr)]))


EDGES = [1, 15, 16, 17, 0, 32, 33, 48, 49, 63, 64, 65, 80, 0, 127, 130]


# fp32: 64-row tiles of 64 weight rows (few tiles) and of 128 (at least two
# tiles per CU, counted from the row bound), K of one part to many blocks
# bf16: widths only these tiles take (K % 128 = 64 among them), short groups
# and one dense group at widths the 128-row ring takes too, and the long-K
# rule's row and tile counts
@pytest.mark.parametrize("dtype,counts,d,F,gather,slack", [
    ("f32", EDGES, 128, 64, True, 0), ("f32", EDGES, 384, 192, False, 9),
    ("f32", EDGES * 3, 1792, 832, True, 0), ("f32", [70], 2048, 64, False, 0),
    ("bf16", EDGES, 128, 64, True, 0), ("bf16", EDGES, 384, 192, True, 9),
    ("bf16", EDGES * 3, 1792, 832, False, 0), ("bf16", EDGES * 2, 512, 256, True, 7),
    ("bf16", [333], 512, 384, False, 0), ("bf16", [1], 256, 128, False, 0),
    ("bf16", [2100], 1152, 704, False, 0), ("bf16", [64], 4096, 2176, False, 0),
    ("bf16", [65], 4096, 2176, False, 0)])
def test_ffn_edges(dtype, counts, d, F, gather, slack):
    X, rows, goff, wgu, wd, n_src = ffn_case(dtype, counts, d, F, gather)
    M = int(goff[-1])
    bound = M + slack
    out = torch.full((n_src, d), float("nan"), device=DEV).to(TORCH[dtype])
    desc = L.make_desc(CONFIGS["tiny"].scaled(hidden=d, ffn=F, dtype=dtype))
    ws = torch.empty((L.fs_workspace_size(desc, L.FS_OP_GROUPED_FFN, bound, F),), dtype=torch.uint8,
                     device=DEV)
    L.fs_grouped_expert_ffn(desc, len(counts), F, X, rows, torch.from_numpy(goff).to(DEV), bound,
                            wgu, wd, out, ws)
    torch.cuda.synchronize()
    check_ffn(dtype, X, rows, goff, wgu, wd, out)


# one dense group on every route its rules lead to (asserted): few rows on the
# skinny, streaming and 64-row kernels, the ring in one round without a K split,
# the ring and the 192-row tiles at equal heights
@pytest.mark.parametrize("rows,d,F,gu,dn", [
    (1, 3072, 1536, R.STREAM, R.SKINNY), (20, 3072, 1536, R.STREAM, R.SKINNY),
    (8, 512, 5120, R.R64, R.SKINNY), (40, 512, 1024, R.R64, R.SKINNY), (50, 1024, 512, R.R64, R.SKINNY),
    (64, 4096, 1024, R.STREAM, R.R64), (1, 2048, 2816, R.R64, R.STREAM), (33, 3072, 1408, R.R64, R.R64),
    (700, 2048, 2816, R.R64, R.R64), (1100, 2048, 2816, R.RING, R.R64), (1000, 5120, 384, R.RING, R.RING),
    (1000, 768, 8192, R.RING, R.RING), (4096, 256, 768, R.RING, R.R64)])
def test_dense_group_routes(rows, d, F, gu, dn):
    assert (R.pass_kind(True, rows, 1, F, d), R.pass_kind(False, rows, 1, F, d)) == (gu, dn)
    X, _, goff, wgu, wd, n_src = ffn_case("bf16", [rows], d, F, False, seed=3)
    out = torch.full((n_src, d), float("nan"), device=DEV).to(torch.bfloat16)
    desc = L.make_desc(CONFIGS["tiny"].scaled(hidden=d, ffn=F, dtype="bf16"))
    ws = torch.empty((L.fs_workspace_size(desc, L.FS_OP_GROUPED_FFN, rows, F),), dtype=torch.uint8,
                     device=DEV)
    L.fs_grouped_expert_ffn(desc, 1, F, X, None, None, rows, wgu, wd, out, ws)
    torch.cuda.synchronize()
    check_ffn("bf16", X, None, goff, wgu, wd, out)


# columns that the 256-wide tiles do not divide, of this pass or of the other one:
# every route (asserted), with groups around tile edges and empty ones
ODD = [200, 0, 193, 1, 450, 64, 129, 563]


@pytest.mark.parametrize("counts,d,F,gather,gu,dn", [
    (ODD, 256, 1472, True, R.STAGED, R.R64), (ODD * 2, 1152, 192, False, R.R64, R.R64),
    (ODD * 3, 1152, 192, True, R.R64, R.RING128), (ODD * 8, 384, 192, True, R.STAGED, R.RING128),
    ([7700], 640, 192, False, R.R64, R.STAGED), ([2100], 1664, 1472, False, R.STAGED, R.RING128),
    ([130] * 63 + [2], 1152, 512, True, R.R192, R.RING128), ([90] * 62 + [128, 3], 384, 512, True, R.RING, R.R64),
    ([130] * 63 + [2], 2048, 320, True, R.STAGED, R.R192), ([130] * 63 + [2], 2048, 192, False, R.R64, R.RING)])
def test_odd_width_routes(counts, d, F, gather, gu, dn):
    M, G = sum(counts), len(counts)
    assert (R.pass_kind(True, M, G, F, d), R.pass_kind(False, M, G, F, d)) == (gu, dn)
    X, rows, goff, wgu, wd, n_src = ffn_case("bf16", counts, d, F, gather, seed=5)
    out = torch.full((n_src, d), float("nan"), device=DEV).to(torch.bfloat16)
    desc = L.make_desc(CONFIGS["tiny"].scaled(hidden=d, ffn=F, dtype="bf16"))
    ws = torch.empty((L.fs_workspace_size(desc, L.FS_OP_GROUPED_FFN, M, F),), dtype=torch.uint8,
                     device=DEV)
    L.fs_grouped_expert_ffn(desc, G, F, X, rows, torch.from_numpy(goff).to(DEV), M, wgu, wd, out, ws)
    torch.cuda.synchronize()
    check_ffn("bf16", X, rows, goff, wgu, wd, out)


# 192-row tiles: every tile height (128 to 192 in steps of 32 and the short
# tiles below) and every largest height that a pass may choose (160, 192, 128),
# groups of one to several equal tiles, one band and more of m-tiles, several
# tiles per workgroup, K of four blocks and more, row bounds above the rows
TALL = [192, 193, 130, 0, 97, 384, 385, 5, 161, 577, 224, 256]


@pytest.mark.parametrize("counts,d,F,gather,slack,gu,dn", [
    (TALL, 2048, 1408, True, 0, 1, 0), (TALL, 512, 3072, False, 31, 1, 0), (TALL * 2, 256, 2816, True, 0, 1, 0),
    ([2048], 768, 2048, False, 0, 1, 0), ([3500, 1], 1280, 1408, True, 5, 1, 0), ([4100], 256, 1024, False, 0, 1, 0),
    ([300] * 8 + [50], 4096, 2048, True, 3, 1, 1),
    # down passes, scattered and in order: K of four blocks, several tiles a workgroup
    (TALL, 2816, 512, True, 0, 0, 1), (TALL * 2, 2816, 768, True, 9, 1, 1), (TALL, 3072, 256, False, 0, 0, 1),
    ([370] * 8 + [100], 4096, 256, True, 0, 0, 1), ([2500, 3], 3328, 640, True, 0, 0, 1), ([4100], 2304, 512, False, 0, 0, 1)])
def test_ffn_tall_tiles(counts, d, F, gather, slack, gu, dn):
    bound, G = sum(counts) + slack, len(counts)
    assert [R.pass_kind(g, bound, G, F, d) == R.R192 for g in (True, False)] == [gu, dn]
    X, rows, goff, wgu, wd, n_src = ffn_case("bf16", counts, d, F, gather, seed=7)
    bound = int(goff[-1]) + slack
    out = torch.full((n_src, d), float("nan"), device=DEV).to(torch.bfloat16)
    desc = L.make_desc(CONFIGS["tiny"].scaled(hidden=d, ffn=F, dtype="bf16"))
    ws = torch.empty((L.fs_workspace_size(desc, L.FS_OP_GROUPED_FFN, bound, F),), dtype=torch.uint8,
                     device=DEV)
    L.fs_grouped_expert_ffn(desc, len(counts), F, X, rows, torch.from_numpy(goff).to(DEV), bound,
                            wgu, wd, out, ws)
    torch.cuda.synchronize()
    check_ffn("bf16", X, rows, goff, wgu, wd, out)


@pytest.mark.parametrize("dtype,m,n,kd", [
    ("bf16", 2300, 3840, 256), ("bf16", 4097, 2048, 384), ("f32", 1, 64, 64), ("f32", 65, 192, 128), ("f32", 129, 4096, 320), ("f32", 1030, 8256, 64),
    ("bf16", 33, 640, 4032), ("bf16", 130, 384, 4096), ("bf16", 1000, 2048, 192),
    ("bf16", 2000, 1152, 320), ("bf16", 1300, 5120, 64)])
def test_dense_linear_edges(dtype, m, n, kd):
    gen = torch.Generator(device=DEV).manual_seed(m + n)
    a = torch.randn((m, kd), generator=gen, device=DEV).to(TORCH[dtype])
    w = (0.05 * torch.randn((n, kd), generator=gen, device=DEV)).to(TORCH[dtype])
    out = torch.full((m, n), float("nan"), device=DEV).to(TORCH[dtype])
    L.fs_dense_linear(L.FS_F32 if dtype == "f32" else L.FS_BF16, m, n, kd, a, w, out)
    torch.cuda.synchronize()
    assert rel_err(out, oracle.dense_linear(f64(a), f64(w))) <= TOL[dtype]


def quant(t):
    c = torch.empty(t.shape, dtype=torch.uint8, device=DEV)
    s = torch.empty(t.shape[:-1], dtype=torch.float32, device=DEV)
    L.fs_quantize_fp8(L.FS_BF16, s.numel(), t.shape[-1], t, c, s)
    return c, s


# FP8 on the 192-row tiles (heights 128 and 192, odd and even K block counts)
# against the fragment-ordered kernel on the same codes: H is the same bits;
# the down pass's fp32 sums may round differently in the last place, so an
# output differs by one bf16 step at most (2^-7 of its value), or, where the
# sum cancels, by the fp32 rounding of its F terms (F 2^-24 of the rms bounds
# it).
@pytest.mark.parametrize("counts,d,F,gather,gu,dn", [
    (TALL, 2048, 1408, True, 1, 0), (TALL * 2, 512, 2816, False, 1, 0), ([2050], 768, 2048, False, 1, 0),
    ([3000, 1], 1280, 1408, True, 1, 0),
    # down passes, scattered and in order: K of four blocks, several tiles a workgroup
    # (gate/up passes that split K would not give the same bits of H)
    (TALL * 3, 2816, 512, True, 1, 1), (TALL * 2, 2816, 768, True, 1, 1), (TALL * 3, 1024, 640, False, 1, 1),
    ([300] * 8 + [50], 4096, 1280, True, 1, 1), ([4100], 2304, 1024, False, 1, 1)])
def test_ffn_fp8_tall_tiles(counts, d, F, gather, gu, dn):
    kinds = [R.pass_kind_fp8(g, sum(counts), len(counts), F, d) for g in (True, False)]
    assert [k == R.R192 for k in kinds] == [gu, dn]
    X, rows, goff, wgu, wd, n_src = ffn_case("bf16", counts, d, F, gather, seed=9)
    G, M = len(counts), int(goff[-1])
    (xc, xs), (gc, gs), (dc, ds) = quant(X), quant(wgu), quant(wd)
    desc = L.make_desc(CONFIGS["tiny"].scaled(hidden=d, ffn=F, dtype="bf16"))
    ws = torch.empty((L.fs_workspace_size(desc, L.FS_OP_GROUPED_FFN_FP8, M, F),), dtype=torch.uint8,
                     device=DEV)
    go = torch.from_numpy(goff).to(DEV)
    out, ref = (torch.full((n_src, d), float("nan"), device=DEV).to(torch.bfloat16) for _ in range(2))
    H = lambda: ws[:2 * M * F].clone()
    L.fs_grouped_expert_ffn_fp8(desc, G, F, xc, xs, rows, go, M, gc, gs, dc, ds, out, ws)
    h_out = H()
    L.fs_grouped_expert_ffn_fp8_fo(desc, G, F, xc, xs, rows, go, M, fragment_ordered_fp8(gc), gs,
                                   fragment_ordered_fp8(dc), ds, ref, ws)
    torch.cuda.synchronize()
    assert torch.equal(h_out, H())
    at = rows.long() if gather else torch.arange(M, device=DEV)
    o, r = out[at].double(), ref[at].double()
    assert torch.all((o - r).abs() <= 2.0 ** -7 * r.abs() + F * 2.0 ** -24 * r.square().mean().sqrt())
    rest = torch.ones(n_src, dtype=torch.bool, device=DEV)
    rest[at] = False
    assert out[rest].isnan().all()


# the ring running on from tile to tile: more tiles than workgroups, gathered rows
# through scalar loads, K of 4 and 8 blocks (FP8: 4), groups too short for the
# 192-row tiles
@pytest.mark.parametrize("d", [256, 512])
@pytest.mark.parametrize("fp8", [False, True])
def test_ffn_ring_many_tiles(d, fp8):
    counts, F = [100] * 31 + [0, 1, 111, 0] + [97] * 31, 1408
    M, G = sum(counts), len(counts)
    kind = R.pass_kind_fp8(True, M, G, F, d) if fp8 else R.pass_kind(True, M, G, F, d)
    assert kind == R.RING and G * (F // 128) > 2 * R.CUS
    X, rows, goff, wgu, wd, n_src = ffn_case("bf16", counts, d, F, True, seed=11)
    desc = L.make_desc(CONFIGS["tiny"].scaled(hidden=d, ffn=F, dtype="bf16"))
    go = torch.from_numpy(goff).to(DEV)
    out = torch.full((n_src, d), float("nan"), device=DEV).to(torch.bfloat16)
    op = L.FS_OP_GROUPED_FFN_FP8 if fp8 else L.FS_OP_GROUPED_FFN
    ws = torch.empty((L.fs_workspace_size(desc, op, M, F),), dtype=torch.uint8, device=DEV)
    if not fp8:
        L.fs_grouped_expert_ffn(desc, G, F, X, rows, go, M, wgu, wd, out, ws)
        torch.cuda.synchronize()
        check_ffn("bf16", X, rows, goff, wgu, wd, out)
        return
    (xc, xs), (gc, gs), (dc, ds) = quant(X), quant(wgu), quant(wd)
    L.fs_grouped_expert_ffn_fp8(desc, G, F, xc, xs, rows, go, M, gc, gs, dc, ds, out, ws)
    h = ws[:2 * M * F].clone()
    ref = torch.empty_like(out)
    L.fs_grouped_expert_ffn_fp8_fo(desc, G, F, xc, xs, rows, go, M, fragment_ordered_fp8(gc), gs,
                                   fragment_ordered_fp8(dc), ds, ref, ws)
    torch.cuda.synchronize()
    assert torch.equal(h, ws[:2 * M * F])   # the gate/up pass, bit for bit


# a row bound of all token slots over the 8 experts of 64 that are here: both
# sides of the tile rule on the rows they likely hold (892 and 900), groups
# far shorter and longer than that
@pytest.mark.parametrize("n_tokens", [1190, 1200])
def test_gathered_loose_bound(n_tokens):
    counts, d, F, bound = [1, 0, 193, 64, 300, 17, 129, 196], 2048, 1408, n_tokens * 6
    X, rows, goff, wgu, wd, _ = ffn_case("bf16", counts, d, F, True)
    desc = L.make_desc(CONFIGS["tiny"].scaled(n_tokens=n_tokens, hidden=d, n_experts=64, top_k=6,
                                              ffn=F, dtype="bf16"))
    y = torch.full((bound, d), float("nan"), dtype=torch.bfloat16, device=DEV)
    ws = torch.empty(L.fs_workspace_size(desc, L.FS_OP_GROUPED_FFN, bound, F), dtype=torch.uint8,
                     device=DEV)
    gat = torch.zeros(bound, dtype=torch.int32, device=DEV)
    gat[:len(rows)] = rows
    L.fs_grouped_expert_ffn_gathered(desc, len(counts), F, X, gat, torch.tensor(goff, device=DEV),
                                     bound, wgu, wd, y, ws)
    torch.cuda.synchronize()
    Xr, M = X[rows.long()], int(goff[-1])
    assert bool(torch.isnan(y[M:]).all())
    check_ffn("bf16", Xr, None, goff, wgu, wd, y[:M])
