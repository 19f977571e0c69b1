"""GPU parity of the tile kernels on ragged shapes (any rows, columns and contraction length, any row pitch) against
the fp64 oracle, at the edges of their tiles; nothing outside the output may be written."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_15306_amd import llmq, synth
from gpu_common import DEV, GEMM_TOL, bf16_to_f64, assert_gemm_close, f32_bits, gpu_amax
from test_gpu_gemm import _rand_codes, _scales
from test_gpu_gemm_bf16 import _check, _rand

pytestmark = pytest.mark.gpu

TILES = ["4x4", "4x2", "2x4", "2x2"]
# (R, C, T): just below, at and above tile edges; T with whole 16-byte chunks (0, 1 and several K steps, with and without
# a tail) and without; widths that are multiples of 8 and odd ones
SHAPES = [(1, 8, 16), (127, 130, 112), (257, 264, 128), (300, 17, 144), (255, 513, 272), (130, 256, 400),
          (1, 1, 17), (33, 40, 31), (129, 255, 127), (256, 136, 129), (270, 260, 250), (513, 24, 393), (40, 300, 1001)]
GUARD = 512      # sentinel elements before and after the output


def _guarded(R, C, init=None):
    buf = torch.full((R * C + 2 * GUARD,), -77.0, dtype=torch.bfloat16, device=DEV)
    c = buf[GUARD:GUARD + R * C].view(R, C)
    c.copy_(torch.full((R, C), float("nan"), dtype=torch.bfloat16) if init is None else init)
    return buf, c


def _untouched(buf, R, C):
    return bool((buf[:GUARD] == -77.0).all() and (buf[GUARD + R * C:] == -77.0).all())


def _operand(codes, layout):
    t = torch.from_numpy(np.ascontiguousarray(codes.T) if layout else codes)
    return t.to(DEV)


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("R,C,T", SHAPES)
def test_ragged_fp8(R, C, T, tile, monkeypatch):
    monkeypatch.setenv("LLMQ_GEMM_EDGE_TILE", tile)
    layouts = [(False, False), (False, True), (True, True)]
    fa = (R + T) % 2
    A, B = _rand_codes((R, T), fa, 7 * R + T), _rand_codes((C, T), 0, 5 * C + T + 1)
    y, S = oracle.gemm_tn(A, fa, B, 0, 3.7, 0.61)
    c0 = _rand((R, C), 5, 30.0)
    first = None
    for ta, tb in layouts:
        print("edge R=%d C=%d T=%d tile=%s ta=%d tb=%d" % (R, C, T, tile, ta, tb), flush=True)
        dsa, dsb = _scales(3.7, 0.61)
        am = torch.full((1,), -1.0, dtype=torch.float32, device=DEV)
        buf, c = _guarded(R, C)
        llmq.llmq_fp8_gemm(_operand(A, ta), fa, ta, _operand(B, tb), 0, tb, dsa, dsb, c, False, am)
        assert_gemm_close(c, y, S, "edge")
        assert _untouched(buf, R, C)
        assert f32_bits(am) == f32_bits(gpu_amax(c.reshape(-1).clone(), 0, want_scale=False)[0])
        buf, acc = _guarded(R, C, c0)
        llmq.llmq_fp8_gemm(_operand(A, ta), fa, ta, _operand(B, tb), 0, tb, dsa, dsb, acc, True, am)
        want = bf16_to_f64(c0) + y
        assert np.all(np.abs(bf16_to_f64(acc) - want) <= GEMM_TOL * S + 2.0 ** -8 * np.abs(want))
        assert _untouched(buf, R, C)
        assert f32_bits(am) == f32_bits(gpu_amax(acc.reshape(-1).clone(), 0, want_scale=False)[0])
        if first is None:
            first = c.clone()
        assert torch.equal(first.view(torch.int16), c.view(torch.int16))      # same sums in every layout


@pytest.mark.parametrize("R,C,T", SHAPES + [(1, 1001, 384), (16, 17, 16), (130, 300, 48), (700, 520, 256), (40, 40, 2000), (2000, 136, 100)])
def test_generic_and_tile_kernel_give_the_same_bytes(R, C, T, monkeypatch):
    """Small problems take the generic kernel, by a rule on sizes, layouts and accumulation: nothing else may depend on it."""
    fa = (R + C) % 2
    A, B = _rand_codes((R, T), fa, 11 * R + T), _rand_codes((C, T), 0, 13 * C + T)
    dsa, dsb = _scales(2.9, 0.37)
    c0 = _rand((R, C), 6, 30.0)
    for ta, tb in ((False, False), (False, True), (True, True)):
        a, b, got = _operand(A, ta), _operand(B, tb), []
        for tile in ("0x0", "2x2", None):
            if tile is None:
                monkeypatch.delenv("LLMQ_GEMM_EDGE_TILE")
            else:
                monkeypatch.setenv("LLMQ_GEMM_EDGE_TILE", tile)
            print("R=%d C=%d T=%d tile=%s ta=%d tb=%d" % (R, C, T, tile, ta, tb), flush=True)
            am = torch.zeros(2, dtype=torch.float32, device=DEV)
            (buf, c), (buf2, acc) = _guarded(R, C), _guarded(R, C, c0)
            llmq.llmq_fp8_gemm(a, fa, ta, b, 0, tb, dsa, dsb, c, False, am[0:1])
            llmq.llmq_fp8_gemm(a, fa, ta, b, 0, tb, dsa, dsb, acc, True, am[1:2])
            assert _untouched(buf, R, C) and _untouched(buf2, R, C)
            got.append((buf.view(torch.int16), buf2.view(torch.int16), am))
        for other in got[1:]:
            assert all(torch.equal(x, y) for x, y in zip(got[0], other))


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("R,C,T", [(257, 264, 136), (130, 8, 8), (40, 300, 500), (255, 129, 63), (300, 520, 257)])
def test_ragged_bf16(R, C, T, tile, monkeypatch):
    monkeypatch.setenv("LLMQ_GEMM_EDGE_TILE", tile)
    print("edge bf16 R=%d C=%d T=%d tile=%s" % (R, C, T, tile), flush=True)
    A, B, prev = _rand((R, T), 100 + R + T), _rand((C, T), 200 + C + T, 0.05), _rand((R, C), 300 + R, 0.5)
    y, S = oracle.gemm_bf16_tn(synth.bf16_bits(A), synth.bf16_bits(B))
    for p in (None, prev):
        buf, c = _guarded(R, C, p)
        llmq.llmq_bf16_gemm_tn(A.to(DEV), B.to(DEV), c, accumulate=p is not None)
        _check(c, y, S, T, "edge", prev=None if p is None else bf16_to_f64(p))
        assert _untouched(buf, R, C)


@pytest.mark.parametrize("tile", [None, "2x2", "4x4", "3x4", "3x2"])
@pytest.mark.parametrize("fa,T", [(0, 272), (1, 272), (0, 275), (1, 275)])
def test_values_beyond_the_operands_do_not_reach_the_results(fa, T, tile, monkeypatch):
    """NaN and Inf codes lie directly behind the operands in memory; one NaN row inside stays one NaN row.  The kernel the sizes choose, and
    the guarded tiles of every height (192 rows: aligned rows only)."""
    if tile:
        monkeypatch.setenv("LLMQ_GEMM_EDGE_TILE", tile)
    R, C = 130, 72
    nan, inf = (0x7F, 0x7F) if fa == 0 else (0x7E, 0x7C)
    A, B = _rand_codes((R, T), fa, 3), _rand_codes((C, T), 0, 4)
    A[5, T - 1] = nan
    bufA = torch.full((R * T + 4096,), inf, dtype=torch.uint8, device=DEV)
    bufB = torch.full((C * T + 4096,), 0x7F, dtype=torch.uint8, device=DEV)
    a, b = bufA[:R * T].view(R, T), bufB[:C * T].view(C, T)
    a.copy_(torch.from_numpy(A))
    b.copy_(torch.from_numpy(B))
    dsa, dsb = _scales(1.5, 0.8)
    am = torch.zeros(1, dtype=torch.float32, device=DEV)
    c = torch.zeros((R, C), dtype=torch.bfloat16, device=DEV)
    llmq.llmq_fp8_gemm_tn(a, fa, b, 0, dsa, dsb, c, False, am)
    bad = torch.isnan(c).all(dim=1)
    assert bad[5] and int(bad.sum()) == 1 and torch.isfinite(c[torch.arange(R, device=DEV) != 5]).all()
    assert f32_bits(am) == 0x7FC00000
    a[5, T - 1] = 0x38
    llmq.llmq_fp8_gemm_tn(a, fa, b, 0, dsa, dsb, c, False, am)
    assert torch.isfinite(c).all() and am.item() == c.float().abs().max().item()


@pytest.mark.parametrize("fa", [0, 1])
@pytest.mark.parametrize("T", [16, 40, 100, 129, 250, 272, 400])
def test_values_beyond_t_major_operands_do_not_reach_the_results(fa, T):
    """The same with the contraction running down the rows: what lies behind the last row and, T no multiple of a K step,
    where the rows of that step would be; widths with and without whole 16-byte chunks."""
    nan, inf = (0x7F, 0x7F) if fa == 0 else (0x7E, 0x7C)
    for R, C in ((144, 80), (130, 72)):
        A, B = _rand_codes((R, T), fa, 3), _rand_codes((C, T), 0, 4)
        bufA = torch.full((R * T + 65536,), inf, dtype=torch.uint8, device=DEV)
        bufB = torch.full((C * T + 65536,), 0x7F, dtype=torch.uint8, device=DEV)
        dsa, dsb = _scales(1.5, 0.8)
        y, S = oracle.gemm_tn(A, fa, B, 0, 1.5, 0.8)
        for ta in (False, True):
            a, b = (bufA[:R * T].view(T, R) if ta else bufA[:R * T].view(R, T)), bufB[:C * T].view(T, C)
            a.copy_(_operand(A, ta))
            b.copy_(_operand(B, True))
            for tile in ("2x2", "4x4", "3x4", "3x2", "0x0"):
                with pytest.MonkeyPatch.context() as mp:
                    mp.setenv("LLMQ_GEMM_EDGE_TILE", tile)
                    print("beyond T-major: fa=%d R=%d C=%d T=%d ta=%d tile=%s" % (fa, R, C, T, ta, tile), flush=True)
                    am, c = torch.zeros(1, dtype=torch.float32, device=DEV), torch.zeros((R, C), dtype=torch.bfloat16, device=DEV)
                    llmq.llmq_fp8_gemm(a, fa, ta, b, 0, True, dsa, dsb, c, False, am)
                    assert_gemm_close(c, y, S, "beyond")
                    assert am.item() == c.float().abs().max().item()


@pytest.mark.parametrize("T", [272, 1001, 4112, 3999])
def test_more_tiles_than_compute_units(T, monkeypatch):
    """Many tiles, bands and rounds, long and short contractions, aligned and unaligned: the tile the library picks, all tiles
    forced, a second run and every layout give the same bytes; sampled rows and columns against the oracle."""
    R, C = 3001, 2888
    A, B = _rand_codes((R, T), 0, T), _rand_codes((C, T), 0, T + 1)
    dsa, dsb = _scales(1.7, 0.9)
    rows, cols = np.r_[0:R:397, R - 1], np.r_[0:C:351, C - 1]
    y, S = oracle.gemm_tn(np.ascontiguousarray(A[rows]), 0, np.ascontiguousarray(B[cols]), 0, 1.7, 0.9)
    first = None
    for ta, tb in ((False, False), (False, True), (True, True)):
        a, b = _operand(A, ta), _operand(B, tb)
        for tile in (None, None) + tuple(TILES if not ta else ()):
            if tile is None:
                monkeypatch.delenv("LLMQ_GEMM_EDGE_TILE", raising=False)
            else:
                monkeypatch.setenv("LLMQ_GEMM_EDGE_TILE", tile)
            print("large T=%d tile=%s ta=%d tb=%d" % (T, tile, ta, tb), flush=True)
            am = torch.zeros(1, dtype=torch.float32, device=DEV)
            buf, c = _guarded(R, C)
            llmq.llmq_fp8_gemm(a, 0, ta, b, 0, tb, dsa, dsb, c, False, am)
            assert _untouched(buf, R, C)
            assert am.item() == c.float().abs().max().item()
            if first is None:
                first = c.clone().view(torch.int16)
                assert_gemm_close(c[torch.from_numpy(rows).to(DEV)][:, torch.from_numpy(cols).to(DEV)], y, S, "large")
            assert torch.equal(first, c.view(torch.int16))


@pytest.mark.parametrize("tile", ["3x4", "3x2"])
@pytest.mark.parametrize("R,C,T", [(1, 8, 16), (191, 130, 112), (192, 17, 144), (193, 264, 400), (400, 256, 272), (577, 513, 128),
                                   (208, 272, 400), (208, 272, 401), (384, 144, 133), (192, 16, 17)])
def test_tiles_of_192_rows(R, C, T, tile, monkeypatch):
    """Below, at and above their edges.  Aligned rows only, which the layouts have by different sizes: operands in rows by T, T-major ones by R
    and C (the last four shapes: whole 16-byte chunks T-major, A in E4M3 and E5M2, T inside a K step); the others keep the tiles of even sides."""
    test_ragged_fp8(R, C, T, tile, monkeypatch)
    test_ragged_bf16(R, C, T, tile, monkeypatch)
