"""GPU parity of the 256 x 320 and 320 x 256 tiles, and of guarded tiles where a smaller one divides the problem, against the fp64 oracle and
against the bytes of the tiles that ran before."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_15306_amd import llmq, synth
from gpu_common import DEV, assert_gemm_close, bf16_to_f64, f32_bits, gpu_amax
from test_gpu_gemm import _rand_codes, _scales
from test_gpu_gemm_bf16 import _check, _rand
from test_gpu_gemm_edge import GEMM_TOL, _guarded, _operand, _untouched
from test_gpu_slab_copies import to_slabs

pytestmark = pytest.mark.gpu

# Whole tiles of one and of both kinds (1 to 4 K steps, an odd number too), shapes just below, at and above their edges, widths that are multiples
# of 8 and odd ones, T inside a K step
SHAPES = [(256, 320, 128), (320, 256, 256), (1280, 1280, 384), (512, 640, 512), (640, 512, 128), (1, 8, 16), (255, 321, 128), (257, 319, 272),
          (320, 264, 144), (321, 17, 400), (300, 320, 256), (640, 336, 112), (528, 1296, 640)]


@pytest.mark.parametrize("tile", ["4x5", "5x4"])
@pytest.mark.parametrize("R,C,T", SHAPES)
def test_large_tiles_fp8(R, C, T, tile, monkeypatch):
    monkeypatch.setenv("LLMQ_GEMM_ANY_TILE", tile)
    fa = (R + T // 16) % 2
    A, B = _rand_codes((R, T), fa, 7 * R + T), _rand_codes((C, T), 0, 5 * C + T + 1)
    y, S = oracle.gemm_tn(A, fa, B, 0, 3.7, 0.61)
    c0 = _rand((R, C), 5, 30.0)
    first = None
    layouts = [(False, False), (False, True), (True, True)] + ([(2, 2), (2, True), (False, 2)] if T % 128 == 0 else [])
    for la, lb in layouts:
        if (la is True and R % 16) or (lb is True and C % 16):
            continue
        print("large R=%d C=%d T=%d tile=%s layouts %s %s" % (R, C, T, tile, la, lb), flush=True)
        a, b = (to_slabs(torch.from_numpy(x).to(DEV)) if l == 2 and l is not True else _operand(x, l) for x, l in ((A, la), (B, lb)))
        dsa, dsb = _scales(3.7, 0.61)
        am = torch.full((1,), -1.0, dtype=torch.float32, device=DEV)
        buf, c = _guarded(R, C)
        llmq.llmq_fp8_gemm(a, fa, la, b, 0, lb, dsa, dsb, c, False, am)
        assert_gemm_close(c, y, S, "large")
        assert _untouched(buf, R, C)
        assert f32_bits(am) == f32_bits(gpu_amax(c.reshape(-1).clone(), 0, want_scale=False)[0])
        buf, acc = _guarded(R, C, c0)
        llmq.llmq_fp8_gemm(a, fa, la, b, 0, lb, dsa, dsb, acc, True, am)
        want = bf16_to_f64(c0) + y
        assert np.all(np.abs(bf16_to_f64(acc) - want) <= GEMM_TOL * S + 2.0 ** -8 * np.abs(want))
        assert _untouched(buf, R, C)
        assert f32_bits(am) == f32_bits(gpu_amax(acc.reshape(-1).clone(), 0, want_scale=False)[0])
        first = c.clone() if first is None else first
        assert torch.equal(first.view(torch.int16), c.view(torch.int16))      # same sums in every layout


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("R,C,T", [(300, 12755, 128), (70, 50257, 272), (1, 16001, 16)])
def test_odd_widths_far_beyond_a_tile(R, C, T, accumulate, monkeypatch):
    """256 x 320 tiles whose outputs leave element by element, with the edge of the output up to 50000 columns away: the bytes of the 256 x 256 tile."""
    a, b = (torch.from_numpy(_rand_codes(s, 0, s[0] + T)).to(DEV) for s in ((R, T), (C, T)))
    dsa, dsb = _scales(1.7, 0.9)
    c0 = _rand((R, C), 6, 30.0).to(DEV)
    got = []
    for tile in ("4x5", "4x4"):
        monkeypatch.setenv("LLMQ_GEMM_ANY_TILE", tile)
        print("wide odd R=%d C=%d T=%d tile=%s accumulate %d" % (R, C, T, tile, accumulate), flush=True)
        am = torch.full((1,), -1.0, dtype=torch.float32, device=DEV)
        buf, c = _guarded(R, C, c0 if accumulate else None)
        llmq.llmq_fp8_gemm(a, 0, False, b, 0, False, dsa, dsb, c, accumulate, am)
        assert _untouched(buf, R, C)
        got.append((c.clone().view(torch.int16), am))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("tile", ["4x5", "5x4"])
@pytest.mark.parametrize("R,C,T", [(256, 320, 64), (640, 640, 192), (257, 264, 136), (130, 8, 8), (255, 129, 72), (330, 520, 256)])
def test_large_tiles_bf16(R, C, T, tile, monkeypatch):
    monkeypatch.setenv("LLMQ_GEMM_ANY_TILE", tile)
    print("large bf16 R=%d C=%d T=%d tile=%s" % (R, C, T, tile), flush=True)
    A, B, prev = _rand((R, T), 100 + R + T), _rand((C, T), 200 + C + T, 0.05), _rand((R, C), 300 + R, 0.5)
    y, S = oracle.gemm_bf16_tn(synth.bf16_bits(A), synth.bf16_bits(B))
    for p in (None, prev):
        buf, c = _guarded(R, C, p)
        llmq.llmq_bf16_gemm_tn(A.to(DEV), B.to(DEV), c, accumulate=p is not None)
        _check(c, y, S, T, "large", prev=None if p is None else bf16_to_f64(p))
        assert _untouched(buf, R, C)


@pytest.mark.parametrize("tile", ["4x5", "5x4"])
@pytest.mark.parametrize("layouts", [(False, False), (False, True), (True, True)])
def test_values_beyond_the_operands_do_not_reach_the_results(tile, layouts, monkeypatch):
    """NaN codes lie directly behind the operands in memory: in guarded tiles, and in whole ones that are one K step long."""
    monkeypatch.setenv("LLMQ_GEMM_ANY_TILE", tile)
    ta, tb = layouts
    for R, C, T in ((336, 272, 272), (320, 320, 144), (1280, 1280, 128)):
        A, B = _rand_codes((R, T), 0, 3), _rand_codes((C, T), 0, 4)
        y, S = oracle.gemm_tn(A, 0, B, 0, 1.5, 0.8)
        ops = []
        for x, t in ((A, ta), (B, tb)):
            buf = torch.full((x.size + 65536,), 0x7F, dtype=torch.uint8, device=DEV)
            o = _operand(x, t)
            view = buf[:x.size].view(o.shape)
            view.copy_(o)
            ops.append(view)
        dsa, dsb = _scales(1.5, 0.8)
        am, c = torch.zeros(1, dtype=torch.float32, device=DEV), torch.zeros((R, C), dtype=torch.bfloat16, device=DEV)
        print("beyond R=%d C=%d T=%d tile=%s layouts %s" % (R, C, T, tile, layouts), flush=True)
        llmq.llmq_fp8_gemm(ops[0], 0, ta, ops[1], 0, tb, dsa, dsb, c, False, am)
        assert_gemm_close(c, y, S, "beyond")
        assert am.item() == c.float().abs().max().item()


@pytest.mark.parametrize("sA,sB", [(3.402823466e38, 1.0), (3.402823466e38, 3.402823466e38), (2.0 ** -100, 2.0 ** -100)])
@pytest.mark.parametrize("tile", ["4x5", "5x4"])
def test_degenerate_scales(sA, sB, tile, monkeypatch):
    """Scales whose product leaves the normal range: the bytes of the 256 x 256 tile."""
    R, C, T = 1280, 1280, 256
    a, b = torch.from_numpy(_rand_codes((R, T), 0, 1)).to(DEV), torch.from_numpy(_rand_codes((C, T), 0, 2)).to(DEV)
    dsa, dsb = _scales(sA, sB)
    got = []
    for t in (tile, "4x4"):
        monkeypatch.setenv("LLMQ_GEMM_ANY_TILE", t)
        print("degenerate %g %g tile=%s" % (sA, sB, t), flush=True)
        c = torch.full((R, C), -7.0, dtype=torch.bfloat16, device=DEV)
        llmq.llmq_fp8_gemm_tn(a, 0, b, 0, dsa, dsb, c)
        got.append(c.view(torch.int16))
    assert torch.equal(*got)


@pytest.mark.parametrize("R,C,T", [(2176, 6400, 1536), (4096, 5120, 512), (2560, 5120, 1296), (8192, 2560, 384), (1984, 8000, 640), (3200, 3904, 256)])
def test_the_chosen_tile_gives_the_bytes_of_the_others(R, C, T, monkeypatch):
    """What the library picks (large tiles, guarded 256 x 256 and 192 x 256 ones) against the tiles that divide the problem or ran before, in every
    layout, with and without addition to the output."""
    A, B = _rand_codes((R, T), 0, T), _rand_codes((C, T), 0, T + 1)
    dsa, dsb = _scales(1.7, 0.9)
    c0 = _rand((R, C), 6, 30.0).to(DEV)
    for ta, tb in ((False, False), (False, True), (True, True)):
        if (ta and R % 16) or (tb and C % 16):
            continue
        a, b = _operand(A, ta), _operand(B, tb)
        got = []
        for tile in (None, "0", "4x4", "3x4", "5x4", "4x5"):
            if tile is None:
                monkeypatch.delenv("LLMQ_GEMM_ANY_TILE", raising=False)
            else:
                monkeypatch.setenv("LLMQ_GEMM_ANY_TILE", tile)
            print("chosen R=%d C=%d T=%d tile=%s ta=%d tb=%d" % (R, C, T, tile, ta, tb), flush=True)
            am = torch.zeros(2, dtype=torch.float32, device=DEV)
            buf, c = _guarded(R, C)
            llmq.llmq_fp8_gemm(a, 0, ta, b, 0, tb, dsa, dsb, c, False, am[:1])
            buf2, acc = _guarded(R, C, c0)
            llmq.llmq_fp8_gemm(a, 0, ta, b, 0, tb, dsa, dsb, acc, True, am[1:])
            assert _untouched(buf, R, C) and _untouched(buf2, R, C)
            got.append((c.view(torch.int16), acc.view(torch.int16), am))
        for g in got[1:]:
            assert all(torch.equal(x, z) for x, z in zip(got[0], g))


@pytest.mark.parametrize("tile", ["4x5", "5x4"])
@pytest.mark.parametrize("layouts", [(False, False), (False, True), (True, True)])
def test_request_of_the_next_tiles_slabs(layouts, tile, monkeypatch):
    """Every workgroup requests lines of the first two slabs of the one 8 ids further on: no byte changes.  Contractions of exactly those slabs
    and longer ones."""
    ta, tb = layouts
    monkeypatch.setenv("LLMQ_GEMM_ANY_TILE", tile)
    monkeypatch.setenv("LLMQ_GEMM_SLOTS", "8")
    dsa, dsb = _scales(2.5, 0.5)
    for R, C, T in ((1280, 2560, 256), (1280, 1280, 640)):
        A, B = _rand_codes((R, T), 0, 71), _rand_codes((C, T), 0, 72)
        a, b = _operand(A, ta), _operand(B, tb)
        got = []
        for on in ("1", "0"):
            monkeypatch.setenv("LLMQ_GEMM_TOUCH_NEXT", on)
            print("next R=%d C=%d T=%d tile=%s layouts %s on %s" % (R, C, T, tile, layouts, on), flush=True)
            c, am = torch.full((R, C), float("nan"), dtype=torch.bfloat16, device=DEV), torch.zeros(1, dtype=torch.float32, device=DEV)
            llmq.llmq_fp8_gemm(a, 0, ta, b, 0, tb, dsa, dsb, c, False, am)
            got.append((c.view(torch.int16), am))
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
        y, S = oracle.gemm_tn(A, 0, B, 0, 2.5, 0.5)
        assert_gemm_close(c, y, S, "next")
