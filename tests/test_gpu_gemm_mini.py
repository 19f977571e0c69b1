"""GPU parity of the contraction on tiles of 64 x 64 and 32 x 32, for problems of few outputs: against the fp64 oracle at the edges of
the tiles, of the K steps and of the stages, and byte for byte against the 128 x 128 tile; nothing outside the output may be written."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_15306_amd import llmq, synth
from gpu_common import DEV, GEMM_TOL, assert_gemm_close, bf16_to_f64, f32_bits, gpu_amax
from test_gpu_gemm import _rand_codes, _scales
from test_gpu_gemm_bf16 import _check, _rand
from test_gpu_gemm_edge import _guarded, _untouched

pytestmark = pytest.mark.gpu

# (R, C, T): tile edges; one K step and less, whole stages of four, a step more and less, more stages than are kept; widths that are
# multiples of 4 and others
SHAPES = [(1, 1, 16), (16, 16, 128), (31, 33, 48), (32, 64, 512), (33, 30, 528), (64, 65, 384), (100, 136, 272), (65, 4, 640), (17, 101, 1024),
          (128, 256, 2048), (40, 96, 2064), (7, 70, 2560), (96, 32, 4224)]


def _slabs(codes):
    """[rows, T] -> [T / 128, rows, 128]"""
    rows, T = codes.shape
    return np.ascontiguousarray(codes.reshape(rows, T // 128, 128).transpose(1, 0, 2))


@pytest.mark.parametrize("side", ["32", "64"])
@pytest.mark.parametrize("R,C,T", SHAPES)
def test_small_tiles_fp8(R, C, T, side, monkeypatch):
    fa, fb = (R + T // 16) % 2, (C // 2) % 2
    print("mini R=%d C=%d T=%d side=%s fa=%d fb=%d" % (R, C, T, side, fa, fb), flush=True)
    A, B = _rand_codes((R, T), fa, 7 * R + T), _rand_codes((C, T), fb, 5 * C + T + 1)
    y, S = oracle.gemm_tn(A, fa, B, fb, 3.7, 0.61)
    c0 = _rand((R, C), 5, 30.0)
    dsa, dsb = _scales(3.7, 0.61)
    got = {}
    for which in (side, "tile"):
        for lay in ((0, 2) if T % 128 == 0 else (0,)):
            a, b = (torch.from_numpy(_slabs(t) if lay else t).to(DEV) for t in (A, B))
            if which == "tile":
                monkeypatch.delenv("LLMQ_GEMM_MINI", raising=False)
                monkeypatch.setenv("LLMQ_GEMM_EDGE_TILE", "2x2")
            else:
                monkeypatch.setenv("LLMQ_GEMM_MINI", which)
            for acc in (False, True):
                am = torch.full((1,), -1.0, dtype=torch.float32, device=DEV)
                buf, c = _guarded(R, C, c0 if acc else None)
                llmq.llmq_fp8_gemm(a, fa, lay, b, fb, lay, dsa, dsb, c, acc, am)
                assert _untouched(buf, R, C)
                assert f32_bits(am) == f32_bits(gpu_amax(c.reshape(-1).clone(), 0, want_scale=False)[0])
                got[which, lay, acc] = c.clone()
    assert_gemm_close(got[side, 0, False], y, S, "mini")
    want = bf16_to_f64(c0) + y
    assert np.all(np.abs(bf16_to_f64(got[side, 0, True]) - want) <= GEMM_TOL * S + 2.0 ** -8 * np.abs(want))
    for (which, lay, acc), c in got.items():
        assert torch.equal(c.view(torch.int16), got["tile", 0, acc].view(torch.int16)), (which, lay, acc)


@pytest.mark.parametrize("side", ["32", "64"])
@pytest.mark.parametrize("R,C,T", [(1, 3, 8), (33, 70, 136), (64, 32, 256), (40, 101, 1032), (130, 64, 1288)])
def test_small_tiles_bf16(R, C, T, side, monkeypatch):
    monkeypatch.setenv("LLMQ_GEMM_MINI", side)
    A, B, prev = _rand((R, T), 100 + R + T), _rand((C, T), 200 + C + T, 0.05), _rand((R, C), 300 + R, 0.5)
    y, S = oracle.gemm_bf16_tn(synth.bf16_bits(A), synth.bf16_bits(B))
    for p in (None, prev):
        buf, c = _guarded(R, C, p)
        llmq.llmq_bf16_gemm_tn(A.to(DEV), B.to(DEV), c, accumulate=p is not None)
        _check(c, y, S, T, "mini", prev=None if p is None else bf16_to_f64(p))
        assert _untouched(buf, R, C)


@pytest.mark.parametrize("R,C,T", [(33, 70, 136), (64, 32, 256), (40, 101, 1032), (130, 64, 1288), (128, 256, 2048)])
def test_small_tiles_bf16_have_the_bytes_of_the_tile_kernel(R, C, T, monkeypatch):
    A, B, prev = _rand((R, T), R + T).to(DEV), _rand((C, T), C + T, 0.05).to(DEV), _rand((R, C), R, 0.5).to(DEV)
    outs = []
    for mini in ("0", "32", "64"):
        monkeypatch.setenv("LLMQ_GEMM_MINI", mini)
        c, acc = torch.zeros((R, C), dtype=torch.bfloat16, device=DEV), prev.clone()
        llmq.llmq_bf16_gemm_tn(A, B, c)
        llmq.llmq_bf16_gemm_tn(A, B, acc, accumulate=True)
        outs.append((c.view(torch.int16), acc.view(torch.int16)))
    assert all(torch.equal(a, b) for o in outs[1:] for a, b in zip(outs[0], o))


@pytest.mark.parametrize("R,C", [(1, 3), (48, 272), (300, 300), (29, 921)])
def test_shortest_bf16_contractions_stay_on_the_generic_kernel(R, C, monkeypatch):
    """Eight elements: one lane per output is the faster kernel, whose sums run along t one by one."""
    A, B = _rand((R, 8), R + 1).to(DEV), _rand((C, 8), C + 2).to(DEV)
    outs = []
    for tile in (None, "0x0"):
        if tile:
            monkeypatch.setenv("LLMQ_GEMM_EDGE_TILE", tile)
        c = torch.zeros((R, C), dtype=torch.bfloat16, device=DEV)
        llmq.llmq_bf16_gemm_tn(A, B, c)
        outs.append(c.view(torch.int16))
    assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("side", ["32", "64"])
def test_values_beyond_the_operands_and_degenerate_scales(side, monkeypatch):
    """NaN and Inf codes lie directly behind the operands; one NaN row stays one NaN row; scales whose product leaves the
    normal range are applied one after the other, as everywhere."""
    monkeypatch.setenv("LLMQ_GEMM_MINI", side)
    R, C, T = 70, 36, 272
    A, B = _rand_codes((R, T), 0, 3), _rand_codes((C, T), 0, 4)
    A[5, T - 1] = 0x7F
    bufA, bufB = (torch.full((n * T + 8192,), 0x7F, dtype=torch.uint8, device=DEV) for n in (R, C))
    a, b = bufA[:R * T].view(R, T), bufB[:C * T].view(C, T)
    a.copy_(torch.from_numpy(A))
    b.copy_(torch.from_numpy(B))
    dsa, dsb = _scales(1.5, 0.8)
    am = torch.zeros(1, dtype=torch.float32, device=DEV)
    c = torch.zeros((R, C), dtype=torch.bfloat16, device=DEV)
    llmq.llmq_fp8_gemm_tn(a, 0, b, 0, dsa, dsb, c, False, am)
    bad = torch.isnan(c).all(dim=1)
    assert bad[5] and int(bad.sum()) == 1 and torch.isfinite(c[torch.arange(R, device=DEV) != 5]).all()
    assert f32_bits(am) == 0x7FC00000
    a[5, T - 1] = 0x38
    for sa, sb in ((1.0, 2.0), (3.402823466e38, 0.5), (1e-30, 1e-20), (3.402823466e38, 3.402823466e38)):
        dsa, dsb = _scales(sa, sb)
        outs = []
        for mini in (side, "0"):
            monkeypatch.setenv("LLMQ_GEMM_MINI", mini)
            out = torch.zeros_like(c)
            llmq.llmq_fp8_gemm_tn(a, 0, b, 0, dsa, dsb, out, False, am)
            outs.append((out.view(torch.int16), am.clone().view(torch.int32)))
        assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1]), (sa, sb)


@pytest.mark.parametrize("R,C,T", [(256, 1024, 512), (256, 512, 1024), (1024, 512, 256), (117, 304, 1440), (128, 96, 6656), (300, 136, 64)])
def test_chosen_kernel_gives_the_same_bytes(R, C, T, monkeypatch):
    """Whatever the dispatch takes for shapes on either side of its lines, the bytes are those of the other kernels."""
    A, B = _rand_codes((R, T), 1, R), _rand_codes((C, T), 0, C)
    dsa, dsb = _scales(2.0, 0.7)
    outs = []
    for mini in (None, "0", "32", "64"):
        if mini is None:
            monkeypatch.delenv("LLMQ_GEMM_MINI", raising=False)
        else:
            monkeypatch.setenv("LLMQ_GEMM_MINI", mini)
        c, am = torch.zeros((R, C), dtype=torch.bfloat16, device=DEV), torch.zeros(1, device=DEV)
        llmq.llmq_fp8_gemm_tn(torch.from_numpy(A).to(DEV), 1, torch.from_numpy(B).to(DEV), 0, dsa, dsb, c, False, am)
        outs.append((c.view(torch.int16), am))
    assert all(torch.equal(o[0], outs[0][0]) and torch.equal(o[1], outs[0][1]) for o in outs)
