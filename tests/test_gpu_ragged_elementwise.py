"""GPU parity of the element-wise kernels at the edges of their tiles (64 x 128 and 128 x 128), vectors and row widths,
byte for byte against the oracle; nothing behind an output may be written."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_15306_amd import llmq, synth
from gpu_common import DEV, f32_bits, np_f32_bits
from test_gpu_rmsnorm import EPS, RSTD_TOL, _case as rms_case, gpu_rmsnorm_fwd
from test_gpu_swiglu import _case as swiglu_case

pytestmark = pytest.mark.gpu
PAD = 256


def _out(n, dtype, fill):
    """n elements followed by PAD sentinels"""
    return torch.full((n + PAD,), fill, dtype=dtype, device=DEV)


def _whole(buf, n, fill):
    assert bool((buf[n:] == fill).all()), "written behind the end"
    return buf[:n]


SHAPES = [(1, 1), (1, 7), (3, 9), (63, 127), (64, 128), (65, 129), (66, 136), (129, 257), (200, 250), (127, 513), (16, 264), (300, 1001)]
FORCED = [(128, 256), (256, 512), (384, 256)]            # whole tiles: both tile kernels, plain and slabs
NARROW = [(16, 8), (128, 64), (144, 40), (272, 16), (1040, 56)]        # whole patches of 16 x 8
# more than one tile row, more tile columns than a band is wide (ragged pitches walk in bands), and every kind of kernel
KINDS = [s + (k,) for s in SHAPES + [(200, 1300), (150, 1152)] for k in "02"] + [s + (k,) for s in NARROW for k in "012"]


def _slabs(qt, rows, cols):
    return qt.reshape(cols, rows // 128, 128).transpose(1, 0, 2).reshape(-1)


@pytest.mark.parametrize("rows,cols,tile,kind", [s + (None, None) for s in SHAPES] + [s + (t, None) for s in FORCED for t in "01"] +
                         [s[:2] + (None, s[2]) for s in KINDS])
@pytest.mark.parametrize("fmt", [0, 1])
def test_codes_of_every_producer(rows, cols, tile, kind, fmt, monkeypatch):
    if tile is not None:
        monkeypatch.setenv("LLMQ_QUANT_TILE", tile)
    if kind is not None:
        monkeypatch.setenv("LLMQ_CODES_KERNEL", kind)
    print("codes rows=%d cols=%d tile=%s kind=%s fmt=%d" % (rows, cols, tile, kind, fmt), flush=True)
    n = rows * cols
    gu, _ = swiglu_case(rows, cols, 31 + rows + cols)
    res, _, w = rms_case(rows, cols, 37 + rows + cols)
    h = oracle.swiglu_fwd(synth.bf16_bits(gu))
    rstd = oracle.rms_rstd(synth.bf16_bits(res), EPS).astype(np.float32)
    y = oracle.rmsnorm_apply(synth.bf16_bits(res), synth.bf16_bits(w), rstd)
    x_d, gu_d, w_d, rstd_d = res.to(DEV), gu.to(DEV), w.to(DEV), torch.from_numpy(rstd).to(DEV)
    for bits, plain, slabs in (
            (synth.bf16_bits(res), lambda s, q, qt: llmq.llmq_quantize_fp8(x_d, s, fmt, q, qt), lambda s, q, qt: llmq.llmq_quantize_fp8_slabs(x_d, s, fmt, q, qt)),
            (h, lambda s, q, qt: llmq.llmq_swiglu_fwd_fp8(gu_d, s, fmt, q, qt, None), lambda s, q, qt: llmq.llmq_swiglu_fwd_fp8_slabs(gu_d, s, fmt, q, qt, None)),
            (y, lambda s, q, qt: llmq.llmq_rmsnorm_apply_fp8(x_d, w_d, rstd_d, s, fmt, q, qt, None), lambda s, q, qt: llmq.llmq_rmsnorm_apply_fp8_slabs(x_d, w_d, rstd_d, s, fmt, q, qt, None))):
        sc = oracle.scale(oracle.amax_bf16(bits), fmt)
        if not np.isfinite(sc) or sc == 0:
            continue
        want_q, want_qt = oracle.quantize(bits.reshape(rows, cols), sc, fmt)
        s_d = torch.tensor([float(sc)], dtype=torch.float32, device=DEV)
        calls = [(plain, want_qt.reshape(-1)), (plain, None)] + ([(slabs, _slabs(want_qt, rows, cols))] if tile is not None else [])
        for call, want in calls:
            q, qt = _out(n, torch.uint8, 0xAA), _out(n, torch.uint8, 0xAA)
            call(s_d, q[:n], None if want is None else qt[:n])
            assert np.array_equal(_whole(q, n, 0xAA).cpu().numpy(), want_q.reshape(-1))
            if want is not None:
                assert np.array_equal(_whole(qt, n, 0xAA).cpu().numpy(), want)


@pytest.mark.parametrize("stream", ["0", "1"])
def test_streamed_results(stream, monkeypatch):
    """Results of rows of whole lines are streamed from 96 or 144 MiB on: every such kernel on small shapes, against the oracle."""
    monkeypatch.setenv("LLMQ_STREAM", stream)
    for rows, cols in FORCED:
        for fmt in (0, 1):
            test_codes_of_every_producer(rows, cols, "1", None, fmt, monkeypatch)
    for M, I in ((8, 64), (16, 576), (4, 128), (36, 320)):                      # eight and four rows per lane
        test_swiglu_forward_and_backward_of_ragged_shapes(M, I, None, monkeypatch)
    monkeypatch.setenv("LLMQ_NORM_KERNEL", "2")
    for M in (1, 6):
        for C in (2112, 4096, 5120, 8192, 8256, 16384):
            for with_x in (True, False):
                test_rmsnorm_forward_at_the_edges_of_its_widths(M, C, with_x)
    for C in (2112, 8192, 16384):
        res, x, w = rms_case(7, C, C)
        out = gpu_rmsnorm_fwd(res, x, w, 0)
        in_place = gpu_rmsnorm_fwd(res, x, w, 0, in_place=True)
        assert all(torch.equal(a, b) for a, b in zip(out, in_place))


@pytest.mark.parametrize("rows,cols", [(200, 1300), (129, 257), (300, 1001)])
def test_launches_in_pieces(rows, cols, monkeypatch):
    """More workgroups than a launch may have (a limit of 8 stands for that of the hardware): the same bytes."""
    monkeypatch.setenv("LLMQ_CODES_KERNEL", "2")
    monkeypatch.setenv("LLMQ_MAX_WORKGROUPS", "8")
    for fmt in (0, 1):
        test_codes_of_every_producer(rows, cols, None, None, fmt, monkeypatch)
    M, K, N = rows, cols, rows + 24
    g = torch.Generator().manual_seed(rows)
    x, w = (torch.randn(s, generator=g).to(torch.bfloat16).to(DEV) for s in ((M, K), (N, K)))
    got = []
    for most in ("8", None):
        if most is None:
            monkeypatch.delenv("LLMQ_MAX_WORKGROUPS")
        ws = torch.zeros(llmq.llmq_fp8_linear_workspace_bytes(M, N, K), dtype=torch.uint8, device=DEV)
        y, s, a = torch.zeros((M, N), dtype=torch.bfloat16, device=DEV), torch.zeros(2, device=DEV), torch.full((1,), 7.0, device=DEV)
        llmq.llmq_fp8_linear_fwd(x, w, M, N, K, s[0:1], s[1:2], y, a, ws, llmq.JIT_X | llmq.JIT_W)
        got.append((ws, y.view(torch.int16), s, a))
    assert all(torch.equal(p, q) for p, q in zip(*got))


@pytest.mark.parametrize("M,I", [(1, 1), (3, 9), (5, 511), (4, 512), (7, 513), (130, 1001), (2, 1030), (64, 8), (36, 32), (4, 40)])
@pytest.mark.parametrize("kind", [None, "0", "2"])
def test_swiglu_forward_and_backward_of_ragged_shapes(M, I, kind, monkeypatch):
    if kind is not None:
        monkeypatch.setenv("LLMQ_CODES_KERNEL", kind)
    gu, dh = swiglu_case(M, I, 3 * M + I)
    gu[0, 0] = -90.0                          # below the range of the short sigmoid, and far below
    if I > 8:
        gu[M - 1, I - 1] = -300.0
        gu[0, 8] = -86.5
    gu_d, dh_d, n = gu.to(DEV), dh.to(DEV), M * I
    ws = torch.full((llmq.llmq_swiglu_workspace_bytes(M, I) + PAD,), 0xFF, dtype=torch.uint8, device=DEV)
    f = torch.zeros(4, dtype=torch.float32, device=DEV)
    h, dgu = _out(n, torch.bfloat16, -7.0), _out(2 * n, torch.bfloat16, -7.0)
    wsv = ws[:ws.numel() - PAD]
    llmq.llmq_swiglu_fwd(gu_d, h[:n], 0, f[0:1], f[1:2], wsv)
    llmq.llmq_swiglu_bwd(dh_d, gu_d, dgu[:2 * n], 1, f[2:3], f[3:4], wsv)
    want_h, want_d = oracle.swiglu_fwd(synth.bf16_bits(gu)), oracle.swiglu_bwd(synth.bf16_bits(dh), synth.bf16_bits(gu))
    assert np.array_equal(synth.bf16_bits(_whole(h, n, -7.0)), want_h.reshape(-1))
    assert np.array_equal(synth.bf16_bits(_whole(dgu, 2 * n, -7.0)), want_d.reshape(-1))
    assert f32_bits(f[0:1]) == np_f32_bits(oracle.amax_bf16(want_h)) and f32_bits(f[2:3]) == np_f32_bits(oracle.amax_bf16(want_d))
    assert bool((ws[-PAD:] == 0xFF).all())


@pytest.mark.parametrize("M", [1, 4, 7])
@pytest.mark.parametrize("C", [1, 511, 512, 2047, 2048, 2049, 4096, 4097, 6144, 6145, 8191, 8192, 8200, 12289, 16384, 16385])
@pytest.mark.parametrize("with_x", [True, False])
def test_rmsnorm_forward_at_the_edges_of_its_widths(M, C, with_x):
    res, x, w = rms_case(M, C, M + C)
    x = x if with_x else None
    n = M * C
    ro, y, rstd = _out(n, torch.bfloat16, -7.0), _out(n, torch.bfloat16, -7.0), _out(M, torch.float32, -7.0)
    f = torch.zeros(2, dtype=torch.float32, device=DEV)
    ws = torch.full((llmq.llmq_rmsnorm_workspace_bytes(M) + PAD,), 0xFF, dtype=torch.uint8, device=DEV)
    llmq.llmq_rmsnorm_fwd(res.to(DEV), None if x is None else x.to(DEV), w.to(DEV), EPS, ro[:n] if with_x else None, y[:n], rstd[:M], 0,
                          f[0:1], f[1:2], ws[:ws.numel() - PAD])
    new = oracle.residual_add(synth.bf16_bits(res), synth.bf16_bits(x)) if with_x else synth.bf16_bits(res)
    if with_x:
        assert np.array_equal(synth.bf16_bits(_whole(ro, n, -7.0)), new.reshape(-1))
    want = oracle.rms_rstd(new, EPS)
    got = _whole(rstd, M, -7.0).cpu().numpy()
    assert np.all(np.abs(got - want) <= RSTD_TOL * want)
    want_y = oracle.rmsnorm_apply(new, synth.bf16_bits(w), got)          # the formula with the statistic the kernel found
    assert np.array_equal(synth.bf16_bits(_whole(y, n, -7.0)), want_y.reshape(-1))
    assert f32_bits(f[0:1]) == np_f32_bits(oracle.amax_bf16(want_y))
    assert bool((ws[-PAD:] == 0xFF).all())


@pytest.mark.parametrize("C", [17, 500, 2047, 2049, 4100, 8193, 16383, 16400])
@pytest.mark.parametrize("with_x", [True, False])
def test_rmsnorm_absmax_of_rows_whose_squares_underflow(C, with_x):
    """eps = 0 and a row of 2^-80: its statistic and its results are infinite, and the absmax is that of what is stored,
    whatever a kernel computes behind the end of a row."""
    M, n = 5, 5 * C
    res, _, w = rms_case(M, C, C)
    res[3] = 2.0 ** -80
    x = torch.zeros((M, C), dtype=torch.bfloat16) if with_x else None
    w.abs_()
    y, ro = _out(n, torch.bfloat16, -7.0), _out(n, torch.bfloat16, -7.0)
    rstd, f = torch.zeros(M, dtype=torch.float32, device=DEV), torch.zeros(4, dtype=torch.float32, device=DEV)
    ws = torch.empty(llmq.llmq_rmsnorm_workspace_bytes(M), dtype=torch.uint8, device=DEV)
    llmq.llmq_rmsnorm_fwd(res.to(DEV), None if x is None else x.to(DEV), w.to(DEV), 0.0, ro[:n] if with_x else None, y[:n], rstd, 0, f[0:1], f[1:2], ws)
    stored = _whole(y, n, -7.0).view(M, C)
    assert bool(torch.isinf(stored[3]).all()) and bool(torch.isfinite(stored[torch.arange(M) != 3]).all())
    llmq.llmq_amax(stored.reshape(-1).clone(), 0, f[2:3], f[3:4], torch.empty(llmq.llmq_amax_workspace_bytes(), dtype=torch.uint8, device=DEV))
    assert f32_bits(f[0:1]) == f32_bits(f[2:3]) == 0x7F800000 and f32_bits(f[1:2]) == f32_bits(f[3:4]) == 0


@pytest.mark.parametrize("k", range(9))
def test_every_remainder_of_rows_and_columns(k, monkeypatch):
    """The last vector of a row holds 1 to 8 elements (of a tensor narrower than a vector, one element too few for the load that
    ends with the row), the last piece of a transposed row 1 to 16 codes."""
    monkeypatch.setenv("LLMQ_CODES_KERNEL", "2")
    for rows, cols in ((48 + k, 128 + k), (64 + 8 + k, 120 + k), (5, max(1, k)), (130 + 2 * k, 8 + k)):
        test_codes_of_every_producer(rows, cols, None, "2", k % 2, monkeypatch)
    for M, I in ((5, 512 + k), (6, 8 + k), (3, max(1, k))):
        test_swiglu_forward_and_backward_of_ragged_shapes(M, I, "2", monkeypatch)
    for C in (max(1, k), 8 + k, 2048 + k):
        for with_x in (True, False):
            test_rmsnorm_forward_at_the_edges_of_its_widths(5, C, with_x)


@pytest.mark.parametrize("rows,cols", [(128, 128), (256, 384)])
@pytest.mark.parametrize("fmt", [0, 1])
def test_whole_tiles_that_are_no_slabs(rows, cols, fmt, monkeypatch):
    """128 x 128 tiles of tensors whose width is no multiple of the 256 columns that slabs come in."""
    monkeypatch.setenv("LLMQ_QUANT_TILE", "1")
    test_codes_of_every_producer(rows, cols, None, None, fmt, monkeypatch)


@pytest.mark.parametrize("rows,cols", [(12545, 8001), (12551, 8008), (9579, 7104)])
def test_large_ragged_codes_are_those_of_their_bands(rows, cols):
    """Above 66M elements in whole vectors (quantize, rows that do not start at lines: 40M) the lanes of the guarded tile lie differently: the
    codes are those of bands of rows by themselves."""
    x = torch.randn(rows, cols, device=DEV).to(torch.bfloat16)
    w = torch.randn(cols, device=DEV).to(torch.bfloat16)
    rstd = torch.rand(rows, device=DEV) + 0.5
    scale = torch.full((1,), 90.0, device=DEV)

    def codes(a, b):
        n = (b - a) * cols
        out = [torch.zeros(n, dtype=torch.uint8, device=DEV) for _ in range(4)]
        llmq.llmq_quantize_fp8(x[a:b], scale, 0, out[0].view(b - a, cols), out[1])
        llmq.llmq_rmsnorm_apply_fp8(x[a:b], w, rstd[a:b], scale, 0, out[2].view(b - a, cols), out[3], None)
        return out[0].view(b - a, cols), out[1].view(cols, b - a), out[2].view(b - a, cols), out[3].view(cols, b - a)

    q, qt, n, nt = codes(0, rows)
    assert torch.equal(qt, q.t()) and torch.equal(nt, n.t())
    for a in range(0, rows, 4000):
        b = min(rows, a + 4000)
        bq, _, bn, _ = codes(a, b)
        assert torch.equal(q[a:b], bq) and torch.equal(n[a:b], bn)
