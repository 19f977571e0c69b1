"""The compiled module behind the calls of a training step: it takes the plain case, gives what the ctypes path gives, and leaves
everything else, errors included, to that path."""
import os
import shutil
import subprocess
import sys

import pytest
import torch

from paper_2512_15306_amd import llmq

DEV = "cuda:0"
M, N, K = 128, 256, 384


def test_module_is_built_and_declines_what_is_not_plain():
    f = llmq._fast
    assert hasattr(f, "__file__") and f.__file__.endswith("_binding.so")
    cpu = torch.zeros((4, 8), dtype=torch.bfloat16)
    one = torch.zeros(1)
    assert f.amax(cpu, 0, one, one, torch.zeros(4096, dtype=torch.uint8)) is None
    assert f.amax() is None and f.linear_fwd(None, None) is None
    with pytest.raises(ValueError, match="must live on the GPU"):
        llmq.llmq_amax(cpu, 0, one, one, torch.zeros(4096, dtype=torch.uint8))


def _package(tmp_path, *files):
    """The binding's Python part in a package of its own, with these files beside it"""
    pkg = tmp_path / "pkg"
    pkg.mkdir()
    (pkg / "__init__.py").write_text("")
    for f in ("llmq.py",) + files:
        shutil.copy(os.path.join(os.path.dirname(llmq.__file__), f), pkg / f)
    return pkg


def _python(tmp_path, code):
    return subprocess.run([sys.executable, "-W", "always", "-c", code], cwd=tmp_path, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)


def test_another_library_gets_every_call(tmp_path):
    """A program that points LIB_PATH at another build of the library has that one called throughout: the module, which calls the one
    beside it, is left out."""
    other = tmp_path / "other"
    other.mkdir()
    shutil.copy(llmq.LIB_PATH, other / "libllmq.so")
    root = os.path.dirname(os.path.dirname(os.path.abspath(llmq.__file__)))
    code = """if 1:
        import sys; sys.path.insert(0, %r)
        from paper_2512_15306_amd import llmq
        assert "_binding" not in "".join(m for m in sys.modules if m.startswith("paper")), "loaded before any call"
        path = llmq.LIB_PATH
        llmq.LIB_PATH = %r
        f = llmq._fast.amax
        print(type(llmq._fast).__name__, llmq.lib()._name, f(1, 2))
        llmq._lib, llmq._fast, llmq.LIB_PATH = None, llmq._UnloadedBinding(), path
        print(llmq._fast.__file__)
        llmq.llmq_amax_workspace_bytes()
        """
    p = _python(tmp_path, code % (root, str(other / "libllmq.so")))
    lines = [l for l in p.stdout.splitlines() if "amdgpu.ids" not in l]
    assert p.returncode == 0 and lines[0] == "_NoBinding %s None" % (other / "libllmq.so") and lines[1].endswith("_binding.so"), p.stdout


def test_a_module_that_does_not_load_is_reported(tmp_path):
    """Not a word where the module is not built; a warning, and the ctypes path, where it is and cannot be loaded."""
    pkg = _package(tmp_path, "libllmq.so")
    code = "from pkg import llmq; print(llmq._fast.amax(1), type(llmq._fast).__name__)"
    p = _python(tmp_path, code)
    assert p.returncode == 0 and "None _NoBinding" in p.stdout and "RuntimeWarning" not in p.stdout, p.stdout
    (pkg / "_binding.so").write_text("of another build")
    p = _python(tmp_path, code)
    assert p.returncode == 0 and "None _NoBinding" in p.stdout and "RuntimeWarning" in p.stdout and "does not load" in p.stdout, p.stdout
    os.remove(pkg / "libllmq.so")
    p = _python(tmp_path, code)
    assert p.returncode != 0 and "libllmq.so is not built" in p.stdout, p.stdout


class Calls:
    """Every call once, on the same inputs."""

    def __init__(self):
        g = torch.Generator(device=DEV).manual_seed(5)
        bf = lambda *s: torch.randn(s, generator=g, device=DEV).to(torch.bfloat16)
        self.x, self.w, self.dy, self.gu, self.nw = bf(M, K), bf(N, K), bf(M, N), bf(M, 2 * N), bf(K)
        self.outs = []

    def _new(self, *shape, dtype=torch.bfloat16):
        t = torch.zeros(shape, dtype=dtype, device=DEV)
        self.outs.append(t)
        return t

    def run(self):
        self.outs = []
        f32 = lambda n=1: self._new(n, dtype=torch.float32)
        u8 = lambda *s: self._new(*s, dtype=torch.uint8)
        ws = torch.zeros(llmq.llmq_fp8_linear_workspace_bytes(M, N, K), dtype=torch.uint8, device=DEV)
        sx, sw, sd = f32(), f32(), f32()
        llmq.llmq_fp8_linear_fwd(self.x, self.w, M, N, K, sx, sw, self._new(M, N), f32(), ws, llmq.JIT_X | llmq.JIT_W)
        llmq.llmq_fp8_linear_dgrad(self.dy, None, M, N, K, sd, sw, llmq.E5M2, self._new(M, K), None, ws, llmq.JIT_DY | llmq.REUSE_W)
        for acc in (False, True):
            llmq.llmq_fp8_linear_wgrad(None, None, M, N, K, sd, sx, llmq.E5M2, self._new(N, K), acc, ws, llmq.REUSE_X | llmq.REUSE_DY)
        a, s, aws = f32(), f32(), torch.zeros(4096, dtype=torch.uint8, device=DEV)
        llmq.llmq_amax(self.x, 0, a, s, aws)
        llmq.llmq_quantize_fp8(self.x, s, 0, u8(M, K), u8(K, M))
        llmq.llmq_quantize_fp8(self.x, s, 0, u8(M, K), None)
        llmq.llmq_quantize_fp8_slabs(self.gu, s, 1, u8(M, 2 * N), u8(2 * N, M))
        llmq.llmq_bf16_gemm_tn(self.x, self.w, self._new(M, N))
        sws = torch.zeros(llmq.llmq_swiglu_workspace_bytes(M, N), dtype=torch.uint8, device=DEV)
        llmq.llmq_swiglu_fwd(self.gu, self._new(M, N), 0, a, s, sws)
        llmq.llmq_swiglu_fwd_fp8(self.gu, s, 0, u8(M, N), u8(N, M), self._new(M, N))
        llmq.llmq_swiglu_fwd_fp8_slabs(self.gu, s, 0, u8(M, N), u8(N, M))
        llmq.llmq_swiglu_bwd(self.dy, self.gu, self._new(M, 2 * N), 1, f32(), None, sws)
        nws = torch.zeros(llmq.llmq_rmsnorm_workspace_bytes(M), dtype=torch.uint8, device=DEV)
        rstd, ny, ns = f32(M), f32(), f32()
        llmq.llmq_rmsnorm_fwd(self.x, self.x, self.nw, 1e-6, self._new(M, K), self._new(M, K), rstd, 0, ny, ns, nws)
        llmq.llmq_rmsnorm_fwd(self.x, None, self.nw, 1e-6, None, self._new(M, K), rstd, 0, ny, ns, nws)
        llmq.llmq_rmsnorm_apply_fp8(self.x, self.nw, rstd, ns, 0, u8(M, K), u8(K, M), self._new(M, K))
        llmq.llmq_rmsnorm_apply_fp8_slabs(self.gu, self.gu[0], rstd, ns, 0, u8(M, 2 * N), u8(2 * N, M))
        return [t.view(torch.uint8).clone() for t in self.outs]


@pytest.mark.gpu
def test_same_as_the_ctypes_path_on_any_stream(monkeypatch):
    calls = Calls()
    fast = calls.run()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        on_side = calls.run()
    side.synchronize()
    monkeypatch.setattr(llmq, "_fast", llmq._NoBinding())
    slow = calls.run()
    assert len(fast) == len(slow) > 30
    for a, b, c in zip(fast, on_side, slow):
        assert torch.equal(a, c) and torch.equal(b, c)


@pytest.mark.gpu
def test_errors_are_those_of_the_ctypes_path(monkeypatch):
    x = torch.zeros((M, K), dtype=torch.bfloat16, device=DEV)
    s, q = torch.ones(1, device=DEV), torch.zeros((M, K), dtype=torch.uint8, device=DEV)
    aws = torch.zeros(4096, dtype=torch.uint8, device=DEV)
    big = torch.zeros((M, 2 * K), dtype=torch.bfloat16, device=DEV)
    ws = torch.zeros(16, dtype=torch.uint8, device=DEV)
    bad = [lambda: llmq.llmq_amax(x.float(), 0, s, s, aws), lambda: llmq.llmq_amax(x.cpu(), 0, s, s, aws), lambda: llmq.llmq_amax(x.t(), 0, s, s, aws),
           lambda: llmq.llmq_amax(x, 7, s, s, aws), lambda: llmq.llmq_amax(x, 0, None, s, aws), lambda: llmq.llmq_amax(x, 0, s, s, aws[:16]),
           lambda: llmq.llmq_amax(x.view(-1)[1:], 0, s, s, aws), lambda: llmq.llmq_amax(x, 0, s, s, None), lambda: llmq.llmq_amax(x, "0", s, s, aws),
           lambda: llmq.llmq_quantize_fp8(x, s, 0, q[:1], None), lambda: llmq.llmq_quantize_fp8(x.view(-1), s, 0, q, None),
           lambda: llmq.llmq_quantize_fp8_slabs(x[:100], s, 0, q[:100], q[:100]), lambda: llmq.llmq_quantize_fp8_slabs(x, s, 0, q, None),
           lambda: llmq.llmq_bf16_gemm_tn(x, big, x), lambda: llmq.llmq_swiglu_fwd(x[:, :3], x, 0, s, s, ws), lambda: llmq.llmq_swiglu_fwd(big, x[:1], 0, s, s, ws),
           lambda: llmq.llmq_rmsnorm_fwd(x, None, x[0], 0, None, x, s, 0, s, s, ws), lambda: llmq.llmq_rmsnorm_apply_fp8(x, x[0, :8], s, s, 0, q, None),
           lambda: llmq.llmq_fp8_linear_fwd(x, x, M, N, K, s, s, x, None, ws, 0), lambda: llmq.llmq_fp8_linear_fwd(x, x, M, N, K, s, s, x, None, None, 0),
           lambda: llmq.llmq_fp8_linear_fwd(x, x, 1 << 40, N, K, s, s, x, None, ws, 0), lambda: llmq.llmq_fp8_linear_fwd(x, x, M, N, K, s, s, x, None, ws, 1 << 20)]
    def outcome(f):
        try:
            f()
        except Exception as e:                  # noqa: BLE001 (whatever it is, it has to be the same)
            return type(e), str(e)
        return None
    got = [outcome(f) for f in bad]
    monkeypatch.setattr(llmq, "_fast", llmq._NoBinding())
    want = [outcome(f) for f in bad]
    assert got == want and all(w is not None for w in want)
