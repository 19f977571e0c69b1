"""The 128 x 128 tile with four LDS stages gives the bytes of the one with two, for every number of K steps around the
number of stages, in every layout and with guarded edges."""
import pytest
import torch

import oracle
from gpu_common import assert_gemm_close
from test_gpu_gemm import _rand_codes, _run_gemm
from test_gpu_gemm_tmajor import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [128, 256, 384, 512, 640, 1024, 1152, 272, 528])
@pytest.mark.parametrize("R,C", [(256, 384), (200, 136)])
def test_four_stages_give_the_same_bytes(R, C, T, monkeypatch):
    monkeypatch.setenv("LLMQ_GEMM_TILE", "2x2")
    monkeypatch.setenv("LLMQ_GEMM_EDGE_TILE", "2x2")
    A, B = _rand_codes((R, T), 1, R + T), _rand_codes((C, T), 0, C + T)
    y, S = oracle.gemm_tn(A, 1, B, 0, 1.9, 0.7)
    c0 = torch.full((R, C), 3.0, dtype=torch.bfloat16, device="cuda:0")
    got = {}
    for deep in "01":
        monkeypatch.setenv("LLMQ_GEMM_DEEP", deep)
        print("deep=%s R=%d C=%d T=%d" % (deep, R, C, T), flush=True)
        c, am = _run_gemm(A, 1, B, 0, 1.9, 0.7, want_amax=True)
        assert_gemm_close(c, y, S, "deep " + deep)
        assert am.item() == c.float().abs().max().item()
        outs = [c, _run_gemm(A, 1, B, 0, 1.9, 0.7, accumulate=True, c_init=c0)[0]]
        outs += [_run(A, 1, ta, B, 0, tb, 1.9, 0.7)[0] for ta, tb in ((False, True), (True, True))]
        got[deep] = [o.view(torch.int16) for o in outs]
    for a, b in zip(got["0"], got["1"]):
        assert torch.equal(a, b)


@pytest.mark.parametrize("T", [1920, 2048, 2064, 3968, 4096, 4112])
def test_four_and_eight_waves_give_the_same_bytes(T, monkeypatch):
    """Contractions on either side of the lines between eight and four waves (operands in rows, T-major)."""
    test_four_stages_give_the_same_bytes(*((256, 384) if T % 128 == 0 else (200, 136)), T, monkeypatch)
