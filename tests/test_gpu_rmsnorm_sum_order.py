"""The row statistic of the RMSNorm forward kernels is a binary32 sum in an order that depends on the width alone: the
same bits from every kernel, batch and release, and with them the same y and the same FP8 codes of everything behind."""
import numpy as np
import pytest
import torch

from paper_2512_15306_amd import llmq, synth
from gpu_common import DEV

pytestmark = pytest.mark.gpu
EPS = np.float32(1e-6)


def _rstd(bits, C):
    """Lane l of `lanes` adds up the vectors of eight (or, unit = 1, the elements) l, l + lanes, ..., a butterfly the 64 lanes
    of a wave, and the waves' sums follow one after the other.  The square of a BF16 number is exact in binary32, so a
    fused multiply-add is the binary32 sum of that square."""
    if C % 8 == 0 and C <= 8192:
        unit, lanes = 8, 64
    elif C <= 2048 or C > 16384:
        unit, lanes = 1, 64
    else:
        unit, lanes = 8, 256
    f = (bits.astype(np.uint32) << 16).view(np.float32)
    f = np.concatenate([f, np.zeros((len(f), -C % unit), dtype=np.float32)], axis=1)       # adding 0 changes nothing
    ss = np.zeros((len(f), lanes), dtype=np.float32)
    for first in range(0, C, lanes * unit):
        part = f[:, first:first + lanes * unit]
        for e in range(unit):
            v = part[:, e::unit]
            ss[:, :v.shape[1]] = ss[:, :v.shape[1]] + v * v
    ss = ss.reshape(len(f), lanes // 64, 64)
    for off in (32, 16, 8, 4, 2, 1):
        ss = ss + ss[:, :, np.arange(64) ^ off]
    total = ss[:, 0, 0]
    for wave in range(1, lanes // 64):
        total = total + ss[:, wave, 0]
    return np.float32(1.0) / np.sqrt(total / np.float32(C) + EPS)


@pytest.mark.parametrize("C", [1, 17, 100, 264, 2040, 2047, 2048, 2049, 2056, 3072, 4095, 4096, 4104, 5120, 6150, 8184, 8191, 8192, 8193, 8200, 12296,
                               16383, 16384, 16385])
@pytest.mark.parametrize("M", [1, 6])
@pytest.mark.parametrize("kernel", ["0", "1", "2"])
def test_row_sum_order(M, C, kernel, monkeypatch):
    monkeypatch.setenv("LLMQ_NORM_KERNEL", kernel)         # where the width allows it
    g = torch.Generator().manual_seed(C + M)
    res = (torch.randn(M, C, generator=g) * 1.3).to(torch.bfloat16)
    res[:, torch.randint(0, C, (max(1, C // 200),), generator=g)] *= 50.0
    x = (torch.randn(M, C, generator=g) * 0.4).to(torch.bfloat16)
    w = torch.ones(C, dtype=torch.bfloat16)
    f = torch.zeros(2, device=DEV)
    ws = torch.empty(llmq.llmq_rmsnorm_workspace_bytes(M), dtype=torch.uint8, device=DEV)
    for add in (False, True):
        rstd, y = torch.zeros(M, device=DEV), torch.empty((M, C), dtype=torch.bfloat16, device=DEV)
        out = torch.empty((M, C), dtype=torch.bfloat16, device=DEV) if add else None
        llmq.llmq_rmsnorm_fwd(res.to(DEV), x.to(DEV) if add else None, w.to(DEV), float(EPS), out, y, rstd, 0, f[0:1], f[1:2], ws)
        summed = synth.bf16_bits(out if add else res).reshape(M, C)
        assert np.array_equal(rstd.cpu().numpy().view(np.uint32), _rstd(summed, C).view(np.uint32)), "C=%d add=%s" % (C, add)
