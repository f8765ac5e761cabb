"""Channel LLRs and error counts on the GPU at the sizes where their vector
accesses begin and end: rows shorter than one access, rows that start off its
boundary, a last partial block."""
import numpy as np
import pytest
import torch

import synth
from paper_1204_0334_amd import ldpc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3, 4, 5, 1000, 1023, 1028])
def test_channel(n):
    sigma2 = synth.ebn0_to_sigma2(2.0, 0.5)
    gpu = ldpc.awgn_llr(n, 9, sigma2, 99, 5, device="cuda").cpu().numpy()
    cpu = synth.bpsk_awgn_llr(None, sigma2, 99, frame0=5, gamma=9, n=n)
    ulp = np.abs(gpu.view(np.int32).astype(np.int64) - cpu.view(np.int32).astype(np.int64))
    assert ulp.max() <= 1
    assert (ulp == 0).mean() > 0.999


@pytest.mark.parametrize("n", [1, 7, 15, 16, 17, 31, 32, 47, 4096, 5003])
@pytest.mark.parametrize("start", [0, 1, 15])
def test_error_counts(n, start):
    rng = np.random.default_rng(n + start)
    b = np.where(rng.random((5, n)) < 0.3, rng.integers(1, 256, size=(5, n)), 0).astype(np.uint8)
    b[3] = 0
    buf = torch.full((start + 5 * n + 32,), 255, dtype=torch.uint8, device="cuda")
    bits = buf[start:start + 5 * n].view(5, n)
    bits.copy_(torch.from_numpy(b))
    totals = torch.zeros((2,), dtype=torch.int64, device="cuda")
    per = ldpc.count_errors(bits, totals=totals)
    want = (b != 0).sum(1)
    assert np.array_equal(per.cpu().numpy(), want)
    assert totals.cpu().tolist() == [int(want.sum()), int((want > 0).sum())]
