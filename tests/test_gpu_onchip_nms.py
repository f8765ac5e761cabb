"""Learned min-sum decoding of the codes with one posterior sum per variable
(rows of weight 9, 18 and 24) on one compute unit: equal to the message
packages bit for bit.  The codes of test_gpu_onchip_wide; a stop after the
first iteration, in the middle and never; weights of either sign and offsets
that cancel a whole message."""
import numpy as np
import pytest
import torch

from paper_1204_0334_amd import ldpc

from test_gpu_onchip_wide import CODES, code

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("J,L,p", CODES)
def test_equals_the_packages(monkeypatch, J, L, p):
    monkeypatch.delenv("LDPC_BLOCK_PATH", raising=False)
    _, llr, g = code(J, L, p, 7, 3.5 + (L > 9))
    llr[0, :7] = [np.inf, -np.inf, 0.0, -0.0, 1e30, -1e-30, 40.0]
    llr[1], llr[2] = -0.0, 40.0
    x = torch.tensor(llr, dtype=torch.float32, device="cuda")
    rng = np.random.default_rng(1)
    w = rng.uniform([0.7, 0.0], [0.9, 0.1], size=(20, J * L, 2))
    w[1, ::5, 0] *= -1.0
    w[2, ::7, 1] = 50.0
    w = torch.tensor(w, dtype=torch.float32, device="cuda")
    for T, early in ((1, False), (1, True), (2, True), (3, False), (20, True), (20, False)):
        print(f"[gpu] {J}x{L} p={p} learned T={T} early={early}", flush=True)
        ldpc.timing_read()
        ldpc.timing_enable(True)
        got = ldpc.nms_decode(g, x, w[:T].contiguous(), early_stop=early)
        torch.cuda.synchronize()
        ldpc.timing_enable(False)
        t = ldpc.timing_read()
        assert t["onchip_decode"][0] == 1 and t["check_node"][0] == 0, t
        monkeypatch.setenv("LDPC_BLOCK_PATH", "packages")
        want = ldpc.nms_decode(g, x, w[:T].contiguous(), early_stop=early)
        monkeypatch.delenv("LDPC_BLOCK_PATH")
        for a, b in zip(got, want):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
