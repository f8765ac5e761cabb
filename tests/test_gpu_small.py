"""Short codes with a frame's packages in LDS against the launch-per-phase
form, bit for bit: rows of weight 18, 24 and 30, one base row, a base column
without edges, an irregular base of 5 rows, circulants of 1, as many edges as the
rule admits, frames from 1 to a few rounds of the chip."""
import numpy as np
import pytest
import torch

import synth
from paper_1204_0334_amd import ldpc

pytestmark = pytest.mark.gpu


def base(kind, p):
    rng = np.random.default_rng(p)
    if kind == "irregular":
        a = rng.integers(0, p, size=(5, 12))
        a[rng.random((5, 12)) < 0.4] = -1
        a[:, 0] = -1                       # a base column without edges
        a[0, 1:3] = 0                      # a row of weight 2 at least
        return a
    J, L = kind
    return rng.integers(0, p, size=(J, L))


@pytest.mark.parametrize("kind,p,gamma", [((3, 18), 1, 3), ((3, 18), 36, 128), ((3, 18), 63, 700), ((4, 24), 60, 33),
                                          ((1, 3), 40, 5), ((2, 30), 101, 17), ((5, 8), 129, 64), ((8, 9), 7, 1),
                                          ((3, 11), 248, 257), ("irregular", 33, 256), ("irregular", 200, 9)])
def test_equals_the_phase_launches(monkeypatch, kind, p, gamma):
    a = base(kind, p)
    g = ldpc.Graph.qc(a, p)
    n = a.shape[1] * p
    sigma2 = synth.ebn0_to_sigma2(3.0, max(0.3, 1.0 - a.shape[0] / a.shape[1]))
    llr = synth.bpsk_awgn_llr(None, sigma2, 70 + p, gamma=gamma, n=n).astype(np.float32)
    llr[0, :3] = [np.inf, -0.0, -1e30]
    llr = torch.tensor(llr, device="cuda")
    for T, early in ((1, True), (2, True), (25, True), (1, False), (8, False)):
        monkeypatch.setenv("LDPC_BLOCK_PATH", "packages")
        want = [x.clone() for x in ldpc.decode(g, llr, T, early_stop=early)]
        monkeypatch.delenv("LDPC_BLOCK_PATH")
        for x, y in zip(want, ldpc.decode(g, llr, T, early_stop=early)):
            assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), (T, early)
