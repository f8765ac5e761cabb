"""Block decodes with a frame on several compute units (few frames of a long
code) against the one-unit decoder, bit for bit: the shortest code of the rule,
a last member with a partial wavefront, the longest codes, rows of weight 6 and
9, one frame to the largest batch of the rule and the first one past it; and
replays of a captured decode."""
import numpy as np
import pytest
import torch

import synth
from paper_1204_0334_amd import ldpc

pytestmark = pytest.mark.gpu


def code(L, p):
    a = np.random.default_rng(L * p).integers(0, p, size=(3, L))
    a[0, 0], a[1, 1], a[2, L - 1] = 0, p - 1, p - 1
    return ldpc.Graph.qc(a, p)


def channel(L, p, gamma):
    sigma2 = synth.ebn0_to_sigma2({6: 1.6, 9: 2.6}[L], 1.0 - 3 / L)
    llr = synth.bpsk_awgn_llr(None, sigma2, 40 + p, gamma=gamma, n=L * p)
    llr[0, :7] = [np.inf, -np.inf, 0.0, -0.0, 1e30, -1e-30, 40.0]
    return torch.tensor(llr, dtype=torch.float32, device="cuda")


@pytest.mark.parametrize("L,p,gamma", [(6, 1800, 1), (6, 2049, 3), (6, 3060, 1), (6, 3072, 16), (6, 3072, 17),
                                       (9, 1801, 2), (9, 2048, 16)])
def test_equals_one_unit(monkeypatch, L, p, gamma):
    g = code(L, p)
    llr = channel(L, p, gamma)
    w = torch.tensor(np.random.default_rng(1).uniform([0.7, 0.0], [0.9, 0.1], size=(6, 3 * L, 2)),
                     dtype=torch.float32, device="cuda")
    runs = [lambda T=T, e=e: ldpc.decode(g, llr, T, early_stop=e)
            for T, e in ((1, True), (2, True), (30, True), (1, False), (7, False))]
    runs += [lambda e=e: ldpc.nms_decode(g, llr, w, early_stop=e) for e in (True, False)]
    for run in runs:
        monkeypatch.setenv("LDPC_BLOCK_PATH", "onchip")
        want = [x.clone() for x in run()]
        monkeypatch.delenv("LDPC_BLOCK_PATH")
        for a, b in zip(want, run()):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


def test_replays(monkeypatch):
    g = code(6, 3060)
    llr = channel(6, 3060, 2)
    ws = ldpc.workspace(g, 2, 20)
    out = tuple(torch.empty(s, dtype=d, device="cuda") for s, d in
                (((2, g.n), torch.float32), ((2, g.n), torch.uint8), ((2,), torch.int32), ((2,), torch.uint8)))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        ldpc.decode(g, llr, 20, early_stop=True, out=out, ws=ws)
    for seed in range(3):
        llr.copy_(channel(6, 3060, 2) * (1.0 + 0.1 * seed))
        graph.replay()
        torch.cuda.synchronize()
        got = [x.clone() for x in out]
        want = ldpc.decode(g, llr, 20, early_stop=True)
        torch.cuda.synchronize()
        for a, b in zip(want, got):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
