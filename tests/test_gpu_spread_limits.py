"""Frames on several compute units when members give up their waits
(LDPC_SPREAD_TRIES sets how soon): the frame is decoded once more by its last
member, with the same results bit for bit.  And decodes in place, which other
kernels take."""
import numpy as np
import pytest
import torch

from paper_1204_0334_amd import ldpc

from test_gpu_decode import qc_case

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(autouse=True)
def default_path(monkeypatch):
    monkeypatch.delenv("LDPC_BLOCK_PATH", raising=False)
    monkeypatch.delenv("LDPC_SPREAD_TRIES", raising=False)


def case(L, p, gamma):
    a, llr, _ = qc_case(3, L, p, 5, gamma, {6: 1.8, 9: 2.8, 18: 3.8}[L], 70 + p)
    w = np.random.default_rng(1).uniform([0.7, 0.0], [0.9, 0.1], size=(6, 3 * L, 2))
    return ldpc.Graph.qc(a, p), torch.from_numpy(llr).to(DEV), torch.tensor(w, dtype=torch.float32, device=DEV)


@pytest.mark.parametrize("L,p,gamma", [(6, 1800, 3), (6, 3060, 16), (6, 4096, 2), (9, 2048, 5), (9, 3073, 1),
                                       (18, 1537, 16), (18, 3600, 2)])
def test_frames_that_members_give_up(monkeypatch, L, p, gamma):
    g, llr, w = case(L, p, gamma)
    runs = [lambda T=T, e=e: ldpc.decode(g, llr, T, early_stop=e)
            for T, e in ((1, True), (2, True), (3, True), (25, True), (1, False), (6, False))]
    runs += [lambda e=e: ldpc.nms_decode(g, llr, w, early_stop=e) for e in (True, False)]
    for i, run in enumerate(runs):
        want = [x.clone() for x in run()]
        for tries in (0, 1, 3, 300):
            print(f"[gpu] spread 3x{L} p={p} gamma={gamma} run {i} tries={tries}", flush=True)
            monkeypatch.setenv("LDPC_SPREAD_TRIES", str(tries))
            got = run()
            monkeypatch.delenv("LDPC_SPREAD_TRIES")
            for a, b in zip(want, got):
                assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.parametrize("L,p,gamma", [(6, 3060, 2), (18, 3600, 3)])
def test_in_place(L, p, gamma):
    # posteriors over the LLRs: results of the kernels that read a frame's LLRs first
    g, llr, _ = case(L, p, gamma)
    for T, early in ((4, False), (25, True)):
        x = torch.cat([llr, llr])   # too many rows for one call: the second half stays
        want = ldpc.decode(g, torch.cat([llr] * 17)[:17], T, early_stop=early)   # 17 frames: one unit each, or launches
        out = (x[:gamma], torch.empty_like(want[1][:gamma]), torch.empty_like(want[2][:gamma]),
               torch.empty_like(want[3][:gamma]))
        got = ldpc.decode(g, x[:gamma], T, early_stop=early, out=out)
        for a, b in zip(got, want):
            assert torch.equal(a.view(torch.uint8), b[:gamma].contiguous().view(torch.uint8))
        assert torch.equal(x[gamma:], llr)


def test_in_place_in_a_plan():
    g, llr, _ = case(18, 1700, 4)
    plan = ldpc.Plan([g], [4], 20, early_stop=True)
    ws, outs = plan.workspace(), plan.outputs()
    want = ldpc.decode(g, torch.cat([llr] * 5)[:17], 20, early_stop=True)
    x = llr.clone()
    outs[0] = (x, *outs[0][1:])
    plan.decode([x], outs=outs, ws=ws)
    for a, b in zip(outs[0], want):
        assert torch.equal(a.view(torch.uint8), b[:4].contiguous().view(torch.uint8))
