"""Frames of codes too long for one compute unit on several (up to 16 frames):
equal to the message packages bit for bit, so that a frame's results do not
depend on its batch, and against the FP64 references with the tolerances of
test_gpu_decode and test_gpu_nnms.  Rows of weight 6, 9 and 18, the shortest
and longest codes of each, a last member with a partial wavefront, one frame to
the largest batch; sum-product and learned min-sum."""
import numpy as np
import pytest
import torch

import oracle
from oracle import nnms as ref_nnms
from paper_1204_0334_amd import ldpc

from test_gpu_decode import check_parity, gpu_decode, qc_case
from test_gpu_nnms import check_decode, gpu_nms, rand_weights, ref_graph

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
EBN0 = {6: 1.8, 9: 2.8, 18: 3.9}


@pytest.fixture(autouse=True)
def default_path(monkeypatch):
    monkeypatch.delenv("LDPC_BLOCK_PATH", raising=False)


def case(L, p, gamma):
    a, llr, _ = qc_case(3, L, p, 5, gamma, EBN0[L], 70 + p)
    llr[0, :7] = [np.inf, -np.inf, 0.0, -0.0, 1e30, -1e-30, 40.0]
    return a, llr, ldpc.Graph.qc(a, p)


def launches(run):
    """The result of run() and whether it took the launches of the packages."""
    ldpc.timing_read()
    ldpc.timing_enable(True)
    out = run()
    torch.cuda.synchronize()
    ldpc.timing_enable(False)
    t = ldpc.timing_read()
    assert (t["check_node"][0] > 0) != (t["onchip_decode"][0] > 0)
    return out, t["check_node"][0] > 0


@pytest.mark.parametrize("L,p,gamma", [(6, 3073, 3), (6, 3090, 1), (6, 4096, 16), (9, 3073, 2), (9, 4096, 5),
                                       (18, 1537, 16), (18, 1700, 1), (18, 3600, 3), (18, 4096, 2)])
def test_equals_the_packages(monkeypatch, L, p, gamma):
    _, llr, g = case(L, p, gamma)
    x = torch.tensor(llr, dtype=torch.float32, device=DEV)
    w = torch.tensor(np.random.default_rng(1).uniform([0.7, 0.0], [0.9, 0.1], size=(6, 3 * L, 2)),
                     dtype=torch.float32, device=DEV)
    runs = [lambda T=T, e=e: ldpc.decode(g, x, T, early_stop=e)
            for T, e in ((1, True), (2, True), (30, True), (1, False), (2, False), (7, False))]
    runs += [lambda e=e: ldpc.nms_decode(g, x, w, early_stop=e) for e in (True, False)]
    for i, run in enumerate(runs):
        print(f"[gpu] 3x{L} p={p} gamma={gamma} run {i}", flush=True)
        got, packages = launches(run)
        assert not packages
        monkeypatch.setenv("LDPC_BLOCK_PATH", "packages")
        want, packages = launches(run)
        monkeypatch.delenv("LDPC_BLOCK_PATH")
        assert packages
        for a, b in zip(got, want):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.parametrize("L,p", [(6, 3073), (9, 3073), (18, 1537)])
def test_a_frame_does_not_depend_on_its_batch(L, p):
    _, llr, g = case(L, p, 17)
    x = torch.tensor(llr, dtype=torch.float32, device=DEV)
    for T, early in ((5, False), (20, True)):
        all_, packages = launches(lambda: ldpc.decode(g, x, T, early_stop=early))
        assert packages
        few = ldpc.decode(g, x[:3], T, early_stop=early)
        for a, b in zip(few, all_):
            assert torch.equal(a.view(torch.uint8), b[:3].contiguous().view(torch.uint8))


@pytest.mark.parametrize("L,p", [(6, 3073), (9, 3073), (18, 1537), (18, 3600)])
def test_against_the_reference(L, p):
    a, llr, _ = qc_case(3, L, p, 5, 4, EBN0[L], 70 + p)
    g = ldpc.Graph.qc(a, p)
    H = oracle.qc_parity_check(a, p)
    for T in (1, 3):
        check_parity(gpu_decode(g, llr, T, False), oracle.decode_block(H, llr, T), True, f"3x{L} p={p} I={T}")
    check_parity(gpu_decode(g, llr, 20, True), oracle.decode_block(H, llr, 20, early_stop=True), False,
                 f"3x{L} p={p} early stop")
    w = rand_weights(3, 3 * L, 11)
    ref = ref_nnms.decode(ref_graph(a, p), llr.astype(np.float64), w[..., 0], w[..., 1], 3)
    check_decode(gpu_nms(g, llr, w), ref, f"3x{L} p={p} learned")
