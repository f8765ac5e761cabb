"""GPU parity of the on-chip decoder with one posterior sum per variable
(rows of weight 9, 18 and 24), against the FP64 references with the tolerances
of test_gpu_decode and test_gpu_nnms: the smallest and the largest circulant
of each instantiation, sizes one row past a wavefront and past a workgroup's
rows, and shifts of 0 and p - 1 (the wrap at either end of a column)."""
import numpy as np
import pytest

import oracle
import synth
from oracle import nnms as ref_nnms
from paper_1204_0334_amd import ldpc

from test_gpu_decode import check_parity, gpu_decode
from test_gpu_nnms import check_decode, gpu_nms, rand_weights, ref_graph

pytestmark = pytest.mark.gpu

# (J, L, p): NQ = 1 rows of weight 24 and 18, NQ = 2 rows of weight 18 (p >
# 1024), NQ = 3 rows of weight 9 (p > 2048)
CODES = [(4, 24, 64), (4, 24, 65), (4, 24, 449), (4, 24, 1024), (3, 18, 64), (3, 18, 127), (3, 18, 1024),
         (3, 18, 1025), (3, 18, 1536), (3, 9, 2049), (3, 9, 3072)]


@pytest.fixture(autouse=True)
def default_path(monkeypatch):
    monkeypatch.delenv("LDPC_BLOCK_PATH", raising=False)


def code(J, L, p, gamma, ebn0):
    a = np.random.default_rng(J * 100 + L + p).integers(0, p, size=(J, L))
    a[0, 0], a[1, 1], a[J - 1, L - 1] = 0, p - 1, p - 1
    llr = synth.bpsk_awgn_llr(None, synth.ebn0_to_sigma2(ebn0, 1.0 - J / L), 900 + p, gamma=gamma, n=L * p)
    g = ldpc.Graph.qc(a, p)
    assert ldpc.decode_path(g) == "onchip"
    return a, llr, g


@pytest.mark.parametrize("J,L,p", CODES)
def test_fixed_iterations_all_frames(J, L, p):
    a, llr, g = code(J, L, p, 5, 3.0 + 0.25 * (L > 9))
    for iters in (1, 2, 3):
        ref = oracle.decode_block(oracle.qc_parity_check(a, p), llr, iters)
        check_parity(gpu_decode(g, llr, iters, False), ref, True, f"{J}x{L} p={p} I={iters}")


@pytest.mark.parametrize("J,L,p", CODES)
def test_early_stop(J, L, p):
    a, llr, g = code(J, L, p, 9, 4.0 + (L > 9))
    llr = llr.copy()
    llr[0] = -0.0       # decides the all-zero word at once
    llr[1] = 40.0       # no decision to change: stops after one iteration
    H = oracle.qc_parity_check(a, p)
    ref = oracle.decode_block(H, llr, 25, early_stop=True)
    gpu = gpu_decode(g, llr, 25, True)
    check_parity(gpu, ref, False, f"{J}x{L} p={p} early stop")
    assert np.array_equal(gpu["converged"].astype(bool), ~H.syndrome(gpu["bits"]).any(1))
    assert gpu["iters"][0] == 1 and gpu["iters"][1] == 1 and not gpu["bits"][:2].any()


@pytest.mark.parametrize("J,L,p", CODES)
def test_learned_min_sum(J, L, p):
    a, llr, g = code(J, L, p, 4, 3.5 + (L > 9))
    w = rand_weights(3, J * L, 11)
    ref = ref_nnms.decode(ref_graph(a, p), llr.astype(np.float64), w[..., 0], w[..., 1], 3)
    check_decode(gpu_nms(g, llr, w), ref, f"{J}x{L} p={p} learned")
