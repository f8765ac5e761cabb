"""The pipelined decoder's sweeps (a stream on one compute unit) against its
launch-per-slot form, bit for bit: processor counts that need one to several
sweeps of every size, chains shorter than a row's reach, open chains, circulant
sizes around a wavefront and at the ends of each instantiation's range, and
batches on either side of one stream per compute unit.  The rate-5/6 code
against the FP64 reference as well."""
import os

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_1204_0334_amd import ldpc

from test_gpu_decode import TOL, gpu_pipeline, rel_err, window_parity

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def shifts(J, L, p):
    a = np.random.default_rng(J * 100 + L + p).integers(0, p, size=(J, L))
    a[0, 0], a[1, 1], a[J - 1, L - 1] = 0, p - 1, p - 1
    return a


def run(path, g, x, I):
    # LDPC_PIPELINE_PATH is read at every call; a launch of the sweeps counts
    # as a check-node launch, and only the launch form has variable-node ones
    if path == "launch":
        os.environ["LDPC_PIPELINE_PATH"] = "launch"
    try:
        ldpc.timing_read()
        ldpc.timing_enable(True)
        post, bits = ldpc.decode_pipeline(g, x, I)
        torch.cuda.synchronize()
        ldpc.timing_enable(False)
        t = ldpc.timing_read()
    finally:
        os.environ.pop("LDPC_PIPELINE_PATH", None)
    assert (t["pipeline_variable_node"][0] > 0) == (path == "launch"), t
    return post, bits


# (J, L, p, positions, terminated, frames, processors)
CASES = [(3, 6, 64, 9, True, 3, 1), (3, 6, 63, 9, True, 5, 4), (3, 6, 65, 10, False, 2, 5), (3, 6, 5, 1, True, 4, 6),
         (3, 6, 70, 2, True, 2, 7), (3, 6, 130, 3, False, 2, 9), (3, 6, 512, 14, True, 3, 11),
         (3, 6, 512, 6, True, 257, 8), (3, 6, 17, 40, True, 300, 20), (3, 6, 33, 25, True, 1, 64),
         (4, 24, 64, 7, True, 3, 1), (4, 24, 63, 1, True, 2, 2), (4, 24, 65, 9, False, 2, 3),
         (4, 24, 426, 6, True, 2, 4), (4, 24, 427, 6, True, 2, 3), (4, 24, 512, 5, True, 2, 2),
         (4, 24, 513, 5, True, 2, 2), (4, 24, 682, 5, True, 1, 2), (4, 24, 683, 5, True, 2, 3),
         (4, 24, 1024, 5, True, 2, 2)]


@pytest.mark.parametrize("J,L,p,positions,terminate,gamma,I", CASES)
def test_sweeps_and_launches_agree_bit_for_bit(J, L, p, positions, terminate, gamma, I):
    g = ldpc.Graph.ldpccc_from_qc(shifts(J, L, p), p, positions, terminate)
    print(f"[gpu] sweep n={g.n} gamma={gamma} I={I}", flush=True)
    x = ldpc.awgn_llr(g.n, gamma, synth.ebn0_to_sigma2(2.0, 1.0 - J / L), 7 + p, 0, device=DEV)
    x[0, ::3] = -0.0
    post, bits = run("sweep", g, x, I)
    post_l, bits_l = run("launch", g, x, I)
    assert torch.equal(bits, bits_l)
    assert torch.equal(post, post_l)


@pytest.mark.parametrize("p,positions,I,gamma", [(64, 9, 3, 5), (65, 8, 10, 6)])
def test_rate_five_sixths_against_the_reference(p, positions, I, gamma):
    a = shifts(4, 24, p)
    Hc, info = oracle.unwrap_qc(a, p, positions)
    llr = synth.bpsk_awgn_llr(None, synth.ebn0_to_sigma2(4.0, 5 / 6), 31, gamma=gamma, n=Hc.n)
    ref = oracle.decode_pipeline(Hc, llr, I, info["ms"])
    gpu = gpu_pipeline(ldpc.Graph.ldpccc_from_qc(a, p, positions), llr, I)
    if I <= 3:
        assert rel_err(gpu["post"], ref["post"]).max() <= TOL
    window_parity(gpu, ref, f"pipeline 4x24 p={p} I={I}", 6 * p)


def test_a_workspace_of_the_ring_alone_still_decodes():
    # 40 positions and 8 processors: the sweeps need more than the ring
    p, positions, I, gamma = 48, 40, 8, 200
    g = ldpc.Graph.ldpccc_from_qc(shifts(3, 6, p), p, positions, True)
    x = ldpc.awgn_llr(g.n, gamma, 0.5, 5, 0, device=DEV)
    full = g.workspace_size(gamma, I, 0)
    os.environ["LDPC_PIPELINE_PATH"] = "launch"
    ring = g.workspace_size(gamma, I, 0)
    os.environ.pop("LDPC_PIPELINE_PATH")
    assert ring < full
    ws = torch.empty(ring, dtype=torch.uint8, device=DEV)
    post, bits = ldpc.decode_pipeline(g, x, I, ws=ws)
    want, _ = ldpc.decode_pipeline(g, x, I)
    assert torch.equal(post, want)
    with pytest.raises(ldpc.LdpcError):
        ldpc.decode_pipeline(g, x, I, ws=ws[:-1])
