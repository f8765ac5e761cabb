"""The message-package kernels of the training step, which take the bases that
no one-unit kernel covers: full rows of weight 4, 8, 12 and 24 with other row
counts, and zero blocks; frames of one tile, of several and of a partial one;
checkpoints every iteration, every few, and at the end.  Against the FP64
reference with the tolerances of test_gpu_nnms."""
import numpy as np
import pytest
import torch

import synth
from oracle import nnms as ref_nnms
from paper_1204_0334_amd import ldpc

from test_gpu_nnms import check_grad, gpu_grad, rand_weights, ref_graph

pytestmark = pytest.mark.gpu

# (J, L, p, zero blocks, frames, iterations)
CASES = [(3, 12, 40, 0, 70, 5), (2, 4, 33, 0, 130, 6), (4, 8, 24, 0, 65, 5), (2, 24, 51, 0, 40, 4), (6, 12, 20, 9, 64, 4)]


def setup(J, L, p, zeros, gamma, T):
    rng = np.random.default_rng(J * L + p)
    a = rng.integers(0, p, size=(J, L))
    a[0, 0], a[1, 1], a[J - 1, L - 1] = 0, p - 1, p - 1
    for l in range(zeros):
        a[l % J, l] = -1
    llr = synth.bpsk_awgn_llr(None, synth.ebn0_to_sigma2(2.5, 1.0 - J / L), 700 + p, gamma=gamma, n=L * p)
    llr[0, :L * p // 2] *= 20.0       # messages beyond the clip
    w = rand_weights(T, int((a >= 0).sum()), 21)
    w[T - 1, 1, 0] = -0.5
    return a, llr, w


def train(g, llr, w, ckpt, coef):
    """Loss and gradient, which must have come from the package kernels."""
    ldpc.timing_read()
    ldpc.timing_enable(True)
    out = gpu_grad(g, llr, w, ckpt, dloss=coef)
    ldpc.timing_enable(False)
    assert ldpc.timing_read()["train_variable_node"][0] > 0
    return out


@pytest.mark.parametrize("J,L,p,zeros,gamma,T", CASES)
def test_loss_and_gradient(J, L, p, zeros, gamma, T):
    a, llr, w = setup(J, L, p, zeros, gamma, T)
    coef = np.linspace(0.5, 1.5, T)
    loss, grad = train(ldpc.Graph.qc(a, p), llr, w, 2, coef)
    G, x = ref_graph(a, p), np.ones_like(llr, dtype=np.float64)
    per = ref_nnms.iteration_losses(G, llr.astype(np.float64), x, torch.tensor(w[..., 0], dtype=torch.float64),
                                    torch.tensor(w[..., 1], dtype=torch.float64), T).numpy()
    np.testing.assert_allclose(loss, per, rtol=1e-5)
    _, gw, gb = ref_nnms.grad(G, llr.astype(np.float64), x, w[..., 0].astype(np.float64),
                              w[..., 1].astype(np.float64), T, coef=coef)
    check_grad(grad, gw, gb, f"{J}x{L} p={p}")


@pytest.mark.parametrize("J,L,p,zeros,gamma,T", CASES)
def test_gradient_independent_of_checkpoint_interval(J, L, p, zeros, gamma, T):
    a, llr, w = setup(J, L, p, zeros, gamma, T)
    g = ldpc.Graph.qc(a, p)
    first = train(g, llr, w, 1, np.ones(T))
    for ckpt in sorted({2, 3, T}):
        again = train(g, llr, w, ckpt, np.ones(T))
        assert np.array_equal(first[0], again[0]) and np.array_equal(first[1], again[1]), ckpt
