"""The sliding-window decoder with messages in registers against the
launch-per-phase form, bit for bit: 1, 2, 3 and 6 layers per thread, windows
that are not a multiple of them, windows longer than the chain, open chains,
and batches on either side of one stream per compute unit."""
import numpy as np
import pytest
import torch

import synth
from paper_1204_0334_amd import ldpc

from test_gpu_decode import window_path

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

# (p, positions, W, K, streams, terminated)
CASES = [(5, 1, 3, 1, 2, True), (64, 9, 6, 3, 3, True), (65, 11, 5, 2, 300, True), (128, 8, 7, 3, 3, False),
         (140, 9, 6, 2, 300, True), (192, 20, 12, 2, 2, True), (320, 4, 9, 2, 3, True), (340, 12, 7, 3, 2, True),
         (340, 20, 12, 2, 3, False), (512, 9, 5, 3, 2, True), (512, 7, 6, 2, 300, False)]


@pytest.mark.parametrize("p,positions,W,K,gamma,terminate", CASES)
def test_register_and_launch_paths_agree_bit_for_bit(p, positions, W, K, gamma, terminate):
    a = np.random.default_rng(p + W).integers(0, p, size=(3, 6))
    a[0, 0], a[1, 1], a[2, 5] = 0, p - 1, p - 1
    g = ldpc.Graph.ldpccc_from_qc(a, p, positions, terminate)
    print(f"[gpu] window n={g.n} gamma={gamma} W={W} K={K}", flush=True)
    x = ldpc.awgn_llr(g.n, gamma, synth.ebn0_to_sigma2(1.75, 0.5), 7 + p, 0, device=DEV)
    x[0, ::3] = -0.0
    post, bits, t = window_path("lds", g, x, W, K)
    want, want_bits, _ = window_path("launch", g, x, W, K)
    assert t["window_lds"][0] == 1 and t["window_check_node"][0] == 0, t
    assert torch.equal(bits, want_bits)
    assert torch.equal(post, want)
