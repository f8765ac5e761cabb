"""The FP32 rounding error of whole decodes against the FP64 reference, as
relative 2-norm over all posteriors: kernels that take the place of the message
packages are no further off than these.

The error of a few iterations is the sum of very many independent roundings, so
its norm over 10^5 values repeats to less than 1 %; 5 % leave room for the
transcendentals' share, which differs between the two check rules."""
import numpy as np
import pytest
import torch

import oracle
from paper_1204_0334_amd import ldpc

from test_gpu_decode import gpu_decode, qc_case

pytestmark = pytest.mark.gpu


def error(post, ref):
    return np.linalg.norm(post.astype(np.float64) - ref) / np.linalg.norm(ref)


@pytest.mark.parametrize("J,L,p,ebn0,iters", [(4, 24, 422, 3.6, 2), (4, 24, 1024, 3.3, 3), (3, 18, 500, 3.6, 2),
                                              (3, 18, 1300, 3.4, 3), (3, 9, 2399, 2.4, 2)])
def test_on_chip_codes_are_as_exact_as_the_packages(monkeypatch, J, L, p, ebn0, iters):
    monkeypatch.delenv("LDPC_BLOCK_PATH", raising=False)
    a, llr, _ = qc_case(J, L, p, 3, 24, ebn0, 90 + p)
    g = ldpc.Graph.qc(a, p)
    assert ldpc.decode_path(g) == "onchip"
    ref = np.clip(oracle.decode_block(oracle.qc_parity_check(a, p), llr, iters)["post"], -30.0, 30.0)
    here = error(gpu_decode(g, llr, iters, False)["post"], ref)
    monkeypatch.setenv("LDPC_BLOCK_PATH", "packages")
    there = error(gpu_decode(g, llr, iters, False)["post"], ref)
    print(f"[gpu] {J}x{L} p={p} iters={iters}: {here:.3e} on chip, {there:.3e} in packages", flush=True)
    assert here <= 1.05 * there
