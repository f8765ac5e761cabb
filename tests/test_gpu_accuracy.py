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
import synth
from paper_1204_0334_amd import ldpc

from test_gpu_decode import gpu_decode, qc_case

pytestmark = pytest.mark.gpu


DEV = "cuda:0"


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


def separate_sums(H, llr, iters):
    """Flooding in FP32 with every beta the sum of the other alphas (base-2
    units, (tanh, 1 - tanh) pairs, the GPU's exponential and logarithm): the
    rounding error that the convolutional decoders have to stay within."""
    f = np.float32
    exp2 = lambda x: torch.exp2(torch.from_numpy(x).to(DEV)).cpu().numpy()  # noqa: E731
    log2 = lambda x: torch.log2(torch.from_numpy(x).to(DEV)).cpu().numpy()  # noqa: E731
    n, deg = llr.shape[1], np.diff(H.row_ptr)
    d = deg.max()
    idx = np.full((len(deg), d), n)           # missing edges: a variable behind the last
    for r in range(len(deg)):
        idx[r, :deg[r]] = H.col_idx[H.row_ptr[r]:H.row_ptr[r + 1]]
    there = idx < n
    # the edges of each variable, by ascending row
    order = np.lexsort((np.nonzero(there)[0], idx[there]))
    flat = np.flatnonzero(there.ravel())[order]
    dv = np.bincount(idx[there], minlength=n)
    slot = np.arange(len(flat)) - np.repeat(np.cumsum(dv) - dv, dv)
    edges = np.full((dv.max(), n), idx.size)  # an alpha of 0 behind the last
    edges[slot, idx.ravel()[flat]] = flat
    fma = lambda a, b, c: (a.astype(np.float64) * b + c).astype(f)  # noqa: E731
    clip = f(30 * np.log2(np.e))
    out = np.empty((llr.shape[0], n))
    for g in range(llr.shape[0]):
        mu = (llr[g].astype(f) * f(np.log2(np.e))).astype(f)
        beta = np.clip(np.append(mu, f(np.inf))[idx], -clip, clip)
        for _ in range(iters):
            e = np.where(there, exp2(-np.abs(beta)), f(0))
            r = f(1) / (f(1) + e)
            t, q = (f(1) - e) * r, (e + e) * r
            P, Q = np.ones(len(deg), f), np.zeros(len(deg), f)
            suf = [None] * d
            for k in range(d - 1, -1, -1):
                suf[k] = (P, Q)
                P, Q = P * t[:, k], fma(Q, t[:, k], q[:, k])
            P, Q = np.ones(len(deg), f), np.zeros(len(deg), f)
            alpha = np.empty_like(beta)
            neg = np.where(beta < 0, f(-1), f(1))
            for k in range(d):
                alpha[:, k] = log2((f(1) + P * suf[k][0]) * (f(1) / fma(suf[k][1], P, Q)))
                P, Q = P * t[:, k], fma(q[:, k], P, Q)
            alpha *= neg.prod(1, keepdims=True) * neg
            a = np.append(alpha.ravel(), f(0))[edges]
            after, S = [None] * len(a), np.zeros(n, f)
            for k in range(len(a) - 1, -1, -1):
                after[k] = S
                S = S + a[k]
            pre, b = np.zeros(n, f), np.empty_like(a)
            for k in range(len(a)):
                b[k] = mu + (pre + after[k])
                pre = pre + a[k]
            flat_beta = np.full(idx.size + 1, clip, f)
            flat_beta[edges] = np.clip(b, -clip, clip)
            beta = flat_beta[:-1].reshape(idx.shape)
        out[g] = np.clip((mu + pre) * f(np.log(2)), -30, 30)
    return out


# The repeatability as above; 3 % for the hardware's reciprocal.
@pytest.mark.parametrize("J,L,p,ebn0,path", [(3, 6, 200, 2.0, "sweep"), (3, 6, 200, 2.0, "launch"),
                                             (4, 24, 100, 4.0, "sweep"), (2, 4, 150, 2.0, "sweep"),
                                             (3, 6, 200, 2.0, "window"), (2, 4, 150, 2.0, "window")])
def test_convolutional_decoders_are_as_exact_as_separate_sums(monkeypatch, J, L, p, ebn0, path):
    positions, iters, gamma = 10, 2, 24
    a, _, _ = qc_case(J, L, p, 3, 1, ebn0, 1)
    H, info = oracle.unwrap_qc(a, p, positions)
    g = ldpc.Graph.ldpccc_from_qc(a, p, positions, True)
    llr = synth.bpsk_awgn_llr(None, synth.ebn0_to_sigma2(ebn0, 1 - J / L), 77, gamma=gamma, n=H.n)
    x = torch.tensor(llr, dtype=torch.float32, device=DEV)
    if path == "window":
        # a window over the whole chain: `iters` iterations until position 0 is decided
        part = slice(0, H.n // positions)
        ref = oracle.decode_window(H, llr, 12, iters)["post"]
        post = ldpc.decode_window(g, x, 12, iters)[0].cpu().numpy()
    else:
        if path == "launch":
            monkeypatch.setenv("LDPC_PIPELINE_PATH", "launch")
        part = slice(0, H.n)
        ref = oracle.decode_pipeline(H, llr, iters, info["ms"])["post"]
        post = ldpc.decode_pipeline(g, x, iters)[0].cpu().numpy()
    ref = np.clip(ref, -30.0, 30.0)[:, part]
    here, there = error(post[:, part], ref), error(separate_sums(H, llr, iters)[:, part], ref)
    print(f"[gpu] {J}x{L} p={p} {path}: {here:.3e} here, {there:.3e} with separate sums", flush=True)
    assert here <= 1.03 * there
