"""The decoding work a user has this library do, as sized cases.

Each case is one pass through the public entry points: block decoding of one
code (from a single codeword to a batch that fills the chip), a batch of the
error-rate simulation (channel, decoder, error count), the two decoders of
convolutional codes, learned min-sum decoding, its training step, and a plan
over several codes.  The codes are regular quasi-cyclic ones of the shapes the
library's benchmark, tests and command line use (3 x 6, 3 x 9, 3 x 18 and
4 x 24 bases), with seeded shifts free of 4-cycles.  Channel values are those
of BPSK over AWGN at signal-to-noise ratios where these codes are used, i.e.
where nearly every frame decodes (training excepted, which runs in the
waterfall region, as `nnms.train` does); simulation and training send the
all-zero codeword, as the library does, the others random codewords.

`listed` gives the fixed cases, `draw` another one of the same ranges,
`prepare` / `run` do a case, `work` counts what it cannot do without, and
`exact` computes its outputs in 64-bit floating point from the definitions.
"""
import functools
import math

import numpy as np
import torch

from paper_1204_0334_amd import ldpc, nnms

CLIP = 30.0

# ----------------------------------------------------------------------------
# cases
# ----------------------------------------------------------------------------

# the mixed batch of the multi-code plan: (J, L, p, frames)
MIX = [(3, 6, 27, 1024), (3, 6, 81, 256), (3, 6, 2700, 64), (3, 9, 72, 512), (3, 9, 2400, 32), (3, 18, 36, 128),
       (3, 18, 3600, 8)]


def listed():
    return [
        # one codeword of the long rate-1/2 code, as a receiver decodes it: latency
        dict(name="one_frame", kind="block", J=3, L=6, p=3060, frames=1, iters=20, early=True),
        # a small batch of a short code: latency of one small launch and of the call
        dict(name="short_code", kind="block", J=3, L=6, p=64, frames=64, iters=20, early=True),
        # the benchmark's code and batch, fixed work
        dict(name="long_code", kind="block", J=3, L=6, p=3060, frames=1024, iters=20, early=False),
        # a ragged batch of a rate-2/3 code, stopping when decoded
        dict(name="ragged_batch", kind="block", J=3, L=9, p=2399, frames=101, iters=30, early=True),
        # the longest of the paper's rate-5/6 codes, throughput decoding
        dict(name="rate56_long", kind="block", J=4, L=24, p=1024, frames=1024, iters=30, early=False),
        # one batch of the error-rate simulation of the paper's shortest rate-5/6 code
        dict(name="simulation", kind="simulate", J=4, L=24, p=422, frames=1024, iters=30, early=True),
        # convolutional code, sliding window (128 positions, 512 streams)
        dict(name="window", kind="window", J=3, L=6, p=512, frames=512, positions=128, window=6, iters=10),
        # the same code and streams through the pipelined decoder with 20 processors
        dict(name="pipeline", kind="pipeline", J=3, L=6, p=512, frames=512, positions=128, iters=20),
        # the rate-5/6 convolutional code of the paper's pipelined decoder
        dict(name="pipeline_rate56", kind="pipeline", J=4, L=24, p=422, frames=256, positions=64, iters=20),
        # learned min-sum decoding of the benchmark's code
        dict(name="learned", kind="learned", J=3, L=6, p=3060, frames=1024, iters=12, early=False),
        # forward and backward of its training step (every iteration kept, the default)
        dict(name="training", kind="train", J=3, L=6, p=3060, frames=1024, iters=12, keep=12),
        # seven codes of three rates in one captured plan
        dict(name="mixed_plan", kind="plan", codes="0123456", scale=1.0, iters=20, early=True, graph=True),
    ]


SHAPES = [(3, 6), (3, 6), (3, 9), (3, 18), (4, 24), (4, 24)]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["block"] * 6 + ["simulate", "window", "pipeline", "pipeline", "learned", "learned", "train",
                                       "train", "plan"])
    early = rng.random() < 0.6
    while True:
        J, L = rng.choice(SHAPES)
        if kind in ("block", "simulate", "learned"):
            c = dict(kind=kind, J=J, L=L, p=_log_int(rng, 2 * L + 12, 24576 // L),
                     frames=_log_int(rng, 1, 1500), iters=rng.randint(10, 30), early=early)
        elif kind == "train":
            c = dict(kind=kind, J=J, L=L, p=_log_int(rng, 2 * L + 12, 18432 // L), frames=_log_int(rng, 16, 1024),
                     iters=rng.randint(5, 18), keep=0)
            c["keep"] = rng.choice([c["iters"], c["iters"], 4])
        elif kind == "window":
            c = dict(kind=kind, J=3, L=6, p=_log_int(rng, 40, 512), frames=_log_int(rng, 1, 512),
                     positions=_log_int(rng, 12, 128), window=rng.choice([5, 6, 6]), iters=rng.randint(5, 12))
        elif kind == "pipeline":
            J, L = rng.choice([(3, 6), (4, 24)])
            c = dict(kind=kind, J=J, L=L, p=_log_int(rng, 2 * L + 12, 512 if L == 6 else 1024),
                     frames=_log_int(rng, 1, 512), positions=_log_int(rng, 12, 128), iters=rng.randint(8, 24))
        else:
            ids = sorted(rng.sample(range(len(MIX)), rng.randint(2, len(MIX))))
            c = dict(kind=kind, codes="".join(map(str, ids)), scale=math.exp(rng.uniform(math.log(0.05), 0.0)),
                     iters=rng.randint(10, 30), early=early, graph=rng.random() < 0.7)
        if _updates(c) <= {"train": 7e8, "window": 1.3e10}.get(kind, 3.1e9):
            return c


# ----------------------------------------------------------------------------
# codes and channel values
# ----------------------------------------------------------------------------


@functools.lru_cache(maxsize=None)
def shift_table(J, L, p):
    """Seeded shifts of a J x L base of p x p circulants without 4-cycles: the
    differences of two rows' shifts are distinct over the columns."""
    rng = np.random.default_rng(J * 1000003 + L * 10007 + p)
    while True:
        rows = [[0] * L for _ in range(J)]
        seen = {(i, j): set() for j in range(J) for i in range(j)}
        for j in range(J):
            for l in range(L):
                for _ in range(200):
                    a = int(rng.integers(p))
                    if all((a - rows[i][l]) % p not in seen[i, j] for i in range(j)):
                        break
                else:
                    break
                rows[j][l] = a
                for i in range(j):
                    seen[i, j].add((a - rows[i][l]) % p)
            else:
                continue
            break
        else:
            return tuple(tuple(r) for r in rows)


def _ebn0_db(kind, J, L, n):
    """Eb/N0 where a code of this rate and length is used (frame error rates
    around 1e-6 and below); short codes need more."""
    base = {(3, 6): 2.7, (3, 9): 3.4, (3, 18): 4.4, (4, 24): 4.3}[(J, L)]
    slope = {(3, 6): 1.6, (3, 9): 1.4, (3, 18): 1.2, (4, 24): 1.2}[(J, L)]
    extra = {"learned": 0.4, "window": 0.6, "pipeline": 0.6}.get(kind, 0.0)
    return base + extra + slope * max(0.0, math.log10(18000.0 / n))


def _sigma2(db, J, L):
    return 1.0 / (2.0 * (1.0 - J / L) * 10.0 ** (db / 10.0))


def _channel(frames, n, sigma2, gen):
    """LLRs 2 y / sigma^2 of the all-zero codeword: float32 [frames, n]."""
    x = torch.randn((frames, n), generator=gen, device=gen.device, dtype=torch.float32)
    return x.mul_(2.0 / math.sqrt(sigma2)).add_(2.0 / sigma2)


def _send_codewords(llr, groups, columns, gen):
    """Turns LLRs of the all-zero codeword into those of a random codeword per
    frame that is constant on the circulant columns: a check meets one
    variable of every column of a base row (of every position, in the
    unwrapped code), so an even number of flipped columns satisfies it."""
    frames = llr.shape[0]
    flip = torch.randint(0, 2, (frames, groups, columns), generator=gen, device=gen.device)
    flip[..., -1] = flip[..., :-1].sum(-1) % 2
    llr.view(frames, groups, columns, -1).mul_((1 - 2 * flip)[..., None].float())
    return llr


def _generator(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return gen


def _inputs(c, seed):
    """What a case's seed decides, on the GPU."""
    gen = _generator(seed)
    kind = c["kind"]
    if kind == "plan":
        return [_send_codewords(_channel(f, L * p, _sigma2(_ebn0_db(kind, J, L, L * p), J, L), gen), 1, L, gen)
                for J, L, p, f in _plan_codes(c)]
    J, L, p = c["J"], c["L"], c["p"]
    n = L * p if "positions" not in c else L // math.gcd(J, L) * p * c["positions"]
    if kind == "train":
        # every run of 64 frames at an Eb/N0 drawn from 1.0-2.5 dB (rate 1/2; higher rates need more)
        lo = {(3, 6): 1.0, (3, 9): 1.8, (3, 18): 3.0, (4, 24): 3.0}[(J, L)]
        llr = torch.empty((c["frames"], n), device="cuda", dtype=torch.float32)
        db = np.random.default_rng(seed).uniform(lo, lo + 1.5, size=(c["frames"] + 63) // 64)
        for k, d in enumerate(db):
            part = llr[64 * k:64 * (k + 1)]
            part.copy_(_channel(part.shape[0], n, _sigma2(float(d), J, L), gen))
        return llr, _weights(c, gen)
    sigma2 = _sigma2(_ebn0_db(kind, J, L, n if "positions" not in c else 8 * n // c["positions"]), J, L)
    if kind == "simulate":
        return sigma2
    llr = _send_codewords(_channel(c["frames"], n, sigma2, gen), c.get("positions", 1),
                          L if "positions" not in c else L // math.gcd(J, L), gen)
    return (llr, _weights(c, gen)) if kind == "learned" else llr


def _weights(c, gen):
    """Scales and offsets as training leaves them: around 0.8 and 0.05, each
    edge class a little different."""
    r = torch.rand((c["iters"], c["J"] * c["L"], 2), generator=gen, device="cuda", dtype=torch.float32)
    r[..., 0].mul_(0.1).add_(0.75)
    r[..., 1].mul_(0.1)
    return r


def _plan_codes(c):
    return [(J, L, p, max(1, int(f * c["scale"]))) for J, L, p, f in (MIX[int(k)] for k in c["codes"])]


# ----------------------------------------------------------------------------
# the passes
# ----------------------------------------------------------------------------


def _decode_outputs(frames, n):
    return (torch.empty((frames, n), device="cuda", dtype=torch.float32),
            torch.empty((frames, n), device="cuda", dtype=torch.uint8),
            torch.empty((frames,), device="cuda", dtype=torch.int32),
            torch.empty((frames,), device="cuda", dtype=torch.uint8))


def prepare(case, seed):
    c, kind = dict(case), case["kind"]
    s = dict(case=c, seed=seed)
    if kind == "plan":
        codes = _plan_codes(c)
        s["llr"] = _inputs(c, seed)
        s["plan"] = ldpc.Plan([ldpc.Graph.qc(shift_table(J, L, p), p) for J, L, p, _ in codes],
                              [f for _, _, _, f in codes], c["iters"], c["early"])
        s["ws"], s["out"] = s["plan"].workspace(), s["plan"].outputs()
        if c["graph"]:
            s["plan"].capture(s["llr"], s["out"], s["ws"])
        return s
    J, L, p, frames, iters = c["J"], c["L"], c["p"], c["frames"], c["iters"]
    table = shift_table(J, L, p)
    if "positions" in c:
        g = s["g"] = ldpc.Graph.ldpccc_from_qc(table, p, c["positions"], True)
        s["llr"] = _inputs(c, seed)
        s["out"] = _decode_outputs(frames, g.n)[:2]
        s["ws"] = ldpc.workspace(g, frames, 1 if kind == "window" else iters, c.get("window", 0))
        return s
    g = s["g"] = ldpc.Graph.qc(table, p)
    if kind == "train":
        s["llr"], w = _inputs(c, seed)
        s["w"] = w.requires_grad_(True)
        s["coef"] = torch.full((iters,), 1.0 / iters, device="cuda")
        s["ws"] = ldpc.nms_train_workspace(g, frames, iters, min(c["keep"], iters))
        return s
    if kind == "learned":
        s["llr"], s["w"] = _inputs(c, seed)
    elif kind == "simulate":
        s["sigma2"] = _inputs(c, seed)
        s["llr"] = torch.empty((frames, g.n), device="cuda", dtype=torch.float32)
        s["errors"] = torch.empty((frames,), device="cuda", dtype=torch.int32)
    else:
        s["llr"] = _inputs(c, seed)
    s["out"] = _decode_outputs(frames, g.n)
    s["ws"] = ldpc.workspace(g, frames, iters, 0)
    return s


def run(s):
    c, kind = s["case"], s["case"]["kind"]
    if kind == "block":
        return ldpc.decode(s["g"], s["llr"], c["iters"], c["early"], out=s["out"], ws=s["ws"])
    if kind == "simulate":
        ldpc.awgn_llr(s["g"].n, c["frames"], s["sigma2"], s["seed"], 0, out=s["llr"])
        out = ldpc.decode(s["g"], s["llr"], c["iters"], c["early"], out=s["out"], ws=s["ws"])
        ldpc.count_errors(out[1], frame_errors=s["errors"])
        return (s["llr"], *out, s["errors"])
    if kind == "window":
        return ldpc.decode_window(s["g"], s["llr"], c["window"], c["iters"], out=s["out"], ws=s["ws"])
    if kind == "pipeline":
        return ldpc.decode_pipeline(s["g"], s["llr"], c["iters"], out=s["out"], ws=s["ws"])
    if kind == "learned":
        return ldpc.nms_decode(s["g"], s["llr"], s["w"], c["early"], out=s["out"], ws=s["ws"])
    if kind == "train":
        losses = nnms.iteration_losses(s["w"], s["g"], s["llr"], min(c["keep"], c["iters"]), s["ws"])
        (grad,) = torch.autograd.grad((s["coef"] * losses).sum(), s["w"])
        return losses.detach(), grad
    if c["graph"]:
        s["plan"].replay()
    else:
        s["plan"].decode(s["llr"], s["out"], s["ws"])
    return s["out"]


# ----------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------


def _edges(c):
    if c["kind"] == "plan":
        return sum(J * L * p * f for J, L, p, f in _plan_codes(c))
    e = c["J"] * c["L"] * c["p"] * c["frames"]
    return e if "positions" not in c else e // math.gcd(c["J"], c["L"]) * c["positions"]


def _iterations(c):
    """Iterations that every frame needs: all of them without early stopping,
    else about 5 at these signal-to-noise ratios."""
    if c["kind"] == "window":
        return c["window"] * c["iters"]
    return min(5, c["iters"]) if c.get("early") else c["iters"]


def _updates(c):
    """Edge updates a pass may need (size cap of drawn cases)."""
    return _edges(c) * (c["window"] if c["kind"] == "window" else 1) * c["iters"]


def work(case):
    c, kind = case, case["kind"]
    if kind == "plan":
        bits = sum(L * p * f for _, L, p, f in _plan_codes(c))
        degree = _edges(c) / sum(J * p * f for J, L, p, f in _plan_codes(c))
    else:
        n = c["L"] * c["p"] * c["frames"]
        bits = n if "positions" not in c else n // math.gcd(c["J"], c["L"]) * c["positions"]
        degree = c["L"]
    # LLRs in, posteriors and decisions out; a training step only reads them
    bytes_ = 4 * bits if kind == "train" else 9 * bits
    if kind == "simulate":
        bytes_ += 4 * bits + bits
    # per edge and iteration: input triple 3, sign 1, two sweeps 10 (short
    # rows less), exponential, reciprocal and logarithm 3, output 4, the
    # variable's sum, difference and clip 4; the minimum rule 9 + 4; its
    # backward as much again
    if kind in ("learned", "train"):
        per = 13 if kind == "learned" else 26
    else:
        per = 15 + 10 * (degree - 2) / degree
    return {"bytes": float(bytes_), "flops": float(per * _edges(c) * _iterations(c))}


# ----------------------------------------------------------------------------
# the same outputs in 64 bits, from the definitions
# ----------------------------------------------------------------------------


def _rows(J, L, p, table, positions=None):
    """Variables of every check: long [checks, weight], and the number of
    variables; for the unwrapped code rows at the two ends are filled up with
    a variable past the last."""
    t = np.asarray(table)
    s = np.arange(p)
    if positions is None:
        rows = [[l * p + (s + t[j, l]) % p for l in range(L)] for j in range(J)]
        v = np.stack([np.stack(r, 1) for r in rows]).reshape(J * p, L)
        return torch.from_numpy(v).cuda(), L * p
    T = math.gcd(J, L)
    Jb, Lb = J // T, L // T
    n = positions * Lb * p
    v = np.full((positions + T - 1, Jb, p, T, Lb), n, dtype=np.int64)
    for lay in range(positions + T - 1):
        for d in range(T):
            q = lay - d
            if 0 <= q < positions:
                for a in range(Jb):
                    for b in range(Lb):
                        v[lay, a, :, d, b] = (q * Lb + b) * p + (s + t[lay % T * Jb + a, q % T * Lb + b]) % p
    return torch.from_numpy(v.reshape(-1, T * Lb)).cuda(), n


def _box(a, b):
    """2 atanh(tanh(a/2) tanh(b/2))."""
    return (torch.sign(a) * torch.sign(b) * torch.minimum(a.abs(), b.abs())
            + torch.log1p(torch.exp(-(a + b).abs())) - torch.log1p(torch.exp(-(a - b).abs())))


def _check_update(beta):
    """Eq. 3 over the second-last axis of beta [..., weight, frames]."""
    x = beta.unbind(-2)
    d = len(x)
    after = [None] * d
    for k in range(d - 2, -1, -1):
        after[k] = x[k + 1] if after[k + 1] is None else _box(x[k + 1], after[k + 1])
    out, before = [], None
    for k in range(d):
        out.append(after[k] if before is None else before if after[k] is None else _box(before, after[k]))
        before = x[k] if before is None else _box(before, x[k])
    return torch.stack(out, -2)


def _min_update(beta, w):
    """The learned rule; w [weight or checks x weight, 2]."""
    mag = beta.abs().clamp(max=CLIP)
    two, at = mag.topk(2, dim=-2, largest=False)
    k = torch.arange(beta.shape[-2], device=beta.device)[:, None]
    m = torch.where(k == at[..., :1, :], two[..., 1:, :], two[..., :1, :])
    neg = beta < 0
    neg = neg ^ (neg.sum(-2, keepdim=True) % 2 == 1)
    a = w[..., 0:1] * (m - w[..., 1:2]).clamp(min=0.0)
    return torch.where(neg, -a, a)


def _flood(rows, n, mu, iters, early, weights=None, p=0):
    """Algorithm 1 on mu [n, frames]: the posteriors before the clip, per
    frame those of the first zero syndrome if `early`, and of every iteration
    if weights need a gradient."""
    idx = rows.reshape(-1)
    pad = (rows == n)[..., None]
    ext = torch.cat([mu, torch.full_like(mu[:1], 1e4)])
    beta = torch.where(pad, 1e4, ext[rows].clamp(-CLIP, CLIP))
    done, kept, every = torch.zeros(mu.shape[1], dtype=torch.bool, device=mu.device), None, []
    for it in range(iters):
        if weights is None:
            alpha = _check_update(beta)
        else:
            alpha = _min_update(beta, weights[it].reshape(-1, 1, rows.shape[1], 2).expand(-1, p, -1, -1).reshape(
                rows.shape[0], rows.shape[1], 2))
        post = ext.index_add(0, idx, torch.where(pad, 0.0, alpha).reshape(idx.numel(), -1))
        every.append(post[:n])
        if weights is None or not weights.requires_grad:
            every = every[-1:]
        kept = post[:n] if kept is None else torch.where(done, kept, post[:n])
        if early:
            done = done | ~((post[rows] < 0).sum(1) % 2 == 1).any(0)
            if bool(done.all()):
                break
        beta = torch.where(pad, 1e4, (post[rows] - alpha).clamp(-CLIP, CLIP))
    return every if weights is not None and weights.requires_grad else kept


def _slide(c, rows, n, mu):
    """The window decoder on mu [n, frames]: posteriors before the clip."""
    P, W, T = c["positions"], c["window"], math.gcd(c["J"], c["L"])
    layers, per = P + T - 1, n // P
    rows = rows.reshape(layers, -1, rows.shape[1])
    frames = mu.shape[1]
    beta = torch.empty((*rows.shape, frames), dtype=mu.dtype, device=mu.device)
    beta.copy_(torch.where((rows == n)[..., None], 1e4, torch.cat([mu, mu[:1]])[rows].clamp(-CLIP, CLIP)))
    pos = rows // per
    out = torch.empty_like(mu)
    for s in range(P):
        hi, top = min(s + W, layers), min(s + W, P)
        lay = slice(s, hi)                       # the window's layers
        reach = slice(s, min(top + T - 1, layers))   # the layers its positions meet
        own = ((pos[reach] >= s) & (pos[reach] < top))[..., None]
        idx = (rows[reach] - s * per).clamp(0, (top - s) * per - 1)
        flat = idx.reshape(-1)
        alpha = torch.zeros((*idx.shape, frames), dtype=mu.dtype, device=mu.device)
        for _ in range(c["iters"]):
            alpha[:hi - s] = _check_update(beta[lay])
            post = mu[s * per:top * per].index_add(0, flat, torch.where(own, alpha, 0.0).reshape(flat.numel(), -1))
            beta[reach] = torch.where(own, (post[idx] - alpha).clamp(-CLIP, CLIP), beta[reach])
        out[s * per:(s + 1) * per] = post[:per]
    return out


def _simulated_llr(n, frames, sigma2, seed):
    """float32 LLRs of the all-zero codeword from Philox-4x32-10 and
    Box-Muller, as `ldpc_awgn_llr` defines them."""
    low, shift = np.uint64(0xFFFFFFFF), np.uint64(32)
    b = (n + 3) // 4
    c0 = np.broadcast_to(np.arange(b, dtype=np.uint64), (frames, b)).copy()
    c1 = np.broadcast_to(np.arange(frames, dtype=np.uint64)[:, None], (frames, b)).copy()
    c2, c3 = np.full_like(c0, 0x4E5A), np.zeros_like(c0)
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32 & 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = c0 * np.uint64(0xD2511F53), c2 * np.uint64(0xCD9E8D57)
        c0, c1 = (p1 >> shift) ^ c1 ^ np.uint64(k0), p1 & low
        c2, c3 = (p0 >> shift) ^ c3 ^ np.uint64(k1), p0 & low
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    u = [torch.from_numpy(((c.astype(np.float64) + 0.5) * 2.0 ** -32)).cuda() for c in (c0, c1, c2, c3)]
    z = []
    for k in (0, 2):
        r = torch.sqrt(-2.0 * torch.log(u[k]))
        z += [r * torch.cos(2 * math.pi * u[k + 1]), r * torch.sin(2 * math.pi * u[k + 1])]
    z = torch.stack(z, -1).reshape(frames, 4 * b)[:, :n]
    return (2.0 * (1.0 + math.sqrt(sigma2) * z) / sigma2).float()


def _posteriors(c, rows, n, llr, weights=None):
    """clip(posterior) [frames, n] in float64, some frames at a time."""
    out = torch.empty(llr.shape, dtype=torch.float64, device=llr.device)
    step = max(1, int(3e7) // rows.numel())
    for f in range(0, llr.shape[0], step):
        mu = llr[f:f + step].double().t().contiguous()
        if c["kind"] == "window":
            post = _slide(c, rows, n, mu)
        else:
            post = _flood(rows, n, mu, c["iters"], c.get("early", False), weights, c["p"])
        out[f:f + step] = post.clamp(-CLIP, CLIP).t()
    return out


def exact(case, seed):
    c, kind = dict(case), case["kind"]
    if kind == "plan":
        outs = []
        for (J, L, p, _), llr in zip(_plan_codes(c), _inputs(c, seed)):
            rows, n = _rows(J, L, p, shift_table(J, L, p))
            outs.append((_posteriors(dict(c, p=p), rows, n, llr), None, None, None))
        return outs
    J, L, p, frames = c["J"], c["L"], c["p"], c["frames"]
    rows, n = _rows(J, L, p, shift_table(J, L, p), c.get("positions"))
    got = _inputs(c, seed)
    if kind == "train":
        llr, w = got
        w = w.double().requires_grad_(True)
        losses = torch.zeros(c["iters"], dtype=torch.float64, device="cuda")
        grad = torch.zeros_like(w)
        step = max(1, int(1.2e8) // (rows.numel() * c["iters"]))
        for f in range(0, frames, step):
            mu = llr[f:f + step].double().t().contiguous()
            every = _flood(rows, n, mu, c["iters"], False, w, p)
            part = torch.stack([torch.nn.functional.softplus(-x).sum() for x in every]) / (frames * n)
            grad += torch.autograd.grad(part.sum() / c["iters"], w)[0]
            losses += part.detach()
        return losses, grad
    if kind == "simulate":
        llr = _simulated_llr(n, frames, got, seed)
        return llr.double(), _posteriors(c, rows, n, llr), None, None, None, None
    if kind == "learned":
        return _posteriors(c, rows, n, got[0], got[1].double()), None, None, None
    post = _posteriors(c, rows, n, got)
    return (post, None) if "positions" in c else (post, None, None, None)
