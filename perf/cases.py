"""Performance cases of the decoder: what a user's program calls, over the sizes it is called with.

Each case is a dict of plain values; `prepare` makes what the program has in hand before the call (syndromes on
the GPU, options, a workspace of its own, network weights), `run` is one pass through the public entry points.
Syndromes are those of i.i.d. Pauli errors (the paper's noise model) at the case's rate.

`exact` evaluates the same outputs in 64 bits with plain torch: blockBP by dense block contraction (where chi
truncates nothing), the boundary MPS with a library SVD, the warm-start network and its gradient by autograd.
"""
import math

import numpy as np
import torch

import paper_2402_04834_amd as bbp
from paper_2402_04834_amd import warm, workload

# chi at which the boundary state of a block of this width is never truncated (dense kernels) ...
EXACT_CHI = {1: 4, 2: 4, 3: 4, 4: 16, 5: 16, 6: 32}
# ... and (block, chi) pairs where it is (truncating sweeps); 7 and 8 always run the truncating sweeps
BINDING = ((3, 2), (4, 4), (5, 4), (6, 8), (6, 12), (7, 8), (8, 16))
EARLY_EXIT_ITERS = 14   # iterations of an early-exit decode counted as work (d = 17, p = 0.10: 14.5 on average)


def listed():
    return [
        # one syndrome of a small code as it arrives: latency and launches
        dict(name="decode d5 k3 x1", kind="decode", d=5, block=3, chi=4, batch=1, p=0.10, precision=0),
        # a real-time decoder's small batches at the headline's distance and options
        dict(name="decode d17 k6 x16 bf16", kind="decode", d=17, block=6, chi=32, batch=16, p=0.10, precision=1),
        # the headline Monte Carlo batch (Sec. IV): throughput
        dict(name="decode d17 k6 x4096 bf16", kind="decode", d=17, block=6, chi=32, batch=4096, p=0.10, precision=1),
        # a threshold scan at a smaller code in plain FP32, a ragged count
        dict(name="decode d11 k4 x1001", kind="decode", d=11, block=4, chi=16, batch=1001, p=0.15, precision=0),
        # syndromes of several code sizes and rates decoded together, replayed as one HIP graph
        dict(name="mixed d9-21 x2048 graph", kind="groups", distances="9,13,17,21", block=6, chi=32, batch=2048,
             precision=1, graph=True),
        # Z-biased noise (four Pauli probabilities), FP32
        dict(name="biased d17 k6 x512", kind="decode", d=17, block=6, chi=32, batch=512, p=0.10, precision=0,
             bias=10.0),
        # naive blockBP with blocks of 2 x 2 tensors
        dict(name="decode d17 k2 x2048", kind="decode", d=17, block=2, chi=4, batch=2048, p=0.10, precision=0),
        # accuracy studies with a binding chi: boundary MPSs compressed after every column
        dict(name="trunc d17 k6 chi8 x32", kind="decode", d=17, block=6, chi=8, batch=32, p=0.10, precision=0),
        dict(name="trunc d13 k8 chi16 x16", kind="decode", d=13, block=8, chi=16, batch=16, p=0.10, precision=0),
        # the single-block boundary-MPS decoder, the accuracy reference
        dict(name="bmps d13 chi16 x32", kind="bmps", d=13, chi=16, batch=32, p=0.10),
        # start messages of a batch by the learned warm start (inference)
        dict(name="warm forward d21 x512 bf16", kind="predict", d=21, block=6, chi=32, batch=512, p=0.10, precision=1),
        # one training step of the warm start: gradient and Adam
        dict(name="warm train d17 x16", kind="train", d=17, block=6, chi=32, batch=16, p=0.10),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))


def draw(rng):
    kind = rng.choice(("decode", "decode", "decode", "small", "groups", "trunc", "bmps", "predict", "train"))
    p = round(rng.uniform(0.05, 0.15), 4)
    if kind == "decode":
        d = rng.choice((3, 5, 7, 9, 11, 13, 15, 17, 19, 21, 23, 25))
        block = rng.choice((3, 4, 5, 6, 6, 6))
        c = dict(kind="decode", d=d, block=block, chi=EXACT_CHI[block], batch=_log_int(rng, 1, 4096 * 200 // max(200, d * d)),
                 p=p, precision=rng.choice((0, 1)))
        extra = rng.choice(("", "", "gate", "bias"))
        if extra == "gate":
            c["gate"] = 1e-5
        elif extra == "bias":
            c.update(precision=0, bias=float(rng.choice((3, 10, 30))))
        return c
    if kind == "small":
        block = rng.choice((1, 2))
        return dict(kind="decode", d=rng.choice((5, 9, 13, 17, 21)), block=block, chi=4, batch=_log_int(rng, 1, 2048), p=p,
                    precision=0)
    if kind == "groups":
        ds = sorted(rng.sample((5, 7, 9, 11, 13, 15, 17, 19, 21), rng.choice((2, 3, 4))))
        return dict(kind="groups", distances=",".join(map(str, ds)), block=6, chi=32, batch=_log_int(rng, 8, 2048),
                    precision=rng.choice((0, 1)), graph=rng.choice((False, True)))
    if kind == "trunc":
        block, chi = rng.choice(BINDING)
        d = rng.choice((7, 9, 11, 13))
        return dict(kind="decode", d=d, block=block, chi=chi, batch=_log_int(rng, 1, 24), p=p, precision=0)
    if kind == "bmps":
        return dict(kind="bmps", d=rng.choice((5, 7, 9, 11, 13)), chi=rng.choice((4, 8, 12, 16)), batch=_log_int(rng, 1, 32), p=p)
    if kind == "predict":
        precision = rng.choice((0, 1, 1, 1))
        return dict(kind="predict", d=rng.choice((9, 13, 17, 21, 25, 27)), block=rng.choice((3, 4, 6)), chi=32,
                    batch=_log_int(rng, 1, 60 if precision == 0 else 400), p=p, precision=precision)
    return dict(kind="train", d=rng.choice((13, 15, 17, 19, 21)), block=6, chi=32, batch=_log_int(rng, 4, 32), p=p)


# ------------------------------------------------------------------------------------------------ inputs
def _noise(case):
    """Probabilities of I, X, Z, Y (code x + 2z)."""
    if "bias" in case:
        return workload.biased_probs(case["p"], case["bias"])
    p = case["p"]
    return (1.0 - p, p / 3.0, p / 3.0, p / 3.0)


def _syndromes(d, pi, count, gen):
    """Syndromes [count, m] of sampled errors; pi: [4] probabilities by code, or [count, 4]."""
    pi = np.atleast_2d(np.asarray(pi, dtype=np.float64))
    edges = np.cumsum(pi, axis=1)[:, None, :3]
    u = gen.random((count, workload.num_qubits(d)))[:, :, None]
    return workload.syndrome_of(d, (u >= edges).sum(axis=2).astype(np.uint8))


def _opts(case):
    return bbp.default_opts(block=case["block"], chi=case["chi"], max_iter=20, precision=case.get("precision", 0),
                            gate=case.get("gate", 0.0), graph=int(case.get("graph", False)))


def _split(case, gen):
    """Per-group distances and per-syndrome rates of a mixed batch, its syndromes shared out evenly."""
    ds = [int(x) for x in case["distances"].split(",")]
    return [(d, gen.uniform(0.05, 0.15, case["batch"] // len(ds) + (k < case["batch"] % len(ds))))
            for k, d in enumerate(ds)]


def _host_inputs(case, seed):
    """The case's inputs as numpy arrays, from the seed alone."""
    gen = np.random.default_rng(seed)
    if case["kind"] == "groups":
        return [(d, ps, _syndromes(d, np.stack([1 - ps, ps / 3, ps / 3, ps / 3], axis=1), len(ps), gen))
                for d, ps in _split(case, gen)]
    syn = _syndromes(case["d"], _noise(case), case["batch"], gen)
    if case["kind"] != "train":
        return syn
    # converged messages put most of their weight on one configuration; most cosets converged
    M, K = _num_messages(case), _message_legs(case)
    peak = gen.integers(0, 1 << 30, size=(case["batch"], 4, M)) % (1 << K)
    t = gen.random((case["batch"], 4, M, 64)).astype(np.float32) * 0.02
    t[np.arange(64)[None, None, None, :] == peak[..., None]] = 1.0
    t *= np.arange(64) < (1 << K)[:, None]
    t /= np.sqrt((t * t).sum(axis=3, keepdims=True))
    use = (gen.random(4 * case["batch"]) < 0.9).astype(np.uint8)
    use[0] = 1
    return syn, t, use


def prepare(case, seed):
    dev = torch.device("cuda")
    host = _host_inputs(case, seed)
    if case["kind"] == "groups":
        groups = [(d, torch.from_numpy(ps).to(dev), torch.from_numpy(s).to(dev)) for d, ps, s in host]
        opts = _opts(case)
        outs = [bbp._outputs(len(ps), workload.num_qubits(d), dev) for d, ps, _ in host]
        sizes = sum(bbp.workspace_size(d, len(ps), opts) + 256 for d, ps, _ in host)
        return dict(case=case, groups=groups, opts=opts, outs=outs, stream=torch.cuda.Stream(),
                    ws=torch.empty(sizes, dtype=torch.uint8, device=dev))
    if case["kind"] == "bmps":
        ws = torch.empty(bbp.bmps_workspace_size(case["d"], case["batch"], case["chi"]), dtype=torch.uint8, device=dev)
        return dict(case=case, syn=torch.from_numpy(host).to(dev), ws=ws)
    opts = _opts(case)
    st = dict(case=case, opts=opts)
    if case["kind"] == "decode":
        st["syn"] = torch.from_numpy(host).to(dev)
        st["noise"] = _noise(case) if "bias" in case else case["p"]
        st["ws"] = torch.empty(bbp.workspace_size(case["d"], case["batch"], opts), dtype=torch.uint8, device=dev)
        return st
    st["params"] = torch.from_numpy(warm.load()).to(dev)
    train = case["kind"] == "train"
    st["ws"] = torch.empty(warm.workspace_size(case["d"], case["batch"], opts, train), dtype=torch.uint8, device=dev)
    if not train:
        st["syn"] = torch.from_numpy(host).to(dev)
        return st
    st["syn"], st["targets"], st["use"] = (torch.from_numpy(x).to(dev) for x in host)
    st["m"], st["v"] = torch.zeros_like(st["params"]), torch.zeros_like(st["params"])
    st["theta"] = st["params"].clone()
    return st


RESULTS = ("loglik", "delta", "iters", "coset", "correction")


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "groups":
        outs, _, _ = bbp.decode_groups(s["groups"], s["opts"], workspace=s["ws"], outs=s["outs"], stream=s["stream"])
        return [{k: o[k] for k in RESULTS} for o in outs]
    if kind == "bmps":
        out = bbp.bmps_decode(case["d"], case["p"], s["syn"], chi=case["chi"], workspace=s["ws"])
        return {k: out[k] for k in ("loglik", "coset", "correction")}
    if kind == "decode":
        if "bias" in case:
            outs, _, _ = bbp.decode_groups([(case["d"], s["noise"], s["syn"])], s["opts"], workspace=s["ws"])
            out = outs[0]
        else:
            out = bbp.decode_device(case["d"], s["noise"], s["syn"], s["opts"], workspace=s["ws"])
        return {k: out[k] for k in RESULTS}
    if kind == "predict":
        return warm.predict(case["d"], case["p"], s["syn"], s["opts"], s["params"], precision=case["precision"],
                            workspace=s["ws"])
    # one training step: the gradient at the parameters, and an optimiser step on the running copy
    loss, grad = warm.loss_grad(case["d"], case["p"], s["syn"], s["opts"], s["params"], s["targets"], s["use"],
                                workspace=s["ws"])
    warm.adam(s["theta"], grad, s["m"], s["v"], 1, 1e-4)
    return loss, grad


# ------------------------------------------------------------------------------------------------ work
def work(case):
    if case["kind"] == "groups":
        ds = [int(x) for x in case["distances"].split(",")]
        parts = [work(dict(case, kind="decode", d=d, batch=case["batch"] / len(ds))) for d in ds]
        return {k: sum(x[k] for x in parts) for k in ("bytes", "flops")}
    d, b = case["d"], case["batch"]
    L, m, n = 2 * d - 1, 2 * d * (d - 1), workload.num_qubits(d)
    if case["kind"] == "bmps":
        # per row and column: absorption, QR, SVD and carry at the natural bonds min(chi, 2^j, 2^(L-j))
        bond = [min(case["chi"], 2 ** min(j, 30), 2 ** min(L - j, 30)) for j in range(L + 1)]
        wide = [min(2 * bond[j], 2 ** min(j, 30), 2 ** min(L - j, 30)) for j in range(L + 1)]
        f = 0.0
        for r in range(L):
            mm, nn = 2 * wide[r], wide[r + 1]
            k = min(wide[r], 2 * bond[r + 1])
            f += 4 * mm * nn * bond[r] + 2 * mm * nn * nn + 4 * mm * bond[r + 1] * min(mm, nn) + 21 * k ** 3
        return {"bytes": b * (m + 33 + n), "flops": 4 * b * (L - 1) * f}
    rows = 4 * b * L * L
    macs = 99 * 64 + 576 * 128 + 1152 * 96
    if case["kind"] in ("predict", "train"):
        M = _num_messages(case)
        out = 4 * b * M * 64 * 4
        if case["kind"] == "predict":
            return {"bytes": b * m + out + 4 * warm.param_count(), "flops": 2.0 * rows * macs}
        return {"bytes": b * m + out + 16 * warm.param_count(), "flops": 2.0 * rows * (3 * macs - 99 * 64)}
    if case["chi"] < EXACT_CHI.get(case["block"], 1 << 30) or case["block"] > 6:
        # a truncating update: per site and column, absorption, QR and SVD at bond 2 chi (about 220 chi^3)
        k, x = case["block"], case["chi"]
        M = _num_messages(case)
        per = 220.0 * x ** 3 * k * (k + 2)
        flops = 4 * b * EARLY_EXIT_ITERS * M * per
    else:
        info = bbp.plan_query(d, _opts(case))
        flops = 4 * b * (EARLY_EXIT_ITERS * info.flops_per_iter + info.flops_bethe)
    return {"bytes": b * (m + 4 * 20 + 1 + n), "flops": flops}


# ------------------------------------------------------------------------------------- 64-bit evaluation
def _extents(L, k):
    return [(s, min(k, L - s)) for s in range(0, L, k)]


MOVES = ((0, 1), (0, -1), (1, 0), (-1, 0))   # E, W, S, N


def _messages(d, k):
    """Directed messages (sender block, receiver block, direction, legs), in the library's order."""
    ext = _extents(2 * d - 1, k)
    nb, out = len(ext), []
    for I in range(nb):
        for J in range(nb):
            for f, (di, dj) in enumerate(MOVES):
                if 0 <= I + di < nb and 0 <= J + dj < nb:
                    out.append(((I, J), (I + di, J + dj), f, ext[I if f < 2 else J][1]))
    return ext, out


def _num_messages(case):
    return len(_messages(case["d"], case["block"])[1])


def _message_legs(case):
    return np.array([K for _, _, _, K in _messages(case["d"], case["block"])[1]])


def _labels(d, syn):
    """x and z bits [batch, 4, L, L] of the coset labels (I, X, Y, Z) of syndromes [batch, m]."""
    L, nz = 2 * d - 1, d * (d - 1)
    s = syn.astype(np.int64)
    x, z = np.zeros((len(s), L, L), np.int64), np.zeros((len(s), L, L), np.int64)
    zc, xc = s[:, :nz].reshape(-1, d, d - 1), s[:, nz:].reshape(-1, d - 1, d)
    # parity of the checks right of / below each horizontal edge
    x[:, ::2, 0:L - 1:2] = np.cumsum(zc[:, :, ::-1], axis=2)[:, :, ::-1] % 2
    z[:, 0:L - 1:2, ::2] = np.cumsum(xc[:, ::-1], axis=1)[:, ::-1] % 2
    xs, zs = np.repeat(x[:, None], 4, 1), np.repeat(z[:, None], 4, 1)
    xs[:, (1, 2), 0, ::2] ^= 1
    zs[:, (2, 3), ::2, 0] ^= 1
    return xs, zs


def _site(x, z, r, c, L, pi):
    """Tensor [jobs, up, left, down, right] of a grid site; legs that leave the grid only take the value 0."""
    n = x.shape[0]
    if (r + c) % 2 == 0:
        b = torch.arange(2, device=pi.device)
        ud = (b[:, None, None, None] ^ b[None, None, :, None]).expand(2, 2, 2, 2)
        lr = (b[None, :, None, None] ^ b[None, None, None, :]).expand(2, 2, 2, 2)
        fx, fz = (ud, lr) if r % 2 == 0 else (lr, ud)
        code = (x[:, r, c].view(-1, 1, 1, 1, 1) ^ fx) + 2 * (z[:, r, c].view(-1, 1, 1, 1, 1) ^ fz)
        t = torch.gather(pi, 1, code.reshape(n, 16)).reshape(n, 2, 2, 2, 2)
    else:
        t = torch.zeros(1, 2, 2, 2, 2, dtype=pi.dtype, device=pi.device)
        for v in range(2):
            t[(0,) + tuple(v if ok else 0 for ok in (r > 0, c > 0, r < L - 1, c < L - 1))] = 1.0
        return t.expand(n, 2, 2, 2, 2)
    keep = t.clone()
    if r == 0:
        keep[:, 1] = 0
    if c == 0:
        keep[:, :, 1] = 0
    if r == L - 1:
        keep[:, :, :, 1] = 0
    if c == L - 1:
        keep[:, :, :, :, 1] = 0
    return keep


def _reversed_legs(m, K):
    return m.reshape((-1,) + (2,) * K).permute((0,) + tuple(range(K, 0, -1))).reshape(-1, 2 ** K)


def _cap(msg, K, t, like):
    """Operator [jobs or 1, old, emitted, new] that absorbs leg t of a K-leg side message (first leg first): the
    bond carries the legs emitted so far up to the middle leg, the legs still to come after it."""
    if msg is None:
        return torch.tensor([1.0, 0.0], dtype=like.dtype, device=like.device).view(1, 1, 2, 1)
    D = K // 2
    if t == D:
        return msg.reshape(-1, 2 ** D, 2, 2 ** (K - D - 1))
    if t < D:
        return torch.eye(2 ** (t + 1), dtype=like.dtype, device=like.device).view(1, 2 ** t, 2, 2 ** (t + 1))
    r = 2 ** (K - t - 1)
    return torch.eye(2 * r, dtype=like.dtype, device=like.device).view(2, r, 2, r).permute(0, 1, 2, 3).reshape(1, 2 * r, 2, r)


def _sweep(tensors, ext, I, J, f, msgs):
    """Contraction of block (I, J) toward side f with its other incoming messages: unit vectors over the crossing
    configurations [jobs, 2^kp] and the natural log of the scale."""
    (r0, kr), (c0, kc) = ext[I], ext[J]
    get = lambda i, j: msgs.get(((i, j), (I, J)))   # noqa: E731
    if f < 2:
        kt, kp = kc, kr
        site = lambda t, i: (r0 + i, c0 + (t if f == 0 else kc - 1 - t))   # noqa: E731
        perm = (0, 1, 2, 3, 4) if f == 0 else (0, 1, 4, 3, 2)
        init, top, bot = get(I, J - 1 if f == 0 else J + 1), get(I - 1, J), get(I + 1, J)
    else:
        kt, kp = kr, kc
        site = lambda t, i: (r0 + (t if f == 2 else kr - 1 - t), c0 + i)   # noqa: E731
        perm = (0, 2, 1, 4, 3) if f == 2 else (0, 2, 3, 4, 1)
        init, top, bot = get(I - 1 if f == 2 else I + 1, J), get(I, J - 1), get(I, J + 1)
    if f in (1, 3):
        top, bot = (None if m is None else _reversed_legs(m, kt) for m in (top, bot))
    like = tensors[0][0]
    n = like.shape[0]
    if init is None:
        psi = torch.zeros(n, 2 ** kp, dtype=like.dtype, device=like.device)
        psi[:, 0] = 1.0
    else:
        psi = init
    psi = psi.reshape(n, 1, 2 ** kp, 1)
    logs = torch.zeros(n, dtype=like.dtype, device=like.device)
    for t in range(kt):
        op = _cap(top, kt, t, like).expand(n, -1, -1, -1)
        S = psi.shape[3]
        N = op.shape[3]
        psi = torch.bmm(op.reshape(n, op.shape[1], -1).transpose(1, 2).contiguous(), psi.reshape(n, op.shape[1], -1))
        psi = psi.reshape(n, 2, N, 2 ** kp * S)
        for i in range(kp):
            r, c = site(t, i)
            T = tensors[r][c].permute(perm).reshape(n, 4, 4)                       # (up, in), (down, out)
            q = psi.reshape(n, 2, N * 2 ** i, 2, -1).permute(0, 1, 3, 2, 4).reshape(n, 4, -1)
            q = torch.bmm(T.transpose(1, 2).contiguous(), q)
            psi = q.reshape(n, 2, 2, N * 2 ** i, -1).permute(0, 1, 3, 2, 4)
        op = _cap(bot, kt, t, like).expand(n, -1, -1, -1)
        psi = psi.reshape(n, 2, N * 2 ** kp, S).permute(0, 2, 3, 1).reshape(n, N * 2 ** kp, S * 2)
        psi = torch.bmm(psi.contiguous(), op.reshape(n, S * 2, -1).contiguous()).reshape(n, N, 2 ** kp, -1)
        nrm = psi.reshape(n, -1).norm(dim=1)
        psi = psi / nrm.view(-1, 1, 1, 1)
        logs = logs + nrm.log()
    return psi.reshape(n, 2 ** kp), logs


def _blockbp(d, block, syn, pi, max_iter=20, delta0=1e-4, eta=0.1, gate=0.0):
    """ln Z and Delta [batch, 4] of blockBP with exact block contractions; pi: [1 or batch, 4] by code x + 2z."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    L = 2 * d - 1
    xs, zs = (torch.from_numpy(a.reshape(-1, L, L)).to(dev) for a in _labels(d, syn))
    n = xs.shape[0]
    pi = torch.from_numpy(np.repeat(np.broadcast_to(np.atleast_2d(np.asarray(pi, np.float64)), (len(syn), 4)), 4, 0)).to(dev)
    T = [[_site(xs, zs, r, c, L, pi) for c in range(L)] for r in range(L)]
    ext, edges = _messages(d, block)
    M = len(edges)
    msgs = {(a, b): torch.full((n, 2 ** K), 2.0 ** (-K / 2), dtype=torch.float64, device=dev) for a, b, _, K in edges}
    terms = {k: torch.full((n,), math.inf, dtype=torch.float64, device=dev) for k in msgs}
    delta = torch.full((n,), math.inf, dtype=torch.float64, device=dev)
    active = torch.ones(n, dtype=torch.bool, device=dev)
    for _ in range(max_iter):
        idx = active.nonzero().ravel()
        if idx.numel() == 0:
            break
        Ts = T if idx.numel() == n else [[t[idx] for t in row] for row in T]
        sub = {k: v[idx] for k, v in msgs.items()}
        for colour in (0, 1):
            fresh = {}
            for a, b, f, _ in edges:
                if (a[0] + a[1]) % 2 != colour:
                    continue
                new, _ = _sweep(Ts, ext, a[0], a[1], f, {k: v for k, v in sub.items() if k[1] == a and k[0] != b})
                old = sub[(a, b)]
                new = new / new.norm(dim=1, keepdim=True)
                new = (1 - eta) * new + eta * old
                new = new / new.norm(dim=1, keepdim=True)
                term = 0.5 * (new - old).square().sum(1) * (new + old).square().sum(1)
                if gate > 0:
                    still = terms[(a, b)][idx] < gate
                    for w, dst, _, _ in edges:
                        if dst == a and w != b:
                            still &= terms[(w, dst)][idx] < gate
                    new, term = torch.where(still[:, None], old, new), torch.where(still, 0.0, term)
                fresh[(a, b)] = (new, term)
            for k, (new, term) in fresh.items():
                sub[k] = new
                msgs[k][idx] = new
                terms[k][idx] = term
        dl = torch.stack([t[idx] for t in terms.values()]).sum(0).clamp(min=0).sqrt() / max(M, 1) if M else torch.zeros(
            idx.numel(), dtype=torch.float64, device=dev)
        delta[idx] = dl
        active[idx] = dl >= delta0
    lnz = torch.zeros(n, dtype=torch.float64, device=dev)
    for I in range(len(ext)):
        for J in range(len(ext)):
            v, ls = _sweep(T, ext, I, J, 0, {k: m for k, m in msgs.items() if k[1] == (I, J) and k[0] != (I, J + 1)})
            close = msgs.get(((I, J + 1), (I, J)))
            lnz += ls + torch.log(v[:, 0] if close is None else (v * close).sum(1))
    for a, b, _, _ in edges:
        if a < b:
            lnz -= torch.log((msgs[(a, b)] * msgs[(b, a)]).sum(1))
    bad = ~torch.isfinite(lnz)
    return lnz.masked_fill(bad, math.nan).reshape(-1, 4), delta.masked_fill(bad, math.inf).reshape(-1, 4)


def _bmps(d, chi, syn, pi):
    """Boundary-MPS estimates of ln Z [batch, 4], compressed to chi after every column but the last."""
    L = 2 * d - 1
    xs, zs = (torch.from_numpy(a.reshape(-1, L, L)) for a in _labels(d, syn))
    n = xs.shape[0]
    pi = torch.tensor(pi, dtype=torch.float64).view(1, 4).expand(n, 4).contiguous()
    A = [torch.ones(n, 1, 1, 1, dtype=torch.float64) for _ in range(L)]
    logs = torch.zeros(n, dtype=torch.float64)
    for c in range(L):
        for r in range(L):
            T = _site(xs, zs, r, c, L, pi)
            T = T[:, :1 if r == 0 else 2, :A[r].shape[2], :1 if r == L - 1 else 2, :1 if c == L - 1 else 2]
            a = torch.einsum("basc,busdt->bautcd", A[r], T)
            A[r] = a.reshape(n, a.shape[1] * a.shape[2], a.shape[3], a.shape[4] * a.shape[5])
        if c == L - 1:
            break
        for r in range(L - 1):
            s = A[r].shape
            Q, R = torch.linalg.qr(A[r].reshape(n, s[1] * s[2], s[3]))
            A[r] = Q.reshape(n, s[1], s[2], -1)
            A[r + 1] = torch.einsum("bij,bjsk->bisk", R, A[r + 1])
            nr = A[r + 1].reshape(n, -1).norm(dim=1)
            A[r + 1] = A[r + 1] / nr.view(-1, 1, 1, 1)
            logs += nr.log()
        for r in range(L - 1, 0, -1):
            s = A[r].shape
            U, S, V = torch.linalg.svd(A[r].reshape(n, s[1], -1), full_matrices=False)
            k = min(chi, S.shape[1])
            A[r] = V[:, :k].reshape(n, k, s[2], s[3])
            A[r - 1] = torch.einsum("basi,bij->basj", A[r - 1], U[:, :, :k] * S[:, None, :k])
            nr = A[r - 1].reshape(n, -1).norm(dim=1)
            A[r - 1] = A[r - 1] / nr.view(-1, 1, 1, 1)
            logs += nr.log()
    v = torch.ones(n, 1, dtype=torch.float64)
    for r in range(L):
        v = torch.einsum("ba,bac->bc", v, A[r][:, :, 0])
        s = v.abs().amax(dim=1)
        v, logs = v / s[:, None], logs + s.log()
    return torch.where(v[:, 0] > 0, logs + v[:, 0].clamp(min=1e-300).log(), math.nan).reshape(-1, 4)


def _channels(d, p, syn):
    """Input channels [jobs, L, L, 11] of the warm-start network."""
    L, nz = 2 * d - 1, d * (d - 1)
    lx, lz = _labels(d, syn)
    X = np.zeros((len(syn), 4, L, L, 11))
    r, c = np.indices((L, L))
    qubit, vertex, plaq = (r + c) % 2 == 0, (r % 2 == 0) & (c % 2 == 1), (r % 2 == 1) & (c % 2 == 0)
    X[..., 0], X[..., 1] = lx, lz
    s = np.zeros((len(syn), L, L))
    s[:, ::2, 1::2] = syn[:, :nz].reshape(-1, d, d - 1)
    s[:, 1::2, ::2] = syn[:, nz:].reshape(-1, d - 1, d)
    X[..., 2] = s[:, None]
    X[..., 3], X[..., 4], X[..., 5] = qubit, vertex, plaq
    X[..., 6], X[..., 7] = p, 1.0
    X[:, (1, 2), ..., 8] = 1.0
    X[:, (2, 3), ..., 9] = 1.0
    hx, hz = lx * ((r % 2 == 0) & (c % 2 == 0)), lz * ((r % 2 == 0) & (c % 2 == 0))
    X[..., 10] = np.where(plaq, np.cumsum(hx, axis=2) % 2, np.where(vertex, np.cumsum(hz, axis=3) % 2, 0))
    return torch.from_numpy(X.reshape(-1, L, L, 11))


def _scores(d, block, X, theta):
    """Scores [jobs, M, 64] of every message configuration (-inf beyond 2^K)."""
    parts, o = [], 0
    shapes = [(99, 64), (64,), (576, 128), (128,), (1152, 96), (96,)] + [(192, 2), (2,), (384, 4), (4,)] * 4
    for s in shapes:
        parts.append(theta[o:o + math.prod(s)].reshape(s))
        o += math.prod(s)
    n, L = X.shape[:2]
    for k in range(3):
        W, b = parts[2 * k], parts[2 * k + 1]
        P = torch.nn.functional.pad(X, (0, 0, 1, 1, 1, 1))
        C = X.shape[3]
        Y = b
        for t in range(9):
            Y = Y + P[:, t // 3:t // 3 + L, t % 3:t % 3 + L].reshape(-1, C) @ W[t * C:(t + 1) * C]
        X = Y.reshape(n, L, L, -1)
        X = X.clamp(min=0) if k < 2 else X
    ext, edges = _messages(d, block)
    out = []
    for (I, J), _, f, K in edges:
        (r0, kr), (c0, kc) = ext[I], ext[J]
        i = torch.arange(K)
        if f < 2:
            r, c = r0 + i, torch.full((K,), c0 + (kc - 1 if f == 0 else 0))
        else:
            r, c = torch.full((K,), r0 + (kr - 1 if f == 2 else 0)), c0 + i
        di, dj = MOVES[f]
        F = torch.cat([X[:, r, c], X[:, r + di, c + dj]], dim=2)                     # [jobs, K, 192]
        Wu, bu, Wp, bp = parts[6 + 4 * f:10 + 4 * f]
        u = F @ Wu + bu
        pr = torch.cat([F[:, :-1], F[:, 1:]], dim=2) @ Wp + bp
        bits = (torch.arange(2 ** K, device=X.device)[:, None] >> torch.arange(K - 1, -1, -1, device=X.device)) & 1
        s = sum(u[:, k, bits[:, k]] for k in range(K))
        s = s + sum((pr[:, k, 2 * bits[:, k] + bits[:, k + 1]] for k in range(K - 1)), torch.zeros_like(s))
        out.append(torch.nn.functional.pad(s, (0, 64 - 2 ** K), value=-math.inf))
    return torch.stack(out, dim=1)


def exact(case, seed):
    # In BF16 a slowly drifting coset can stop an iteration or more away from where it stops in 64 bits, on another
    # distance: that distance has no 64-bit value to be held to.
    host = _host_inputs(case, seed)
    kind = case["kind"]
    bf16 = case.get("precision", 0) == 1
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    if kind == "groups":
        if case["batch"] > 1024:
            return None
        out = []
        for d, ps, syn in host:
            ll, dl = _blockbp(d, case["block"], syn, np.stack([1 - ps, ps / 3, ps / 3, ps / 3], axis=1))
            out.append(dict(loglik=ll, delta=None if bf16 else dl, iters=None, coset=None, correction=None))
        return out
    if kind == "bmps":
        if 4 * case["batch"] * (2 * case["d"] - 1) ** 2 > 90000:
            return None
        return dict(loglik=_bmps(case["d"], case["chi"], host, _noise(case)), coset=None, correction=None)
    if kind == "decode":
        if case["chi"] < EXACT_CHI.get(case["block"], 1 << 30) or case["block"] > 6:
            return None   # a compression in every block update
        blocks = len(_extents(2 * case["d"] - 1, case["block"])) ** 2
        if case["batch"] * case["d"] ** 2 > 300000 or blocks > 150:
            return None
        ll, dl = _blockbp(case["d"], case["block"], host, _noise(case), gate=case.get("gate", 0.0))
        return dict(loglik=ll, delta=None if bf16 else dl, iters=None, coset=None, correction=None)
    theta = torch.from_numpy(warm.load()).double().to(dev)
    if kind == "predict":
        out = []
        step = max(1, 4000 // case["d"] ** 2)
        for b in range(0, case["batch"], step):
            s = _scores(case["d"], case["block"], _channels(case["d"], case["p"], host[b:b + step]).to(dev), theta)
            m = torch.exp(s - s.amax(dim=2, keepdim=True))
            out.append(m / m.norm(dim=2, keepdim=True))
        return torch.cat(out).reshape(case["batch"], 4, -1, 64)
    syn, targets, use = host
    theta.requires_grad_(True)
    idx = np.flatnonzero(use)
    X = _channels(case["d"], case["p"], syn)[idx]
    t = torch.from_numpy(targets.reshape((-1,) + targets.shape[2:])[idx]).double()
    count, total, step = len(idx) * t.shape[1], 0.0, 16
    for b in range(0, len(idx), step):
        logp = torch.log_softmax(_scores(case["d"], case["block"], X[b:b + step].to(dev), theta), dim=2)
        q = t[b:b + step].to(dev)
        q = q / q.sum(dim=2, keepdim=True)
        part = torch.where(q > 0, q * (q.clamp(min=1e-300).log() - logp.masked_fill(q <= 0, 0.0)), 0.0).sum() / count
        part.backward()
        total = total + part.detach()
    return total.reshape(1), theta.grad
