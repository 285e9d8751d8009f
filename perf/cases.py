"""The calls of this framework that its speed is judged by: GreedyLore steps
as a training program makes them.

A program keeps one compressor and calls step() once per training step; a
step is one of three kinds, and each is a case of its own here:

  select   a step between refreshes: the r columns of the kept basis U are
           chosen by their scores (tau - 1 of every tau steps)
  refresh  a step with t mod tau == 0: the complete singular basis of the
           worker mean is computed anew, warm-started from the previous one
  tau1     tau = 1, every step a refresh of the leading block only

prepare() builds what such a program holds in the middle of its training and
restores it through write_state() / resume(), as a resume from a checkpoint
does: optimizer state, error buffers and their mean, and an orthonormal basis
U whose leading rows are the planted directions of the gradients (the weights
are zero, so that what a step adds to them can be compared; the time does not
depend on them).  The gradients are a planted low-rank part shared by the workers
(r directions falling from 10 to 1, then as many again at 1/3, so that the
leading r are determined by the data) plus fresh Gaussian noise per worker.
A refresh or tau1 state alternates between two gradient batches of opposite
noise and tail: what is refreshed differs from pass to pass, as it does in
training, and the error buffers stay bounded however many passes are made.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2507_08784_amd as glr

LR, BETA1, BETA2, EPS = 1e-3, 0.9, 0.999, 1e-8
NOISE = 1.0 / 3.0          # largest singular value of the worker mean's noise
T0 = 3                     # refresh periods behind a restored state


# ----------------------------------------------------------------------------
# the cases
# ----------------------------------------------------------------------------
def _conv_shapes(count):
    """The reshaped convolution kernels of the repository's 50-layer workload:
    {64..512} output channels by {576..2304} inputs times taps."""
    rng = np.random.default_rng([0, 0x5EED0003])
    ds = rng.choice([64, 128, 256, 512], size=count)
    Ds = rng.choice([576, 1152, 2304], size=count)
    return ",".join(f"{a}x{b}" for a, b in zip(ds, Ds))


def _case(name, step, shapes, workers, rank, tau, opt, select="approx", store="fp32"):
    c = {"step": step, "shapes": shapes, "workers": workers, "rank": rank, "tau": tau, "opt": opt,
         "select": select, "store": store}
    if name:
        c["name"] = name
    return c


def listed():
    conv = _conv_shapes(50)
    # the six weight matrices of one encoder layer of width 768: four square
    # ones and a wide and a tall one, so the sides differ inside one step
    enc = "768x768,768x768,768x768,768x768,3072x768,768x3072"
    return [
        # the smallest real layer: launches and latency are all there is
        _case("select_256x128", "select", "256x128", 4, 4, 5, "msgd"),
        _case("refresh_256x128", "refresh", "256x128", 4, 4, 5, "msgd"),
        # all fifty convolution layers of a residual network in one step
        _case("select_conv50", "select", conv, 16, 8, 20, "msgd"),
        _case("refresh_conv50", "refresh", conv, 16, 8, 20, "msgd"),
        # one encoder layer in one step, matrices of both orientations
        _case("select_encoder768", "select", enc, 4, 16, 10, "adam"),
        # a layer whose sides are multiples of nothing, scored exactly
        _case("select_1011x2053_exact", "select", "1011x2053", 3, 50, 10, "adam", select="exact"),
        # the square attention weight of a transformer of width 4096
        _case("select_4096", "select", "4096x4096", 8, 64, 10, "msgd"),
        _case("refresh_4096", "refresh", "4096x4096", 8, 64, 10, "msgd"),
        # its feed-forward weights, tall in fp32 and wide with bf16 gradients
        _case("select_11008x4096", "select", "11008x4096", 8, 128, 10, "adam"),
        _case("select_4096x11008_bf16", "select", "4096x11008", 8, 128, 10, "adam", store="bf16"),
        # every step a refresh: a small feed-forward weight, and the largest
        # weight of the repository's benchmark
        _case("tau1_768x3072", "tau1", "768x3072", 4, 32, 1, "adam"),
        _case("tau1_8192x28672", "tau1", "8192x28672", 4, 256, 1, "adam"),
    ]


def draw(rng):
    """One step of the same ranges: one to eight matrices, min(m, n) from 40
    to 4096, aspect ratios up to four, ranks from 2 to 256, one worker (a
    communication hook's case) to sixteen, odd sizes as often as round ones."""
    step = rng.choice(["select", "select", "refresh", "tau1"])
    count = rng.choice([1, 1, 1, 2, 5, 8])
    top = 4096 if count == 1 else 1024
    base = math.exp(rng.uniform(math.log(40), math.log(top)))
    workers = rng.choice([1, 2, 3, 4, 8, 16])
    unit = rng.choice([1, 1, 2, 32, 64])
    shapes = []
    for _ in range(count):
        d = min(top, max(40, base * rng.uniform(0.7, 1.3)))
        D = d * math.exp(rng.uniform(0.0, math.log(4.0)))
        d, D = (max(unit, int(round(x / unit)) * unit) for x in (d, D))
        d, D = max(d, 40), max(D, d, 40)
        while workers > 1 and workers * d * D > 8 * 4096 * 11008:
            workers //= 2
        shapes.append(f"{D}x{d}" if rng.random() < 0.5 else f"{d}x{D}")
    dmin = min(min(int(a) for a in s.split("x")) for s in shapes)
    rank = int(round(math.exp(rng.uniform(math.log(2), math.log(min(256, dmin // 4))))))
    opt = rng.choice(["msgd", "adam"])
    store = rng.choice(["fp32", "fp32", "bf16"])
    select = rng.choice(["approx", "approx", "exact", "approx_bf16"]) if step == "select" else "approx"
    tau = 1 if step == "tau1" else rng.choice([5, 10, 20])
    return _case(None, step, ",".join(shapes), workers, rank, tau, opt, select, store)


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------
def _shapes(case):
    return [tuple(int(x) for x in s.split("x")) for s in case["shapes"].split(",")]


def _orthonormal(d, gen):
    """d x d orthonormal rows (fp64): a cosine basis with random signs, its
    rows permuted, after one random reflection."""
    n = torch.arange(d, dtype=torch.float64, device="cuda")
    B = torch.cos(math.pi / d * torch.outer(n, n + 0.5)).mul_(math.sqrt(2.0 / d))
    B[0] *= math.sqrt(0.5)
    B *= (torch.randint(0, 2, (d,), generator=gen, device="cuda", dtype=torch.float64) * 2 - 1)
    B = B[torch.randperm(d, generator=gen, device="cuda")]
    v = torch.randn(d, generator=gen, device="cuda", dtype=torch.float64)
    v /= v.norm()
    B -= torch.outer(2.0 * (B @ v), v)
    return B


def _matrix(case, shape, gen, batches):
    """Everything a program holds for one matrix."""
    m, n = shape
    d, D = min(m, n), max(m, n)
    N, r = case["workers"], min(case["rank"], d)
    right = m > n
    f32 = dict(device="cuda", dtype=torch.float32)
    gdt = torch.bfloat16 if case["store"] == "bf16" else torch.float32
    B = _orthonormal(d, gen)
    k = min(2 * r, d // 2)
    s = torch.tensor([10.0 ** (1.0 - j / r) if j < r else 1.0 / 3.0 for j in range(k)], **f32)
    L = B[:k].float()
    R = torch.randn(k, D, generator=gen, **f32) / math.sqrt(D)

    def part(w):
        A = (L * w[:, None]).T @ R
        return A.T if right else A

    first = torch.arange(k, device="cuda") < r
    lead, tail = part(torch.where(first, s, 0.0)), part(torch.where(first, 0.0, s))
    nu = NOISE * math.sqrt(N) / (math.sqrt(d) + math.sqrt(D))

    def workers(base, sd):
        out = torch.empty(N, m, n, device="cuda", dtype=gdt)
        for i in range(N):
            out[i] = base + sd * torch.randn(m, n, generator=gen, **f32)
        return out

    G = [workers(lead + tail, nu)]
    if batches == 2:
        G.append(torch.empty_like(G[0]))
        for i in range(N):
            G[1][i] = 2.0 * lead - G[0][i]
    E = workers(0.5 * tail, 0.7 * nu)
    Ebar = torch.zeros(m, n, device="cuda", dtype=torch.float64)
    for i in range(N):
        Ebar += E[i]
    gs = 10.0 / math.sqrt(m * n)      # size of a gradient element
    S1 = gs * torch.randn(m, n, generator=gen, **f32)
    S2 = gs * gs * (0.5 + torch.rand(m, n, generator=gen, **f32)) if case["opt"] == "adam" else None
    return {"G": G, "E": E, "Ebar": (Ebar / N).float(), "U": B.float(), "S1": S1, "S2": S2}


def _first_step(case):
    t = T0 * case["tau"]
    return t + 1 if case["step"] == "select" else t


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return [_matrix(case, s, gen, 1 if case["step"] == "select" else 2) for s in _shapes(case)]


def prepare(case, seed):
    mats = _inputs(case, seed)
    comp = glr.GreedyLore(_shapes(case), case["workers"], case["rank"], case["tau"], opt=case["opt"], lr=LR,
                          beta1=BETA1, beta2=BETA2, eps=EPS, select=case["select"], seed=1234 + seed % 1000,
                          store=case["store"])
    for l, a in enumerate(mats):
        parts = {"E": a.pop("E"), "Ebar": a.pop("Ebar"), "Ut": a.pop("U"), "S1": a.pop("S1")}
        S2 = a.pop("S2")
        if S2 is not None:
            parts["S2"] = S2
        comp.write_state(l, **parts)
        torch.cuda.current_stream().synchronize()   # before `parts` is freed
    # the weights lie side by side in one buffer, each 256-byte aligned
    sizes = [(m * n + 63) // 64 * 64 for m, n in _shapes(case)]
    weights = torch.zeros(sum(sizes), device="cuda")
    X, at = [], 0
    for (m, n), size in zip(_shapes(case), sizes):
        X.append(weights[at:at + m * n].view(m, n))
        at += size
    t = _first_step(case)
    comp.resume(t)
    return {"comp": comp, "case": case, "t": t, "pass": 0, "weights": weights, "X": X, "G": [a["G"] for a in mats]}


def run(state):
    comp, case, t = state["comp"], state["case"], state["t"]
    G = [g[state["pass"] % len(g)] for g in state["G"]]
    comp.step(state["X"], G, t)
    # the next step of the same kind
    tau = case["tau"]
    state["pass"] += 1
    if case["step"] == "select":
        state["t"] = t + 1 if (t + 1) % tau else t + 2
    else:
        state["t"] = t + tau
    if state["t"] != t + 1:
        comp.resume(state["t"])
    return _outputs(comp, case, state["weights"])


def _many(case):
    """More matrices than eight: fewer outputs of each."""
    return case["shapes"].count(",") >= 8


def _outputs(comp, case, weights):
    """The weights and the state that the step updated.  The basis of a
    refresh is left out (its columns have no sign, and those inside the noise
    no order of their own); the weights, the residuals and the singular values
    follow from it.  Of many matrices, each gives its error buffers and their
    mean in one piece (they are neighbours in the state)."""
    outs = [weights]
    for l, L in enumerate(comp.layouts):
        if _many(case):
            at = (-comp.state.data_ptr()) % 256
            outs.append(comp.state[at + L.off_E:at + L.off_Ebar + 4 * L.m * L.n].view(torch.float32))
            continue
        out = {"E": comp.E(l), "Ebar": comp.Ebar(l), "S1": comp.S1(l)}
        if case["opt"] == "adam":
            out["S2"] = comp.S2(l)
        if case["step"] == "select":
            out["score"] = comp.score(l)
            out["Rbar"] = comp.Rbar(l)
        elif case["step"] == "refresh":
            out["sigma"] = comp.sigma(l)
        outs.append(out)
    return outs


# ----------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------
def work(case):
    """Bytes: the gradients once, the error buffers, their mean, the weights
    and the optimizer state in and out, the basis in (and out at a refresh).
    Flops: the projection, the residuals and the reconstruction; the scores
    2 d^2 D; a refresh the Gram d^2 D and 16/3 d^3 for a dense symmetric
    eigenproblem with vectors (reduction 4/3, vectors 2, back transformation
    2); tau = 1 one pass of the block through M and back, 4 r d D."""
    nbytes = flops = 0.0
    N, es = case["workers"], 2 if case["store"] == "bf16" else 4
    for m, n in _shapes(case):
        d, D = min(m, n), max(m, n)
        r = min(case["rank"], d)
        mn = m * n
        nbytes += 3.0 * N * mn * es + 8.0 * mn * (3 + (case["opt"] == "adam"))
        flops += 2.0 * r * mn * (2 * N + 1)
        if case["step"] == "select":
            nbytes += 4.0 * d * d
            flops += 2.0 * d * d * D
        elif case["step"] == "refresh":
            nbytes += 8.0 * d * d
            flops += 1.0 * d * d * D + 16.0 / 3.0 * d ** 3
        else:
            nbytes += 8.0 * r * d
            flops += 4.0 * r * mn
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the error against exact(), the largest of all outputs:
    a selection step 1e-7 .. 1.8e-6 (the scores are squares of cancelling
    sums), a refresh 1e-6 .. 2.5e-6 (the noise of Ebar is 1 / sqrt(N) of the
    workers'), a tau = 1 step 1e-4 .. 6e-4 (its block iteration stops when the
    leading subspace moves by less than 1e-5, and E is a hundredth of M).
    Buffers in bf16 add the rounding of the few elements that lie between two
    values: 7e-5, an element by one step of 2^-8."""
    if case["step"] == "tau1":
        return {"rel": 2.5e-3, "max": 0.1}
    if case["store"] == "bf16":
        return {"rel": 3e-4, "max": 0.01}
    return {"rel": 1e-5 if case["step"] == "select" else 2e-5}


# ----------------------------------------------------------------------------
# the same step in 64 bits
# ----------------------------------------------------------------------------
def _philox(c, j, mat, t, key):
    """Philox4x32-10 (Salmon et al., SC'11) on int64 tensors."""
    M32 = 0xFFFFFFFF
    x0, x1, x2, x3 = torch.broadcast_tensors(c, j, torch.full_like(c, mat), torch.full_like(c, t))
    k0, k1 = key & M32, (key >> 32) & M32
    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
        pa, pb = x0 * 0xD2511F53, x2 * 0xCD9E8D57
        x0, x1, x2, x3 = (((pb >> 32) & M32) ^ x1) ^ k0, pb & M32, (((pa >> 32) & M32) ^ x3) ^ k1, pa & M32
    return x0, x1, x2, x3


def _normals(j0, j1, D, mat, t, key):
    """Rows j0..j1 of the random vectors of step t: standard normals by
    Box-Muller, rounded to fp32."""
    c = torch.arange((D + 3) // 4, device="cuda", dtype=torch.int64)[None, :]
    j = torch.arange(j0, j1, device="cuda", dtype=torch.int64)[:, None]
    x = _philox(c, j, mat, t, key)
    u = [(a >> 9).double() * 2.0 ** -23 + 2.0 ** -24 for a in x]
    out = []
    for a, b in ((u[0], u[1]), (u[2], u[3])):
        rho = torch.sqrt(-2.0 * torch.log(a))
        out += [rho * torch.cos(2.0 * math.pi * b), rho * torch.sin(2.0 * math.pi * b)]
    return torch.stack(out, dim=2).reshape(j1 - j0, -1)[:, :D].float().double()


def _scores(case, U, Mo, mat, t, key):
    d, D = Mo.shape
    if case["select"] == "approx_bf16":
        U, Mo = U.bfloat16().double(), Mo.float().bfloat16().double()
    out = torch.empty(d, device="cuda", dtype=torch.float64)
    step = max(1, 4_000_000 // D)
    for j0 in range(0, d, step):
        j1 = min(d, j0 + step)
        C = U[j0:j1] @ Mo
        if case["select"] == "exact":
            out[j0:j1] = C.square().sum(1)
        else:
            out[j0:j1] = (C * _normals(j0, j1, D, mat, t, key)).sum(1).square()
    return out


def _leading(Mo, r):
    """The leading r left singular vectors (columns) of Mo, by subspace
    iteration on a doubled block."""
    d = Mo.shape[0]
    A = Mo @ Mo.T
    K = min(d, 2 * r + 32)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    Q = torch.linalg.qr(torch.randn(d, K, generator=gen, device="cuda", dtype=torch.float64))[0]
    for _ in range(60):
        Q = torch.linalg.qr(A @ Q)[0]
    w, V = torch.linalg.eigh((Q.T @ (A @ Q)).cpu())
    return Q @ V.to(Q.device).flip(1)[:, :r]


def exact(case, seed):
    shapes = _shapes(case)
    if max(min(s) for s in shapes) > 4096:
        return None
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    t, key = _first_step(case), 1234 + seed % 1000
    outs, weights = [], []
    for l, shape in enumerate(shapes):
        a = _matrix(case, shape, gen, 1 if case["step"] == "select" else 2)
        out = _exact_one(case, shape, a, l, t, key)
        del a
        X = out.pop("X").reshape(-1)
        weights.append(torch.nn.functional.pad(X, (0, (-X.numel()) % 64)))
        if _many(case):
            out = torch.cat([out["E"].reshape(-1), out["Ebar"].reshape(-1)])
        outs.append(out)
    return [torch.cat(weights)] + outs


def _exact_one(case, shape, a, mat, t, key):
    m, n = shape
    d, D = min(m, n), max(m, n)
    N, r, right = case["workers"], min(case["rank"], d), m > n
    G, E = a["G"][0], a["E"]

    def orient(x):
        return x.T if right else x

    Mbar = a["Ebar"].double()
    for i in range(N):
        Mbar = Mbar + G[i].double() / N
    Mo = orient(Mbar)
    out = {}
    if case["step"] == "select":
        U = a["U"].double()
        out["score"] = _scores(case, U, Mo, mat, t, key)
        J = torch.sort(torch.topk(out["score"], r).indices).values
        P = U[J].T.contiguous()
    else:
        P = _leading(Mo, r)
        if case["step"] == "refresh":
            out["sigma"] = None
            if d <= 1536:
                out["sigma"] = torch.linalg.eigvalsh((Mo @ Mo.T).cpu()).flip(0).clamp(min=0).sqrt()
    Enew = torch.empty_like(E)                       # in the storage type: what a buffer can hold
    if E.dtype == torch.float32:
        Enew = Enew.double()
    Ebar = torch.zeros(m, n, device="cuda", dtype=torch.float64)
    Rbar = torch.zeros(r, D, device="cuda", dtype=torch.float64)
    for i in range(N):
        M = orient(G[i].double() + E[i].double())
        Q = P.T @ M
        Enew[i] = orient(M - P @ Q)
        Ebar += Enew[i].double() / N
        Rbar += Q / N
    gh = orient(P @ Rbar)
    b1, b2 = float(np.float32(BETA1)), float(np.float32(BETA2))
    lr, eps = float(np.float32(LR)), float(np.float32(EPS))
    S1 = b1 * a["S1"].double() + (1.0 - b1) * gh
    if case["opt"] == "adam":
        S2 = b2 * a["S2"].double() + (1.0 - b2) * gh * gh
        out["S2"] = S2
        out["X"] = -lr * S1 / (S2.sqrt() + eps)
    else:
        out["X"] = -lr * S1
    out.update(E=Enew, Ebar=Ebar, S1=S1)
    if case["step"] == "select":
        out["Rbar"] = Rbar
    return out
