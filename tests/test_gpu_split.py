"""Products on the 16-bit matrix cores from split fp32 operands, at the edges
of their tiles and of the operands' range, against fp64."""
import ctypes

import numpy as np
import pytest
import torch

from oracle.philox import gaussian_vectors
from synth import get_workload, gradient_batch, planted_matrix

pytestmark = pytest.mark.gpu


def _orthonormal(d, rng):
    return np.linalg.qr(rng.standard_normal((d, d)))[0]


# d and D around the 64-wide tiles, the 32-deep slices and the 256-deep
# flush; rows of 1 to 3 elements past a quad; operands far from 1, with
# columns of very different size, and zero
@pytest.mark.parametrize("shape", [(1, 37), (2, 3), (31, 33), (33, 130), (127, 129), (128, 128), (257, 300), (300, 257),
                                   (130, 33), (290, 1023)])
@pytest.mark.parametrize("select", ["exact", "approx"])
@pytest.mark.parametrize("scale", [1.0, 1e-15, 1e15, 0.0])
def test_scores_against_fp64(gpu_lib, shape, select, scale):
    m, n = shape
    d, D = min(shape), max(shape)
    rng = np.random.default_rng([m, n])
    U = _orthonormal(d, rng).astype(np.float32)              # row j: u_j
    M = rng.standard_normal((d, D)) * 10.0 ** rng.uniform(-3, 0, D)
    G = ((M.T if m > n else M) * scale).astype(np.float32)
    comp = gpu_lib.GreedyLore([shape], 1, max(1, d // 2), 1000, select=select, seed=11)
    comp.write_state(0, Ut=torch.from_numpy(U).cuda())
    comp.resume(1)
    comp.step([torch.zeros(m, n, device="cuda")], [torch.from_numpy(G)[None].cuda().contiguous()], 1)
    got = comp.score(0).double().cpu().numpy()
    comp.check_status()
    if d == 1:
        return                                               # every direction kept: no scores
    Mo = G.astype(np.float64)
    Mo = Mo.T if m > n else Mo
    C = U.astype(np.float64) @ Mo
    fro = np.linalg.norm(Mo)
    # a split product is within 2^-21 of |a b|, so a row of C within 2^-21 |u|
    # |M|_F of its own; the fold over D sums in fp32 (1e-5 of its terms' norm)
    if select == "exact":
        ref = (C ** 2).sum(1)
        bound = 2 * 2.0 ** -21 * np.sqrt(ref) * fro + (2.0 ** -21 * fro) ** 2 + 1e-5 * ref
    else:
        v = gaussian_vectors(11, 1, 0, range(d), D).astype(np.float64)
        ref = np.abs((C * v).sum(1))
        bound = (2.0 ** -21 * fro + 1e-5 * np.linalg.norm(C, axis=1)) * np.linalg.norm(v, axis=1)
        got = np.sqrt(got)
    assert np.all(np.abs(got - ref) <= bound)


# at least 256 tiles of 128 x 128, which then run (fewer: 64 x 64 ones): d past
# a tile, D a few columns and more than half a tile past one, odd rows; against
# fp64 of the operands as the mode rounds them
@pytest.mark.parametrize("shape", [(1930, 1953), (1953, 1930), (1931, 2040), (2040, 1930)])
@pytest.mark.parametrize("select", ["exact", "approx", "approx_bf16"])
def test_scores_in_large_tiles(gpu_lib, shape, select):
    m, n = shape
    d, D = min(shape), max(shape)
    gen = torch.Generator(device="cuda").manual_seed(d + n)
    U = torch.linalg.qr(torch.randn(d, d, generator=gen, device="cuda", dtype=torch.float64))[0].float().contiguous()
    G = torch.randn(1, m, n, generator=gen, device="cuda") * torch.logspace(0, -2, n, device="cuda")
    comp = gpu_lib.GreedyLore([shape], 1, 4, 1000, select=select, seed=11)
    comp.write_state(0, Ut=U)
    comp.resume(1)
    comp.step([torch.zeros(m, n, device="cuda")], [G], 1)
    comp.check_status()
    got = comp.score(0).double()
    Mo = G[0].T if m > n else G[0]
    if select == "approx_bf16":
        U, Mo = U.bfloat16(), Mo.bfloat16()
    C = U.double() @ Mo.double()
    fro = float(Mo.double().norm())
    # as for the small tiles (exact products of bf16 operands in the bf16 mode,
    # their fp32 sums of up to 2000 terms within 1e-5 of the terms' norm)
    if select == "exact":
        ref = C.square().sum(1)
        bound = 2 * 2.0 ** -21 * ref.sqrt() * fro + (2.0 ** -21 * fro) ** 2 + 1e-5 * ref
    else:
        v = torch.from_numpy(np.asarray(gaussian_vectors(11, 1, 0, range(d), D), dtype=np.float64)).cuda()
        ref = (C * v).sum(1).abs()
        bound = (2.0 ** -21 * fro + 1e-5 * C.norm(dim=1)) * v.norm(dim=1)
        got = got.sqrt()
    assert bool(((got - ref).abs() <= bound).all())


# a group of at least 256 large tiles whose matrices have fewer each: the bits of
# the small tiles that they take alone
@pytest.mark.parametrize("select", ["exact", "approx", "approx_bf16"])
@pytest.mark.parametrize("right", [False, True])
def test_grouped_scores_across_the_tile_sizes(gpu_lib, monkeypatch, select, right):
    shapes = [(768, 768)] * 4 + [(700, 790), (640, 1100), (513, 911), (129, 3000)]
    assert sum(-(-a // 128) * -(-b // 128) for a, b in shapes) >= 256
    if right:
        shapes = [(b, a) for a, b in shapes if b > a] * 3
    gen = torch.Generator(device="cuda").manual_seed(int(right))
    G = [torch.randn(1, m, n, generator=gen, device="cuda") for m, n in shapes]
    U = [torch.linalg.qr(torch.randn(min(s), min(s), generator=gen, device="cuda"))[0].contiguous() for s in shapes]
    runs = []
    for grouped in ("0", None):
        if grouped is None:
            monkeypatch.delenv("GLR_GROUPED", raising=False)
        else:
            monkeypatch.setenv("GLR_GROUPED", grouped)
        comp = gpu_lib.GreedyLore(shapes, 1, 12, 1000, select=select)
        for l, u in enumerate(U):
            comp.write_state(l, Ut=u)
        comp.resume(1)
        comp.step([torch.zeros(m, n, device="cuda") for m, n in shapes], G, 1)
        comp.check_status()
        runs.append(comp)
    for l in range(len(shapes)):
        assert torch.equal(runs[0].score(l), runs[1].score(l)) and torch.equal(runs[0].J(l), runs[1].J(l))
        assert torch.equal(runs[0].E(l), runs[1].E(l))


# hundreds of partials a column: their fold adds no error of its own.  A
# partial of 64 rows is within about 2^-23 of its squares' sum, of either sign,
# so 313 and 1094 of them leave 7e-9; the rounding of the stored score is 2.5e-8
# rms.  (Folded in fp32: 2e-7.)
@pytest.mark.parametrize("d,D", [(256, 20000), (40, 70003)])
def test_score_fold_over_many_partials(gpu_lib, d, D):
    rng = np.random.default_rng(D)
    U = torch.from_numpy(_orthonormal(d, rng).astype(np.float32)).cuda()
    G = torch.from_numpy(rng.standard_normal((1, d, D)).astype(np.float32)).cuda()
    comp = gpu_lib.GreedyLore([(d, D)], 1, 2, 1000, select="exact")
    comp.write_state(0, Ut=U)
    comp.resume(1)
    comp.step([torch.zeros(d, D, device="cuda")], [G], 1)
    comp.check_status()
    ref = (U.double() @ G[0].double()).square().sum(1)
    assert float((comp.score(0).double() - ref).norm() / ref.norm()) < 4e-8


# ranks around the 16-deep steps and their powers of two (one to sixteen steps,
# and the fp32 pass above rank 256); ragged tiles on both sides; columns of
# very different size, whose residuals are held to their own column's size
@pytest.mark.parametrize("rank", [1, 15, 16, 17, 33, 64, 65, 128, 130, 256, 257])
@pytest.mark.parametrize("shape", [(299, 330), (330, 299), (297, 331)])
@pytest.mark.parametrize("workers,store", [(1, "fp32"), (3, "fp32"), (5, "bf16")])
def test_residual_against_fp64(gpu_lib, rank, shape, workers, store):
    m, n = shape
    d, D = min(shape), max(shape)
    rng = np.random.default_rng([m, rank, workers])
    U = _orthonormal(d, rng).astype(np.float32)
    M = rng.standard_normal((workers, d, D)) * 10.0 ** rng.uniform(-12, 3, D)
    dt = torch.bfloat16 if store == "bf16" else torch.float32
    G = torch.from_numpy((M.transpose(0, 2, 1) if m > n else M).astype(np.float32)).to(dt)
    comp = gpu_lib.GreedyLore([shape], workers, rank, 1000, opt="msgd", lr=1.0, beta1=0.0, select="exact", store=store)
    comp.write_state(0, Ut=torch.from_numpy(U).cuda())
    comp.resume(1)
    X = torch.zeros(m, n, device="cuda")
    comp.step([X], [G.cuda().contiguous()], 1)
    comp.check_status()

    def oriented(x):
        x = x.double().cpu().numpy()
        return np.swapaxes(x, -1, -2) if m > n else x

    P = U[comp.J(0).cpu().numpy()].astype(np.float64).T
    Mo = oriented(G)
    C = P @ (P.T @ Mo)
    col = np.linalg.norm(Mo, axis=1, keepdims=True)          # of each worker's columns
    # fp32 sums over d of products within 2^-21: 4e-6 of the column, and the
    # rounding of the stored residual
    E = oriented(comp.E(0))
    assert np.all(np.abs(E - (Mo - C)) <= 4e-6 * col + (2.0 ** -8 if store == "bf16" else 2.0 ** -22) * np.abs(Mo - C))
    assert np.all(np.abs(-oriented(X) - C.mean(0)) <= 4e-6 * col.max(0))
    assert np.all(np.abs(oriented(comp.Ebar(0)) - E.mean(0)) <= 1e-6 * np.abs(E).max(0) + 1e-37)


# a second, ragged slice of the projection above rank 64 (slices of 1024 terms of
# d), with odd rows
@pytest.mark.parametrize("rank", [65, 130])
@pytest.mark.parametrize("shape", [(1031, 1100), (1101, 1031), (1033, 1061)])
@pytest.mark.parametrize("store", ["fp32", "bf16"])
def test_residual_of_two_projection_slices(gpu_lib, rank, shape, store):
    m, n = shape
    d, N = min(shape), 2
    gen = torch.Generator(device="cuda").manual_seed(rank + n)
    U = torch.linalg.qr(torch.randn(d, d, generator=gen, device="cuda", dtype=torch.float64))[0].float().contiguous()
    G = torch.randn(N, m, n, generator=gen, device="cuda").to(torch.bfloat16 if store == "bf16" else torch.float32)
    comp = gpu_lib.GreedyLore([shape], N, rank, 1000, opt="msgd", lr=1.0, beta1=0.0, select="exact", store=store)
    comp.write_state(0, Ut=U)
    comp.resume(1)
    X = torch.zeros(m, n, device="cuda")
    comp.step([X], [G], 1)
    comp.check_status()
    o = (lambda x: x.double().transpose(-1, -2)) if m > n else (lambda x: x.double())
    P, Mo = U.double()[comp.J(0).long()].T, o(G)
    C = P @ (P.T @ Mo)
    col = Mo.norm(dim=1, keepdim=True)
    rounding = (2.0 ** -8 if store == "bf16" else 2.0 ** -22) * (Mo - C).abs()
    assert bool(((o(comp.E(0)) - (Mo - C)).abs() <= 4e-6 * col + rounding).all())
    assert bool(((-o(X) - C.mean(0)).abs() <= 4e-6 * col.amax(0)).all())
    assert bool(((o(comp.Rbar(0)) if m <= n else comp.Rbar(0).double()) - (P.T @ Mo).mean(0)).abs().max() <= 4e-6 * col.max())


# rows of P (and of M) from 1 down to 1e-9 of the largest: the reconstruction of
# a row is held to that row's own size
@pytest.mark.parametrize("rank", [5, 17, 64, 128, 200])
@pytest.mark.parametrize("shape", [(299, 330), (330, 299)])
@pytest.mark.parametrize("store", ["fp32", "bf16"])
def test_reconstruction_of_small_rows(gpu_lib, rank, shape, store):
    m, n = shape
    d, D, N = min(shape), max(shape), 3
    rng = np.random.default_rng([m, rank])
    size = 10.0 ** rng.uniform(-9, 0, d)
    U = (_orthonormal(d, rng) * size).astype(np.float32)          # row j: u_j
    M = rng.standard_normal((N, d, D)) * size[:, None]
    dt = torch.bfloat16 if store == "bf16" else torch.float32
    G = torch.from_numpy((M.transpose(0, 2, 1) if m > n else M).astype(np.float32)).to(dt)
    comp = gpu_lib.GreedyLore([shape], N, rank, 1000, opt="msgd", lr=1.0, beta1=0.0, select="exact", store=store)
    comp.write_state(0, Ut=torch.from_numpy(U).cuda())
    comp.resume(1)
    X = torch.zeros(m, n, device="cuda")
    comp.step([X], [G.cuda().contiguous()], 1)
    comp.check_status()

    def oriented(x):
        x = x.double().cpu().numpy()
        return np.swapaxes(x, -1, -2) if m > n else x

    P = U[comp.J(0).cpu().numpy()].astype(np.float64).T
    Mo = oriented(G)
    C = P @ (P.T @ Mo)
    # Q within 4e-6 of |M_b| (|P| <= 1), each product of a row within 2^-21
    bound = 5e-6 * np.linalg.norm(P, axis=1)[:, None] * np.linalg.norm(Mo, axis=1, keepdims=True)
    assert np.all(np.abs(-oriented(X) - C.mean(0)) <= bound.max(0))
    if store == "fp32":
        assert np.all(np.abs(oriented(comp.E(0)) - (Mo - C)) <= bound + 2.0 ** -22 * np.abs(Mo - C))


# a basis far above 1 written into the state (a multiple of an orthonormal one:
# the scores and residuals scale with it, and the span that a tau = 1 refresh
# starts from is the same): no overflow, the same relative bounds
@pytest.mark.parametrize("scale", [1.0, 3000.0, 2.0 ** 20])
@pytest.mark.parametrize("shape", [(150, 333), (333, 150)])
@pytest.mark.parametrize("rank", [7, 40])
def test_basis_of_large_entries(gpu_lib, scale, shape, rank):
    m, n = shape
    d, D = min(shape), max(shape)
    rng = np.random.default_rng([m, rank])
    U = (_orthonormal(d, rng) * scale).astype(np.float32)
    M = rng.standard_normal((d, D))
    G = torch.from_numpy((M.T if m > n else M).astype(np.float32))[None].cuda().contiguous()
    Mo = G[0].double().cpu().numpy()
    Mo = Mo.T if m > n else Mo
    comp = gpu_lib.GreedyLore([shape], 1, rank, 1000, lr=1.0, beta1=0.0, select="exact")
    comp.write_state(0, Ut=torch.from_numpy(U).cuda())
    comp.resume(1)
    X = torch.zeros(m, n, device="cuda")
    comp.step([X], [G], 1)
    comp.check_status()
    ref = ((U.astype(np.float64) @ Mo) ** 2).sum(1)
    assert np.all(np.abs(comp.score(0).double().cpu().numpy() - ref) <= 1e-5 * ref)
    P = U[comp.J(0).cpu().numpy()].astype(np.float64).T
    C = P @ (P.T @ Mo)
    x = -X.double().cpu().numpy()
    bound = 5e-6 * scale * scale * np.linalg.norm(Mo, axis=0)
    assert np.all(np.abs((x.T if m > n else x) - C) <= bound)
    # tau = 1: the refreshed basis is that of the orthonormal start, and the
    # handle's later steps are
    low = (P[:, :rank] / scale) @ rng.standard_normal((rank, D)) * 30
    runs = []
    for s in (1.0, scale):
        comp = gpu_lib.GreedyLore([shape], 1, rank, 1, lr=1.0, beta1=0.0)
        comp.write_state(0, Ut=torch.from_numpy((U / scale * s).astype(np.float32)).cuda(),
                         sigma=torch.linspace(2.0, 1.0, d, device="cuda"))
        comp.resume(1)
        x = Mo + low
        g = torch.from_numpy((x.T if m > n else x).astype(np.float32))[None].cuda().contiguous()
        for t in (1, 2):
            comp.step([X], [g], t)
        assert comp.sync_status() in (0, 7)
        V = comp.Ut(0).double()[:rank]
        assert bool(torch.isfinite(V).all())
        assert float((V @ V.T - torch.eye(rank, device="cuda", dtype=torch.float64)).abs().max()) < 1e-5
        runs.append(V.T @ V)
    assert float((runs[0] - runs[1]).norm()) < 1e-3 * rank ** 0.5


# more row tiles than a grid's y extent holds (65535): the rows on both sides of
# that tile, against fp64
def test_residual_of_more_row_tiles_than_a_grid_extent(gpu_lib):
    m, n, r = 65535 * 64 + 129, 130, 129
    gen = torch.Generator(device="cuda").manual_seed(3)
    U = torch.from_numpy(_orthonormal(n, np.random.default_rng(3)).astype(np.float32)).cuda()
    G = torch.randn(1, m, n, generator=gen, device="cuda")
    comp = gpu_lib.GreedyLore([(m, n)], 1, r, 1000, lr=1.0, beta1=0.0, select="exact")
    comp.write_state(0, Ut=U)
    comp.resume(1)
    X = torch.zeros(m, n, device="cuda")
    comp.step([X], [G], 1)
    comp.check_status()
    P = U.double()[comp.J(0).long()]
    for a in (0, 65535 * 64 - 64, m - 193, m - 64):
        M = G[0, a:a + 64].double()
        C = (M @ P.T) @ P
        col = M.norm(dim=1, keepdim=True)
        assert bool(((comp.E(0)[0, a:a + 64].double() - (M - C)).abs() <= 4e-6 * col).all())
        assert bool(((X[a:a + 64].double() + C).abs() <= 4e-6 * col).all())


# fp32 Q^(i) below rank 257, where the packed operands would take too much (a
# configuration that fits the static scratch only so; long rows): against fp64,
# and a static handle against one with its own workspace
@pytest.mark.parametrize("shape,workers,rank,opt,select", [((588, 2356), 16, 181, "adam", "approx"),
                                                           ((2613, 467), 32, 128, "msgd", "exact"),
                                                           ((3, 900_001), 2, 2, "adam", "exact"),
                                                           ((900_001, 1), 2, 1, "msgd", "approx")])
def test_residual_without_packed_operands(gpu_lib, shape, workers, rank, opt, select):
    m, n = shape
    d, D = min(shape), max(shape)
    gen = torch.Generator(device="cuda").manual_seed(d)
    U = torch.from_numpy(_orthonormal(d, np.random.default_rng(d)).astype(np.float32)).cuda()
    G = torch.randn(workers, m, n, generator=gen, device="cuda")
    lib, runs = gpu_lib.load(), []
    cfg, _keep = gpu_lib.make_config([shape], workers, rank, 1000, opt=opt, lr=1.0, beta1=0.0, select=select, seed=3)
    sb, wb = gpu_lib.workspace_bytes(cfg)
    comp = gpu_lib.GreedyLore([shape], workers, rank, 1000, opt=opt, lr=1.0, beta1=0.0, select=select, seed=3)
    comp.write_state(0, Ut=U)
    comp.resume(1)
    X = torch.zeros(m, n, device="cuda")
    comp.step([X], [G], 1)
    comp.check_status()
    P = U.double()[comp.J(0).long()].T
    o = (lambda x: x.transpose(-1, -2)) if m > n else (lambda x: x)
    for w in range(workers):
        M = o(G[w].double())
        R = M - P @ (P.T @ M)
        assert bool(((o(comp.E(0)[w]).double() - R).abs() <= 4e-6 * M.norm(dim=0)).all())
    if wb > gpu_lib.STATIC_SCRATCH_BYTES:
        return
    state = torch.empty(sb + 256, dtype=torch.uint8, device="cuda")
    s0 = (-state.data_ptr()) % 256
    stream, h = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream), ctypes.c_void_p()
    assert lib.glr_create_static(ctypes.byref(cfg), ctypes.c_void_p(state.data_ptr() + s0), sb, stream,
                                 ctypes.byref(h)) == 0
    try:
        view = gpu_lib.StateView(Ut=ctypes.c_void_p(U.data_ptr()))
        assert lib.glr_write_state(h, 0, ctypes.byref(view), stream) == 0 and lib.glr_resume(h, 1) == 0
        X2 = torch.zeros(m, n, device="cuda")
        assert lib.glr_step(h, (ctypes.c_void_p * 1)(X2.data_ptr()), (ctypes.c_void_p * 1)(G.data_ptr()), 1, stream) == 0
        assert lib.glr_sync_status(h, stream) == 0
        assert torch.equal(X, X2)
    finally:
        assert lib.glr_destroy(h) == 0


# one and several keys a thread, the fold inside and outside the selecting
# workgroup, ties (equal scores go to the smaller index) and extremes
@pytest.mark.parametrize("d,D", [(2, 3), (127, 300), (1023, 1100), (1025, 1500), (2050, 2100), (1030, 9000)])
@pytest.mark.parametrize("rank", [1, 7, 400])
def test_top_r_order(gpu_lib, d, D, rank):
    if rank >= d:
        pytest.skip("every direction kept")
    rng = np.random.default_rng([d, rank])
    # U = I and one entry per row of M: the exact scores are these squares, with
    # ties (all above (2^-39 max |M|)^2, what one scale for the matrix resolves)
    vals = rng.choice([0.0, 1e-6, 0.5, 1.0, 2.0, 3.0], size=d).astype(np.float32)
    G = np.zeros((1, d, D), np.float32)
    G[0, np.arange(d), rng.integers(0, D, d)] = vals
    comp = gpu_lib.GreedyLore([(d, D)], 1, rank, 1000, select="exact")
    comp.resume(1)
    comp.step([torch.zeros(d, D, device="cuda")], [torch.from_numpy(G).cuda()], 1)
    comp.check_status()
    score = comp.score(0).cpu().numpy()
    assert np.allclose(score, vals.astype(np.float64) ** 2, rtol=1e-6, atol=1e-30)
    want = np.sort(np.argsort(-score, kind="stable")[:rank])
    assert np.array_equal(comp.J(0).cpu().numpy(), want)


# a set with both sides: one grouped part per side, bitwise the per-matrix launches
@pytest.mark.parametrize("rank,opt", [(5, "msgd"), (12, "adam"), (40, "adam")])
def test_grouped_selection_with_both_sides(gpu_lib, monkeypatch, rank, opt):
    shapes = [(90, 200), (200, 90), (64, 64), (333, 130), (70, 71)]
    rng = np.random.default_rng(rank)
    G = [[torch.from_numpy(rng.standard_normal((3, m, n)).astype(np.float32)).cuda() for m, n in shapes]
         for _ in range(3)]
    runs = []
    for grouped in ("0", None):
        if grouped is None:
            monkeypatch.delenv("GLR_GROUPED", raising=False)
        else:
            monkeypatch.setenv("GLR_GROUPED", grouped)
        comp = gpu_lib.GreedyLore(shapes, 3, rank, 1000, opt=opt)
        comp.resume(1)
        X = [torch.zeros(m, n, device="cuda") for m, n in shapes]
        for t in range(3):
            comp.step(X, G[t], t + 1)
        comp.check_status()
        runs.append((comp, X))
    (c1, x1), (c2, x2) = runs
    for l in range(len(shapes)):
        assert torch.equal(x1[l], x2[l]) and torch.equal(c1.E(l), c2.E(l)) and torch.equal(c1.J(l), c2.J(l))
        assert torch.equal(c1.score(l), c2.score(l)) and torch.equal(c1.Rbar(l), c2.Rbar(l))


# A refresh whose enqueued sweeps end before it converges is finished by the
# trailing launch with the bits of enqueued sweeps.  A diagonal batch takes one
# sweep, so the handle that has seen it enqueues two (four above d = 128) of the
# random batch's seven to nine, and the trailing launch the rest (odd and even
# counts); a new handle in the same state enqueues sixteen.
@pytest.mark.parametrize("shapes,tau", [([(40, 70)], 2), ([(128, 200)], 2), ([(190, 130)], 2), ([(330, 340)], 2),
                                        ([(97, 64), (64, 70), (150, 90)], 2), ([(140, 200), (60, 80)], 2),
                                        ([(300, 500)], 1), ([(500, 170)], 1)])
@pytest.mark.parametrize("opt", ["msgd", "adam"])
def test_trailing_sweeps_finish_a_refresh(gpu_lib, shapes, tau, opt):
    r = 20
    gen = torch.Generator(device="cuda").manual_seed(len(shapes))
    hard = [torch.randn(2, m, n, generator=gen, device="cuda") for m, n in shapes]
    runs, trailing = [], None
    for seen in (True, False):
        comp = gpu_lib.GreedyLore(shapes, 2, r, tau, opt=opt)
        X = [torch.zeros(m, n, device="cuda") for m, n in shapes]
        if seen:
            easy = []
            for m, n in shapes:
                g = torch.zeros(2, m, n, device="cuda")
                i = torch.arange(min(m, n), device="cuda")
                g[:, i, i] = torch.linspace(2.0, 1.0, min(m, n), device="cuda")
                easy.append(g)
            comp.resume(tau)                 # (a warm refresh from U = I)
            comp.step(X, easy, tau)
            torch.cuda.synchronize()
            assert all(comp.sweep_history(l)[:2] == (1, True) for l in range(len(shapes)))
        # the same state for both handles
        for l, (m, n) in enumerate(shapes):
            d = min(m, n)
            parts = {"E": torch.zeros(2, m, n, device="cuda"), "Ebar": torch.zeros(m, n, device="cuda"),
                     "Ut": torch.eye(d, device="cuda"), "sigma": torch.linspace(2.0, 1.0, d, device="cuda"),
                     "S1": torch.zeros(m, n, device="cuda")}
            if opt == "adam":
                parts["S2"] = torch.zeros(m, n, device="cuda")
            comp.write_state(l, **parts)
            torch.cuda.synchronize()
            X[l].zero_()
        comp.resume(2 * tau)
        torch.cuda.synchronize()
        comp.step(X, hard, 2 * tau)
        comp.sync_status()                   # (two tau = 1 iterations may not converge)
        runs.append((comp, X))
    (a, xa), (b, xb) = runs
    for l, (m, n) in enumerate(shapes):
        d = min(m, n)
        K = d if tau > 1 else min(d, r + 32)
        sweeps, conv, hist = a.sweep_history(l)
        assert conv and 2 + (2 if K > 128 else 0) < sweeps <= 16
        assert hist[1] > 1e-3                # far from diagonal where the trailing launch takes over
        assert a.sweep_history(l) == b.sweep_history(l)
        assert torch.equal(xa[l], xb[l]) and torch.equal(a.E(l), b.E(l)) and torch.equal(a.Ebar(l), b.Ebar(l))
        assert torch.equal(a.Ut(l)[:K], b.Ut(l)[:K]) and torch.equal(a.sigma(l)[:K], b.sigma(l)[:K])
        assert torch.equal(a.J(l), b.J(l)) and torch.equal(a.S1(l), b.S1(l))
        U = a.Ut(l).double()[:K]
        assert float((U @ U.T - torch.eye(K, device="cuda", dtype=torch.float64)).abs().max()) < 1e-5


# a captured selection step of a set (of one side and of both) replays on the
# buffers it was captured with, whatever steps ran since, and those steps are
# none the worse for the capture
@pytest.mark.parametrize("shapes", [[(90, 200), (200, 90), (64, 64)], [(90, 200), (64, 130)]])
def test_captured_selection_step_of_a_set(gpu_lib, shapes):
    gen = torch.Generator(device="cuda").manual_seed(len(shapes))
    G = [[torch.randn(2, m, n, generator=gen, device="cuda") for m, n in shapes] for _ in range(4)]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        comp, ref = (gpu_lib.GreedyLore(shapes, 2, 8, 1000, select="exact") for _ in range(2))
        Xa, Xb, Ya, Yb = ([torch.zeros(m, n, device="cuda") for m, n in shapes] for _ in range(4))
        for c, x in ((comp, Xa), (ref, Ya)):
            c.resume(1)
            c.step(x, G[0], 1)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            comp.step(Xa, G[1], 2)
        t = 3
        for _ in range(4):
            graph.replay()
            torch.cuda.synchronize()
            ref.resume(t - 1)
            ref.step(Ya, G[1], t - 1)
            for k in (2, 3):                       # other buffers, both slots of the table
                comp.step(Xb, G[k], t)
                ref.step(Yb, G[k], t)
                t += 1
            torch.cuda.synchronize()
            for l in range(len(shapes)):
                assert torch.equal(Xa[l], Ya[l]) and torch.equal(Xb[l], Yb[l]) and torch.equal(comp.E(l), ref.E(l))


# the convergence measure does not depend on the order in which the groups of a
# launch run: the same refresh many times over, in shared launches and alone,
# to the last bit of its record
def test_refresh_records_repeat(gpu_lib, monkeypatch):
    wl = get_workload("mixed_small")
    planted = [planted_matrix(wl, l) for l in range(len(wl.shapes))]
    G = [torch.from_numpy(gradient_batch(wl, l, 0, planted[l])).cuda() for l in range(len(wl.shapes))]
    seen = set()
    for i in range(120):
        if i % 2:
            monkeypatch.setenv("GLR_JAC_JOINT", "0")
        else:
            monkeypatch.delenv("GLR_JAC_JOINT", raising=False)
        comp = gpu_lib.GreedyLore(wl.shapes, wl.workers, wl.rank, wl.tau, seed=wl.seed)
        comp.step([torch.zeros(m, n, device="cuda") for m, n in wl.shapes], G, 0)
        torch.cuda.synchronize()
        seen.add(tuple(tuple(comp.info(l).cpu().tolist()) for l in range(len(wl.shapes))))
    assert len(seen) == 1
