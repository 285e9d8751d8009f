"""Products on the 16-bit matrix cores from split fp32 operands, at the edges
of their tiles and of the operands' range, against fp64."""
import numpy as np
import pytest
import torch

from oracle.philox import gaussian_vectors

pytestmark = pytest.mark.gpu


def _orthonormal(d, rng):
    return np.linalg.qr(rng.standard_normal((d, d)))[0]


# d and D around the 128-wide tiles, the 32-deep slices and the 256-deep
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


# ranks around the 16-deep steps and their powers of two (one to sixteen steps,
# and the fp32 pass above rank 256); ragged tiles on both sides; columns of
# very different size, whose residuals are held to their own column's size
@pytest.mark.parametrize("rank", [1, 15, 16, 17, 33, 64, 65, 128, 130, 256, 257])
@pytest.mark.parametrize("shape", [(299, 330), (330, 299)])
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
