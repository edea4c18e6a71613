"""GPU parity of the general action where its products run fused, or on the
plain kernels, against the oracle: extents at the edges of the 16-row and
4-step tiles, rectangular products (two LDS images) and square ones (in
place), factors per operand, strided and packed storage, slices of operands
that are too large, and a batch that ends inside a tile."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

DT = {"f32": torch.float32, "f64": torch.float64, "c32": torch.complex64, "c64": torch.complex128}
TOL = {"f32": 1e-5, "c32": 1e-5, "f64": 1e-13, "c64": 1e-13}
# (m, n): in place, two images, one column, n beyond 32 and 64, more products than images hold (slices)
SHAPES = [([16, 16], [16, 16]), ([17, 4], [4, 17]), ([1, 33], [33, 1]), ([40, 3], [36, 65]), ([5, 16, 9], [7, 16, 4]),
          ([16, 16, 16], [16, 16, 16]), ([12, 12, 12], [12, 12, 12]), ([20, 24, 24], [20, 24, 24]), ([3] * 5, [2] * 5),
          ([16] * 4, [16] * 4)]


@pytest.mark.parametrize("varying", [False, True])
@pytest.mark.parametrize("shape", range(len(SHAPES)))
@pytest.mark.parametrize("tag", list(DT))
def test_nd_fused(tag, shape, varying):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1304_7054_amd as kron
    m, n = SHAPES[shape]
    d, nx, ny = len(m), int(np.prod(n)), int(np.prod(m))
    cplx = tag[0] == "c"
    rng = np.random.default_rng(50 + shape)
    ops = "".join(rng.choice(list("NTC"), d))
    npdt = {"f32": np.float32, "f64": np.float64, "c32": np.complex64, "c64": np.complex128}[tag]

    def draw(size):
        v = rng.standard_normal(size)
        return (v + 1j * rng.standard_normal(size)).astype(npdt) if cplx else v.astype(npdt)

    for batch in (1, 3 if nx > 5000 else 301):
        count = batch if varying else 1
        fac = [draw(count * a * b) for a, b in zip(m, n)]
        ldfp = [a * b if varying else 0 for a, b in zip(m, n)]
        X, Y0 = draw(batch * nx), draw(batch * ny)
        for alpha, beta in ((1.0, 0.0), (0.5 - 1.5j if cplx else -1.5, 0.75)):
            ty = torch.from_numpy(Y0).cuda() if beta else torch.full((batch * ny,), float("nan"), dtype=DT[tag], device="cuda")
            getattr(kron, f"kron_nd_batched_{tag}")(m, n, ops, alpha, [torch.from_numpy(f).cuda() for f in fac],
                                                    torch.from_numpy(X).cuda(), beta, ty, batch, ldfp=ldfp)
            torch.cuda.synchronize()
            want = oracle.kron_nd(m, n, ops, alpha, fac, X, beta, Y0 if beta else np.zeros(batch * ny), batch, ldfp=ldfp)
            got = ty.cpu().numpy()
            assert np.all(np.isfinite(got)), (batch, ops)
            assert np.linalg.norm(got - want) <= TOL[tag] * np.linalg.norm(want), (batch, ops, alpha, beta)


@pytest.mark.parametrize("tag", ["f32", "c64"])
@pytest.mark.parametrize("opX", ["N", "T", "C"])
def test_rect2_storage(tag, opX):
    """TKRON2 through the same kernels: padded and packed storage of X and Y,
    op on the operands; the elements between the addressed ones stay."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1304_7054_amd as kron
    cplx = tag[0] == "c"
    npdt = np.complex128 if cplx else np.float32
    rng = np.random.default_rng(9)
    for ma, na, mb, nb, pad, batch in ((6, 9, 11, 5, 3, 77), (16, 16, 16, 16, 0, 40), (8, 8, 8, 8, 1, 33)):
        rows, cols = (nb, na) if opX == "N" else (na, nb)
        ldx, ldy = rows + pad, mb + pad
        lxp, lyp = ldx * cols, ldy * ma

        def draw(size):
            v = rng.standard_normal(size)
            return (v + 1j * rng.standard_normal(size)).astype(npdt) if cplx else v.astype(npdt)

        A, B, X, Y0 = draw(ma * na), draw(mb * nb), draw(batch * lxp), draw(batch * lyp)
        ty = torch.from_numpy(Y0).cuda()
        getattr(kron, f"kron2d_batched_rect_{tag}")("N", "T", opX, ma, na, mb, nb, batch, 2.0, torch.from_numpy(A).cuda(),
                                                    ma, torch.from_numpy(B).cuda(), nb, torch.from_numpy(X).cuda(), ldx,
                                                    lxp, 0.0, ty, ldy, lyp)
        torch.cuda.synchronize()
        Xp = X.reshape(batch, cols, ldx)[:, :, :rows].transpose(0, 2, 1)  # stored matrices
        Xop = Xp if opX == "N" else Xp.transpose(0, 2, 1) if opX == "T" else Xp.conj().transpose(0, 2, 1)
        Ao, Bo = A.reshape(na, ma).T.astype(np.complex128), B.reshape(mb, nb).astype(np.complex128)
        want = 2.0 * Bo @ Xop.astype(np.complex128) @ Ao.T
        got = ty.cpu().numpy().reshape(batch, ma, ldy)
        assert np.array_equal(got[:, :, mb:], Y0.reshape(batch, ma, ldy)[:, :, mb:])
        g = got[:, :, :mb].transpose(0, 2, 1)
        assert np.linalg.norm(g - want) <= TOL[tag] * np.linalg.norm(want), (ma, pad)
