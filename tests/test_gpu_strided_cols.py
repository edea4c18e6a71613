"""The strided action on columns in LDS (operands close together) against the
general strided kernel (the same operands so far apart that a tile's offsets
leave 32 bits) and an FP64 contraction: every n, both types, both dimensions,
op on 2-D operands, beta, odd strides, rows for 16-byte vectors, the strides
of a transposed array, one operand, ragged tiles and results long enough to
bypass the cache.  Tolerances are those of the strided tests."""
import pytest
import torch

import paper_1304_7054_amd as kron

pytestmark = pytest.mark.gpu
DT = {"f32": torch.float32, "f64": torch.float64}
TOL = {"f32": 1e-5, "f64": 1e-13}


def _view(buf, strides, batch, n, dim):
    """(operand, slow .., fast) view of a strided buffer."""
    return buf.as_strided([batch] + [n] * dim, list(strides[::-1]) + [1])


def _strided(x, strides):
    """A buffer holding x (batch, n, ..) at the strides; gaps are 5."""
    batch, n, dim = x.shape[0], x.shape[1], x.dim() - 1
    last = (batch - 1) * strides[-1] + (n - 1) * (1 + sum(strides[:-1])) + 1
    buf = torch.empty(last, dtype=x.dtype, device="cuda")
    if last < 1 << 24:
        buf.fill_(5.0)
    _view(buf, strides, batch, n, dim).copy_(x)
    return buf


def _call(mode, n, ops, mats, X, xs, beta, Y0, ys, batch):
    dim = len(mats)
    Y = _strided(Y0, ys)
    args = [a for m in mats for a in (m, n)]
    getattr(kron, f"kron{dim}d_batched_strided_{mode}")(n, *ops, 0.75, *args, _strided(X, xs), *xs, beta, Y, *ys, batch)
    torch.cuda.synchronize()
    if Y.numel() < 1 << 24:
        keep = torch.ones_like(Y, dtype=torch.bool)
        _view(keep, ys, batch, n, dim).fill_(False)
        assert bool((Y[keep] == 5.0).all()), "a gap was written"
    return _view(Y, ys, batch, n, dim).clone()


def _exact(ops, mats, X, beta, Y0, n):
    """alpha op(A) on the slowest axis, the last factor on the fastest."""
    out = X.double()
    dim = len(mats)
    if dim == 2 and ops[2] == "T":
        out = out.transpose(1, 2)
    for k, (m, op) in enumerate(zip(mats, ops)):
        M = m.double().view(n, n)                       # M[j, i]: column-major storage
        M = M if op == "T" else M.t()
        out = torch.movedim(torch.movedim(out, 1 + k, -1) @ M.t().contiguous(), -1, 1 + k)
    return 0.75 * out + beta * Y0.double()


@pytest.mark.parametrize("mode", ["f32", "f64"])
@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("n", range(1, 17))
def test_columns_against_the_general_kernel(mode, dim, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda").manual_seed(100 * n + dim)
    dt = DT[mode]
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda", dtype=dt)
    cases = [(1, 1, "NTN", 0.0), (2 * 256 // n + 3, 3, "TNT", -1.25), (2000 // n ** (dim - 1) + 5, 4 * (n % 4 == 0), "TTN", 0.0),
             (3, 2, "NNT", 0.5)]
    for k, (batch, pad, ops, beta) in enumerate(cases):
        mats = [rand(n * n) for _ in range(dim)]
        X, Y0 = rand(batch, *[n] * dim), rand(batch, *[n] * dim)
        xs = [(n + pad) * (n + k) ** d for d in range(dim)]
        ys = [(n + pad + 1) * (n + 1) ** d for d in range(dim)]
        if k == 2:  # X stored with its middle and slow (2-D: operand) strides the other way round
            xs = [n * batch, n] if dim == 2 else [n * n, n, n ** 3]
        got = _call(mode, n, ops, mats, X, xs, beta, Y0, ys, batch)
        want = _exact(ops, mats, X, beta, Y0, n)
        err = float((got.double() - want).norm() / want.norm())
        assert err <= TOL[mode], (k, "columns", err)
        few = min(batch, 2)
        far = ys[:-1] + [(1 << 29) // (256 if n == 1 else 1 if n > 11 else 2)]
        if n in (1, 7, 12, 15, 16) and k in (0, 3):
            got = _call(mode, n, ops, mats, X[:few], xs, beta, Y0[:few], far, few)
            err = float((got.double() - want[:few]).norm() / want[:few].norm())
            assert err <= TOL[mode], (k, "general", err)


@pytest.mark.parametrize("mode,dim,n", [("f32", 3, 10), ("f64", 2, 5), ("f32", 2, 16), ("f64", 3, 16)])
def test_results_longer_than_the_cache(mode, dim, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda").manual_seed(3)
    dt = DT[mode]
    ld = [(n + 1) * n ** d for d in range(dim)]
    batch = (180 << 20) // (ld[-1] * torch.empty(0, dtype=dt).element_size())
    mats = [torch.randn(n * n, generator=g, device="cuda", dtype=dt) for _ in range(dim)]
    X = torch.randn(batch, *[n] * dim, generator=g, device="cuda", dtype=dt)
    for beta in (0.0, 2.0):
        got = _call(mode, n, "TNN", mats, X, ld, beta, X, ld, batch)
        want = _exact("TNN", mats, X, beta, X, n)
        assert float((got.double() - want).norm() / want.norm()) <= TOL[mode]
