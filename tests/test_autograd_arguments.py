"""What the autograd front end refuses, and the factor layouts it takes."""
import pytest
import torch

import paper_1304_7054_amd as kron
from paper_1304_7054_amd import autograd


@pytest.mark.parametrize("n", [0, 17])
@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("device", ["cpu", pytest.param("cuda", marks=pytest.mark.gpu)])
@pytest.mark.parametrize("dtype,mode", [(torch.float32, "f32"), (torch.float32, "bf16x3"), (torch.float64, "f64")])
def test_extent_out_of_range_is_a_value_error(dtype, mode, device, dim, n):
    if device == "cuda" and not torch.cuda.is_available():
        pytest.skip("no GPU")
    X = torch.zeros([2] + [n] * dim, dtype=dtype, device=device)
    mats = [torch.zeros(n, n, dtype=dtype, device=device) for _ in range(dim)]
    with pytest.raises(ValueError, match="n must be in 1..16"):
        (autograd.kron2d if dim == 2 else autograd.kron3d)(X, *mats, mode=mode)


def _layouts(M):
    """M's values in the layouts a factor may come in."""
    n = M.shape[0]
    wide = torch.zeros(2 * n, 2 * n, dtype=M.dtype, device=M.device)
    wide[::2, ::2] = M
    return {"rows": M.clone(), "columns": M.t().contiguous().t(), "strided": wide[::2, ::2],
            "negated": torch.complex(torch.zeros_like(M), -M).conj().imag}


@pytest.mark.gpu
@pytest.mark.parametrize("kinds", [("columns", "rows", "columns"), ("rows", "columns", "strided"),
                                   ("negated", "strided", "columns")])
@pytest.mark.parametrize("dim,n", [(2, 5), (2, 16), (3, 4), (3, 11)])
@pytest.mark.parametrize("dtype,tol", [(torch.float32, 1e-5), (torch.float64, 1e-13)])
def test_factor_layouts(dtype, tol, dim, n, kinds):
    """Row-major, column-major, strided and lazily negated factors, mixed:
    results and gradients against products in FP64."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda").manual_seed(31)
    X, dY = (torch.randn(23, *[n] * dim, generator=g, device="cuda", dtype=dtype) for _ in range(2))
    plain = [torch.randn(n, n, generator=g, device="cuda", dtype=dtype) for _ in range(dim)]
    mats = [_layouts(M)[k] for M, k in zip(plain, kinds)]
    leaves = [X.clone().requires_grad_()] + [M.detach().requires_grad_() for M in mats]
    Y = (autograd.kron2d if dim == 2 else autograd.kron3d)(*leaves)
    got = [Y.detach(), *torch.autograd.grad(Y, leaves, dY)]
    wide = [X.double().requires_grad_()] + [M.double().requires_grad_() for M in plain]
    out = wide[0]
    for axis, M in enumerate(wide[1:]):
        out = torch.movedim(torch.movedim(out, 1 + axis, -1) @ M.t(), -1, 1 + axis)
    want = [out.detach(), *torch.autograd.grad(out, wide, dY.double())]
    for name, a, b in zip(("Y", "dX", "dA", "dB", "dC"), got, want):
        assert float((a.double() - b).norm() / b.norm()) <= tol, name
