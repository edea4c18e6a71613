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
