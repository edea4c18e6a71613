"""n = 16 with rows that 16-byte vectors can take: the strided entry points
equal the extended ones on packed storage to the last bit, with and without
beta, because both contract the axes in the same order."""
import pytest
import torch

import paper_1304_7054_amd as kron

pytestmark = pytest.mark.gpu
DT = {"f32": torch.float32, "f64": torch.float64}


@pytest.mark.parametrize("beta", [0.0, 2.0])
@pytest.mark.parametrize("pad", [0, 4])
@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("mode", list(DT))
def test_strided_equals_ex(mode, dim, pad, beta):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, batch = 16, 37
    g = torch.Generator(device="cuda").manual_seed(21)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda", dtype=DT[mode])
    mats, X, Y0 = [rand(n * n) for _ in range(dim)], rand(batch, *[n] * dim), rand(batch, *[n] * dim)
    ops = "TNN" if dim == 2 else "TNT"
    Y = Y0.clone()
    getattr(kron, f"kron{dim}d_batched_ex_{mode}")(n, *ops, 0.5, *mats, X.view(-1), beta, Y.view(-1), batch)
    ld = [(n + pad) * n ** k for k in range(dim)]
    view = lambda buf: buf.as_strided(X.shape, ld[::-1] + [1])
    Xs, Ys = (torch.zeros(batch * ld[-1], dtype=DT[mode], device="cuda") for _ in range(2))
    view(Xs).copy_(X)
    view(Ys).copy_(Y0)
    getattr(kron, f"kron{dim}d_batched_strided_{mode}")(n, *ops, 0.5, *[v for m in mats for v in (m, n)], Xs, *ld, beta,
                                                        Ys, *ld, batch)
    torch.cuda.synchronize()
    assert torch.equal(view(Ys), Y)
