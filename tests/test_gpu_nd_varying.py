"""Factors per operand at small sizes, where a workgroup takes many operands
with their own factors: results against the oracle, at batches that end inside
a tile, and a bound on the time of a large batch."""
import numpy as np
import pytest
import torch

import oracle
import paper_1304_7054_amd as kron

pytestmark = pytest.mark.gpu

DT = {"f32": torch.float32, "f64": torch.float64, "c32": torch.complex64, "c64": torch.complex128}
NP = {"f32": np.float32, "f64": np.float64, "c32": np.complex64, "c64": np.complex128}
TOL = {"f32": 1e-5, "c32": 1e-5, "f64": 1e-13, "c64": 1e-13}
# (m, n): one column, odd extents, several row blocks, blocks of 32 columns and
# one more, an operand near a workgroup's LDS, slices of operands (20^3: the last)
SHAPES = [([2, 2], [2, 2]), ([1, 1, 9], [1, 1, 9]), ([5, 7], [7, 5]), ([17, 3], [3, 18]), ([2, 33], [33, 2]),
          ([4, 4, 4], [4, 4, 4]), ([3, 5, 2], [2, 4, 3]), ([2] * 6, [2] * 6), ([16, 16], [16, 16]), ([40, 40], [40, 40]),
          ([20, 20, 20], [20, 20, 20])]


def _draw(rng, tag, size):
    v = rng.standard_normal(size)
    return (v + 1j * rng.standard_normal(size)).astype(NP[tag]) if tag[0] == "c" else v.astype(NP[tag])


@pytest.mark.parametrize("shape", range(len(SHAPES)))
@pytest.mark.parametrize("tag", list(DT))
def test_varying_factors(tag, shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m, n = SHAPES[shape]
    d, nx, ny = len(m), int(np.prod(n)), int(np.prod(m))
    rng = np.random.default_rng(70 + shape)
    ops = "".join(rng.choice(list("NTC"), d))
    # enough operands that every workgroup has a full tile, and a ragged end
    for batch in (1, 2, 60001 if nx <= 16 and tag == "f32" else 5003 if nx <= 64 else 701 if nx <= 600 else 7):
        # the last factor is shared
        ldfp = [a * b if k < d - 1 else 0 for k, (a, b) in enumerate(zip(m, n))]
        fac = [_draw(rng, tag, (batch if p else 1) * a * b) for a, b, p in zip(m, n, ldfp)]
        X, Y0 = _draw(rng, tag, batch * nx), _draw(rng, tag, batch * ny)
        alpha = 0.5 - 1.5j if tag[0] == "c" else -1.5
        for beta in (0.0, 0.75):
            ty = torch.from_numpy(Y0).cuda() if beta else torch.full((batch * ny,), float("nan"), dtype=DT[tag], device="cuda")
            getattr(kron, f"kron_nd_batched_{tag}")(m, n, ops, alpha, [torch.from_numpy(f).cuda() for f in fac],
                                                    torch.from_numpy(X).cuda(), beta, ty, batch, ldfp=ldfp)
            torch.cuda.synchronize()
            want = oracle.kron_nd(m, n, ops, alpha, fac, X, beta, Y0 if beta else np.zeros(batch * ny), batch, ldfp=ldfp)
            got = ty.cpu().numpy()
            assert np.all(np.isfinite(got)), (batch, ops)
            assert np.linalg.norm(got - want) <= TOL[tag] * np.linalg.norm(want), (batch, ops, beta)


# batches that give every workgroup tiles of several operands, or of several
# slices of one operand (20^3 and 24^3), and end inside a tile
FULL = [([2, 33], [33, 2], 3001), ([17, 17], [16, 16], 2077), ([16, 16], [16, 16], 3500), ([40, 3], [36, 5], 2600),
        ([20, 20, 20], [20, 20, 20], 131), ([24, 24, 24], [24, 24, 24], 90), ([3, 20, 20], [2, 24, 20], 700)]


@pytest.mark.parametrize("shape", range(len(FULL)))
@pytest.mark.parametrize("tag", list(DT))
def test_varying_factors_in_full_tiles(tag, shape):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m, n, batch = FULL[shape]
    d, nx, ny = len(m), int(np.prod(n)), int(np.prod(m))
    rng = np.random.default_rng(90 + shape)
    ops = "".join(rng.choice(list("NTC"), d))
    ldfp = [a * b + 3 * k for k, (a, b) in enumerate(zip(m, n))]
    fac = [_draw(rng, tag, batch * p) for p in ldfp]
    X = _draw(rng, tag, batch * nx)
    ty = torch.full((batch * ny,), float("nan"), dtype=DT[tag], device="cuda")
    getattr(kron, f"kron_nd_batched_{tag}")(m, n, ops, 1.0, [torch.from_numpy(f).cuda() for f in fac],
                                            torch.from_numpy(X).cuda(), 0.0, ty, batch, ldfp=ldfp)
    torch.cuda.synchronize()
    want = oracle.kron_nd(m, n, ops, 1.0, fac, X, 0.0, np.zeros(batch * ny), batch, ldfp=ldfp)
    got = ty.cpu().numpy()
    assert np.all(np.isfinite(got)), ops
    assert np.linalg.norm(got - want) <= TOL[tag] * np.linalg.norm(want), ops


def test_many_small_operands_share_workgroups():
    """700,000 2 x 2 operands take less time than three 1 GiB copies; with a
    workgroup each they took six."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    batch = 700000
    rand = lambda k: torch.randn(k, device="cuda")
    fac, X, Y = [rand(4 * batch), rand(4 * batch)], rand(4 * batch), torch.empty(4 * batch, device="cuda")
    ws = torch.empty(kron.kron_nd_workspace_size([2, 2], [2, 2], batch, kron.MODE_F32), dtype=torch.uint8, device="cuda")
    a, b = (torch.empty(1 << 30, dtype=torch.uint8, device="cuda") for _ in range(2))

    def best(fn):
        times = []
        for _ in range(6):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            fn()
            end.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(end))
        return min(times)

    copy = best(lambda: kron.kron_copy_bytes(a, b))
    call = best(lambda: kron.kron_nd_batched_f32([2, 2], [2, 2], "NN", 1.0, fac, X, 0.0, Y, batch, ldfp=[4, 4], ws=ws))
    assert call < 3 * copy, (call, copy)
