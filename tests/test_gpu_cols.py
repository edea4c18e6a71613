"""GPU parity of the 3-D column kernels (the built-in default of their sizes)
against the CPU oracle where they can go wrong: a single operand, a ragged
last tile, several tiles per workgroup, and operand arrays that start off a
16-byte boundary (the shifted tile of odd n, the element-wise stores of even
n).  Tolerances are those of the forward tests."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import gpu_util as gu

# one n of every lane layout: vector width along the fast axis, padded planes
# and rows, scalar and matrix FP64 products
CASES = ([("f32", n) for n in (1, 3, 4, 6, 8, 12, 15)] + [("f64", n) for n in (1, 5, 8, 9, 11, 16)] +
         [("bf16", n) for n in (3, 6, 10)])


@pytest.mark.parametrize("mode,n", CASES)
def test_columns_at_tile_edges(mode, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1304_7054_amd as kron
    code = {"f32": kron.MODE_F32, "f64": kron.MODE_F64, "bf16": kron.MODE_BF16}[mode]
    kron.kron_set_launch(code, 3, n, -1, 0)
    # the last batch keeps every resident workgroup on its second tile or later
    for batch, xo, yo in ((1, 0, 0), (2, 1, 0), (517, 0, 1), (519, 3, 2), ((1 << 23) // n ** 3 + 3, 0, 0)):
        rng = np.random.default_rng(7 * n + batch)
        mats = [rng.uniform(-1, 1, n * n).astype(np.float32) for _ in range(3)]
        X = rng.standard_normal(batch * n ** 3).astype(np.float32)
        got = gu.run(mode, 3, n, mats, X, batch, x_offset=xo, y_offset=yo)
        exact = gu.rounded_inputs(mode, mats + [X])
        want = oracle.kron3d(n, *exact[:-1], exact[-1], batch, "f64")
        assert np.all(np.isfinite(got)), (batch, xo, yo)
        assert gu.errors(got, want, batch)[0] <= gu.TOL[mode], (batch, xo, yo)
