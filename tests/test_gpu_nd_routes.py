"""The general action on packed real cubes up to n = 16, whose products the
plain 2-D / 3-D kernels can take, against the oracle: scales that leave the
type's range when they meet a factor, but not when they meet the result; and
the launches of a call."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_1304_7054_amd as kron

pytestmark = pytest.mark.gpu

NP = {"f32": np.float32, "f64": np.float64}
TOL = {"f32": 1e-5, "f64": 1e-13}


def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _call(mode, d, n, ops, alpha, factors, X, beta, Y, batch):
    ty = torch.from_numpy(Y.copy()).cuda()
    getattr(kron, f"kron_nd_batched_{mode}")([n] * d, [n] * d, ops, alpha, [torch.from_numpy(f).cuda() for f in factors],
                                             torch.from_numpy(X).cuda(), beta, ty, batch)
    torch.cuda.synchronize()
    return ty.cpu().numpy()


@pytest.mark.parametrize("large", [False, True])
@pytest.mark.parametrize("d,n", [(2, 4), (2, 16), (3, 10), (3, 16)])
@pytest.mark.parametrize("mode", list(NP))
def test_alpha_scales_the_result(mode, d, n, large):
    """alpha * F_0 overflows (large) or is subnormal; the products and the
    scaled result are ordinary numbers."""
    _need_gpu()
    dt = NP[mode]
    alpha, f0, x = {("f32", True): (1e25, 1e20, 1e-30), ("f32", False): (1e-25, 1e-18, 1e30),
                    ("f64", True): (1e200, 1e150, 1e-250), ("f64", False): (1e-200, 1e-120, 1e250)}[mode, large]
    rng = np.random.default_rng(17)
    factors = [rng.uniform(-1, 1, n * n).astype(dt) for _ in range(d)]
    factors[0] = (factors[0] * f0).astype(dt)
    for batch in (1, 40):
        X = (rng.standard_normal(batch * n ** d) * x).astype(dt)
        got = _call(mode, d, n, "NT" if d == 2 else "TNC", alpha, factors, X, 0.0, np.zeros(batch * n ** d, dt), batch)
        want = oracle.kron_nd([n] * d, [n] * d, "NT" if d == 2 else "TNC", float(dt(alpha)), factors, X, 0.0,
                              np.zeros(batch * n ** d), batch)
        scale = np.abs(want).max()
        assert np.all(np.isfinite(got)), batch
        err = np.linalg.norm(got / scale - want / scale) / np.linalg.norm(want / scale)
        assert err <= TOL[mode], (batch, err)


def _captured_nodes(fn):
    """Nodes of the graph that one call records."""
    fn()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        fn()
    count = ctypes.c_size_t(0)
    hip = kron.lib()  # its symbols include the HIP runtime it is linked to
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(count)) == 0
    return count.value


@pytest.mark.parametrize("mode,d,n", [("f32", 2, 12), ("f32", 3, 7), ("f64", 2, 16), ("f64", 3, 3)])
def test_beta_in_one_launch(mode, d, n):
    """beta != 0 at sizes whose beta kernel pads its tiles or moves single
    elements: one launch of the fused kernel, without prepared factors."""
    _need_gpu()
    dt = NP[mode]
    rng = np.random.default_rng(18)
    batch, ops = 50, "TN" if d == 2 else "NTC"
    factors = [rng.standard_normal(n * n).astype(dt) for _ in range(d)]
    X, Y0 = (rng.standard_normal(batch * n ** d).astype(dt) for _ in range(2))
    tf, tx, ty = [torch.from_numpy(f).cuda() for f in factors], torch.from_numpy(X).cuda(), torch.from_numpy(Y0).cuda()
    code = kron.MODE_F32 if mode == "f32" else kron.MODE_F64
    ws = torch.empty(kron.kron_nd_workspace_size([n] * d, [n] * d, batch, code), dtype=torch.uint8, device="cuda")
    fn = getattr(kron, f"kron_nd_batched_{mode}")
    assert _captured_nodes(lambda: fn([n] * d, [n] * d, ops, 1.0, tf, tx, 0.5, ty, batch, ws=ws)) == 1
    got = _call(mode, d, n, ops, 1.0, factors, X, 0.5, Y0, batch)
    want = oracle.kron_nd([n] * d, [n] * d, ops, 1.0, factors, X, 0.5, Y0, batch)
    assert np.linalg.norm(got - want) <= TOL[mode] * np.linalg.norm(want)


@pytest.mark.parametrize("n", [1, 4, 6, 11, 16])
@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("mode", list(NP))
def test_result_does_not_depend_on_the_batch(mode, d, n):
    """One operand alone, in the workspace that the query names for it, gives
    the bits that it has inside a batch."""
    _need_gpu()
    dt = NP[mode]
    rng = np.random.default_rng(19)
    factors = [rng.standard_normal(n * n).astype(dt) for _ in range(d)]
    e = n ** d
    X = rng.standard_normal(5 * e).astype(dt)
    for ops in ("NNN", "TNT", "CCC"):
        whole = _call(mode, d, n, ops[:d], 1.0, factors, X, 0.0, np.zeros_like(X), 5)
        for p in (0, 4):
            one = _call(mode, d, n, ops[:d], 1.0, factors, X[p * e:(p + 1) * e].copy(), 0.0, np.zeros(e, dt), 1)
            assert np.array_equal(one, whole[p * e:(p + 1) * e]), (ops, p)
