"""A grouped backward that mixes groups with factor gradients and groups that
ask for dX alone: the two kinds do not wait for each other, and the results are
those of the single-group calls."""
import ctypes

import pytest
import torch

import paper_1304_7054_amd as kron

pytestmark = pytest.mark.gpu
SHAPES = [(2, 5), (3, 4), (2, 16), (3, 9), (3, 16), (2, 10)]


def _groups(count):
    """Every second group asks for dX alone."""
    g = torch.Generator(device="cuda").manual_seed(29)
    rand = lambda k: torch.randn(k, generator=g, device="cuda")
    groups = []
    for i, (dim, n) in enumerate(SHAPES):
        grp = {"dim": dim, "n": n, "count": count, "X": rand(count * n ** dim), "dY": rand(count * n ** dim)}
        grp["dX"] = torch.zeros_like(grp["X"])
        for k in "ABC"[:dim]:
            grp[k] = rand(n * n)
            if i % 2 == 0:
                grp["d" + k] = torch.zeros(n * n, device="cuda")
        groups.append(grp)
    return groups


def test_the_kinds_are_independent():
    """In a captured call, kernels of both kinds have no kernel before them."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    groups = _groups(20)
    ws = torch.empty(kron.kron_grouped_backward_workspace_size(groups), dtype=torch.uint8, device="cuda")
    kron.kron_grouped_backward(groups, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        kron.kron_grouped_backward(groups, ws)
    roots = ctypes.c_size_t(0)
    hip = kron.lib()  # its symbols include the HIP runtime it is linked to
    assert hip.hipGraphGetRootNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(roots)) == 0
    dx_only = len(SHAPES) // 2
    assert roots.value == dx_only + 1  # the first of the launches that the others share, and each dX-only one
    graph.instantiate()
    want = [{k: v.clone() for k, v in grp.items() if k[0] == "d" and k not in ("dim", "dY")} for grp in groups]
    for rep in range(4):
        for grp, w in zip(groups, want):
            for k in w:
                grp[k].zero_()
        graph.replay()
        torch.cuda.synchronize()
        for grp, w in zip(groups, want):
            for k in w:
                assert torch.equal(grp[k], w[k]), (rep, grp["dim"], grp["n"], k)


@pytest.mark.parametrize("count", [1, 300])
def test_results_are_the_single_calls(count):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    groups = _groups(count)
    kron.kron_grouped_backward(groups)
    for grp in groups:
        dim, n = grp["dim"], grp["n"]
        want = {k: torch.zeros_like(grp[k]) for k in ("dX", "dA", "dB", "dC") if k in grp}
        getattr(kron, f"kron{dim}d_backward_f32")(n, *[grp[k] for k in "ABC"[:dim]], grp["X"], grp["dY"], want["dX"],
                                                  *[want.get("d" + k) for k in "ABC"[:dim]], count)
        torch.cuda.synchronize()
        for k, w in want.items():
            assert torch.equal(grp[k], w), (dim, n, k)
