"""Shared launches of the grouped backward: more groups than one launch holds,
both types, every size class, empty groups and every mix of outputs give what
the single-group calls give, bit for bit, also from a captured graph."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _group(kron, g, i, dtype):
    dim, n = 2 + i % 2, 1 + i % 16
    count = (0, 1, 7, 300, 5000 // n)[i % 5]
    rand = lambda k: torch.randn(k, generator=g, dtype=dtype).cuda()
    d = {"dim": dim, "n": n, "count": count, "mode": kron.MODE_F32 if dtype == torch.float32 else kron.MODE_F64,
         "X": rand(count * n ** dim), "dY": rand(count * n ** dim)}
    for f, k in enumerate("ABC"[:dim]):
        d[k] = rand(n * n)
        d["d" + k] = torch.full((n * n,), 7.0, dtype=dtype, device="cuda") if (i >> f) % 3 != 1 else None
    d["dX"] = torch.full_like(d["X"], 7.0) if i % 7 != 3 else None
    return d


@pytest.mark.parametrize("ngroups", [1, 33, 150])
def test_shared_launches_equal_single_calls(ngroups):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1304_7054_amd as kron
    g = torch.Generator().manual_seed(ngroups)
    groups = [_group(kron, g, i, torch.float64 if i % 4 == 3 else torch.float32) for i in range(ngroups)]
    out = [(d, k) for d in groups for k in ("dX", "dA", "dB", "dC") if d.get(k) is not None]
    for d in groups:
        t = "f32" if d["mode"] == kron.MODE_F32 else "f64"
        names = "ABC"[:d["dim"]]
        ws = torch.empty(max(1, kron.kron_backward_workspace_size(d["dim"], d["n"], d["count"], d["mode"])),
                         dtype=torch.uint8, device="cuda")
        getattr(kron, f"kron{d['dim']}d_backward_{t}")(d["n"], *[d[k] for k in names], d["X"], d["dY"], d["dX"],
                                                        *[d["d" + k] for k in names], d["count"], ws)
    torch.cuda.synchronize()
    want = [d[k].clone() for d, k in out]
    ws = torch.empty(kron.kron_grouped_backward_workspace_size(groups), dtype=torch.uint8, device="cuda")

    def check():
        torch.cuda.synchronize()
        for (d, k), w in zip(out, want):
            assert torch.equal(d[k], w), (d["dim"], d["n"], d["count"], k)
            d[k].fill_(7.0)
        torch.cuda.synchronize()

    for d, k in out:
        d[k].fill_(7.0)
    kron.kron_grouped_backward(groups, ws)
    check()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        kron.kron_grouped_backward(groups, ws)
    for _ in range(3):
        graph.replay()
        check()
