"""The measured cases: what programs have this library do, through its public entry points.

A case is a dict of plain values.  `kind` names the entry points:

  fwd       kron{2,3}d_batched_* in one of the five precision modes
  step      one training step of the autograd front end: Y, dX and the factor gradients
  grouped   one prepared launch over a batch that mixes sizes and 2-D / 3-D operands
  groupedb  the backward of such a batch
  nd        kron_nd_batched_*: any number of dimensions, rectangular, complex, factors per operand
  strided   kron{2,3}d_batched_strided_*: alpha, op and leading dimensions

Factors are U[-1, 1] and operands N(0, 1), the distributions of the repository's workloads.
"""
import math

import numpy as np
import torch

import paper_1304_7054_amd as kron
from paper_1304_7054_amd import autograd

DTYPE = {"f32": torch.float32, "f64": torch.float64, "bf16x3": torch.float32, "bf16x6": torch.float32,
         "bf16": torch.bfloat16, "c32": torch.complex64, "c64": torch.complex128}
SUFFIX = {"f32": "f32", "f64": "f64", "bf16x3": "f32_bf16x3", "bf16x6": "f32_bf16x6", "bf16": "bf16"}
ESIZE = {"f32": 4, "f64": 8, "bf16x3": 4, "bf16x6": 4, "bf16": 2, "c32": 8, "c64": 16}
ND_CODE = {"f32": kron.MODE_F32, "f64": kron.MODE_F64, "c32": kron.KRON_TYPE_C32, "c64": kron.KRON_TYPE_C64}


def listed():
    return [
        # the smallest call: 2-D n = 4, 4096 operands, bound by the launch
        dict(name="fwd2d_n4_f32_small", kind="fwd", dim=2, n=4, mode="f32", batch=4096),
        # the two 1 GiB sizes of the 3-D action in single precision
        dict(name="fwd3d_n16_f32", kind="fwd", dim=3, n=16, mode="f32", batch=65536),
        dict(name="fwd3d_n10_f32", kind="fwd", dim=3, n=10, mode="f32", batch=268435),
        # double precision at the paper's batch of 50,000 arrays
        dict(name="fwd3d_n12_f64", kind="fwd", dim=3, n=12, mode="f64", batch=50000),
        # bf16 storage, an odd size and a ragged batch
        dict(name="fwd3d_n7_bf16", kind="fwd", dim=3, n=7, mode="bf16", batch=100003),
        # half a million small operands of 30 sizes in one launch, and their backward
        dict(name="grouped_mixed", kind="grouped", count=500000),
        dict(name="grouped_backward_mixed", kind="groupedb", count=500000),
        # training steps: a large 3-D one and the paper's 100,000 2-D matrices
        dict(name="step3d_n16_f32", kind="step", dim=3, n=16, mode="f32", batch=32768),
        dict(name="step2d_n10_f32", kind="step", dim=2, n=10, mode="f32", batch=100000),
        # the general action: factors beyond 16, and complex arrays with a conjugate transpose
        dict(name="nd2d_n32_f32", kind="nd", type="f32", m="32,32", n="32,32", ops="NN", varying=False, batch=131072),
        dict(name="nd3d_n16_c32", kind="nd", type="c32", m="16,16,16", n="16,16,16", ops="NCT", varying=False,
             batch=16384),
        # padded leading dimensions with transposed factors and a scale
        dict(name="strided3d_n16_f32_ld20", kind="strided", dim=3, n=16, mode="f32", ops="TNT", pad=4, batch=32768),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    kind = rng.choice(["fwd", "fwd", "fwd", "step", "step", "nd", "nd", "strided", "grouped", "groupedb"])
    if kind in ("grouped", "groupedb"):
        return dict(kind=kind, count=_log_int(rng, 2000, 400000))
    if kind == "nd":
        typ = rng.choice(["f32", "f32", "f64", "c32", "c64"])
        d = rng.choice([1, 2, 2, 3, 3, 4])
        hi = {1: 64, 2: 48, 3: 20, 4: 16}[d]
        n = [rng.randint(2, hi) for _ in range(d)]
        m = list(n) if rng.random() < 0.5 else [rng.randint(2, hi) for _ in range(d)]
        varying = rng.random() < 0.2
        per = max(math.prod(n), math.prod(m)) * ESIZE[typ]
        if varying:
            per += sum(a * b for a, b in zip(m, n)) * ESIZE[typ]
        total = _log_int(rng, 1 << 20, 1 << 28)
        return dict(kind=kind, type=typ, m=",".join(map(str, m)), n=",".join(map(str, n)),
                    ops="".join(rng.choice("NTC") for _ in range(d)), varying=varying, batch=max(1, total // per))
    dim, n = rng.choice([2, 3]), rng.randint(1, 16)
    if kind == "fwd":
        mode = rng.choice(["f32", "f32", "f32", "f64", "f64", "bf16", "bf16x3", "bf16x6"])
        total = _log_int(rng, 1 << 16, 1 << 29)
        return dict(kind=kind, dim=dim, n=n, mode=mode, batch=max(1, total // (n ** dim * ESIZE[mode])))
    mode = rng.choice(["f32", "f32", "f64"])
    if kind == "step":
        n = max(n, 2)
        total = _log_int(rng, 1 << 18, 1 << 27)
        return dict(kind=kind, dim=dim, n=n, mode=mode, batch=max(1, total // (n ** dim * ESIZE[mode])))
    total = _log_int(rng, 1 << 18, 1 << 28)
    return dict(kind=kind, dim=dim, n=n, mode=mode, ops="".join(rng.choice("NT") for _ in range(dim)),
                pad=rng.choice([0, 1, 2, 4]), batch=max(1, total // ((n + 4) * n ** (dim - 1) * ESIZE[mode])))


# ---- inputs -------------------------------------------------------------------


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _uniform(g, count, dtype):
    if dtype.is_complex:
        real = torch.float32 if dtype == torch.complex64 else torch.float64
        return torch.view_as_complex(torch.rand(count, 2, generator=g, device="cuda", dtype=real) * 2 - 1)
    if dtype == torch.bfloat16:
        return (torch.rand(count, generator=g, device="cuda") * 2 - 1).to(dtype)
    return torch.rand(count, generator=g, device="cuda", dtype=dtype) * 2 - 1


def _normal(g, count, dtype):
    return torch.randn(count, generator=g, device="cuda", dtype=dtype)


def _dense_inputs(case, seed):
    g, dt, n = _gen(seed), DTYPE[case["mode"]], case["n"]
    mats = [_uniform(g, n * n, dt) for _ in range(case["dim"])]
    X = _normal(g, case["batch"] * n ** case["dim"], dt)
    return mats, X, g


def _group_sizes(count):
    """(dim, n, operands) of a mixed batch: n in 2..16 with weight 3 on 6..10 and 1 elsewhere, 70 % 2-D."""
    weight = {n: 3 if 6 <= n <= 10 else 1 for n in range(2, 17)}
    total = sum(weight.values())
    return [(dim, n, max(1, round(count * share * weight[n] / total)))
            for dim, share in ((2, 0.7), (3, 0.3)) for n in range(2, 17)]


def _group_inputs(case, seed):
    g, out = _gen(seed), []
    for dim, n, b in _group_sizes(case["count"]):
        grp = {"dim": dim, "n": n, "count": b}
        for k in "ABC"[:dim]:
            grp[k] = _uniform(g, n * n, torch.float32)
        grp["X"] = _normal(g, b * n ** dim, torch.float32)
        if case["kind"] == "groupedb":
            grp["dY"] = _normal(g, b * n ** dim, torch.float32)
        out.append(grp)
    return out


def _flat_outputs(groups, dtype):
    """Each group's dX, dA, dB (and dC) as 256-byte aligned slices of one array per output, which it returns."""
    out = []
    for k, source in (("dX", "X"), ("dA", "A"), ("dB", "B"), ("dC", "C")):
        users = [grp for grp in groups if source in grp]
        flat = torch.zeros(sum(-(-grp[source].numel() // 64) * 64 for grp in users), dtype=dtype, device="cuda")
        at = 0
        for grp in users:
            grp[k] = flat[at:at + grp[source].numel()]
            at += -(-grp[source].numel() // 64) * 64
        out.append(flat)
    return out


def _nd_shape(case):
    return [int(v) for v in case["m"].split(",")], [int(v) for v in case["n"].split(",")]


def _nd_inputs(case, seed):
    g, dt = _gen(seed), DTYPE[case["type"]]
    m, n = _nd_shape(case)
    count = case["batch"] if case["varying"] else 1
    factors = [_uniform(g, count * a * b, dt) for a, b in zip(m, n)]
    return factors, _normal(g, case["batch"] * math.prod(n), dt)


def _strides(case):
    """Leading dimension, plane and operand strides with `pad` unused elements per row."""
    n, ld = case["n"], case["n"] + case["pad"]
    return [ld * n ** k for k in range(case["dim"])]


def _strided_inputs(case, seed):
    g, dt, n = _gen(seed), DTYPE[case["mode"]], case["n"]
    mats = [_uniform(g, n * n, dt) for _ in range(case["dim"])]
    return mats, _normal(g, case["batch"] * _strides(case)[-1], dt)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "fwd":
        mats, X, _ = _dense_inputs(case, seed)
        fn = getattr(kron, f"kron{case['dim']}d_batched_{SUFFIX[case['mode']]}")
        return dict(kind=kind, fn=fn, n=case["n"], mats=mats, X=X, Y=torch.empty_like(X), batch=case["batch"])
    if kind == "step":
        mats, X, g = _dense_inputs(case, seed)
        dim, n, b = case["dim"], case["n"], case["batch"]
        leaves = [X.view([b] + [n] * dim)] + [M.view(n, n) for M in mats]
        dY = _normal(g, X.numel(), X.dtype).view(leaves[0].shape)
        return dict(kind=kind, fn=autograd.kron2d if dim == 2 else autograd.kron3d,
                    leaves=[t.requires_grad_() for t in leaves], dY=dY)
    if kind == "grouped":
        groups = _group_inputs(case, seed)
        for grp in groups:
            grp["Y"] = torch.empty_like(grp["X"])
        ws = torch.empty(kron.kron_grouped_workspace_size(groups), dtype=torch.uint8, device="cuda")
        kron.kron_grouped_prepare(groups, ws)
        return dict(kind=kind, groups=groups, ws=ws)
    if kind == "groupedb":
        groups = _group_inputs(case, seed)
        out = _flat_outputs(groups, torch.float32)
        ws = torch.empty(kron.kron_grouped_backward_workspace_size(groups), dtype=torch.uint8, device="cuda")
        return dict(kind=kind, groups=groups, out=out, ws=ws)
    if kind == "nd":
        m, n = _nd_shape(case)
        factors, X = _nd_inputs(case, seed)
        need = kron.kron_nd_workspace_size(m, n, case["batch"], ND_CODE[case["type"]])
        return dict(kind=kind, fn=getattr(kron, f"kron_nd_batched_{case['type']}"), m=m, n=n, ops=case["ops"],
                    factors=factors, ldfp=[a * b if case["varying"] else 0 for a, b in zip(m, n)], X=X,
                    Y=torch.empty(case["batch"] * math.prod(m), dtype=X.dtype, device="cuda"), batch=case["batch"],
                    ws=torch.empty(max(1, need), dtype=torch.uint8, device="cuda"))
    mats, X = _strided_inputs(case, seed)
    code = kron.MODE_F64 if case["mode"] == "f64" else kron.MODE_F32
    return dict(kind=kind, fn=getattr(kron, f"kron{case['dim']}d_batched_strided_{case['mode']}"), n=case["n"],
                ops=case["ops"] + "N" * (3 - case["dim"]), mats=mats, X=X, Y=torch.zeros_like(X), ld=_strides(case),
                batch=case["batch"], ws=torch.empty(kron.kron_ex_workspace_size(case["dim"], case["n"], code),
                                                    dtype=torch.uint8, device="cuda"))


def run(s):
    kind = s["kind"]
    if kind == "fwd":
        s["fn"](s["n"], *s["mats"], s["X"], s["Y"], s["batch"])
        return s["Y"]
    if kind == "step":
        Y = s["fn"](*s["leaves"])
        return [Y.detach(), *torch.autograd.grad(Y, s["leaves"], s["dY"])]
    if kind == "grouped":
        kron.kron_grouped_launch(s["ws"])
        return [grp["Y"] for grp in s["groups"]]
    if kind == "groupedb":
        kron.kron_grouped_backward(s["groups"], s["ws"])
        return s["out"]
    if kind == "nd":
        s["fn"](s["m"], s["n"], s["ops"], 1.0, s["factors"], s["X"], 0.0, s["Y"], s["batch"], ldfp=s["ldfp"],
                ws=s["ws"])
        return s["Y"]
    factors = [v for M in s["mats"] for v in (M, s["n"])]
    s["fn"](s["n"], *s["ops"], -1.5, *factors, s["X"], *s["ld"], 0.0, s["Y"], *s["ld"], s["batch"], ws=s["ws"])
    return s["Y"]


# ---- work ---------------------------------------------------------------------


def _products(m, n):
    """Multiply-adds of one operand's mode products, fastest index first."""
    total = 0
    for k in range(len(n) - 1, -1, -1):
        total += math.prod(n[:k]) * m[k] * n[k] * math.prod(m[k + 1:])
    return total


def work(case):
    kind = case["kind"]
    if kind in ("grouped", "groupedb"):
        elems = sum(b * n ** dim for dim, n, b in _group_sizes(case["count"]))
        mads = sum(b * dim * n ** (dim + 1) for dim, n, b in _group_sizes(case["count"]))
        if kind == "grouped":
            return {"bytes": 8 * elems, "flops": 2 * mads}
        return {"bytes": 12 * elems, "flops": 5 * mads}
    if kind == "nd":
        m, n = _nd_shape(case)
        e = ESIZE[case["type"]]
        fac = sum(a * b for a, b in zip(m, n)) * e * (case["batch"] if case["varying"] else 1)
        return {"bytes": case["batch"] * (math.prod(n) + math.prod(m)) * e + fac,
                "flops": case["batch"] * _products(m, n) * (8 if case["type"][0] == "c" else 2)}
    dim, n, b, e = case["dim"], case["n"], case["batch"], ESIZE[case["mode"]]
    mads = b * dim * n ** (dim + 1)
    if kind == "step":  # forward: X in, Y out; backward: X and dY in, dX out
        return {"bytes": 5 * b * n ** dim * e, "flops": 7 * mads}
    return {"bytes": 2 * b * n ** dim * e, "flops": 2 * mads}


# ---- the values in 64 bits ------------------------------------------------------


def _wide(t):
    return t.to(torch.complex128 if t.is_complex() else torch.float64)


def _along(X, M, axis):
    """sum_a M(i, a) X(.., a, ..) on one axis of X; M may carry one matrix per leading index of X."""
    moved = X.movedim(axis, -1).contiguous()
    if M.dim() == 3:
        out = torch.bmm(moved.reshape(M.shape[0], -1, M.shape[2]), M.transpose(1, 2).contiguous())
    else:
        out = moved.reshape(-1, M.shape[1]) @ M.t().contiguous()
    return out.reshape(moved.shape[:-1] + (M.shape[-2],)).movedim(-1, axis)


def _apply(X, mats):
    for k, M in enumerate(mats):
        X = _along(X, M, k + 1)
    return X


def _colmajor(v, rows, cols):
    return _wide(v).reshape(cols, rows).t()


def _factor_gradients(X, dY, mats):
    out = []
    for k in range(len(mats)):
        T = X
        for j, M in enumerate(mats):
            if j != k:
                T = _along(T, M, j + 1)
        n = mats[k].shape[0]
        out.append(dY.movedim(k + 1, 0).reshape(n, -1) @ T.movedim(k + 1, 0).reshape(n, -1).t())
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("fwd", "step"):
        mats, X, g = _dense_inputs(case, seed)
        dim, n, b = case["dim"], case["n"], case["batch"]
        shape = [b] + [n] * dim
        if kind == "fwd":
            return _apply(_wide(X).view(shape), [_colmajor(M, n, n) for M in mats]).reshape(-1)
        dY = _wide(_normal(g, X.numel(), X.dtype)).view(shape)
        X, F = _wide(X).view(shape), [_wide(M).view(n, n) for M in mats]
        return [_apply(X, F), _apply(dY, [M.t() for M in F]), *_factor_gradients(X, dY, F)]
    if kind in ("grouped", "groupedb"):
        groups = _group_inputs(case, seed)
        out = _flat_outputs(groups, torch.float64) if kind == "groupedb" else []
        for grp in groups:
            dim, n = grp["dim"], grp["n"]
            F = [_colmajor(grp[k], n, n) for k in "ABC"[:dim]]
            X = _wide(grp["X"]).view([grp["count"]] + [n] * dim)
            if kind == "grouped":
                out.append(_apply(X, F).reshape(-1))
                continue
            dY = _wide(grp["dY"]).view(X.shape)
            grp["dX"].copy_(_apply(dY, [M.t() for M in F]).reshape(-1))
            for k, G in zip("ABC", _factor_gradients(X, dY, F)):
                grp["d" + k].copy_(G.t().reshape(-1))
        return out
    if kind == "nd":
        m, n = _nd_shape(case)
        factors, X = _nd_inputs(case, seed)
        mats = []
        for k, v in enumerate(factors):
            rows, cols = (m[k], n[k]) if case["ops"][k] == "N" else (n[k], m[k])
            M = _wide(v).reshape(-1, cols, rows).transpose(1, 2)
            if case["ops"][k] != "N":
                M = M.transpose(1, 2)
            if case["ops"][k] == "C":
                M = M.conj().resolve_conj()
            mats.append(M if case["varying"] else M[0])
        return _apply(_wide(X).view([case["batch"]] + n), mats).reshape(-1)
    mats, X = _strided_inputs(case, seed)
    dim, n, b = case["dim"], case["n"], case["batch"]
    shape, ld = [b] + [n] * dim, _strides(case)
    strides = [ld[-1]] + ld[:-1][::-1] + [1]
    F = [_colmajor(M, n, n) for M in mats]
    F = [M.t() if op == "T" else M for M, op in zip(F, case["ops"])]
    Y = torch.zeros(X.numel(), dtype=torch.float64, device="cuda")
    Y.as_strided(shape, strides).copy_(-1.5 * _apply(_wide(X).as_strided(shape, strides), F))
    return Y
