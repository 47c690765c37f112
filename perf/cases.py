"""The work that a user of this library has it do, at the sizes it is used at.

Four kinds of work, all through the public calls of the package:
  spmm    Z = op(A X) and Z' = op(A^T X) on one matrix (both directions: forward propagates with A^T, backward with A)
  epoch   one full-batch training epoch: forward, loss, backward, W <- W - lr Y
  layers  the same pass composed by the caller from the per-layer calls, with bias vectors and their gradients
  build   an edge list turned into the compressed, normalised matrix and its transpose

Graphs are drawn on the GPU from the seed with the recipes of `synth` (Erdos-Renyi, R-MAT, Chung-Lu; endpoints renamed at
random), so vertex numbers carry no locality, as in the paper's runs.  Dense operands are uniform in [-1, 1) or standard
normal, labels uniform, weights Glorot-uniform.
"""
from __future__ import annotations

import math

import torch

import paper_2005_03300_amd as g

_CHUNK = 1 << 24          # endpoint pairs drawn at one time

_SPMM = dict(kind="spmm", norm="sym", slice=1, epilogue="none")
_EPOCH = dict(kind="epoch", norm="sym", labelled=1.0, preaggregated=False, lr=0.05)


def listed():
    return [
        # A neighbourhood-sized graph: one product on it is launches and host work, nothing else.
        dict(_SPMM, name="spmm_small", graph="er", n=1000, pairs=8000, f=16),
        # The toy model: an epoch whose kernels are all shorter than their launches.
        dict(_EPOCH, name="epoch_tiny", graph="er", n=4096, pairs=32768, dims="64-16-8"),
        # Stand-alone product with a wide operand on a skewed sparse graph.
        dict(_SPMM, name="spmm_rmat20_f128", graph="rmat", n=1 << 20, pairs=16 << 20, f=128),
        # Directed graph, odd vertex count, width that is no multiple of four, backward's mask: nothing is aligned.
        dict(_SPMM, name="spmm_directed_f41", graph="rmat", n=150_001, pairs=2_400_000, f=41, norm="row", epilogue="mask"),
        # One process's block row of eight (1D distribution) at hidden width 64: rectangular, values given by the caller.
        dict(_SPMM, name="spmm_block_row_f64", graph="rmat", n=1 << 20, pairs=16 << 20, f=64, slice=8, epilogue="relu"),
        # Dense power-law graph (mean degree 490): long rows, operand close to the caches' size, 602 features.
        dict(_EPOCH, name="epoch_dense_graph", graph="chunglu", n=232_965, pairs=59_450_000, gamma=2.1, max_degree=20_000.0,
             dims="602-16-16-41"),
        # Large sparse graph (mean degree 17): 17 GB of features, operand far beyond the caches.
        dict(_EPOCH, name="epoch_sparse_graph", graph="rmat", n=14_249_639, pairs=121_500_000, dims="300-16-16-24"),
        # The billion-edge graph at half its size, so that three of them fit one GPU: mean degree 150, 256 classes.
        dict(_EPOCH, name="epoch_large_graph", graph="chunglu", n=4_372_771, pairs=328_250_000, gamma=2.3, max_degree=50_000.0,
             dims="128-16-16-256"),
        # Hidden width 64 with a training split: the last layer is wide too, most rows of the loss are masked.
        dict(_EPOCH, name="epoch_hidden64_split", graph="chunglu", n=120_007, pairs=3_000_000, gamma=2.3, max_degree=4_000.0,
             dims="256-64-64-41", labelled=0.3),
        # Many epochs on fixed features: A^T H0 is computed once, the first layer is dense only.
        dict(_EPOCH, name="epoch_preaggregated", graph="rmat", n=1_781_204, pairs=15_187_500, dims="300-16-16-24", labelled=0.6,
             preaggregated=True),
        # A model of the caller's own making: two layers with biases on a directed graph, through the per-layer calls.
        dict(kind="layers", name="layers_bias", graph="rmat", n=200_003, pairs=3_200_000, norm="row", dims="128-64-41",
             labelled=0.5),
        # A new graph: sort, deduplicate, normalise, transpose.
        dict(kind="build", name="build_rmat20", graph="rmat", n=1 << 20, pairs=16 << 20, norm="sym"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["spmm", "epoch", "layers", "build"], [4, 4, 2, 1])[0]
    most = {"spmm": 100e6, "epoch": 60e6, "layers": 30e6, "build": 40e6}[kind]      # endpoint pairs
    n = _log(rng, 1000, 4_000_000)
    case = dict(kind=kind, graph=rng.choice(["er", "rmat", "chunglu"]), n=n)
    case["pairs"] = max(1000, int(n * min(_log(rng, 3, 250), most / n)))
    if case["graph"] == "chunglu":
        case["gamma"] = round(rng.uniform(2.1, 2.6), 2)
        case["max_degree"] = float(max(int(5 * case["pairs"] / n) + 8, min(n // 12, 20_000)))
    norm = rng.choice(["sym", "sym", "row"])
    if kind == "spmm":
        # the hidden widths in use, and any width at all; wide operands only while they stay below 2 GB
        f = rng.choice([16, 16, 32, 64, 128]) if rng.random() < 0.5 else _log(rng, 1, 300)
        case.update(f=max(1, min(f, int(5e8 // n))), norm=norm, slice=rng.choice([1, 1, 1, 4, 8]),
                    epilogue=rng.choice(["none", "relu", "mask"]))
    elif kind == "build":
        case.update(norm=norm)
    else:
        f0 = max(8, min(_log(rng, 16, 602), int(8e8 // n)))
        hidden, classes = rng.choice([16, 16, 32, 64]), _log(rng, 2, 256)
        dims = [f0] + [hidden] * rng.choice([1, 2, 2]) + [classes]
        if n * sum(dims) > 12e8:
            dims = [f0, 16, 16, min(classes, 64)]
        labelled = rng.choice([1.0, 0.1, 0.5])
        case.update(dims="-".join(map(str, dims)), norm=norm, labelled=labelled)
        if kind == "epoch":
            case.update(preaggregated=rng.random() < 0.25, lr=rng.choice([0.0, 0.05]))
    return case


# ---- inputs ------------------------------------------------------------------------------------------------------

def _dims(case):
    return [int(d) for d in case["dims"].split("-")]


def _rmat(scale, count, gen):
    """Each pair picks one quadrant per bit level with probabilities 0.57, 0.19, 0.19, 0.05."""
    u = torch.zeros(count, dtype=torch.int32, device="cuda")
    v = torch.zeros(count, dtype=torch.int32, device="cuda")
    for _ in range(scale):
        r = torch.rand(count, generator=gen, device="cuda")
        ubit = r >= 0.76
        u.mul_(2).add_(ubit)
        v.mul_(2).add_(((r >= 0.57) ^ ubit) | (r >= 0.95))
    return u, v


def _chung_lu_sampler(n, pairs, gamma, max_degree):
    """Endpoints with probability proportional to (i + i0)^(-1/(gamma-1)), by the closed form of the inverse of its
    integral; i0 is set so that the heaviest vertex expects `max_degree` pairs at the most."""
    b = 1.0 - 1.0 / (gamma - 1.0)

    def top(i0):
        return 2.0 * pairs * ((1 + i0) ** b - i0 ** b) / ((n + i0) ** b - i0 ** b)
    lo, hi = 1e-9, 1.0
    while top(hi) > max_degree and hi < 1e12:
        hi *= 2.0
    for _ in range(80):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if top(mid) > max_degree else (lo, mid)
    base, span = hi ** b, (n + hi) ** b - hi ** b

    def sample(count, gen):
        t = torch.rand(count, generator=gen, device="cuda", dtype=torch.float64).mul_(span).add_(base)
        return t.pow_(1.0 / b).sub_(hi).clamp_(0, n - 1).to(torch.int32)
    return sample


def _edges(case, seed):
    n, pairs, kind = case["n"], case["pairs"], case["graph"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    perm = torch.randperm(n, generator=gen, device="cuda").to(torch.int32)
    sample = _chung_lu_sampler(n, pairs, case["gamma"], case["max_degree"]) if kind == "chunglu" else None
    src, dst = [], []
    for first in range(0, pairs, _CHUNK):
        k = min(_CHUNK, pairs - first)
        if kind == "rmat":
            u, v = _rmat(max(1, (n - 1).bit_length()), k, gen)
            if n & (n - 1):
                keep = (u < n) & (v < n)
                u, v = u[keep], v[keep]
        elif kind == "chunglu":
            u, v = sample(k, gen), sample(k, gen)
        else:
            u = torch.randint(n, (k,), generator=gen, device="cuda", dtype=torch.int32)
            v = torch.randint(n, (k,), generator=gen, device="cuda", dtype=torch.int32)
        src.append(perm[u])
        dst.append(perm[v])
    return torch.cat(src), torch.cat(dst)


def _flags(case):
    if case["norm"] == "row":          # directed: A and A^T differ
        return g.ADD_SELF_LOOPS | g.NORM_ROW | g.BUILD_TRANSPOSE
    return g.SYMMETRISE | g.ADD_SELF_LOOPS | g.NORM_SYM | g.BUILD_TRANSPOSE


def _matrix(case, seed):
    src, dst = _edges(case, seed)
    torch.cuda.empty_cache()           # the library allocates for itself
    a = g.gcn_csr_create(case["n"], src, dst, _flags(case))
    parts = case.get("slice", 1)
    if parts > 1:
        rows = max(1, case["n"] // parts)
        rowptr, colidx, val, _ = a.arrays()
        end = int(rowptr[rows])
        a.close()
        a = g.gcn_csr_create_from_csr_rect(rows, case["n"], rowptr[:rows + 1].clone(), colidx[:end].clone(),
                                           val[:end].clone(), g.BUILD_TRANSPOSE)
    return a


def _uniform(rows, cols, gen):
    return torch.rand(rows, cols, generator=gen, device="cuda").mul_(2.0).sub_(1.0)


def prepare(case, seed):
    if case["kind"] == "build":
        src, dst = _edges(case, seed)
        torch.cuda.empty_cache()
        # the caller's own arrays, sized for the case that no pair repeats
        most = case["n"] + (1 if case["norm"] == "row" else 2) * case["pairs"]
        arrays = [(torch.zeros(most, dtype=torch.int32, device="cuda"), torch.zeros(most, device="cuda")) for _ in range(2)]
        return dict(case=case, src=src, dst=dst, arrays=arrays)
    a = _matrix(case, seed)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed + 1_000_003)
    if case["kind"] == "spmm":
        f = case["f"]
        st = dict(case=case, a=a, X=_uniform(a.n_cols, f, gen), Xt=_uniform(a.n_rows, f, gen),
                  Z=torch.empty(a.n_rows, f, device="cuda"), Zt=torch.empty(a.n_cols, f, device="cuda"), M=None, Mt=None)
        if case["epilogue"] == "mask":
            st["M"], st["Mt"] = _uniform(a.n_rows, f, gen), _uniform(a.n_cols, f, gen)
        g.gcn_spmm_prepare(a, 0, f)
        g.gcn_spmm_prepare(a, 1, f)
        return st
    n, dims = case["n"], _dims(case)
    labels = torch.randint(dims[-1], (n,), generator=gen, device="cuda", dtype=torch.int32)
    count = n
    if case["labelled"] < 1.0:
        labels[torch.rand(n, generator=gen, device="cuda") >= case["labelled"]] = -1
        labels[0] = 0
        count = int((labels >= 0).sum())
    H0 = torch.randn(n, dims[0], generator=gen, device="cuda")
    W = [_uniform(fi, fo, gen).mul_(math.sqrt(6.0 / (fi + fo))) for fi, fo in zip(dims, dims[1:])]
    st = dict(case=case, a=a, dims=dims, labels=labels, count=count, H0=H0, W=W, Y=[torch.empty_like(w) for w in W],
              loss=torch.zeros(1, device="cuda"))
    if case["kind"] == "layers":
        # gemm-first layers keep T n x f_out, the others n x f_in
        mats = [[torch.empty(n, k, device="cuda") for k in (fo, fo, min(fi, fo), min(fi, fo), fo)]
                for fi, fo in zip(dims, dims[1:])]
        st["Z"], st["H"], st["T"], st["S"], st["G"] = (list(m) for m in zip(*mats))
        st["b"] = [_uniform(1, fo, gen).view(-1) for fo in dims[1:]]
        st["db"] = [torch.empty_like(b) for b in st["b"]]
        for fi, fo in zip(dims, dims[1:]):
            g.gcn_spmm_prepare(a, 0, min(fi, fo))
            g.gcn_spmm_prepare(a, 1, min(fi, fo))
        return st
    if case["preaggregated"]:
        st["H0"] = g.gcn_spmm(a, 1, H0, torch.empty_like(H0))
    st["ws"] = torch.empty(g.gcn_epoch_workspace_bytes(n, dims), dtype=torch.uint8, device="cuda")
    g.gcn_epoch_prepare(a, dims)
    return st


# ---- one pass ----------------------------------------------------------------------------------------------------

def _run_layers(st):
    a, dims, W, b, Z, H, T, S, G = (st[k] for k in ("a", "dims", "W", "b", "Z", "H", "T", "S", "G"))
    last = len(W) - 1
    x = st["H0"]
    for l in range(last + 1):
        if l < last:
            g.gcn_layer_forward(a, x, W[l], Z[l], H[l], T[l], bias=b[l])
        else:
            g.gcn_layer_forward(a, x, W[l], Z[l], None, T[l], act=g.ACT_NONE, bias=b[l])
        x = H[l]
    g.gcn_softmax_nll_masked(Z[last], st["labels"], st["count"], st["loss"], G[last])
    for l in range(last, -1, -1):
        g.gcn_layer_backward(a, H[l - 1] if l else st["H0"], Z[l - 1] if l else None, W[l], G[l], T[l], S[l], st["Y"][l],
                             G[l - 1] if l else None, dbias=st["db"][l])
    return [st["loss"], Z[last], st["Y"], st["db"], G[0]]


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "spmm":
        epi = {"none": g.EPI_NONE, "relu": g.EPI_RELU, "mask": g.EPI_MASK}[case["epilogue"]]
        g.gcn_spmm(st["a"], 0, st["X"], st["Z"], epi, st["M"])
        g.gcn_spmm(st["a"], 1, st["Xt"], st["Zt"], epi, st["Mt"])
        return [st["Z"], st["Zt"]]
    if kind == "epoch":
        args = (st["W"], st["Y"], case["lr"], st["loss"], st["ws"])
        if case["preaggregated"]:
            g.gcn_epoch_preaggregated(st["a"], st["dims"], st["H0"], st["labels"], st["count"], *args)
        elif case["labelled"] < 1.0:
            g.gcn_epoch_masked(st["a"], st["dims"], st["H0"], st["labels"], st["count"], *args)
        else:
            g.gcn_epoch(st["a"], st["dims"], st["H0"], st["labels"], *args)
        return [st["loss"], st["Y"], st["W"]]
    if kind == "layers":
        return _run_layers(st)
    a = g.gcn_csr_create(case["n"], st["src"], st["dst"], _flags(case))
    out = []
    for transposed, (columns, values) in enumerate(st["arrays"]):
        rowptr, colidx, val, deg = a.arrays(bool(transposed))
        columns[:a.nnz].copy_(colidx)
        values[:a.nnz].copy_(val)
        out.append([rowptr, columns, values, deg])
    a.close()
    return out


# ---- what a pass cannot do without -------------------------------------------------------------------------------

def _entries(case):
    """Stored entries of the whole matrix: both directions of every pair (one when directed) and the diagonal, less the
    pairs that repeat (about 7 % on the skewed graphs at these sizes)."""
    per_pair = 1 if case["norm"] == "row" else 2
    keep = 1.0 if case["graph"] == "er" else 0.93
    return min(case["n"] + per_pair * case["pairs"] * keep, 0.9 * case["n"] ** 2)


def work(case):
    n, nnz = case["n"], _entries(case)
    if case["kind"] == "build":
        # the pairs once; A and A^T (row pointers, columns, values) and the degrees, written and exported
        return {"bytes": 8 * case["pairs"] + 2 * (2 * (8 * n + 8 * nnz) + 4 * n), "flops": 2 * nnz}
    if case["kind"] == "spmm":
        # a matrix normalised here needs its columns and degrees, one given by the caller its values too
        parts, f = case["slice"], case["f"]
        nnz, rows = nnz / parts, n // parts
        per_entry = 8 if parts > 1 else 4
        mask = 4 * f * (n + rows) if case["epilogue"] == "mask" else 0
        return {"bytes": 2 * per_entry * nnz + 8 * (n + rows) + 2 * 4 * f * (n + rows) + mask, "flops": 2 * 2 * nnz * f}
    dims = _dims(case)
    b, fl = 4.0 * n, 0.0                                            # the labels
    for l, (fi, fo) in enumerate(zip(dims, dims[1:])):
        w = min(fi, fo)
        sparse = 0 if l == 0 and case.get("preaggregated") else 2   # forward and backward
        b += sparse * (4 * nnz + 8 * n + 8 * n * w)
        fl += sparse * 2 * nnz * w
        b += 2 * 4 * n * fi if l == 0 else 3 * 4 * n * fi           # layer inputs: forward, weight gradient, mask
        fl += (2 if l == 0 else 3) * 2 * n * fi * fo
    return {"bytes": b, "flops": fl}


def tolerance(case):
    if case["kind"] == "build":
        return "exact"
    if case["kind"] == "spmm":
        return {"rel": 1e-5}
    # fp32 sums over all vertices; a hidden activation that is zero to rounding may fall on either side of the ReLU
    return {"rel": 1e-4, "max": 0.01}
