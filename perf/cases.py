"""The work that users of this library have it do, as measurable cases.

Each case is one pass through the public entry points (``api.Plan.run``,
``api.spmm_submit`` / ``api.spmm_wait``, ``api.Plan.on_device``) on seeded
inputs made on the GPU.  ``listed()`` names the fixed cases, ``draw(rng)``
gives another one of the same ranges, ``prepare`` makes what a program holds
before the call, ``run`` is the call, ``work`` what it cannot do without, and
``exact`` the product in 64 bits.

Kinds of matrices (the shapes this library is measured on):
  uniform    a fixed number of random columns in every row; small, so that
             latency and launches count
  graph      Chung-Lu power-law graph (GNN aggregation; vector path)
  block      16x16 community blocks at 30% fill in a band, plus two stray
             columns a row (tiles for the matrix cores and a remainder)
  mask       block-sparse attention mask: 64x64 blocks at 10% and a sliding
             window of 512 (dense tiles)
  batch      uneven power-law graphs in one submission
  minibatch  a sampled bipartite layer, planned for this batch alone, run
             forward with A and backward with A transposed
"""
import math

import torch

from paper_2606_22482_amd import api

DEV = "cuda"
TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
SIZE = {"f32": 4, "bf16": 2, "f16": 2}
BLOCK_OPTS = dict(mode="mixed", row_order="original_ranges")
MASK_OPTS = dict(mode="mixed", row_order="original_ranges", window_h=64)


def listed():
    return [
        # the smallest call: one layer on a small graph, bound by latency
        dict(name="uniform_4k_n32", kind="uniform", m=4096, k=4096, per_row=16, n=32, vals="f32", b="f32"),
        # GNN aggregation in training at full size, forward (its graph is symmetric, so backward is the same)
        dict(name="graph_1m_n128", kind="graph", m=1 << 20, mean=16.0, gamma=2.1, n=128, vals="f32", b="f32"),
        # the last layer of a GNN: as many columns as there are classes, an odd number
        dict(name="graph_200k_n47", kind="graph", m=200003, mean=14.0, gamma=2.1, n=47, vals="f32", b="f32"),
        # serving on a resident graph with 16-bit features
        dict(name="graph_500k_n256_bf16", kind="graph", m=500000, mean=16.0, gamma=2.1, n=256, vals="f32", b="bf16"),
        # wide features on a middling graph
        dict(name="graph_100k_n512", kind="graph", m=100000, mean=16.0, gamma=2.1, n=512, vals="f32", b="f32"),
        # community-clustered matrix, 16-bit features on the matrix cores
        dict(name="block_262k_n256_bf16", kind="block", m=262144, n=256, vals="f32", b="bf16"),
        # attention over a long sequence (prefill), 16-bit weights and values
        dict(name="mask_32k_n256_bf16", kind="mask", m=32768, n=256, vals="bf16", b="bf16"),
        # attention with f32 weights and f32 values at one head's width
        dict(name="mask_16k_n64_f32", kind="mask", m=16384, n=64, vals="f32", b="f32"),
        # attention over a short, ragged sequence: few windows for the chip
        dict(name="mask_3k_n128_bf16", kind="mask", m=3001, n=128, vals="f32", b="bf16"),
        # many uneven matrices in one submission (throughput)
        dict(name="batch_64_f16", kind="batch", count=64, lo=1000, hi=200000, spec=4, vals="f16", b="f16"),
        # a serving loop's batch of small requests (latency)
        dict(name="batch_16_small", kind="batch", count=16, lo=1000, hi=20000, spec=5, vals="f32", b="f32"),
        # mini-batch training: both directions' plans, forward and backward
        dict(name="minibatch_10k_n100", kind="minibatch", m=10000, k=60000, per_row=15, n=100, vals="f32", b="f32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A width: half of the time one of the usual ones, else any, odd ones among them."""
    usual = [w for w in (16, 32, 64, 128, 256, 512) if lo <= w <= hi]
    return rng.choice(usual) if rng.random() < 0.5 else _log(rng, lo, hi)


def draw(rng):
    kind = rng.choice(["uniform", "graph", "graph", "graph", "block", "mask", "mask", "batch", "minibatch"])
    if kind == "uniform":
        return dict(kind=kind, m=_log(rng, 1000, 16000), k=_log(rng, 1000, 16000), per_row=rng.randint(8, 32),
                    n=_width(rng, 16, 128), vals="f32", b="f32")
    if kind == "graph":
        m, mean, n = _log(rng, 2000, 1 << 20), rng.uniform(8, 24), _width(rng, 16, 512)
        vals, b = rng.choice([("f32", "f32"), ("f32", "bf16"), ("bf16", "bf16"), ("f16", "f16")])
        n = max(16, min(n, int(2.1e9 / (m * mean))))  # at most the work of the largest
        return dict(kind=kind, m=m, mean=round(mean, 2), gamma=round(rng.uniform(2.1, 2.4), 2), n=n, vals=vals, b=b)
    if kind == "block":
        vals, b = rng.choice([("f32", "bf16"), ("bf16", "bf16"), ("f16", "f16")])
        return dict(kind=kind, m=16 * _log(rng, 1024, 16384), n=_width(rng, 32, 256), vals=vals, b=b)
    if kind == "mask":
        vals, b = rng.choice([("bf16", "bf16"), ("f32", "bf16"), ("f16", "f16"), ("f32", "f32")])
        return dict(kind=kind, m=_log(rng, 1000, 32768), n=_width(rng, 32, 256), vals=vals, b=b)
    if kind == "batch":
        vals, b = rng.choice([("f16", "f16"), ("f32", "f32"), ("f32", "bf16")])
        return dict(kind=kind, count=_log(rng, 4, 48), lo=1000, hi=_log(rng, 8000, 150000), spec=rng.randint(10, 10 ** 6),
                    vals=vals, b=b)
    m = _log(rng, 1000, 40000)
    return dict(kind=kind, m=m, k=m * rng.randint(2, 8) + rng.randint(0, 7), per_row=rng.randint(5, 20), n=_width(rng, 16, 256),
                vals="f32", b="f32")


# --------------------------------------------------------------------------------------------
# inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _values(g, n, kind, lo=-1.0, hi=1.0):
    return (torch.rand(n, generator=g, device=DEV) * (hi - lo) + lo).to(TORCH[kind])


def _dense(g, rows, n, kind):
    return torch.randn(rows, n, generator=g, device=DEV).to(TORCH[kind])


def _csr(key, m, k):
    """Row pointers and columns of the sorted, distinct keys row * k + column."""
    rows = torch.div(key, k, rounding_mode="floor")
    ptr = torch.zeros(m + 1, dtype=torch.int64, device=DEV)
    ptr[1:] = torch.cumsum(torch.bincount(rows, minlength=m), 0)
    return ptr, (key - rows * k).to(torch.int32), rows


def _power(n, gamma, mean, wmax):
    """Expected degrees c (i + i0)^(-1/(gamma - 1)) with the given mean and largest."""
    i = torch.arange(n, dtype=torch.float64, device=DEV)
    beta, lo, hi = -1.0 / (gamma - 1.0), 1e-6, float(n)
    for _ in range(40):
        f = (i + math.sqrt(lo * hi)) ** beta
        if float(f[0] / f.mean()) > wmax / mean:
            lo = math.sqrt(lo * hi)
        else:
            hi = math.sqrt(lo * hi)
    f = (i + math.sqrt(lo * hi)) ** beta
    return f * (mean / f.mean())


def _pick(g, weights, shape):
    """Indices drawn in proportion to the weights (in whole numbers: sums of floats may differ from run to run)."""
    cdf = torch.cumsum((weights * (1 << 24)).long() + 1, 0)
    at = (torch.rand(shape, generator=g, device=DEV, dtype=torch.float64) * cdf[-1].double()).long()
    return torch.searchsorted(cdf, at, right=True).clamp_(max=weights.numel() - 1)


def _graph(g, m, mean, gamma, vals):
    w = _power(m, gamma, mean, min(20000.0, m / 8.0))
    e = int(m * mean / 2)
    u, v = _pick(g, w, e), _pick(g, w, e)
    perm = torch.randperm(m, generator=g, device=DEV)
    u, v = perm[u[u != v]], perm[v[u != v]]
    ptr, col, rows = _csr(torch.unique(torch.cat([u * m + v, v * m + u])), m, m)
    if vals == "f32":  # symmetric normalisation
        d = (ptr[1:] - ptr[:-1]).double()
        return ptr, col, (d[rows] * d[col.long()]).rsqrt().float()
    return ptr, col, _values(g, col.numel(), vals)


def _uniform(g, m, k, per_row, vals):
    key = torch.arange(m, device=DEV)[:, None] * k + torch.randint(0, k, (m, per_row), generator=g, device=DEV)
    ptr, col, _ = _csr(torch.unique(key), m, k)
    return ptr, col, _values(g, col.numel(), vals)


def _block(g, m, vals):
    nb = m // 16
    pick = torch.rand(nb, 64, generator=g, device=DEV).argsort(dim=1, stable=True)[:, :8]
    bc = (torch.arange(nb, device=DEV)[:, None] - 32 + pick) % nb
    br, j, r, c = torch.nonzero(torch.rand(nb, 8, 16, 16, generator=g, device=DEV) < 0.3, as_tuple=True)
    key = (br * 16 + r) * m + bc[br, j] * 16 + c
    stray = torch.arange(m, device=DEV)[:, None] * m + torch.randint(0, m, (m, 2), generator=g, device=DEV)
    ptr, col, _ = _csr(torch.unique(torch.cat([key, stray.reshape(-1)])), m, m)
    return ptr, col, _values(g, col.numel(), vals)


def _mask(g, m, vals):
    nb = -(-m // 64)
    on = torch.rand(nb, nb, generator=g, device=DEV).argsort(dim=1, stable=True) < math.ceil(0.1 * nb)
    i = torch.arange(m, device=DEV)
    cols, lens = [], []
    for r0 in range(0, m, 2048):
        r = i[r0:r0 + 2048, None]
        at = on[(r // 64).squeeze(1)].repeat_interleave(64, 1)[:, :m] | ((i >= r - 256) & (i < r + 256))
        lens.append(at.sum(1))
        cols.append(torch.nonzero(at)[:, 1].to(torch.int32))
    ptr = torch.zeros(m + 1, dtype=torch.int64, device=DEV)
    ptr[1:] = torch.cumsum(torch.cat(lens), 0)
    col = torch.cat(cols)
    return ptr, col, _values(g, col.numel(), vals, 0.0, 1.0)


def _specs(case):
    """(rows, mean degree, width) of a batch's matrices, the same for every seed."""
    import random
    r = random.Random(case["spec"])
    return [(_log(r, case["lo"], case["hi"]), r.uniform(8, 32) if case["vals"] == "f16" else 16.0, r.choice([32, 64, 128]))
            for _ in range(case["count"])]


def _inputs(case, seed):
    """[(rowptr, colidx, vals, m, k, B)], one for each product of the case."""
    g, kind = _gen(seed), case["kind"]
    if kind == "batch":
        gamma = 2.3 if case["vals"] == "f16" else 2.1
        got = []
        for m, mean, n in _specs(case):
            a = _graph(g, m, mean, gamma, case["vals"])
            got.append(a + (m, m, _dense(g, m, n, case["b"])))
        return got
    m, n = case["m"], case["n"]
    if kind == "minibatch":
        k = case["k"]
        # columns by popularity: neighbours of a sample are power-law distributed
        col = _pick(g, _power(k, 2.1, 1.0, k / 64.0), (m, case["per_row"]))
        key = torch.unique(torch.arange(m, device=DEV)[:, None] * k + col)
        ptr, col, rows = _csr(key, m, k)
        deg = ptr[1:] - ptr[:-1]
        val = 1.0 / deg[rows].float()
        back, order = torch.sort(col.long() * m + rows)
        tptr, tcol, _ = _csr(back, k, m)
        return [(ptr, col, val, m, k, _dense(g, k, n, "f32")), (tptr, tcol, val[order].contiguous(), k, m, _dense(g, m, n, "f32"))]
    k = case.get("k", m)
    if kind == "uniform":
        a = _uniform(g, m, k, case["per_row"], case["vals"])
    elif kind == "graph":
        a = _graph(g, m, case["mean"], case["gamma"], case["vals"])
    elif kind == "block":
        a = _block(g, m, case["vals"])
    else:
        a = _mask(g, m, case["vals"])
    return [a + (m, k, _dense(g, k, n, case["b"]))]


def prepare(case, seed):
    opts = {"block": BLOCK_OPTS, "mask": MASK_OPTS}.get(case["kind"], {})
    o = api.default_opts(**opts)
    state = {"case": case, "products": []}
    for ptr, col, val, m, k, B in _inputs(case, seed):
        C = torch.empty(m, B.shape[1], dtype=torch.float32, device=DEV)
        if case["kind"] == "minibatch":  # planned in the pass
            state["products"].append((ptr, col, val, m, k, B, C))
        else:
            state["products"].append((api.Plan.on_device(ptr, col, val, m, k, B.shape[1], case["b"], o), B, C))
    if case["kind"] == "batch":
        state["items"] = [api.WorkItem(*p) for p in state["products"]]
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "batch":
        api.spmm_wait(api.spmm_submit(state["items"]))
        return [C for _, _, C in state["products"]]
    if case["kind"] == "minibatch":
        out = []
        for ptr, col, val, m, k, B, C in state["products"]:
            plan = api.Plan.on_device(ptr, col, val, m, k, B.shape[1], "f32")
            plan.run(B, C)
            plan.destroy()
            out.append(C)
        return out
    plan, B, C = state["products"][0]
    plan.run(B, C)
    return C


def _nnz(case):
    """Expected entries of a single matrix."""
    m, kind = case["m"], case["kind"]
    if kind in ("uniform", "minibatch"):
        return m * case["per_row"]
    if kind == "graph":
        return 0.97 * m * case["mean"]
    if kind == "block":
        return m * (8 * 16 * 0.3 + 2)
    nb = -(-m // 64)
    return m * (64 * math.ceil(0.1 * nb) + 0.9 * min(512, m))


def work(case):
    sv, sb = SIZE[case["vals"]], SIZE[case["b"]]
    if case["kind"] == "batch":
        nnz = [(m, 0.97 * m * mean, n) for m, mean, n in _specs(case)]
        return {"bytes": sum(4 * m + e * (4 + sv) + m * n * (sb + 4) for m, e, n in nnz),
                "flops": sum(2 * e * n for _, e, n in nnz)}
    m, k, n, e = case["m"], case.get("k", case["m"]), case["n"], _nnz(case)
    if case["kind"] == "minibatch":  # two plans (each reads and writes its CSR once) and two products
        used = min(k, 0.6 * e)  # columns that the sample reaches
        return {"bytes": 2 * (2 * e * 8 + 8 * (m + k)) + 4 * n * (used + m + m + k), "flops": 4 * e * n}
    # entries: a column and a value each; in tiles a 16-bit value and its bit of the bitmap
    per = {"block": 2.5, "mask": 2.15}.get(case["kind"], 4 + sv)
    return {"bytes": 4 * m + e * per + k * n * sb + m * n * 4, "flops": 2 * e * n}


def exact(case, seed):
    out = []
    for ptr, col, val, m, k, B in _inputs(case, seed):
        A = torch.sparse_csr_tensor(ptr, col.long(), val.double(), size=(m, k))
        out.append((A @ B.double()).contiguous())
    return out if case["kind"] in ("batch", "minibatch") else out[0]
