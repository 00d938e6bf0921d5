"""What a user of this library has it do, as measured cases.

A case names a kind of pass, a synthetic graph and a width:

* ``spmm``      one C = A*B on a handle that was built before, with the parameters the
                library picks (features -> select -> build), as every epoch of a training run
                or every request to a server does it;
* ``train``     forward and backward of a GCN / GIN model on a PcsrOperator: the shape the
                library is embedded in (5 layers, 16 input and output features);
* ``fresh``     a graph that has just arrived in device memory (sampled, filtered or otherwise
                made there) and is used once: features, selection, PCSR generation, one product;
* ``operator``  a graph in host memory becomes a PcsrOperator and does its first forward and
                backward product: what a program pays at its start;
* ``reorder``   the locality pre-step on host arrays: relabelling plus the permuted CSR.

Graphs are drawn on the GPU from the seed alone, in the shape classes of the benchmark's own
generators (Poisson, road-like, power-law, communities, cliques).
"""
import math

import torch

import paper_2605_15695_amd as pc
from paper_2605_15695_amd.gnn import PcsrOperator, make_model

RMAT_A, RMAT_B, RMAT_C = 0.57, 0.19, 0.19


def listed():
    return [
        # the smallest call: 33 K nonzeros, a few microseconds on the GPU, so launches and the
        # host path count (small molecules' or batched mini-graphs' adjacency)
        dict(name="spmm_poisson_4k_k32", kind="spmm", graph="poisson", n=4096, deg=8.0, K=32),
        # road network: rows of 3, wide features, streaming-bound
        dict(name="spmm_road_2m_k128", kind="spmm", graph="road", n=2_000_000, width=2000, deg=2.1, K=128),
        # communities with contiguous ids: what a graph looks like after the pre-step
        dict(name="spmm_sbm_250k_k256", kind="spmm", graph="sbm", n=250_000, block=500, deg=50.0, intra=0.9,
             shuffled=False, K=256),
        # the same graph with its ids in random order: what it looks like without the pre-step
        dict(name="spmm_shuffled_250k_k256", kind="spmm", graph="sbm", n=250_000, block=500, deg=50.0, intra=0.9,
             shuffled=True, K=256),
        # co-authorship-like cliques, an odd width (class scores): nothing is 16-byte aligned
        dict(name="spmm_cliques_300k_k75", kind="spmm", graph="cliques", n=300_000, size=24.0, noise=0.1, K=75),
        # large power-law graph, the narrowest layers of a model
        dict(name="spmm_rmat22_k16", kind="spmm", graph="rmat", n=1 << 22, edges=16, symmetric=True, permute=False,
             K=16),
        # the same graph at the widest layers: the largest product, the benchmark's default
        dict(name="spmm_rmat22_k512", kind="spmm", graph="rmat", n=1 << 22, edges=16, symmetric=True, permute=False,
             K=512),
        # GCN training on a directed power-law graph (forward on A, backward on its transpose)
        dict(name="train_gcn_rmat20_h64", kind="train", model="gcn", graph="rmat", n=1 << 20, edges=16,
             symmetric=False, permute=True, layers=5, features=16, hidden=64),
        # GIN training on a road-like graph (symmetric: one handle for both directions)
        dict(name="train_gin_road_h64", kind="train", model="gin", graph="road", n=2_000_000, width=2000, deg=2.1,
             layers=5, features=16, hidden=64),
        # a power-law graph made on the GPU and multiplied once
        dict(name="fresh_rmat20_k64", kind="fresh", graph="rmat", n=1 << 20, edges=16, symmetric=False, permute=True,
             K=64),
        # start of a training program on a directed community graph held by the host
        dict(name="operator_sbm_250k_k128", kind="operator", graph="sbm", n=250_000, block=500, deg=50.0, intra=0.9,
             shuffled=False, K=128),
        # the pre-step on a community graph whose ids carry no locality
        dict(name="reorder_shuffled_250k", kind="reorder", by="cluster", graph="sbm", n=250_000, block=500, deg=50.0,
             intra=0.9, shuffled=True),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_graph(rng, n_lo, n_hi, nnz_hi):
    """A graph of one of the shape classes with between n_lo and n_hi rows and about nnz_hi
    nonzeros at most."""
    n = max(64, int(_log(rng, n_lo, n_hi)))
    graph = rng.choice(["poisson", "road", "rmat", "sbm", "cliques"])
    room = max(2.0, nnz_hi / n)
    if graph == "poisson":
        return dict(graph=graph, n=n, deg=round(_log(rng, 4.0, min(160.0, max(4.5, room))), 2))
    if graph == "road":
        width = max(8, int(math.sqrt(n) * rng.uniform(0.5, 3.0)))
        return dict(graph=graph, n=max(8, n // width) * width, width=width, deg=round(rng.uniform(1.6, 5.0), 2))
    if graph == "rmat":
        symmetric = rng.random() < 0.5
        most = min(64.0, room / (2 if symmetric else 1))
        return dict(graph=graph, n=n, edges=max(2, int(_log(rng, 4.0, max(4.5, most)))), symmetric=symmetric,
                    permute=rng.random() < 0.5)
    if graph == "sbm":
        return dict(graph=graph, n=n, block=min(n, int(_log(rng, 50, 2000))),
                    deg=round(_log(rng, 12.0, min(90.0, max(12.5, room))), 2), intra=round(rng.uniform(0.7, 0.95), 2),
                    shuffled=rng.random() < 0.5)
    size = round(_log(rng, 8.0, min(64.0, max(8.5, room / 1.5))), 1)
    return dict(graph=graph, n=n, size=size, noise=round(rng.uniform(0.0, 0.5), 2))


def draw(rng):
    kind = rng.choice(["spmm"] * 7 + ["train"] * 2 + ["fresh", "operator", "reorder"])
    if kind == "spmm":
        c = dict(kind=kind, **_draw_graph(rng, 1000, 1 << 22, 1.2e8))
        most = min(512.0, 2.0 ** 31 / c["n"], 5e10 / (c["n"] * max(3.0, _mean_degree(c))))
        c["K"] = int(_log(rng, 8.0, max(16.0, most)))
        return c
    if kind == "train":
        return dict(kind=kind, model=rng.choice(["gcn", "gin"]), **_draw_graph(rng, 4000, 1.5e6, 2e7),
                    layers=rng.randint(2, 5), features=rng.choice([8, 16, 16, 32]),
                    hidden=rng.choice([16, 24, 32, 48, 64, 64, 96, 128]))
    if kind == "fresh":
        return dict(kind=kind, **_draw_graph(rng, 2000, 2e6, 3e7), K=int(_log(rng, 8.0, 128.0)))
    if kind == "operator":
        return dict(kind=kind, **_draw_graph(rng, 2000, 1e6, 1.2e7), K=int(_log(rng, 8.0, 128.0)))
    return dict(kind=kind, by=rng.choice(["cluster", "cluster", "degree"]), **_draw_graph(rng, 4000, 2.5e5, 1.2e7))


# ------------------------------------------------------------------------------ graphs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda")


def _randint(g, hi, n):
    """n integers in [0, hi); hi: a number or a tensor of n of them."""
    r = torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * hi
    return torch.minimum(r.long(), torch.as_tensor(hi, device="cuda").long() - 1)


def _poisson(g, mean, n):
    return torch.poisson(torch.full((n,), float(mean), device="cuda"), generator=g).long()


def _csr(n, src, dst, most=None, g=None):
    """rowptr int32[n+1], colidx int32 (sorted, no duplicates) of the pairs, of `most` of them."""
    key = torch.sort(src * n + dst).values
    if key.numel():
        keep = torch.ones(key.numel(), dtype=torch.bool, device="cuda")
        keep[1:] = key[1:] != key[:-1]
        key = key[keep]
    if most is not None and most < key.numel():
        key = key[torch.sort(torch.randperm(key.numel(), generator=g, device="cuda")[:most]).values]
    rows = torch.div(key, n, rounding_mode="floor")
    colidx = (key - rows * n).to(torch.int32)
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rowptr[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
    return rowptr.to(torch.int32), colidx


def _graph(case, seed):
    """(rowptr, colidx, vals) on the GPU; mean-aggregation or GCN values as the class has them."""
    g, n, kind = _gen(seed), case["n"], case["graph"]
    gcn = kind in ("road", "rmat")
    if kind == "poisson":
        src = torch.repeat_interleave(torch.arange(n, device="cuda"), _poisson(g, case["deg"], n))
        dst = _randint(g, n, src.numel())
    elif kind == "road":
        src, dst = _road_edges(g, n, case["width"], case["deg"])
    elif kind == "rmat":
        src, dst = _rmat_edges(g, n, case["edges"])
        if case["permute"]:
            perm = torch.randperm(n, generator=g, device="cuda")
            src, dst = perm[src], perm[dst]
        if case["symmetric"]:
            src, dst = torch.cat([src, dst]), torch.cat([dst, src])
    elif kind == "sbm":
        src = torch.repeat_interleave(torch.arange(n, device="cuda"), _poisson(g, case["deg"], n))
        first = torch.div(src, case["block"], rounding_mode="floor") * case["block"]
        inside = first + _randint(g, torch.clamp(n - first, max=case["block"]).double(), src.numel())
        dst = torch.where(_rand(g, src.numel()) < case["intra"], inside, _randint(g, n, src.numel()))
        if case["shuffled"]:
            perm = torch.randperm(n, generator=g, device="cuda")
            src, dst = perm[src], perm[dst]
    else:  # cliques of consecutive ids, with some random columns per row
        sizes = 4 + _poisson(g, max(case["size"] - 4.0, 0.0), int(n / case["size"] * 1.3) + 16)
        ends = torch.cumsum(sizes, 0)
        ids = torch.arange(n, device="cuda")
        of = torch.clamp(torch.searchsorted(ends, ids, right=True), max=sizes.numel() - 1)
        first = torch.clamp((ends - sizes)[of], max=n - 1)
        size = torch.clamp(torch.minimum(ends[of], torch.full_like(ids, n)) - first, min=1)
        src = torch.repeat_interleave(ids, size)
        start = torch.cumsum(size, 0) - size
        dst = first[src] + (torch.arange(src.numel(), device="cuda") - start[src])
        extra = torch.poisson(case["noise"] * size.float(), generator=g).long()
        src2 = torch.repeat_interleave(ids, extra)
        src, dst = torch.cat([src, src2]), torch.cat([dst, _randint(g, n, src2.numel())])
    rowptr, colidx = _csr(n, src, dst, _kept(case), g)
    del src, dst
    deg = (rowptr[1:] - rowptr[:-1]).long()
    if gcn:
        indeg = torch.clamp(torch.bincount(colidx, minlength=n), min=1).float()
        out = torch.clamp(deg, min=1).float()
        vals = torch.rsqrt(torch.repeat_interleave(out, deg) * indeg[colidx.long()])
    else:
        vals = torch.repeat_interleave(1.0 / torch.clamp(deg, min=1).float(), deg)
    return rowptr, colidx, vals


def _rmat_edges(g, n, edges):
    scale, count = max(1, (n - 1).bit_length()), n * edges
    src = torch.zeros(count, dtype=torch.int64, device="cuda")
    dst = torch.zeros(count, dtype=torch.int64, device="cuda")
    for _ in range(scale):
        r = _rand(g, count)
        sbit = r >= RMAT_A + RMAT_B
        dbit = ((r >= RMAT_A) & ~sbit) | (r >= RMAT_A + RMAT_B + RMAT_C)
        src.mul_(2).add_(sbit)
        dst.mul_(2).add_(dbit)
    if n != 1 << scale:  # other sizes: ids are scaled down to [0, n)
        src, dst = (src * n) >> scale, (dst * n) >> scale
    return src, dst


def _road_edges(g, n, width, draw_mean):
    """Jittered grid, row-major ids; a node links to its Poisson(draw_mean) nearest neighbours
    among the 8 surrounding cells, both ways."""
    height = n // width
    ids = torch.arange(n, device="cuda")
    x, y = ids % width, torch.div(ids, width, rounding_mode="floor")
    jx, jy = (_rand(g, n) - 0.5) * 0.8, (_rand(g, n) - 0.5) * 0.8
    m = _poisson(g, draw_mean, n)
    near, other = [], []
    for dx, dy in ((-1, -1), (0, -1), (1, -1), (-1, 0), (1, 0), (-1, 1), (0, 1), (1, 1)):
        nx, ny = x + dx, y + dy
        ok = (nx >= 0) & (nx < width) & (ny >= 0) & (ny < height)
        nid = torch.where(ok, ny * width + nx, 0)
        d2 = (dx + jx[nid] - jx) ** 2 + (dy + jy[nid] - jy) ** 2
        near.append(torch.where(ok, d2, math.inf))
        other.append(nid)
    near, order = torch.sort(torch.stack(near, 1), dim=1, stable=True)
    other = torch.gather(torch.stack(other, 1), 1, order)
    take = (torch.arange(8, device="cuda")[None, :] < m[:, None]) & torch.isfinite(near)
    u, v = ids[:, None].expand(n, 8)[take], other[take]
    return torch.cat([u, v]), torch.cat([v, u])


# ------------------------------------------------------------------------------ passes
def _select_and_build(rowptr, colidx, vals, n, K):
    p = pc.pcsr_select(pc.pcsr_features(n, n, rowptr, colidx), K)
    return pc.pcsr_build(n, n, rowptr, colidx, vals, p)


def prepare(case, seed):
    n, kind = case["n"], case["kind"]
    rowptr, colidx, vals = _graph(case, seed)
    g = _gen(seed + 0x5EED)
    s = dict(case, rowptr=rowptr, colidx=colidx, vals=vals)
    if kind == "spmm":
        s["handle"] = _select_and_build(rowptr, colidx, vals, n, case["K"])
        pc.pcsr_reserve_workspace(s["handle"], case["K"])
        for name in ("rowptr", "colidx", "vals"):  # the handle owns its own arrays
            del s[name]
        s["B"] = torch.randn(n, case["K"], generator=g, device="cuda")
        s["C"] = torch.empty(n, case["K"], device="cuda")
    elif kind == "fresh":
        s["B"] = torch.randn(n, case["K"], generator=g, device="cuda")
    else:
        host = [t.cpu().numpy() for t in (rowptr, colidx, vals)]
        s["rowptr"], s["colidx"], s["vals"] = host
        if kind == "operator":
            s["B"] = torch.randn(n, case["K"], generator=g, device="cuda").requires_grad_(True)
            s["dC"] = torch.randn(n, case["K"], generator=g, device="cuda")
        elif kind == "train":
            op = PcsrOperator(n, n, *host, symmetric=_symmetric(case), K_hint=case["hidden"])
            torch.manual_seed(seed)
            s["model"] = make_model(case["model"], op, case["features"], case["hidden"], case["features"],
                                    case["layers"]).cuda()
            s["X"] = torch.randn(n, case["features"], generator=g, device="cuda")
            s["Y"] = torch.randn(n, case["features"], generator=g, device="cuda")
    return s


def run(s):
    kind, n = s["kind"], s["n"]
    if kind == "spmm":
        pc.pcsr_spmm(s["handle"], s["B"], s["C"], s["K"], torch.cuda.current_stream())
        return s["C"]
    if kind == "fresh":
        h = _select_and_build(s["rowptr"], s["colidx"], s["vals"], n, s["K"])
        C = torch.empty(n, s["K"], device="cuda")
        stream = torch.cuda.current_stream()
        pc.pcsr_spmm(h, s["B"], C, s["K"], stream)
        stream.synchronize()  # the handle may only be freed once its product is done
        h.close()
        return C
    if kind == "operator":
        op = PcsrOperator(n, n, s["rowptr"], s["colidx"], s["vals"], K_hint=s["K"])
        B = s["B"].detach().requires_grad_(True)
        C = op(B)
        C.backward(s["dC"])
        torch.cuda.current_stream().synchronize()  # the operator goes out of scope here
        return [C.detach(), B.grad]
    if kind == "reorder":
        if s["by"] == "degree":
            perm = pc.pcsr_reorder_by_degree(n, s["rowptr"], s["colidx"])
        else:
            perm, _ = pc.pcsr_reorder(n, s["rowptr"], s["colidx"])
        return [perm, *pc.pcsr_permute_csr(n, s["rowptr"], s["colidx"], s["vals"], perm)]
    model = s["model"]
    model.zero_grad(set_to_none=True)
    out = model(s["X"])
    torch.nn.functional.mse_loss(out, s["Y"]).backward()
    return [out.detach(), *(p.grad for p in model.parameters())]


# ------------------------------------------------------------------------------ work
def _symmetric(case):
    """Whether the drawn matrix equals its transpose."""
    return case["graph"] == "road" or (case["graph"] == "rmat" and case["symmetric"])


def _mean_degree(case):
    kind = case["graph"]
    if kind in ("poisson", "sbm"):
        return case["deg"]
    if kind == "road":
        return 1.43 * case["deg"]
    if kind == "rmat":
        return case["edges"] * (2.0 if case["symmetric"] else 1.0)
    # the clique a node is in: E[s^2]/E[s] with s = 4 + Poisson(size - 4)
    return case["size"] + (case["size"] - 4.0) / case["size"] + case["noise"] * case["size"]


def _expected(case):
    """Expected (nonzeros, referenced columns) after duplicates are dropped."""
    n, kind = case["n"], case["graph"]
    if kind == "road":
        return n * _mean_degree(case), n * 0.99
    if kind == "sbm":
        b, lam = min(case["block"], n), case["deg"] * case["intra"]
        nnz = n * (b * -math.expm1(-lam / b) + case["deg"] - lam)
        return nnz, n * -math.expm1(-nnz / n)
    if kind == "rmat":
        scale, draws = max(1, (n - 1).bit_length()), n * case["edges"] * (2.0 if case["symmetric"] else 1.0)
        d, cells, cols = 1.0 - RMAT_A - RMAT_B - RMAT_C, 0.0, 0.0
        for i in range(scale + 1):  # i zero bits of a pair, j bits in one of the two off-diagonal quadrants
            for j in range(scale - i + 1):
                k = scale - i - j
                p = RMAT_A ** i * RMAT_B ** j * d ** k
                cells += math.comb(scale, i) * math.comb(scale - i, j) * 2.0 ** j * -math.expm1(-draws * p)
            p = (RMAT_A + RMAT_C) ** i * (RMAT_B + d) ** (scale - i)
            cols += math.comb(scale, i) * -math.expm1(-draws * p)
        return cells, cols * n / (1 << scale)
    if kind == "poisson":
        return n * n * -math.expm1(-case["deg"] / n), n * -math.expm1(-case["deg"])
    return n * _mean_degree(case), float(n)


def _kept(case):
    """The relabelled matrix is an output: its number of nonzeros is the same for every seed (a
    random part of those drawn), everywhere else it varies."""
    return int(0.85 * _expected(case)[0]) if case["kind"] == "reorder" else None


def _spmm_work(n, nnz, refs, K):
    """A, every referenced row of B and C, each once; one multiply-add per nonzero and column."""
    return nnz * 8.0 + (n + 1) * 4.0 + (refs + n) * K * 4.0, 2.0 * nnz * K


def work(case):
    n, kind = case["n"], case["kind"]
    nnz, refs = _expected(case)
    nnz = _kept(case) or nnz
    csr = nnz * 8.0 + (n + 1) * 4.0
    if kind in ("spmm", "fresh"):
        b, f = _spmm_work(n, nnz, refs, case["K"])
        return dict(bytes=b, flops=f)
    if kind == "operator":  # A once, B and dC in, C and dB out
        b, f = _spmm_work(n, nnz, refs, case["K"])
        return dict(bytes=b + n * case["K"] * 8.0, flops=2 * f)
    if kind == "reorder":  # pattern in (values too for the permuted matrix), matrix and permutation out
        return dict(bytes=2 * csr + n * 4.0, flops=0)
    # Training.  A layer's output exceeds what the caches keep, so each aggregation has to read
    # its operand and write its result, forward and backward, and each dense layer likewise;
    # the first layer needs no gradient of its input.
    dims = [case["features"]] + [case["hidden"]] * (case["layers"] - 1) + [case["features"]]
    total, flops = 0.0, 0.0
    for i in range(case["layers"]):
        a, b = dims[i], dims[i + 1]
        agg = min(a, b) if case["model"] == "gcn" else a
        dense = [(a, b)] if case["model"] == "gcn" else [(a, b), (b, b)]
        times = 1 if i == 0 and (case["model"] == "gin" or a < b) else 2
        by, fl = _spmm_work(n, nnz, refs, agg)
        total, flops = total + times * by, flops + times * fl
        for p, q in dense:
            total += n * (p + q) * 4.0 * 2.0
            flops += 2.0 * n * p * q * 3.0
    return dict(bytes=total, flops=flops)


def tolerance(case):
    if case["kind"] == "reorder":
        return "exact"
    if case["kind"] == "train":
        # 32-bit sums in every layer, and weight gradients that add up to a few million rows
        return {"rel": 1e-4, "max": 2e-2}
    return {"rel": 1e-5, "max": 1e-3}
