"""Relabelling, transpose and window blocks on the GPU against numpy restatements and the host
builder: the integers and bytes have to be the same."""
import numpy as np
import pytest

import paper_2605_15695_amd as pc
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _mix(x, r):
    x = x.astype(np.uint64)
    m = np.uint64(0xffffffff)
    x ^= np.uint64((r * 0x9E3779B9) & 0xffffffff)
    x ^= x >> np.uint64(16)
    x = (x * np.uint64(0x7feb352d)) & m
    x ^= x >> np.uint64(15)
    x = (x * np.uint64(0x846ca68b)) & m
    x ^= x >> np.uint64(16)
    return x


def _label_propagation(n, rp, ci, rounds=8):
    """Most frequent neighbour label; ties: the node's own, else the smallest salted hash."""
    rows = np.repeat(np.arange(n), np.diff(rp))
    lab = np.arange(n)
    for r in range(rounds):
        key, cnt = np.unique(rows * np.int64(n) + lab[ci], return_counts=True)
        row, label = key // n, key % n
        order = np.lexsort((_mix(label, r), label != lab[row], -cnt, row))
        first = np.ones(order.size, bool)
        first[1:] = row[order][1:] != row[order][:-1]
        nxt = lab.copy()
        nxt[row[order][first]] = label[order][first]
        moved = int((nxt != lab).sum())
        lab = nxt
        if moved * 200 < n:
            break
    perm = np.empty(n, np.int32)
    perm[np.argsort(lab, kind="stable")] = np.arange(n)
    return perm, np.unique(lab).size


def _case(name):
    if name == "sbm":
        g = synth.sbm(12_000, 24, mean_deg=40.0, shuffled=True)
        return g.n_rows, g.rowptr, g.colidx, g.vals
    if name == "power":                     # rows of every class, the longest over several passes
        g = synth.rmat(14, 24, symmetric=True, permute=True)
        return g.n_rows, g.rowptr, g.colidx, g.vals
    rng = np.random.default_rng(3)          # a few rows with nearly every column, many empty ones
    n = 30_011
    lengths = np.where(rng.random(n) < 0.6, 0, rng.integers(0, 20, n))
    lengths[[5, 77, n - 1]] = [n, 25_000, 9_000]
    lengths[100:140] = [64, 65] * 10 + [1024, 1025] * 10
    rp = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    ci = np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in lengths if k]).astype(np.int32)
    return n, rp, ci, rng.standard_normal(ci.size).astype(np.float32)


@pytest.mark.parametrize("name", ["sbm", "power", "uneven"])
def test_reorder_permute_transpose(name):
    n, rp, ci, va = _case(name)
    assert ci.size >= 200_000               # enough for the GPU side to be taken
    for rounds in (0, 3):
        perm, clusters = pc.pcsr_reorder(n, rp, ci, rounds)
        ref, ref_clusters = _label_propagation(n, rp, ci, rounds or 8)
        assert clusters == ref_clusters and np.array_equal(perm, ref)
    refs = np.bincount(ci, minlength=n)
    by_degree = np.empty(n, np.int32)
    by_degree[np.argsort(-refs, kind="stable")] = np.arange(n)
    assert np.array_equal(pc.pcsr_reorder_by_degree(n, rp, ci), by_degree)

    rows = np.repeat(np.arange(n), np.diff(rp))
    order = np.lexsort((perm[ci], perm[rows]))
    got = pc.pcsr_permute_csr(n, rp, ci, va, perm)
    assert np.array_equal(got[0], np.concatenate([[0], np.cumsum(np.bincount(perm[rows], minlength=n))]))
    assert np.array_equal(got[1], perm[ci][order]) and np.array_equal(got[2].view(np.uint32), va[order].view(np.uint32))

    for m in (n, n + 1000):                 # a rectangular one with empty columns at the end
        order = np.lexsort((rows, ci))
        t = pc.pcsr_transpose_csr(n, m, rp, ci, va)
        assert np.array_equal(t[0], np.concatenate([[0], np.cumsum(np.bincount(ci, minlength=m))]))
        assert np.array_equal(t[1], rows[order]) and np.array_equal(t[2].view(np.uint32), va[order].view(np.uint32))


@pytest.mark.parametrize("longest", [63, 64, 65, 1024, 1025, 8192, 8193])
@pytest.mark.parametrize("twice", [False, True])
def test_permuted_rows_of_every_class(longest, twice):
    """Rows up to and beyond what a wavefront, a workgroup and LDS sort, and a column that comes twice in one of them."""
    rng = np.random.default_rng(longest)
    n = 10_001
    lengths = rng.integers(0, 45, n)
    lengths[[0, 4000, n - 1]] = [longest, 0, longest]
    rp = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    ci = np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in lengths]).astype(np.int32)
    assert ci.size >= 200_000               # enough for the GPU side to be taken
    va = rng.standard_normal(ci.size).astype(np.float32)
    if twice:
        ci[longest - 1] = ci[longest // 2]
    perm = rng.permutation(n).astype(np.int32)
    rows = np.repeat(np.arange(n), lengths)
    order = np.lexsort((va, perm[ci], perm[rows]))
    got = pc.pcsr_permute_csr(n, rp, ci, va, perm)
    assert np.array_equal(got[0], np.concatenate([[0], np.cumsum(np.bincount(perm[rows], minlength=n))]))
    assert np.array_equal(got[1], perm[ci][order])
    at = np.repeat(np.arange(n), np.diff(got[0]))
    if twice:                               # which of the two comes first is not said
        assert np.array_equal(got[2][np.lexsort((got[2], got[1], at))], va[order])
    else:
        assert np.array_equal(got[2].view(np.uint32), va[order].view(np.uint32))


@pytest.mark.parametrize("n,m,nnz,kind", [
    (250_001, 250_007, 1_500_001, ""), (3, 2, 1 << 20, ""), (5000, 3, 1_100_000, ""), (70_000, 1 << 20, (1 << 20) + 1, ""),
    (70_000, 1000, (1 << 18) - 1, ""), (70_000, 1000, 1 << 18, ""),  # around the least it is used for
    (70_000, (1 << 20) + 1, (1 << 20) + 1, ""),     # one bit more than two passes take
    ((1 << 22) - 5, 1_000_000, 1_200_000, "gap"),   # more rows than a tile looks at between two nonzeros
    ((1 << 22) + 5, 1_000_000, 1_200_000, ""),      # rows too many for the word beside the digit
    (100_000, 100_000, 1_300_000, "hub"), (8192, 1025, 1 << 20, "last"), (4096, 512, (1 << 20) - 1, ""),
])
def test_transpose_of_every_size(n, m, nnz, kind):
    """Columns of 1 to 21 bits, tiles that are full to the last nonzero and one over, rows of any length, a column with half
    of the nonzeros, a column that comes more than once in a row (in its order there)."""
    rng = np.random.default_rng(nnz + m)
    rows = np.sort(rng.integers(0, n, nnz))
    if kind == "gap":
        rows[:nnz // 2] //= 1000
        rows = np.sort(rows)
    ci = rng.integers(0, m, nnz).astype(np.int32)
    if kind == "hub":
        ci[rng.random(nnz) < 0.5] = m // 3
    if kind == "last":
        ci[:] = m - 1
    ci = ci[np.lexsort((ci, rows))]
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int32)
    va = rng.standard_normal(nnz).astype(np.float32)
    order = np.argsort(ci, kind="stable")
    got = pc.pcsr_transpose_csr(n, m, rp, ci, va)
    assert np.array_equal(got[0], np.concatenate([[0], np.cumsum(np.bincount(ci, minlength=m))]))
    assert np.array_equal(got[1], rows[order]) and np.array_equal(got[2].view(np.uint32), va[order].view(np.uint32))


def test_refusals_are_those_of_the_host():
    n, rp, ci, va = _case("sbm")
    bad = ci.copy()
    bad[150_000] = n
    for call in (lambda: pc.pcsr_reorder(n, rp, bad), lambda: pc.pcsr_reorder_by_degree(n, rp, bad),
                 lambda: pc.pcsr_permute_csr(n, rp, bad, va, np.arange(n, dtype=np.int32)),
                 lambda: pc.pcsr_transpose_csr(n, n, rp, bad, va)):
        with pytest.raises(pc.PcsrError) as e:
            call()
        assert e.value.code == pc.binding.PCSR_E_BAD_CSR
    perm = np.arange(n, dtype=np.int32)
    perm[7] = 8
    with pytest.raises(pc.PcsrError) as e:
        pc.pcsr_permute_csr(n, rp, ci, va, perm)
    assert e.value.code == pc.binding.PCSR_E_INVALID_ARG


@pytest.mark.parametrize("wc", [256, 512, 1024, 2048])
@pytest.mark.parametrize("V", [1, 2])
@pytest.mark.parametrize("name", ["sbm", "sbm_shuffled", "cliques", "road", "uneven"])
def test_windows_are_those_of_the_host_builder(name, V, wc):
    if name == "uneven":
        n, rp, ci, va = _case("uneven")
    else:
        g = {"sbm": lambda: synth.sbm(20_000, 40, mean_deg=50.0),
             "sbm_shuffled": lambda: synth.sbm(12_000, 24, shuffled=True),
             "cliques": lambda: synth.cliques(20_011, 40.0, 0.3, 5),
             "road": lambda: synth.road_grid(307, 251)}[name]()
        n, rp, ci, va = g.n_rows, g.rowptr, g.colidx, g.vals
    host = pc.pcsr_build(n, n, rp, ci, va, pc.make_params(V=V, col_window=wc, flags=pc.PCSR_FLAG_HOST_ONLY))
    dev = pc.pcsr_build(n, n, *(torch.from_numpy(x).cuda() for x in (rp, ci, va)), pc.make_params(V=V, col_window=wc))
    assert pc.pcsr_window_stats(host) == pc.pcsr_window_stats(dev)
    B = torch.from_numpy(synth.dense_operand(n, 16, "normal", 2)).cuda()
    C = torch.full((n, 16), float("nan"), device="cuda")
    if wc == 2048:                          # the auto slice of this window exceeds the LDS
        pc.pcsr_set_kernel_params(dev, 4, 2, 1, 16)
    pc.pcsr_spmm(dev, B, C, 16)
    plain = pc.pcsr_build(n, n, rp, ci, va, pc.make_params(V=V))
    D = torch.empty_like(C)
    pc.pcsr_spmm(plain, B, D, 16)
    assert float((C - D).norm() / D.norm()) < 1e-6
    host.close(), dev.close(), plain.close()


def _window_case(name, wc, rng):
    """Rows whose densest window is where the search for it can go wrong."""
    n, m = 600, 40 * wc
    if name == "wide":                      # more stretches of wc columns than the search counts in LDS
        m = 6200 * wc + 7
    rows = []
    for i in range(n):
        g = i // 150                        # blocks of 150 rows
        if name == "ties":                  # the same columns in four places, two of them side by side
            base = rng.choice(wc // 2, 10, replace=False)
            c = np.concatenate([base + k * wc for k in (3 * g, 3 * g + 1, 20, 33)])
        elif name == "edges":               # runs of wc - 1, wc and wc + 1 columns across a multiple of wc, both ends
            first = (0, 5 * wc - 1, 9 * wc + 1 - wc // 2, m - wc - 1)[g]
            c = np.concatenate([first + rng.choice(wc - 1, 30, replace=False), [first, first + wc + (g % 3) - 2]])
        elif name == "scattered":           # no window stands out
            c = rng.choice(m, 20, replace=False)
        else:
            c = np.concatenate([(m // 5) * (g + 1) + rng.choice(wc, 40, replace=False), rng.choice(m, 5)])
        rows.append(np.unique(c))
    rp = np.concatenate([[0], np.cumsum([len(c) for c in rows])]).astype(np.int32)
    ci = np.concatenate(rows).astype(np.int32)
    return n, m, rp, ci, rng.standard_normal(ci.shape[0]).astype(np.float32)


@pytest.mark.parametrize("wc", [256, 2048])
@pytest.mark.parametrize("name", ["ties", "edges", "scattered", "wide"])
def test_window_search_at_its_edges(name, wc):
    n, m, rp, ci, va = _window_case(name, wc, np.random.default_rng(wc))
    host = pc.pcsr_build(n, m, rp, ci, va, pc.make_params(col_window=wc, flags=pc.PCSR_FLAG_HOST_ONLY))
    dev = pc.pcsr_build(n, m, *(torch.from_numpy(x).cuda() for x in (rp, ci, va)), pc.make_params(col_window=wc))
    assert pc.pcsr_window_stats(host) == pc.pcsr_window_stats(dev)
    B = torch.from_numpy(synth.dense_operand(m, 8, "normal", 2)).cuda()
    C = torch.full((n, 8), float("nan"), device="cuda")
    pc.pcsr_set_kernel_params(dev, 4, 2, 1, 16)
    pc.pcsr_spmm(dev, B, C, 8)
    plain = pc.pcsr_build(n, m, rp, ci, va, pc.make_params())
    D = torch.empty_like(C)
    pc.pcsr_spmm(plain, B, D, 8)
    assert float((C - D).norm() / D.norm()) < 1e-6
    host.close(), dev.close(), plain.close()


def test_operator_takes_device_arrays_and_refuses_bad_ones():
    from paper_2605_15695_amd.gnn import PcsrOperator

    n, rp, ci, va = _case("power")
    a = PcsrOperator(n, n, rp, ci, va, K_hint=32)
    b = PcsrOperator(n, n, *(torch.from_numpy(x).cuda() for x in (rp, ci, va)), K_hint=32)
    B = torch.from_numpy(synth.dense_operand(n, 32, "normal", 2)).cuda()
    assert torch.equal(a(B), b(B))
    assert torch.equal(a._run(a.bwd, n, B), b._run(b.bwd, n, B))
    bad = ci.copy()
    bad[3] = bad[2]
    with pytest.raises(pc.PcsrError) as e:
        PcsrOperator(n, n, rp, bad, va)
    assert e.value.code == pc.binding.PCSR_E_BAD_CSR


@pytest.mark.parametrize("shared", ["rowptr", "colidx", "vals", "all inputs"])
def test_permuted_matrix_may_take_the_place_of_its_inputs(shared):
    """Outputs in memory that an input is read from, the values among them, which are uploaded beside the work."""
    rng = np.random.default_rng(5)
    n = 1_300_000
    lengths = rng.integers(1, 3, n)                       # more row pointers than a copying thread is done with at once
    rp = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    ci = rng.integers(0, n // 2, n)
    ci = np.stack([ci, ci + 1 + rng.integers(0, n // 2 - 1, n)], 1)[np.arange(2)[None, :] < lengths[:, None]].astype(np.int32)
    va = rng.standard_normal(ci.size).astype(np.float32)
    perm = rng.permutation(n).astype(np.int32)
    want = pc.pcsr_permute_csr(n, rp, ci, va, perm)
    at = va.copy()                                        # the values' own memory, for an output or two
    ins = [rp.copy(), ci.copy(), at]
    outs = [np.empty_like(x) for x in want]
    if shared == "rowptr":
        outs[0] = at.view(np.int32)[-(n + 1):]
    elif shared == "colidx":
        outs[1] = at.view(np.int32)
    elif shared == "vals":
        outs[2] = at
    else:
        outs = ins
    rc = pc.binding._lib().pcsr_permute_csr(n, *(x.ctypes.data for x in ins), perm.ctypes.data, *(x.ctypes.data for x in outs))
    assert rc == 0
    for k in range(3):
        assert np.array_equal(outs[k].view(np.uint32), want[k].view(np.uint32)), k
