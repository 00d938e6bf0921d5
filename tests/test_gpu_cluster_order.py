"""PCSR_FLAG_CLUSTER_IF_USEFUL: rows of communities with shuffled ids run side by side, and everything else stays as it
is without the flag."""
import numpy as np
import pytest

import oracle
import paper_2605_15695_amd as pc
from tests.helpers import column_ordered_schedule

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
FLAG = pc.PCSR_FLAG_CLUSTER_IF_USEFUL


def _planted(n, block, inner, outer, seed, extra=()):
    """Rows with `inner` columns in their own block of `block` nodes and `outer` anywhere, ids shuffled; extra: (row,
    length) of rows with that many uniform columns in place of their own."""
    rng = np.random.default_rng(seed)
    of = rng.permutation(n) // block
    members = [np.nonzero(of == b)[0] for b in range(int(of.max()) + 1)]
    rows = []
    for i in range(n):
        own = members[of[i]]
        rows.append(np.unique(np.concatenate([rng.choice(own, min(inner, own.shape[0]), replace=False),
                                              rng.integers(0, n, outer)])))
    for r, length in extra:
        rows[r] = np.sort(rng.choice(n, length, replace=False))
    rp = np.concatenate([[0], np.cumsum([len(c) for c in rows])]).astype(np.int32)
    ci = np.concatenate(rows).astype(np.int32)
    return n, rp, ci, rng.standard_normal(ci.shape[0]).astype(np.float32), of


def _device(*arrays):
    return [torch.from_numpy(a).cuda() for a in arrays]


def _check_product(h, n, rp, ci, va, K):
    B = np.random.default_rng(K).uniform(-1, 1, (n, K)).astype(np.float32)
    C = torch.full((n, K), float("nan"), device="cuda")
    pc.pcsr_spmm(h, torch.from_numpy(B).cuda(), C, K)
    ref, bound = oracle.spmm(rp, ci, va, B)
    ok, worst = oracle.within_tolerance(C.cpu().numpy(), ref, bound)
    assert ok, (K, worst)


@pytest.mark.parametrize("S", [0, 1])
@pytest.mark.parametrize("n,block,inner,outer,extra", [
    (6001, 100, 20, 2, ()),                                   # blocks of 100, rows of about 22
    (5003, 50, 40, 6, ((7, 0), (8, 1), (5002, 0), (4000, 3))),  # empty and short rows among them
    (8192, 512, 30, 5, ((0, 1025), (5, 1024), (8191, 4000))),   # rows longer than an item
])
def test_rows_of_a_community_run_side_by_side(n, block, inner, outer, extra, S):
    n, rp, ci, va, of = _planted(n, block, inner, outer, n, extra)
    prm = pc.make_params(S=S, SG=32 if S else 0, flags=FLAG | (pc.PCSR_FLAG_COLUMN_ORDER if S else 0),
                         lanes_per_row=16, vec=2)
    h = pc.pcsr_build(n, n, *_device(rp, ci, va), prm)
    e, got = pc.pcsr_export(h), pc.pcsr_export_schedule(h)
    sched, xb = got["sched"], got["xcd_bounds"]
    assert e["SG"] == 1024 and np.array_equal(e["colidx"], ci) and np.array_equal(e["val"], va)
    lengths = np.diff(rp)
    assert e["M"] == int(np.maximum(1, -(-lengths // 1024)).sum()) == sched.shape[0]
    # every item once, and where it was
    order = np.lexsort((sched[:, 0], sched[:, 2]))
    items = np.lexsort((e["rowptr"][:-1], e["trow"]))
    assert np.array_equal(sched[order, 0][lengths[sched[order, 2]] > 0], e["rowptr"][:-1][items][lengths[e["trow"][items]] > 0])
    assert np.array_equal(np.bincount(sched[:, 2], weights=sched[:, 1], minlength=n).astype(int), lengths)
    # positions one after another within an XCD's range mostly belong to one community: its own rows and at most a few others
    # that its key is shared with
    runs = 0
    for x in range(8):
        rows = sched[xb[x]:xb[x + 1], 2]
        c = of[rows[sched[xb[x]:xb[x + 1], 3] < 0]]
        for k in range(0, c.shape[0] - block, block):
            runs += np.unique(c[k:k + block], return_counts=True)[1].max() >= 0.3 * block
    assert runs >= 0.8 * (n // block - 16)
    work = np.add.reduceat(sched[:, 1] + 8, xb[:-1])
    assert work.max() - work.min() <= 2 * (1024 + 8)
    again = pc.pcsr_build(n, n, *_device(rp, ci, va), prm)
    assert np.array_equal(pc.pcsr_export_schedule(again)["sched"], sched)
    for K in (1, 7, 16, 33, 64, 100, 256, 300, 516):
        _check_product(h, n, rp, ci, va, K)
    h.close(), again.close()


def test_shape_is_chosen_for_the_order_the_build_found():
    n, rp, ci, va, _ = _planted(6001, 100, 20, 2, 1)
    h = pc.pcsr_build(n, n, *_device(rp, ci, va), pc.make_params(flags=FLAG, lanes_per_row=32, vec=2, rep=1, waves_per_wg=2))
    for K, shape in ((64, (16, 4, 1)), (128, (32, 4, 1)), (256, (64, 4, 1)), (512, (64, 4, 2)), (2048, (64, 4, 2))):
        q = pc.pcsr_query_kernel(h, K)
        assert (q["lanes_per_row"], q["vec"], q["rep"], q["waves_per_wg"]) == shape + (4,)
    h.close()


def _uniform(n, m, k, seed):
    rng = np.random.default_rng(seed)
    ci = np.sort(np.argsort(rng.random((n, m)), axis=1)[:, :k].astype(np.int32), axis=1).ravel()
    return np.arange(0, n * k + 1, k, dtype=np.int32), ci, rng.standard_normal(ci.shape[0]).astype(np.float32)


@pytest.mark.parametrize("name", ["uniform", "one_clique", "rectangular", "paired", "empty"])
def test_nothing_changes_without_communities(name):
    n = m = 3000
    V = 2 if name == "paired" else 1
    if name == "uniform":
        rp, ci, va = _uniform(n, n, 20, 1)
    elif name == "one_clique":                       # every row the same columns: one label for all
        rp, ci, va = _uniform(1, n, 24, 2)
        rp, ci, va = np.arange(0, 24 * n + 1, 24, dtype=np.int32), np.tile(ci, n), np.tile(va, n)
    elif name == "rectangular":
        _, rp, ci, va, _ = _planted(n, 100, 20, 2, 3)
        m = n + 1
    elif name == "paired":
        _, rp, ci, va, _ = _planted(n, 100, 20, 2, 4)
    else:
        rp, ci, va = np.zeros(n + 1, np.int32), np.zeros(0, np.int32), np.zeros(0, np.float32)
    for S in (0, 1):
        flags = pc.PCSR_FLAG_COLUMN_ORDER if S else 0
        a, b = (pc.pcsr_build(n, m, *_device(rp, ci, va), pc.make_params(V=V, S=S, SG=8 if S else 0, flags=flags | f))
                for f in (0, FLAG))
        x, y = pc.pcsr_export(a), pc.pcsr_export(b)
        assert all(np.array_equal(x[k], y[k]) for k in x)
        x, y = pc.pcsr_export_schedule(a), pc.pcsr_export_schedule(b)
        assert np.array_equal(x["xcd_bounds"], y["xcd_bounds"])
        assert (x["sched"] is None) == (y["sched"] is None) and (not S or np.array_equal(x["sched"], y["sched"]))
        if S and n == m and ci.size:
            sched, _ = column_ordered_schedule(pc.pcsr_export(b)["rowptr"], pc.pcsr_export(b)["colidx"],
                                               pc.pcsr_export(b)["trow"], pc.pcsr_export(b)["P"])
            assert np.array_equal(y["sched"], sched)
        a.close(), b.close()


def test_a_training_layer_on_such_an_operator():
    """Forward and backward at several widths."""
    from paper_2605_15695_amd.gnn import PcsrOperator

    n, rp, ci, va, _ = _planted(6001, 100, 20, 2, 9)
    prm = pc.make_params(flags=FLAG)
    a = PcsrOperator(n, n, *_device(rp, ci, va), params=prm)
    b = PcsrOperator(n, n, *_device(rp, ci, va), params=pc.make_params())
    assert pc.pcsr_export(a.fwd)["SG"] == 1024
    for K in (16, 30, 128, 600):
        X = torch.randn(n, K, device="cuda")
        x, y = X.clone().requires_grad_(True), X.clone().requires_grad_(True)
        u, v = a(x), b(y)
        u.backward(X), v.backward(X)
        for got, want in ((u.detach(), v.detach()), (x.grad, y.grad)):
            assert float((got - want).norm() / want.norm()) < 1e-6


def test_selector_asks_where_one_product_pays_for_the_search():
    f = np.zeros(len(pc.FEATURE_NAMES))
    f[0] = f[1] = 250_000
    f[2], f[4], f[5], f[6], f[7], f[15], f[16] = 12e6, 48.0, 48.0, 80.0, 0.15, 0.5, 0.004
    assert not pc.pcsr_select(f, 64).flags & FLAG and pc.pcsr_select(f, 128).flags & FLAG
    f[2], f[4], f[5] = 3e6, 12.0, 12.0                          # rows of 12: from K = 334 on
    assert not pc.pcsr_select(f, 256).flags & FLAG and pc.pcsr_select(f, 512).flags & FLAG
    f[16] = 0.5                                                # local columns
    assert not pc.pcsr_select(f, 512).flags & FLAG


WINDOWS = pc.PCSR_FLAG_CLUSTER_WINDOWS


@pytest.mark.parametrize("n,block,inner,outer,extra,windows", [
    (6001, 100, 20, 2, (), True),                                    # several communities to a block of the product
    (5003, 50, 40, 6, ((7, 0), (8, 1), (5002, 0), (4000, 3)), True),  # empty and short rows among them
    (5003, 256, 50, 3, (), True), (5003, 257, 50, 3, (), True),      # the largest that shares a block, the smallest alone
    (8192, 512, 60, 0, (), True), (8210, 513, 60, 1, (), True),      # a block's most rows, a community of two pieces
    (6000, 700, 60, 1, (), None), (20000, 1000, 40, 2, (), False),   # ever fewer vectors inside
    (8192, 512, 30, 5, ((5, 1024), (8191, 1000)), True),             # the longest rows that are one item
    (8192, 512, 30, 5, ((5, 1025),), False),                         # one of two items
])
def test_windows_of_communities(n, block, inner, outer, extra, windows):
    n, rp, ci, va, _ = _planted(n, block, inner, outer, n + block, extra)
    arrays = _device(rp, ci, va)
    plain, h = (pc.pcsr_build(n, n, *arrays, pc.make_params(flags=FLAG | f)) for f in (0, WINDOWS))
    x, y = pc.pcsr_export(plain), pc.pcsr_export(h)
    assert y["SG"] == 1024 and all(np.array_equal(x[k], y[k]) for k in x)
    has = pc.pcsr_query_launch(h, 64)["lds_bytes"] > 0
    assert windows is None or has == windows
    for K in (60, 64, 66, 68, 100, 256, 300, 516):
        q = pc.pcsr_query_launch(h, K)
        assert (q["lds_bytes"] > 0) == (has and K % 4 == 0 and K >= 64)
        _check_product(h, n, rp, ci, va, K)
    # a row of B reaches the rows that refer to it and no others, NaN included
    K, j = 64, int(ci[rp[n // 2]])
    B = torch.randn(n, K, device="cuda")
    B[j] = float("nan")
    C = torch.empty(n, K, device="cuda")
    pc.pcsr_spmm(h, B, C, K)
    refer = np.zeros(n, bool)
    refer[np.repeat(np.arange(n), np.diff(rp))[ci == j]] = True
    assert np.array_equal(torch.isnan(C).any(1).cpu().numpy(), refer) and np.array_equal(torch.isnan(C).all(1).cpu().numpy(), refer)
    # the same bits on another build, in the hardware's order of workgroups and with the caller's own shape once it is taken back
    again = pc.pcsr_build(n, n, *arrays, pc.make_params(flags=FLAG | WINDOWS))
    D = torch.empty(n, K, device="cuda")
    pc.pcsr_set_kernel_params(again, lanes_per_row=16, vec=4, rep=1)
    assert pc.pcsr_query_launch(again, K)["lds_bytes"] == 0
    pc.pcsr_spmm(again, B.nan_to_num(), D, K)
    E = torch.empty_like(D)
    pc.pcsr_spmm(plain, B.nan_to_num(), E, K)
    assert torch.equal(D, E)
    pc.pcsr_set_kernel_params(again, flags=pc.PCSR_FLAG_NO_XCD_REMAP)
    pc.pcsr_spmm(again, B, D, K)
    assert torch.equal(torch.nan_to_num(C), torch.nan_to_num(D))
    # from host arrays, whose values are still under way when the rest of the build is done
    late = pc.pcsr_build(n, n, rp, ci, va, pc.make_params(flags=FLAG | WINDOWS | pc.PCSR_FLAG_GPU_BUILD))
    pc.pcsr_spmm(late, B, D, K)
    assert torch.equal(torch.nan_to_num(C), torch.nan_to_num(D))
    for handle in (plain, h, again, late):
        handle.close()


def test_windows_of_communities_in_a_graph_and_a_layer():
    """The first product of all is captured and replayed beside eager ones; a layer with its elementwise tail agrees with
    one on an ordinary handle."""
    n, rp, ci, va, _ = _planted(6001, 300, 40, 3, 11)
    arrays, K = _device(rp, ci, va), 192
    h = pc.pcsr_build(n, n, *arrays, pc.make_params(flags=FLAG | WINDOWS))
    assert pc.pcsr_query_launch(h, K)["lds_bytes"] > 0
    B, C = torch.randn(n, K, device="cuda"), torch.zeros(n, K, device="cuda")
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        pc.pcsr_spmm(h, B, C, K, torch.cuda.current_stream())
    for k in range(4):
        B.normal_()
        want = torch.empty_like(C)
        pc.pcsr_spmm(h, B, want, K)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(C, want), k
    h.close()

    from paper_2605_15695_amd.gnn import PcsrOperator, make_model

    models = []
    for prm in (pc.make_params(flags=FLAG | WINDOWS), pc.make_params()):
        torch.manual_seed(1)
        op = PcsrOperator(n, n, *arrays, params=prm)
        models.append(make_model("gcn", op, 64, 128, 64, 3).cuda())
    X = torch.randn(n, 64, device="cuda")
    outs = [m(X) for m in models]
    for o in outs:
        o.square().mean().backward()
    for got, want in [(outs[0].detach(), outs[1].detach())] + [(a.grad, b.grad) for a, b in zip(*(m.parameters() for m in models))]:
        assert float((got - want).norm() / want.norm()) < 1e-5


def test_selector_asks_for_windows_where_one_product_pays_for_them():
    f = np.zeros(len(pc.FEATURE_NAMES))
    f[0] = f[1] = 250_000
    f[2], f[4], f[5], f[6], f[7], f[15], f[16] = 12e6, 48.0, 48.0, 80.0, 0.15, 0.5, 0.004
    assert [bool(pc.pcsr_select(f, K).flags & WINDOWS) for K in (128, 192, 256, 258, 512)] == [False, False, True, False, True]
    f[2], f[4], f[5] = 4.5e6, 18.0, 18.0                       # short rows
    assert not pc.pcsr_select(f, 1024).flags & WINDOWS


@pytest.fixture(scope="module")
def long_rows():
    """Rows of a length in communities that hold them, with equal values and with random ones."""
    made = {}

    def get(length):
        if length not in made:
            block = max(100, length + length // 4)
            n, rp, ci, va, _ = _planted(10 * block + 1, block, length, length // 12, length)
            made[length] = n, rp, ci, (np.full_like(va, 1.0 / length), va)
        return made[length]

    return get


def _rms(params, n, rp, ci, va, B, ref, bound):
    """Of the differences from 64 bits, relative to each element's sum of magnitudes."""
    h = pc.pcsr_build(n, n, *_device(rp, ci, va), params)
    C = torch.full(B.shape, float("nan"), device="cuda")
    pc.pcsr_spmm(h, torch.from_numpy(B).cuda(), C, B.shape[1])
    e = (C.cpu().numpy().astype(np.float64) - ref) / np.maximum(bound, 1e-30)
    made = pc.pcsr_format(h)["SG"], pc.pcsr_query_kernel(h, B.shape[1])
    h.close()
    return float(np.sqrt(np.mean(e * e))), made


# The fewest independent squares (rows of 48, K = 8: 8000) have a mean within 5 % of its expectation at three standard
# deviations (their kurtosis is about 3); the root halves that, and the two sides share inputs: 1.04.
@pytest.mark.parametrize("length", [48, 100, 300, 1000])
@pytest.mark.parametrize("K", [8, 32, 64, 256])
def test_long_rows_are_as_exact_as_split_ones(long_rows, length, K):
    """Against 64 bits: no further off than items of 32 vectors whose sums are added by the second pass."""
    n, rp, ci, values = long_rows(length)
    for va in values:
        B = np.random.default_rng(K).uniform(-1, 1, (n, K)).astype(np.float32)
        ref, bound = oracle.spmm(rp, ci, va, B)
        split, _ = _rms(pc.make_params(S=1, SG=32, flags=pc.PCSR_FLAG_COLUMN_ORDER), n, rp, ci, va, B, ref, bound)
        whole, (SG, shape) = _rms(pc.make_params(flags=FLAG), n, rp, ci, va, B, ref, bound)
        print(f"rms of rows of {length}, K={K}: {whole:.3e}, split {split:.3e} {shape}", flush=True)
        assert SG == 1024 and whole <= 1.04 * split, (length, K, whole, split, shape)


@pytest.mark.parametrize("V", [1, 2])
@pytest.mark.parametrize("lanes", [4, 32, 64])
def test_long_items_are_as_exact_as_short_ones(long_rows, V, lanes):
    n, rp, ci, values = long_rows(300)
    B = np.random.default_rng(lanes).uniform(-1, 1, (n, 128)).astype(np.float32)
    for va in values:
        ref, bound = oracle.spmm(rp, ci, va, B)
        short, long = (_rms(pc.make_params(V=V, S=1, SG=SG, lanes_per_row=lanes, vec=2, rep=1, waves_per_wg=8), n, rp, ci, va, B,
                            ref, bound)[0] for SG in (32, 1024))
        print(f"rms V={V}, {lanes} lanes: {long:.3e}, items of 32 {short:.3e}", flush=True)
        assert lanes < 32 or long <= 1.04 * short, (V, lanes, long, short)


@pytest.mark.parametrize("length", [48, 100, 300, 400])
@pytest.mark.parametrize("K", [64, 256])
def test_long_rows_from_windows_of_communities_are_as_exact(long_rows, length, K):
    n, rp, ci, values = long_rows(length)
    for va in values:
        B = np.random.default_rng(K).uniform(-1, 1, (n, K)).astype(np.float32)
        ref, bound = oracle.spmm(rp, ci, va, B)
        split, _ = _rms(pc.make_params(S=1, SG=32, flags=pc.PCSR_FLAG_COLUMN_ORDER), n, rp, ci, va, B, ref, bound)
        staged, (SG, shape) = _rms(pc.make_params(flags=FLAG | WINDOWS), n, rp, ci, va, B, ref, bound)
        print(f"rms of rows of {length}, K={K}: staged {staged:.3e}, split {split:.3e} {shape}", flush=True)
        assert SG == 1024 and shape["lds_bytes"] > 0 and staged <= 1.04 * split, (length, K, staged, split, shape)


@pytest.mark.parametrize("V", [1, 2])
@pytest.mark.parametrize("length", [48, 100, 400])
@pytest.mark.parametrize("wc,kern", [(512, dict(lanes_per_row=16, vec=4, rep=1)), (256, dict(lanes_per_row=32, vec=2, rep=1)),
                                     (256, dict(lanes_per_row=64, vec=1, rep=1)), (256, dict(lanes_per_row=4, vec=4, rep=4)),
                                     (256, dict(lanes_per_row=8, vec=2, rep=4))])
def test_rows_from_column_windows_are_as_exact_as_from_memory(long_rows, V, length, wc, kern):
    """Rows of a community brought together; steps of 16 vectors down to 2, chunks of 4 to 64, on both sides of the rule for long rows."""
    n, rp, ci, values = long_rows(length)
    perm, _ = pc.pcsr_reorder(n, rp, ci)
    K = 128
    for va in values:
        prp, pci, pva = pc.pcsr_permute_csr(n, rp, ci, va, perm)
        B = np.random.default_rng(V).uniform(-1, 1, (n, K)).astype(np.float32)
        ref, bound = oracle.spmm(prp, pci, pva, B)
        plain, _ = _rms(pc.make_params(V=V, **kern), n, prp, pci, pva, B, ref, bound)
        staged, (_, shape) = _rms(pc.make_params(V=V, col_window=wc, **kern), n, prp, pci, pva, B, ref, bound)
        # the vectors outside the window are a sum of their own: one more rounding of the whole, of rms 2^-23 / sqrt(24)
        # (uniform within half a unit, mantissas from 1 to 2)
        whole = 2.0 ** -23 / 24 ** 0.5 * float(np.sqrt(np.mean((ref / np.maximum(bound, 1e-30)) ** 2)))
        limit = 1.04 * (plain ** 2 + whole ** 2) ** 0.5
        print(f"case rows of {length}, V={V}, window of {wc} {kern}: staged {staged:.3e}, plain {plain:.3e}, {limit:.3e}", flush=True)
        assert shape["lds_bytes"] > 0 and staged <= limit, (V, wc, kern, staged, plain, limit)


@pytest.mark.parametrize("vec", [1, 2])
@pytest.mark.parametrize("flags", [FLAG, FLAG | WINDOWS])
def test_alignment_asked_for_is_that_of_the_parameters(vec, flags):
    """What pcsr_select returns for scattered rows of 8 to 40 has vec = 2 (1 at K up to 32): operands at such addresses are taken
    whatever order the build finds, others refused."""
    n, rp, ci, va, _ = _planted(6001, 300, 30, 2, 21)
    h = pc.pcsr_build(n, n, *_device(rp, ci, va), pc.make_params(lanes_per_row=32, vec=vec, rep=1, flags=flags))
    assert pc.pcsr_format(h)["SG"] == 1024
    for K in (32, 64, 128):
        B, S = torch.randn(n, K, device="cuda"), torch.randn(n, K, device="cuda")
        want, tailed = torch.empty_like(B), torch.empty_like(B)
        pc.pcsr_spmm(h, B, want, K)

        def at(offset, source=None):
            t = torch.full((n * K + 4,), float("nan"), device="cuda")[offset:offset + n * K].view(n, K)
            return t if source is None else t.copy_(source)

        def epilogue(B, C, S):
            e = pc.binding.pcsr_epilogue_t(None, S.data_ptr(), None, None, 0, 0)
            return pc.binding._lib().pcsr_spmm_epilogue(h.raw, B.data_ptr(), C.data_ptr(), K, pc.binding.ctypes.byref(e), None)

        assert epilogue(B, tailed, S) == 0
        C = at(vec)
        pc.pcsr_spmm(h, at(vec, B), C, K)
        assert torch.equal(C, want)
        C = at(vec)
        assert epilogue(at(vec, B), C, at(vec, S)) == 0 and torch.equal(C, tailed)
        if vec == 2:
            assert epilogue(at(2, B), at(2), at(1, S)) == pc.binding.PCSR_E_INVALID_ARG
            for b, c in ((1, 2), (2, 1)):
                with pytest.raises(pc.PcsrError) as err:
                    pc.pcsr_spmm(h, at(b, B), at(c), K)
                assert err.value.code == pc.binding.PCSR_E_INVALID_ARG
        pc.pcsr_set_kernel_params(h)
        with pytest.raises(pc.PcsrError):
            pc.pcsr_spmm(h, at(vec, B), want, K)
        h.close()
        h = pc.pcsr_build(n, n, *_device(rp, ci, va), pc.make_params(lanes_per_row=32, vec=vec, rep=1, flags=flags))
    h.close()


def test_first_product_from_column_windows_over_long_rows_may_be_captured(long_rows):
    """Beside products of a handle with short rows, whose kernel is another one."""
    n, rp, ci, values = long_rows(300)
    perm, _ = pc.pcsr_reorder(n, rp, ci)
    rp, ci, va = pc.pcsr_permute_csr(n, rp, ci, values[1], perm)
    m, srp, sci, svalues = long_rows(48)
    sperm, _ = pc.pcsr_reorder(m, srp, sci)
    short = pc.pcsr_build(m, m, *pc.pcsr_permute_csr(m, srp, sci, svalues[1], sperm), pc.make_params(col_window=256))
    h = pc.pcsr_build(n, n, rp, ci, va, pc.make_params(col_window=256))
    K = 128
    assert all(pc.pcsr_query_launch(x, K)["lanes_per_row"] == 32 and pc.pcsr_query_launch(x, K)["lds_bytes"] for x in (short, h))
    pc.pcsr_spmm(short, torch.randn(m, K, device="cuda"), torch.empty(m, K, device="cuda"), K)
    B, C = torch.randn(n, K, device="cuda"), torch.zeros(n, K, device="cuda")
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        pc.pcsr_spmm(h, B, C, K, torch.cuda.current_stream())
    for _ in range(3):
        B.normal_()
        want = torch.empty_like(C)
        pc.pcsr_spmm(h, B, want, K)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(C, want)
    short.close(), h.close()
