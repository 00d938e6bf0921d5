"""B as a buffer: 32-bit offsets up to their last byte, slots and lanes past the end."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_15695_amd as pc
from tests.test_gpu_cluster_order import _device, _planted

pytestmark = pytest.mark.gpu

NEAR_BYTES = 0xE0000000  # pcsr_kernels.hip: kNearBytes


def _rows(rng, lengths, columns):
    """CSR of rows of these lengths, columns drawn from `columns`."""
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    colidx = np.concatenate([np.sort(rng.choice(columns, m, replace=False)) for m in lengths]).astype(np.int32)
    return rowptr, colidx, rng.standard_normal(colidx.size).astype(np.float32)


def _tail(h, B, K, rng):
    """C = relu((1 + eps) S + A B + bias) with a mask, and a reference for an A B that is known."""
    from paper_2605_15695_amd.gnn import _Dense

    n = h.n_rows
    S, bias = rng.standard_normal((n, K)).astype(np.float32), rng.standard_normal(K).astype(np.float32)
    mask = rng.standard_normal((n, K)).astype(np.float32)
    d = _Dense(torch.empty(1, device="cuda"), [(1, 1)])
    C = d.spmm(h, n, B, bias=torch.from_numpy(bias).cuda(), relu=True, self_term=torch.from_numpy(S).cuda(),
               eps=torch.tensor(0.5, device="cuda"), mask=torch.from_numpy(mask).cuda())
    return C, lambda ref, bound: (np.where(mask > 0, np.maximum(ref + 1.5 * S + bias, 0), 0), bound + 1.5 * np.abs(S) + np.abs(bias))


@pytest.mark.parametrize("form,lanes,vec,K", [("plain", 16, 1, 16), ("plain", 32, 1, 32), ("plain", 16, 4, 64), ("plain", 8, 4, 32),
                                              ("tail", 0, 0, 16), ("tail", 0, 0, 64), ("tail", 0, 0, 128), ("window", 16, 4, 64)])
@pytest.mark.parametrize("over", [0, 1])
def test_operands_at_the_limit(form, lanes, vec, K, over):
    """The largest B that is addressed in 32 bits, and one row more."""
    n_cols, n = NEAR_BYTES // (4 * K) + over, 300
    rng = np.random.default_rng(K + over)
    rowptr, colidx, vals = _rows(rng, rng.integers(0, 40, n), n_cols)
    colidx[rowptr[1:][np.diff(rowptr) > 0] - 1] = n_cols - 1  # every row reads the last one of B
    h = pc.pcsr_build(n, n_cols, rowptr, colidx, vals, pc.make_params(lanes_per_row=lanes, vec=vec, rep=1 if lanes else 0,
                                                                      col_window=256 if form == "window" else 0))
    assert (pc.pcsr_query_launch(h, K)["lds_bytes"] > 0) == (form == "window")
    B = torch.full((n_cols, K), float("nan"), device="cuda")  # rows that nobody references must not be seen
    cols, inv = np.unique(colidx, return_inverse=True)
    rows = rng.standard_normal((cols.size, K)).astype(np.float32)
    B[torch.from_numpy(cols.astype(np.int64)).cuda()] = torch.from_numpy(rows).cuda()
    ref, bound = oracle.spmm(rowptr, inv.astype(np.int32), vals, rows)
    if form == "tail":
        C, expect = _tail(h, B, K, rng)
        ref, bound = expect(ref, bound)
    else:
        C = torch.empty(n, K, device="cuda")
        pc.pcsr_spmm(h, B, C, K)
    torch.cuda.synchronize()
    ok, worst = oracle.within_tolerance(C.cpu().numpy(), ref, bound)
    assert ok, worst
    h.close()
    del B
    torch.cuda.empty_cache()


SHORT, MIXED, LONG = (0, 8), (0, 70), (10, 400)  # least and most vectors of a row
FORMS = [  # parameters of the handle, lengths of its rows, widths
    *((dict(V=V), lengths, (8, 12, 16, 24, 32, 48, 64, 75, 128)) for V in (1, 2) for lengths in (SHORT, MIXED)),
    (dict(V=1, lanes_per_row=16, vec=1, rep=2), MIXED, (18, 31)), (dict(V=1, lanes_per_row=32, vec=2, rep=1), MIXED, (64, 130)),
    (dict(V=2, lanes_per_row=16, vec=4, rep=2), MIXED, (128,)), (dict(V=1, lanes_per_row=4, vec=1, rep=1), LONG, (3, 9)),
    # items of up to 8 and 40 vectors, and of more than 64, whose sums are put apart in 32 lanes
    *((dict(V=V, S=1, SG=SG, flags=pc.PCSR_FLAG_COLUMN_ORDER), LONG, (12, 16, 32, 64, 100)) for V in (1, 2) for SG in (8, 40)),
    *((dict(V=V, S=1, SG=200, lanes_per_row=32, vec=4, rep=1), LONG, (64, 128)) for V in (1, 2)),
    (dict(V=1, S=1, SG=200, lanes_per_row=16, vec=1, rep=1), LONG, (12, 16)),
    # column windows, rows of up to 256 vectors and of more
    *((dict(V=V, col_window=256, lanes_per_row=16, vec=4, rep=1), lengths, (64, 68, 192)) for V in (1, 2) for lengths in (MIXED, LONG)),
]


@pytest.mark.parametrize("k", range(len(FORMS)))
def test_offsets_of_32_and_of_64_bits(k):
    """The kernels of a B of any size on a small one, beside those it gets by its size: the same sums in the same order."""
    prm, (least, most), widths = FORMS[k]
    n = 1501
    rng = np.random.default_rng(k)
    cols = np.flatnonzero(np.arange(n) % 5)  # every fifth row of B is referenced by nobody
    lengths = rng.integers(least, most + 1, n)
    if prm.get("col_window"):
        # rows that gather from around their own number, and some vectors elsewhere
        lists = [np.unique(cols[np.concatenate([(i * 4 // 5 + rng.integers(0, 200, m)) % cols.size, rng.integers(0, cols.size, m // 6)])])
                 for i, m in enumerate(lengths)]
        rowptr, colidx = np.concatenate([[0], np.cumsum([len(c) for c in lists])]).astype(np.int32), np.concatenate(lists).astype(np.int32)
        vals = rng.standard_normal(colidx.size).astype(np.float32)
    else:
        rowptr, colidx, vals = _rows(rng, lengths, cols)
    _both(n, rowptr, colidx, vals, prm, widths, rng)


@pytest.mark.parametrize("windows", [0, pc.PCSR_FLAG_CLUSTER_WINDOWS])
@pytest.mark.parametrize("extra", [(), ((5, 1024), (700, 100))])  # rows of more than 32 (no windows) and 88 vectors among them
def test_offsets_of_32_and_of_64_bits_in_communities(windows, extra):
    n, rowptr, colidx, vals, _ = _planted(5003, 200, 40, 3, 1, extra)
    prm = dict(flags=pc.PCSR_FLAG_CLUSTER_IF_USEFUL | windows)
    h = _both(n, *_device(rowptr, colidx, vals), prm, (16, 32, 64, 68, 128, 200), np.random.default_rng(2), host=(rowptr, colidx, vals))
    assert h["SG"] == 1024 and h["windows"] == bool(windows)


def _both(n, rowptr, colidx, vals, prm, widths, rng, host=None):
    prm = dict(prm)
    flags = prm.pop("flags", 0)
    near, far = (pc.pcsr_build(n, n, rowptr, colidx, vals, pc.make_params(flags=flags | f, **prm)) for f in (0, pc.PCSR_FLAG_FAR_OFFSETS))
    again = pc.pcsr_build(n, n, rowptr, colidx, vals, pc.make_params(flags=flags, **prm))
    pc.pcsr_set_kernel_params(again, *(prm.get(f, 0) for f in ("lanes_per_row", "vec", "rep")), flags=pc.PCSR_FLAG_FAR_OFFSETS)
    rowptr, colidx, vals = host or (rowptr, colidx, vals)
    for K in widths:
        B = rng.standard_normal((n, K)).astype(np.float32)
        ref, bound = oracle.spmm(rowptr, colidx, vals, B)
        if host is None:
            B[::5] = np.nan
        B = torch.from_numpy(B).cuda()
        out = []
        for h in (near, far, again):
            C = torch.full((n, K), float("nan"), device="cuda")
            pc.pcsr_spmm(h, B, C, K)
            D, expect = _tail(h, B, K, np.random.default_rng(K))
            out.append((C, D))
        ok, worst = oracle.within_tolerance(out[0][0].cpu().numpy(), ref, bound)
        assert ok, (K, worst)
        ok, worst = oracle.within_tolerance(out[0][1].cpu().numpy(), *expect(ref, bound))
        assert ok, (K, worst)
        for C, D in out[1:]:
            assert torch.equal(C, out[0][0]) and torch.equal(D, out[0][1]), K
    q = dict(SG=pc.pcsr_export(near)["SG"], windows=pc.pcsr_query_launch(near, 64)["lds_bytes"] > 0)
    if prm.get("col_window"):
        assert q["windows"]
    for h in (near, far, again):
        h.close()
    return q


SHAPES = [(16, 1, 1), (16, 1, 2), (32, 1, 1), (8, 1, 2), (4, 1, 1), (16, 2, 1), (32, 4, 1)]  # lanes, vec, rep


@pytest.mark.parametrize("V,S", [(1, 0), (2, 0), (1, 1), (2, 1)])
@pytest.mark.parametrize("lanes,vec,rep,K", [(*shape, K) for shape in SHAPES for K in (9, 16, 18, 31, 32, 68) if K % shape[1] == 0])
@pytest.mark.parametrize("longest", [36, 9])  # items of less than 16 vectors on average have some forms without the buffer
def test_slots_and_columns_past_the_end(V, S, lanes, vec, rep, K, longest):
    """Rows that end within a step and widths that end within a group of lanes; what is read there is zeros, or a row's own
    last column, and never a row of B that the item does not reference."""
    n = 257
    rng = np.random.default_rng(K + lanes)
    cols = np.flatnonzero(np.arange(n) % 5)  # every fifth row of B is referenced by nobody
    rowptr = np.concatenate([[0], np.cumsum(np.arange(n) % (longest + 1))]).astype(np.int32)
    colidx = np.concatenate([np.sort(rng.choice(cols, m, replace=False)) for m in np.diff(rowptr)]).astype(np.int32)
    vals = rng.standard_normal(colidx.size).astype(np.float32)
    B = rng.standard_normal((n, K)).astype(np.float32)
    B[::5] = np.nan
    h = pc.pcsr_build(n, n, rowptr, colidx, vals,
                      pc.make_params(V=V, S=S, SG=8 if S else 0, lanes_per_row=lanes, vec=vec, rep=rep))
    C = torch.full((n, K), float("nan"), device="cuda")
    pc.pcsr_spmm(h, torch.from_numpy(B).cuda(), C, K)
    torch.cuda.synchronize()
    ref, bound = oracle.spmm(rowptr, colidx, vals, np.nan_to_num(B))
    ok, worst = oracle.within_tolerance(C.cpu().numpy(), ref, bound)
    assert ok, worst
    h.close()
