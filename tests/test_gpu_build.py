"""GPU-side generation and features where their workgroup splits can go wrong: rows far longer
than a slice of nonzeros, long runs of empty rows, panels of thousands of items; and the
library's memory cache."""
import numpy as np
import pytest

import paper_2605_15695_amd as pc
from tests.helpers import column_ordered_schedule, near_diagonal_share
from oracle import pcsr_format as pf

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _csr(n, lengths, seed):
    rng = np.random.default_rng(seed)
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    colidx = np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in lengths] + [[]]).astype(np.int32)
    return rowptr, colidx, rng.standard_normal(colidx.shape[0]).astype(np.float32)


def _case(name):
    n = 6001
    if name == "around_the_limits":               # panels of 0, 1, 8, 9, 64 and 300 beside 256 and 257 nonzeros
        n = 1301
    lengths = np.zeros(n, np.int64)
    if name == "long_rows":                       # several slices of 1024 inside one row
        lengths[[0, 1, 2, 3000, n - 1]] = [5000, 4096, 1, 6001, 2500]
    elif name == "empty_runs":                    # thousands of row starts inside one slice
        lengths[::1999] = 700
    elif name == "one_per_row":
        lengths[:] = 1
    elif name == "around_the_limits":
        pairs = [(a, b) for a in (0, 1, 8, 9, 64, 300) for b in (255, 256, 257, 1024, 1300)]
        lengths = np.zeros(n, np.int64)
        flat = np.array(pairs + [p[::-1] for p in pairs]).ravel()
        lengths[:flat.shape[0]] = flat
        lengths[n - 1] = 700
    elif name == "mixed":
        lengths = np.random.default_rng(1).integers(0, 60, n)
        lengths[17] = 3000
    return (n,) + _csr(n, lengths, len(name))


@pytest.mark.parametrize("name", ["long_rows", "empty_runs", "one_per_row", "mixed", "around_the_limits"])
def test_features_and_arrays(name):
    n, rp, ci, va = _case(name)
    d = [torch.from_numpy(x).cuda() for x in (rp, ci, va)]
    f = pc.pcsr_features(n, n, d[0], d[1], 64)
    assert np.allclose(f[:16], pf.features(n, n, rp, ci, 64), rtol=1e-11, atol=0)
    assert f[16] == pytest.approx(near_diagonal_share(rp, ci), rel=1e-12)
    for V, S, SG in [(1, 0, 0), (2, 0, 0), (1, 1, 1), (1, 1, 32), (2, 1, 7)]:
        h = pc.pcsr_build(n, n, *d, pc.make_params(V=V, S=S, SG=SG, flags=pc.PCSR_FLAG_COLUMN_ORDER if S else 0))
        e, r = pc.pcsr_export(h), pf.pcsr_ref(n, rp, ci, va, V, S, SG, 64)
        for k in ("rowptr", "colidx", "trow"):
            assert np.array_equal(e[k], r[k]), (V, S, k)
        assert np.array_equal(e["val"].view(np.uint32), r["val"].view(np.uint32))
        if S:
            got = pc.pcsr_export_schedule(h)
            sched, xb = column_ordered_schedule(e["rowptr"], e["colidx"], e["trow"], e["P"])
            assert np.array_equal(got["xcd_bounds"], xb) and np.array_equal(got["sched"], sched)
        B = torch.randn(n, 8, device="cuda")
        C = torch.full((n, 8), float("nan"), device="cuda")
        pc.pcsr_spmm(h, B, C, 8)
        A = torch.sparse_csr_tensor(d[0].long(), d[1].long(), d[2].double(), size=(n, n))
        ref = A @ B.double()
        assert float((C.double() - ref).norm() / ref.norm()) < 1e-5
        h.close()


@pytest.mark.parametrize("place", [0, 1, 1023, 1024, 4999, 5000])
def test_one_wrong_column_is_found_wherever_it_is(place):
    n, rp, ci, va = _case("long_rows")
    bad = ci.copy()
    bad[place] = bad[place - 1] if place not in (0, 5000) else n   # a duplicate, or out of range
    with pytest.raises(pc.PcsrError) as e:
        pc.pcsr_build(n, n, *(torch.from_numpy(x).cuda() for x in (rp, bad, va)), pc.make_params())
    assert e.value.code == pc.binding.PCSR_E_BAD_CSR


def test_freed_memory_is_kept_within_a_bound_and_reused():
    n, rp, ci, va = _case("mixed")
    B, C = torch.ones(n, 64, device="cuda"), torch.empty(n, 64, device="cuda")

    def once():
        h = pc.pcsr_build(n, n, rp, ci, va, pc.make_params(S=1, SG=4))
        pc.pcsr_spmm(h, B, C, 64)
        h.close()                                   # waits for the product
        return C.clone()

    first = once()
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    for _ in range(20):
        assert torch.equal(once(), first)
    assert free0 - torch.cuda.mem_get_info()[0] <= 64 << 20
    big = 40_000_000                                # 5 x 320 MB of arrays: more than the cache may keep
    rpb = torch.arange(big + 1, dtype=torch.int32, device="cuda")
    cib = torch.arange(big, dtype=torch.int32, device="cuda")
    vab = torch.ones(big, device="cuda")
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    hs = [pc.pcsr_build(big, big, rpb, cib, vab, pc.make_params()) for _ in range(5)]
    for h in hs:
        h.close()
    assert before - torch.cuda.mem_get_info()[0] <= (1 << 30) + (64 << 20)


@pytest.mark.parametrize("n_items", [1, 16_383, 16_384, 70_001, 1 << 21, (1 << 21) + 1])
@pytest.mark.parametrize("bits", [1, 11, 21])
def test_items_come_in_column_order_whatever_their_number(n_items, bits):
    """The sort behind the column-ordered schedule: rows of two nonzeros cut into items of one."""
    rng = np.random.default_rng(n_items + bits)
    n_cols = (1 << bits) + 1
    first = np.minimum(rng.integers(0, n_cols - 1, n_items), rng.integers(0, n_cols - 1, n_items))
    rp = torch.arange(0, 2 * n_items + 1, 2, dtype=torch.int32, device="cuda")
    ci = torch.from_numpy(np.stack([first, np.full(n_items, n_cols - 1)], 1).ravel().astype(np.int32)).cuda()
    h = pc.pcsr_build(n_items, n_cols, rp, ci, torch.ones(2 * n_items, device="cuda"),
                      pc.make_params(S=1, SG=1, flags=pc.PCSR_FLAG_COLUMN_ORDER))
    e, got = pc.pcsr_export(h), pc.pcsr_export_schedule(h)
    sched, xb = column_ordered_schedule(e["rowptr"], e["colidx"], e["trow"], e["P"])
    assert np.array_equal(got["xcd_bounds"], xb) and np.array_equal(got["sched"], sched)
    h.close()


def _device_build_fails(n, m, rp, ci, flags=0):
    with pytest.raises(pc.PcsrError) as err:
        pc.pcsr_build(n, m, *(torch.from_numpy(x).cuda() for x in (rp, ci, np.ones(ci.shape[0], np.float32))),
                      pc.make_params(flags=flags))
    return err.value.code == pc.binding.PCSR_E_BAD_CSR


@pytest.mark.parametrize("where", [0, 1, 3, 1023, 1024, 1025, 2047, 2499])
def test_one_wrong_column_is_found_wherever_it_is(where):
    """Rows of 1, 2, 3, ... nonzeros with runs of empty ones, so that row starts fall everywhere in a slice."""
    lengths = np.concatenate([np.tile(np.arange(8), 90), np.zeros(2000, np.int64)])
    rp = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    n, m = lengths.shape[0], 50
    ci = np.concatenate([5 + 3 * np.arange(k) for k in lengths]).astype(np.int32)
    h = pc.pcsr_build(n, m, *(torch.from_numpy(x).cuda() for x in (rp, ci, np.ones(ci.shape[0], np.float32))))
    assert np.array_equal(pc.pcsr_export(h)["colidx"], ci)
    h.close()
    starts = set(rp.tolist())
    for value in (m, -1) + (() if where in starts else (int(ci[where - 1]), int(ci[where - 1]) - 1)):
        bad = ci.copy()
        bad[where] = value
        assert _device_build_fails(n, m, rp, bad), value
    pointer = rp.copy()
    row = int(np.searchsorted(rp, where, side="right"))
    pointer[row] = rp[-1] + 1
    assert _device_build_fails(n, m, pointer, ci)
    pointer[row] = -3
    assert _device_build_fails(n, m, pointer, ci)


def _same_handle(a, b):
    assert pc.pcsr_format(a) == pc.pcsr_format(b)
    x, y = pc.pcsr_export(a), pc.pcsr_export(b)
    assert x.keys() == y.keys()
    for k in x:
        assert np.array_equal(np.asarray(x[k]).view(np.uint32) if k == "val" else x[k],
                              np.asarray(y[k]).view(np.uint32) if k == "val" else y[k]), k


# both directions at once: values on a thread of their own from 4 MB on (1,048,576 nonzeros), the transpose in two passes from 262,144 on
# and up to 2^20 columns, on the host below 10,000; from device memory too, and from four threads
@pytest.mark.parametrize("rows,cols,nnz", [(301, 257, 9000), (3001, 9001, 12000), (20001, 15013, 300000), (20001, 15013, 1048575),
                                           (40001, 30011, 1048577), (30011, (1 << 20) + 5, 1200000), (70001, 513, 2000003)])
@pytest.mark.parametrize("params", [None, dict(V=1), dict(V=2), dict(V=1, S=1, SG=8, flags=pc.PCSR_FLAG_COLUMN_ORDER)])
@pytest.mark.parametrize("threads", [1, 4])
def test_both_directions_at_once(rows, cols, nnz, params, threads):
    from concurrent.futures import ThreadPoolExecutor

    from paper_2605_15695_amd import binding

    rng = np.random.default_rng(nnz + rows)
    key = np.unique(rng.integers(0, rows * cols, int(nnz * (1.02 + 0.6 * nnz / (rows * cols)))))
    key = key[np.sort(rng.permutation(key.shape[0])[:nnz])]
    rp = np.searchsorted(key, np.arange(rows + 1) * cols).astype(np.int32)
    ci, va = (key % cols).astype(np.int32), rng.standard_normal(key.shape[0]).astype(np.float32)
    forward, backward = (rows, cols, rp, ci, va), (cols, rows, *pc.pcsr_transpose_csr(rows, cols, rp, ci, va))

    def alone(m):
        p = pc.make_params(**params) if params is not None else pc.pcsr_select(pc.pcsr_features(*m[:4]), 24)
        if params is None:
            p.lanes_per_row = p.vec = p.rep = 0
        p.flags |= pc.PCSR_FLAG_GPU_BUILD
        return pc.pcsr_build(*m, p)

    want = alone(forward), alone(backward)

    def one(on_device):
        arrays = [torch.from_numpy(x).cuda() for x in (rp, ci, va)] if on_device else (rp, ci, va)
        torch.cuda.synchronize()
        return binding.pcsr_operator_build(rows, cols, *arrays, pc.make_params(**params) if params is not None else None, 24, True)

    with ThreadPoolExecutor(threads) as pool:
        for made in pool.map(one, [False, True] * threads):
            for h, w in zip(made, want):
                _same_handle(h, w)
                h.close()
