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
    lengths = np.zeros(n, np.int64)
    if name == "long_rows":                       # several slices of 1024 inside one row
        lengths[[0, 1, 2, 3000, n - 1]] = [5000, 4096, 1, 6001, 2500]
    elif name == "empty_runs":                    # thousands of row starts inside one slice
        lengths[::1999] = 700
    elif name == "one_per_row":
        lengths[:] = 1
    elif name == "mixed":
        lengths = np.random.default_rng(1).integers(0, 60, n)
        lengths[17] = 3000
    return (n,) + _csr(n, lengths, len(name))


@pytest.mark.parametrize("name", ["long_rows", "empty_runs", "one_per_row", "mixed"])
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
