"""B as a buffer: 32-bit offsets up to their last byte, slots and lanes past the end."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_15695_amd as pc

pytestmark = pytest.mark.gpu

NEAR_BYTES = 0xE0000000  # pcsr_kernels.hip: kNearBytes


@pytest.mark.parametrize("lanes,vec,K", [(16, 1, 16), (32, 1, 32), (16, 4, 64), (8, 4, 32)])
@pytest.mark.parametrize("over", [0, 1])
def test_operands_at_the_limit(lanes, vec, K, over):
    """The largest B that is addressed in 32 bits, and one row more."""
    n_cols, n = NEAR_BYTES // (4 * K) + over, 300
    rng = np.random.default_rng(K + over)
    rowptr = np.concatenate([[0], np.cumsum(rng.integers(0, 40, n))]).astype(np.int32)
    colidx = np.concatenate([np.sort(rng.choice(n_cols, m, replace=False)) for m in np.diff(rowptr)]).astype(np.int32)
    colidx[rowptr[1:][np.diff(rowptr) > 0] - 1] = n_cols - 1  # every row reads the last one of B
    vals = rng.standard_normal(colidx.size).astype(np.float32)
    h = pc.pcsr_build(n, n_cols, rowptr, colidx, vals, pc.make_params(lanes_per_row=lanes, vec=vec, rep=1))
    B = torch.full((n_cols, K), float("nan"), device="cuda")  # rows that nobody references must not be seen
    cols, inv = np.unique(colidx, return_inverse=True)
    rows = rng.standard_normal((cols.size, K)).astype(np.float32)
    B[torch.from_numpy(cols.astype(np.int64)).cuda()] = torch.from_numpy(rows).cuda()
    C = torch.empty(n, K, device="cuda")
    pc.pcsr_spmm(h, B, C, K)
    torch.cuda.synchronize()
    ref, bound = oracle.spmm(rowptr, inv.astype(np.int32), vals, rows)
    ok, worst = oracle.within_tolerance(C.cpu().numpy(), ref, bound)
    assert ok, worst
    h.close()
    del B
    torch.cuda.empty_cache()


@pytest.mark.parametrize("V,S", [(1, 0), (2, 0), (1, 1), (2, 1)])
@pytest.mark.parametrize("lanes,vec,rep", [(16, 1, 1), (16, 1, 2), (32, 1, 1), (8, 1, 2), (4, 1, 1), (16, 2, 1), (32, 4, 1)])
@pytest.mark.parametrize("K", [9, 16, 18, 31, 32, 68])
@pytest.mark.parametrize("longest", [36, 9])  # items of less than 16 vectors on average have some forms without the buffer
def test_slots_and_columns_past_the_end(V, S, lanes, vec, rep, K, longest):
    """Rows that end within a step and widths that end within a group of lanes; what is read there is zeros, or a row's own
    last column, and never a row of B that the item does not reference."""
    if K % vec:
        pytest.skip("K is no multiple of vec")
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
