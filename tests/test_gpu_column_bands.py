"""Products in bands of columns (PCSR_FLAG_COLUMN_BANDS): against the oracle, in one pass, and where the bands do not apply."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_15695_amd as pc
from tests.test_gpu_near_operand import _tail

pytestmark = pytest.mark.gpu

BANDS = pc.PCSR_FLAG_COLUMN_BANDS
N, N_COLS = 30000, 30011  # B of 8 MB from K = 64 on


def _graph(seed=3):
    """Scattered rows of 0 to 240, empty ones at both ends and some whose columns are all in one band."""
    rng = np.random.default_rng(seed)
    deg = rng.integers(60, 240, N)
    deg[[0, 1, N - 1]] = 0
    deg[rng.integers(0, N, N // 50)] = 0
    step = N_COLS // 240
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    k = np.arange(rowptr[-1]) - np.repeat(rowptr[:-1], deg)
    colidx = k * step + rng.integers(0, step, rowptr[-1])  # ascending, one in each part
    for r in rng.integers(2, N - 1, 200):
        m = rowptr[r + 1] - rowptr[r]
        colidx[rowptr[r]:rowptr[r + 1]] = (N_COLS - 240 if r % 2 else 0) + np.arange(m)
    return rowptr, colidx.astype(np.int32), rng.standard_normal(rowptr[-1]).astype(np.float32)


@pytest.fixture(scope="module")
def graph():
    return _graph()


def _dev(*arrays):
    return [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in arrays]


# every tile the kernel exists for, remainders of it, and several slices
@pytest.mark.parametrize("shape,K", [((8, 1, 1), 5), ((8, 4, 1), 32), ((8, 4, 1), 20), ((16, 1, 1), 9), ((16, 1, 1), 16), ((32, 1, 1), 24),
                                     ((16, 4, 1), 48), ((16, 4, 1), 96), ((32, 2, 1), 66), ((32, 4, 1), 100), ((64, 4, 1), 200)])
def test_bands_against_the_oracle(graph, shape, K):
    rowptr, colidx, vals = graph
    B = np.random.default_rng(K).standard_normal((N_COLS, K)).astype(np.float32)
    kw = dict(lanes_per_row=shape[0], vec=shape[1], rep=shape[2])
    dev, (b,) = _dev(rowptr, colidx, vals), _dev(B)
    ref, bound = oracle.spmm(rowptr, colidx, vals, B)
    got = []
    for csr in (dev, (rowptr, colidx, vals)):
        for flags in (BANDS, BANDS | pc.PCSR_FLAG_FAR_OFFSETS):
            h = pc.pcsr_build(N, N_COLS, *csr, pc.make_params(flags=flags, **kw))
            C = torch.full((N, K), float("nan"), device="cuda")  # what C held is not read
            pc.pcsr_spmm(h, b, C, K)
            got.append(C.cpu().numpy())
            h.close()
    ok, worst = oracle.within_tolerance(got[0], ref, bound)
    assert ok, worst
    for x in got[1:]:
        assert np.array_equal(x, got[0])


# a handle selected for one width at another, which its stand-in shape would cover in slices that share columns
@pytest.mark.parametrize("hint,K", [(33, 65), (50, 66), (62, 126), (66, 130), (75, 131), (126, 134), (66, 258), (50, 514)])
def test_slices_that_share_columns(graph, hint, K):
    rowptr, colidx, vals = graph
    f = np.array(pc.pcsr_features(N, N_COLS, rowptr, colidx), dtype=np.float64)
    f[:2], f[2], f[4:7], f[16] = 300_000, 300_000 * 134, 134, 0.0
    p = pc.pcsr_select(f, hint)
    p.flags &= ~(pc.PCSR_FLAG_CLUSTER_IF_USEFUL | pc.PCSR_FLAG_CLUSTER_WINDOWS)
    assert (p.V, p.S) == (1, 0) and p.flags & BANDS
    h = pc.pcsr_build(N, N_COLS, *_dev(rowptr, colidx, vals), p)
    q = pc.pcsr_query_kernel(h, K)
    assert K % q["vec"] and (q["grid_y"] > 1) == (K > 512)
    B = np.random.default_rng(K).standard_normal((N_COLS, K)).astype(np.float32)
    b, got = _dev(B)[0], []
    for _ in range(3):
        C = torch.full((N, K), float("nan"), device="cuda")
        pc.pcsr_spmm(h, b, C, K)
        got.append(C.cpu().numpy())
    ok, worst = oracle.within_tolerance(got[0], *oracle.spmm(rowptr, colidx, vals, B))
    assert ok, worst
    assert all(np.array_equal(x, got[0]) for x in got)
    h.close()


# auto shapes, as operators have them: tiles of the whole row, slices of 64 and 512 columns, and more than one tile holds
@pytest.mark.parametrize("K", [64, 100, 128, 200, 260, 300, 512, 515, 640, 1000])
def test_wide_rows_are_as_exact_as_items_of_32(graph, K):
    """Rows of 60 to 240 numbers between 0 and 1, rms difference from 64 bits beside that of the same rows split into items of 32 in
    column order: sums of 8, in sums of 32 or 64, in that of the row, are about as many roundings."""
    rowptr, colidx, vals = graph
    dev = _dev(rowptr, colidx, np.abs(vals))
    B = torch.rand(N_COLS, K, device="cuda", generator=torch.Generator("cuda").manual_seed(K))
    rows = np.arange(2, N - 1, 97)
    at = np.concatenate([np.arange(rowptr[r], rowptr[r + 1]) for r in rows])
    part = dev[2][torch.from_numpy(at).cuda()].double()[:, None] * B[dev[1][torch.from_numpy(at).cuda()].long()].double()
    ref = torch.zeros(rows.size, K, dtype=torch.float64, device="cuda").index_add_(
        0, torch.from_numpy(np.repeat(np.arange(rows.size), np.diff(rowptr)[rows])).cuda(), part)
    full = (ref > 0).all(1)
    rms = []
    for kw in (dict(flags=BANDS), dict(S=1, SG=32, flags=pc.PCSR_FLAG_COLUMN_ORDER)):
        h = pc.pcsr_build(N, N_COLS, *dev, pc.make_params(**kw))
        C = torch.empty(N, K, device="cuda")
        pc.pcsr_spmm(h, B, C, K)
        off = ((C[torch.from_numpy(rows).cuda()].double() - ref)[full] / ref[full])
        rms.append(float(off.square().mean().sqrt()))
        h.close()
    assert rms[0] < 1.15 * rms[1], rms


def _launches(f):
    from torch.profiler import ProfilerActivity, profile

    f()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        f()
        torch.cuda.synchronize()
    return sum("spmm_kernel" in e.name for e in p.events())


def test_bands_are_what_runs(graph):
    """Several launches where B outgrows L2, one where it does not, where C is a row of the tail, and where the host built the handle."""
    rowptr, colidx, vals = graph
    dev = _dev(rowptr, colidx, vals)
    h = pc.pcsr_build(N, N_COLS, *dev, pc.make_params(flags=BANDS))
    plain = pc.pcsr_build(N, N_COLS, *dev, pc.make_params())
    host = pc.pcsr_build(N, N_COLS, rowptr, colidx, vals, pc.make_params(flags=BANDS | pc.PCSR_FLAG_HOST_ONLY))
    exported, ref = pc.pcsr_export(host), pc.pcsr_export(plain)
    assert all(np.array_equal(exported[k], ref[k]) for k in ref)
    host.close()
    for K, several in ((64, True), (128, True), (9, False)):
        B, C = torch.randn(N_COLS, K, device="cuda"), torch.empty(N, K, device="cuda")
        assert (_launches(lambda: pc.pcsr_spmm(h, B, C, K)) > 1) == several
        assert _launches(lambda: pc.pcsr_spmm(plain, B, C, K)) == 1
    pc.pcsr_set_kernel_params(h, lanes_per_row=16, vec=4, rep=4, waves_per_wg=4)  # a shape without a kernel for bands
    B, C = torch.randn(N_COLS, 256, device="cuda"), torch.empty(N, 256, device="cuda")
    assert _launches(lambda: pc.pcsr_spmm(h, B, C, 256)) == 1
    h.close()
    plain.close()


@pytest.mark.parametrize("K", [16, 48, 64, 100])
def test_tails(graph, K):
    rowptr, colidx, vals = graph
    rng = np.random.default_rng(K)
    B = rng.standard_normal((N_COLS, K)).astype(np.float32)
    h = pc.pcsr_build(N, N_COLS, *_dev(rowptr, colidx, vals), pc.make_params(flags=BANDS))
    C, expect = _tail(h, _dev(B)[0], K, rng)
    ref, bound = expect(*oracle.spmm(rowptr, colidx, vals, B))
    ok, worst = oracle.within_tolerance(C.cpu().numpy(), ref, bound)
    assert ok, worst
    h.close()


def test_a_tail_that_reads_c(graph):
    """C += A B, the self term being C itself, as products in one pass have it."""
    import ctypes

    from paper_2605_15695_amd import binding

    rowptr, colidx, vals = graph
    K, rng = 64, np.random.default_rng(0)
    B, S = rng.standard_normal((N_COLS, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
    h = pc.pcsr_build(N, N_COLS, *_dev(rowptr, colidx, vals), pc.make_params(flags=BANDS))
    b, C = _dev(B, S)
    epi = binding.pcsr_epilogue_t(None, C.data_ptr(), None, None, 0, 0)
    stream = torch.cuda.current_stream().cuda_stream
    assert binding._lib().pcsr_spmm_epilogue(h.raw, b.data_ptr(), C.data_ptr(), K, ctypes.byref(epi), stream) == 0
    ref, bound = oracle.spmm(rowptr, colidx, vals, B)
    ok, worst = oracle.within_tolerance(C.cpu().numpy(), ref + S, bound + np.abs(S))
    assert ok, worst
    h.close()


def test_not_finite(graph):
    """A row of B that is no number shows in the rows that read it and in no other."""
    rowptr, colidx, vals = graph
    K = 64
    B = torch.randn(N_COLS, K, device="cuda")
    touched = np.zeros(N, bool)
    for col, x in ((17, float("nan")), (N_COLS // 2, float("inf")), (N_COLS - 3, float("-inf"))):
        B[col] = x
        touched[np.searchsorted(rowptr, np.flatnonzero(colidx == col), "right") - 1] = True
    h = pc.pcsr_build(N, N_COLS, *_dev(rowptr, colidx, vals), pc.make_params(flags=BANDS))
    C = torch.empty(N, K, device="cuda")
    pc.pcsr_spmm(h, B, C, K)
    assert np.array_equal(~np.isfinite(C.cpu().numpy()).all(1), touched)
    h.close()


def test_capture_and_streams(graph):
    """The first product of a handle is captured, needs no workspace, and is the same bits on replays and on two streams at once."""
    rowptr, colidx, vals = graph
    K = 64
    h = pc.pcsr_build(N, N_COLS, *_dev(rowptr, colidx, vals), pc.make_params(flags=BANDS))
    B = torch.randn(N_COLS, K, device="cuda")
    C = [torch.empty(N, K, device="cuda") for _ in range(3)]
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        pc.pcsr_spmm_static(h, B, C[0], K, torch.cuda.current_stream())
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        streams = [torch.cuda.Stream() for _ in range(2)]
        for s, c in zip(streams, C[1:]):
            with torch.cuda.stream(s):
                pc.pcsr_spmm(h, B, c, K, s)
        torch.cuda.synchronize()
        assert torch.equal(C[0], C[1]) and torch.equal(C[0], C[2])
        B.mul_(-1.5)
        torch.cuda.synchronize()
    h.close()


def test_columns_in_any_order(graph):
    """Without the check of the CSR a row's columns may come in any order: every vector is in one band all the same."""
    rowptr, colidx, vals = graph
    K, rng = 64, np.random.default_rng(1)
    order = np.lexsort((rng.random(colidx.size), np.repeat(np.arange(N), np.diff(rowptr))))
    B = rng.standard_normal((N_COLS, K)).astype(np.float32)
    h = pc.pcsr_build(N, N_COLS, *_dev(rowptr, colidx[order], vals[order]), pc.make_params(flags=BANDS | pc.PCSR_FLAG_NO_VALIDATE))
    C = torch.empty(N, K, device="cuda")
    pc.pcsr_spmm(h, _dev(B)[0], C, K)
    ok, worst = oracle.within_tolerance(C.cpu().numpy(), *oracle.spmm(rowptr, colidx, vals, B))
    assert ok, worst
    h.close()
