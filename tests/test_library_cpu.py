"""CPU-side checks of the C-ABI library: exported symbols, host PCSR generation bit-exact
against the numpy format reference, feature extraction, error paths.  No GPU calls."""
import ctypes
import pathlib
import re

import numpy as np
import pytest

import paper_2605_15695_amd as pc
from oracle import pcsr_format as pf
import synth
from paper_2605_15695_amd import binding
from tests.helpers import column_ordered_schedule, near_diagonal_share, random_csr

ROOT = pathlib.Path(__file__).resolve().parent.parent
HOST = pc.PCSR_FLAG_HOST_ONLY


def _bits(a):
    return a.view(np.uint32) if a.dtype == np.float32 else a


def _assert_same(e, r):
    for k in ("P", "M", "nnz_v", "V", "SG"):
        assert e[k] == r[k], k
    for k in ("rowptr", "colidx", "val", "trow"):
        assert e[k].dtype == r[k].dtype and np.array_equal(_bits(e[k]), _bits(r[k])), k


def test_every_declared_symbol_is_exported():
    header = (ROOT / "include" / "pcsr.h").read_text()
    names = set(re.findall(r"^(?:int|int32_t|int64_t|const char \*)\s*(pcsr_[a-z_]+)\(", header, re.M))
    assert len(names) >= 11
    assert {"pcsr_build", "pcsr_spmm", "pcsr_free"} <= names
    lib = ctypes.CDLL(str(binding.LIB_PATH))
    for n in sorted(names):
        assert hasattr(lib, n), n


@pytest.mark.parametrize("name", ["poisson", "road", "rmat20", "sbm", "sbm_shuffled", "rmat22"])
@pytest.mark.parametrize("V", [1, 2])
@pytest.mark.parametrize("S,SG,omega", [(0, 0, 0), (1, 0, 0), (1, 0, 32), (1, 5, 0)])
def test_host_generation_bit_exact(name, V, S, SG, omega):
    g = synth.workload(name, "small")
    h = pc.pcsr_build(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals,
                      pc.make_params(V=V, S=S, SG=SG, omega=omega, flags=HOST))
    _assert_same(pc.pcsr_export(h), pf.pcsr_ref(g.n_rows, g.rowptr, g.colidx, g.vals, V, S, SG, omega or 64))
    h.close()


@pytest.mark.parametrize("n", [0, 1, 2, 3, 17])
@pytest.mark.parametrize("V", [1, 2])
@pytest.mark.parametrize("S", [0, 1])
def test_host_generation_tiny_and_degenerate(n, V, S):
    rng = np.random.default_rng(n + 7)
    if n == 0:
        rowptr, colidx, vals = np.zeros(1, np.int32), np.zeros(0, np.int32), np.zeros(0, np.float32)
    else:
        rowptr, colidx, vals, _ = random_csr(rng, n, n + 2, 0.4, empty_rows=(0,) if n > 1 else ())
    h = pc.pcsr_build(n, n + 2, rowptr, colidx, vals, pc.make_params(V=V, S=S, SG=2 if S else 0, flags=HOST))
    _assert_same(pc.pcsr_export(h), pf.pcsr_ref(n, rowptr, colidx, vals, V, S, 2 if S else 0, 64))


def test_explicit_zero_is_kept_as_a_vector():
    rowptr = np.array([0, 2, 3], np.int32)
    colidx = np.array([1, 4, 2], np.int32)
    vals = np.array([0.0, 3.0, -0.0], np.float32)
    for V in (1, 2):
        h = pc.pcsr_build(2, 5, rowptr, colidx, vals, pc.make_params(V=V, flags=HOST))
        e = pc.pcsr_export(h)
        _assert_same(e, pf.pcsr_ref(2, rowptr, colidx, vals, V, 0))
        assert e["nnz_v"] == 3


@pytest.mark.parametrize("name", ["poisson", "road", "rmat20", "sbm"])
@pytest.mark.parametrize("omega", [32, 64])
def test_features_match_reference(name, omega):
    g = synth.workload(name, "small")
    f = pc.pcsr_features(g.n_rows, g.n_cols, g.rowptr, g.colidx, omega)
    r = pf.features(g.n_rows, g.n_cols, g.rowptr, g.colidx, omega)
    assert np.allclose(f[:16], r, rtol=1e-12, atol=0)          # Table 3
    assert f[14] == 0.0 and 0.0 <= f[15] <= 0.5 and f[9] >= 1.0 and f[10] >= 1.0
    assert f[16] == pytest.approx(near_diagonal_share(g.rowptr, g.colidx), rel=1e-12)   # the library's own


def test_near_diagonal_feature_closed_forms():
    n = 3000
    eye_rp, eye_ci = np.arange(n + 1, dtype=np.int32), np.arange(n, dtype=np.int32)
    assert pc.pcsr_features(n, n, eye_rp, eye_ci)[16] == 1.0
    far = ((np.arange(n) + 512) % n).astype(np.int32)            # every nonzero exactly 512 (or more) away
    assert pc.pcsr_features(n, n, eye_rp, far)[16] == 0.0
    near = ((np.arange(n) + 511) % n).astype(np.int32)
    assert pc.pcsr_features(n, n, eye_rp, near)[16] == pytest.approx((n - 511) / n)
    assert pc.pcsr_features(3, 5, np.zeros(4, np.int32), np.zeros(0, np.int32))[16] == 0.0


def test_gap_export_matches_table2():
    for line in (ROOT / "tests/golden/table2_gap.txt").read_text().splitlines():
        if line.strip() and not line.startswith("#"):
            dim, F, gap = map(int, line.split())
            assert pc.pcsr_mac_job_gap(dim, F, 32) == gap
    assert pc.pcsr_mac_job_gap(0, 1, 32) == -1


def _expect(code, *args, **kw):
    with pytest.raises(pc.PcsrError) as ei:
        pc.pcsr_build(*args, **kw)
    assert ei.value.code == code


def test_error_paths():
    rp = np.array([0, 2, 3], np.int32)
    ci = np.array([0, 1, 2], np.int32)
    va = np.ones(3, np.float32)
    P = lambda **k: pc.make_params(flags=HOST, **k)  # noqa: E731
    _expect(binding.PCSR_E_UNSUPPORTED, 2, 3, rp, ci, va, P(V=3))
    _expect(binding.PCSR_E_UNSUPPORTED, 2, 3, rp, ci, va, P(S=2))
    _expect(binding.PCSR_E_UNSUPPORTED, 2, 3, rp, ci, va, P(lanes_per_row=3))
    _expect(binding.PCSR_E_UNSUPPORTED, 2, 3, rp, ci, va, P(vec=3))
    _expect(binding.PCSR_E_UNSUPPORTED, 2, 3, rp, ci, va, P(waves_per_wg=3))
    _expect(binding.PCSR_E_INVALID_ARG, 2, 3, rp, ci, va, P(SG=-1))
    # malformed CSR
    _expect(binding.PCSR_E_BAD_CSR, 2, 3, np.array([0, 3, 2], np.int32), ci, va, P())        # not monotone
    _expect(binding.PCSR_E_BAD_CSR, 2, 3, np.array([1, 2, 3], np.int32), ci, va, P())        # start != 0
    _expect(binding.PCSR_E_BAD_CSR, 2, 3, np.array([0, 2, 2], np.int32), ci, va, P())        # end != nnz
    _expect(binding.PCSR_E_BAD_CSR, 2, 3, rp, np.array([0, 3, 2], np.int32), va, P())        # col >= n_cols
    _expect(binding.PCSR_E_BAD_CSR, 2, 3, rp, np.array([0, -1, 2], np.int32), va, P())       # negative col
    _expect(binding.PCSR_E_BAD_CSR, 2, 3, rp, np.array([1, 0, 2], np.int32), va, P())        # unsorted
    _expect(binding.PCSR_E_BAD_CSR, 2, 3, rp, np.array([1, 1, 2], np.int32), va, P())        # duplicate
    # reserved must be zero
    p = P()
    p.reserved[0] = 5
    _expect(binding.PCSR_E_INVALID_ARG, 2, 3, rp, ci, va, p)
    # SpMM on a host-only handle is refused, never silently computed elsewhere
    h = pc.pcsr_build(2, 3, rp, ci, va, P())
    lib = binding._lib()
    assert lib.pcsr_spmm(h.raw, None, None, 4, None) == binding.PCSR_E_UNSUPPORTED
    assert lib.pcsr_spmm(None, None, None, 4, None) == binding.PCSR_E_INVALID_ARG
    assert lib.pcsr_free(None) == 0
    assert "CSR" in pc.pcsr_strerror(binding.PCSR_E_BAD_CSR)


def test_launch_resolution():
    g = synth.workload("poisson", "small")
    h = pc.pcsr_build(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, pc.make_params(flags=HOST))
    q = pc.pcsr_query_launch(h, 8)
    assert (q["lanes_per_row"], q["vec"], q["rep"]) == (4, 4, 1) and q["grid_y"] == 1
    q = pc.pcsr_query_launch(h, 16)                      # rows of 8 on average: 16 lanes of one dword
    assert (q["lanes_per_row"], q["vec"], q["rep"]) == (16, 1, 1) and q["grid_y"] == 1
    per_wg = q["waves_per_wg"] * 4
    # one work-balanced item range per XCD: 8 x the workgroups of the longest range
    assert q["grid_x"] % 8 == 0 and -(-g.n_rows // per_wg) <= q["grid_x"] <= -(-g.n_rows // per_wg) + 64
    pc.pcsr_set_kernel_params(h, flags=pc.PCSR_FLAG_NO_XCD_REMAP)
    assert pc.pcsr_query_launch(h, 16)["grid_x"] == -(-g.n_rows // per_wg)
    pc.pcsr_set_kernel_params(h)
    q = pc.pcsr_query_launch(h, 512)
    assert q["lanes_per_row"] * q["vec"] * q["rep"] * q["grid_y"] >= 512
    q = pc.pcsr_query_launch(h, 33)
    assert q["vec"] == 1 and q["lanes_per_row"] * q["rep"] * q["grid_y"] >= 33
    pc.pcsr_set_kernel_params(h, 8, 2, 2, 1)
    q = pc.pcsr_query_launch(h, 128)
    assert (q["lanes_per_row"], q["vec"], q["rep"], q["waves_per_wg"], q["grid_y"]) == (8, 2, 2, 1, 4)
    with pytest.raises(pc.PcsrError):
        pc.pcsr_query_launch(h, 33)          # vec = 2 does not divide 33
    with pytest.raises(pc.PcsrError):
        pc.pcsr_set_kernel_params(h, 5, 0, 0, 0)
    with pytest.raises(pc.PcsrError):
        pc.pcsr_set_kernel_params(h, items_per_group=3)
    pc.pcsr_set_kernel_params(h, 32, 4, 1, 4, 4)
    q = pc.pcsr_query_launch(h, 128)
    assert q["items_per_group"] == 4 and q["grid_x"] % 8 == 0
    assert -(-g.n_rows // (4 * 2 * 4)) <= q["grid_x"] <= -(-g.n_rows // (4 * 2 * 4)) + 64
    pc.pcsr_set_kernel_params(h, 4, 4, 1, 4, 4)          # items_per_group must be < lanes_per_row
    with pytest.raises(pc.PcsrError):
        pc.pcsr_query_launch(h, 16)


def test_select_returns_valid_tuple():
    for name in ("road", "rmat20", "sbm"):
        g = synth.workload(name, "small")
        f = pc.pcsr_features(g.n_rows, g.n_cols, g.rowptr, g.colidx)
        p = pc.pcsr_select(f, 64)
        assert p.V in (1, 2) and p.S in (0, 1)
    assert pc.pcsr_select(pc.pcsr_features(*(lambda g: (g.n_rows, g.n_cols, g.rowptr, g.colidx))(
        synth.workload("road", "small"))), 64).S == 0


def test_select_always_returns_a_tuple_the_library_can_launch():
    """Whatever the features (random, extreme, non-finite) and the width, the rule returns
    parameters inside the documented domains, and a handle built from them resolves to a
    launch shape that exists."""
    rng = np.random.default_rng(11)
    g = synth.workload("sbm", "small")
    base = np.array(pc.pcsr_features(g.n_rows, g.n_cols, g.rowptr, g.colidx), dtype=np.float64)
    handles = {}
    for trial in range(400):
        f = base.copy()
        if trial % 4:
            f[0] = f[1] = float(rng.choice([1, 50, 4096, 90_000, 250_000, 4_000_000, 2**31 - 1]))
            f[4] = f[5] = float(rng.choice([0.0, 1.0, 3.0, 7.9, 12.0, 39.9, 40.0, 200.0, 1e5]))
            f[6] = f[5] * float(rng.choice([1.0, 2.0, 100.0, 1e4]))
            f[7] = f[8] = float(rng.choice([0.0, 0.1, 1.49, 1.51, 8.0]))
            f[15] = float(rng.choice([0.0, 0.1, 0.19, 0.2, 0.3, 0.45, 0.5]))
            f[16] = float(rng.choice([0.0, 1e-4, 0.01, 0.3, 0.6, 0.9, 1.0]))
        if trial % 50 == 49:
            f[int(rng.integers(0, f.shape[0]))] = float(rng.choice([np.nan, np.inf, -np.inf, -1.0]))
        K = int(rng.choice([1, 2, 3, 7, 8, 9, 12, 16, 17, 24, 32, 33, 48, 64, 96, 100, 128, 255, 256, 512, 2048]))
        p = pc.pcsr_select(f, K)
        assert p.V in (1, 2) and p.S in (0, 1) and p.SG >= 0 and p.omega in (0, 32, 64)
        assert p.lanes_per_row in (4, 8, 16, 32, 64) and p.vec in (1, 2, 4) and K % p.vec == 0
        assert p.rep in (1, 2, 4) and 1 <= p.waves_per_wg <= 16 and p.items_per_group in (0, 1)
        assert p.col_window in (0, 512)
        if p.col_window:
            assert (p.col_window + 1) * (p.lanes_per_row * p.vec * p.rep + 4) * 4 <= 160 * 1024
            assert p.S == 0 and p.V == 1 and p.flags & pc.PCSR_FLAG_WINDOW_IF_USEFUL
        if p.flags & pc.PCSR_FLAG_COLUMN_ORDER:
            assert p.S == 1
        # the launch shape exists for a handle of that format (built once per format)
        key = (p.V, p.S, min(p.SG, 64), p.col_window, p.flags & pc.PCSR_FLAG_COLUMN_ORDER)
        if key not in handles:
            handles[key] = pc.pcsr_build(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, pc.make_params(
                V=p.V, S=p.S, SG=key[2], col_window=p.col_window, flags=HOST | key[4]))
        h = handles[key]
        pc.pcsr_set_kernel_params(h, p.lanes_per_row, p.vec, p.rep, p.waves_per_wg, 0)
        q = pc.pcsr_query_launch(h, K)
        assert q["lanes_per_row"] == p.lanes_per_row and q["vec"] == p.vec and q["grid_y"] >= 1
        assert q["lanes_per_row"] * q["vec"] * q["rep"] * q["grid_y"] >= K
    for h in handles.values():
        h.close()


def test_reorder_is_a_permutation_and_recovers_planted_clusters():
    g = synth.workload("sbm_shuffled", "small")          # 24 blocks of 500, ids shuffled
    perm, ncl = pc.pcsr_reorder(g.n_rows, g.rowptr, g.colidx)
    assert np.array_equal(np.sort(perm), np.arange(g.n_rows))
    assert ncl == 24
    perm2, _ = pc.pcsr_reorder(g.n_rows, g.rowptr, g.colidx)
    assert np.array_equal(perm, perm2)                   # deterministic
    rp, ci, va = pc.pcsr_permute_csr(g.n_rows, g.rowptr, g.colidx, g.vals, perm)
    # the relabelled matrix is P A P^T: compare with scipy
    import scipy.sparse as sp
    A = sp.csr_matrix((g.vals, g.colidx, g.rowptr), shape=(g.n_rows, g.n_cols)).tocoo()
    A2 = sp.csr_matrix((A.data, (perm[A.row], perm[A.col])), shape=A.shape)
    A2.sort_indices()
    assert np.array_equal(rp, A2.indptr) and np.array_equal(ci, A2.indices)
    assert np.array_equal(va.view(np.uint32), A2.data.astype(np.float32).view(np.uint32))
    # rows of one planted block end up contiguous: the average row bandwidth collapses
    b_before = pc.pcsr_features(g.n_rows, g.n_cols, g.rowptr, g.colidx)[12]
    b_after = pc.pcsr_features(g.n_rows, g.n_cols, rp, ci)[12]
    assert b_after < 0.8 * b_before
    h = pc.pcsr_build(g.n_rows, g.n_cols, rp, ci, va, pc.make_params(col_window=1024, flags=HOST))
    assert pc.pcsr_window_stats(h)["hit_fraction"] > 0.85


def test_reorder_error_paths_and_degenerate_inputs():
    perm, ncl = pc.pcsr_reorder(0, np.zeros(1, np.int32), np.zeros(0, np.int32))
    assert perm.size == 0 and ncl == 0
    perm, ncl = pc.pcsr_reorder(5, np.zeros(6, np.int32), np.zeros(0, np.int32))
    assert np.array_equal(perm, np.arange(5)) and ncl == 5
    with pytest.raises(pc.PcsrError):
        pc.pcsr_reorder(2, np.array([0, 1, 2], np.int32), np.array([0, 5], np.int32))
    with pytest.raises(pc.PcsrError):
        pc.pcsr_permute_csr(2, np.array([0, 1, 2], np.int32), np.array([0, 1], np.int32),
                            np.ones(2, np.float32), np.array([0, 0], np.int32))
    # a column outside [0, n) cannot be relabelled: an error, not a silently wrong row
    for bad in (5, -1):
        with pytest.raises(pc.PcsrError) as ei:
            pc.pcsr_permute_csr(2, np.array([0, 1, 2], np.int32), np.array([0, bad], np.int32),
                                np.ones(2, np.float32), np.array([1, 0], np.int32))
        assert ei.value.code == binding.PCSR_E_BAD_CSR


def test_workspace_size_of_the_balanced_write_back():
    """V*K floats per work item of every panel that was split; nothing without balancing or
    with the atomic write-back."""
    g = synth.workload("rmat20", "small")
    for V in (1, 2):
        h = pc.pcsr_build(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, pc.make_params(V=V, S=1, SG=16, flags=HOST))
        r = pf.pcsr_ref(g.n_rows, g.rowptr, g.colidx, g.vals, V, 1, 16, 64)
        per_panel = np.bincount(r["trow"], minlength=r["P"])
        slots = int(per_panel[per_panel > 1].sum())
        assert slots > 0
        assert pc.pcsr_workspace_bytes(h, 40) == slots * V * 40 * 4
        pc.pcsr_set_kernel_params(h, flags=pc.PCSR_FLAG_ATOMIC_SPLIT)
        assert pc.pcsr_workspace_bytes(h, 40) == 0
        with pytest.raises(pc.PcsrError):
            pc.pcsr_reserve_workspace(h, 40)              # host-only handle: nothing to reserve on
        h.close()
    h = pc.pcsr_build(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, pc.make_params(V=1, S=0, flags=HOST))
    assert pc.pcsr_workspace_bytes(h, 40) == 0
    h.close()


def test_transpose_csr_host():
    import scipy.sparse as sp
    rng = np.random.default_rng(4)
    rowptr, colidx, vals, dense = random_csr(rng, 13, 29, 0.3, empty_rows=(2,))
    trp, tci, tva = pc.pcsr_transpose_csr(13, 29, rowptr, colidx, vals)
    At = sp.csr_matrix(dense.T)
    At.sort_indices()
    assert np.array_equal(trp, At.indptr) and np.array_equal(tci, At.indices)
    assert np.array_equal(tva, At.data)
    with pytest.raises(pc.PcsrError):
        pc.pcsr_transpose_csr(2, 2, np.array([0, 1, 2], np.int32), np.array([0, 7], np.int32),
                              np.ones(2, np.float32))


@pytest.mark.parametrize("name", ["rmat20", "rmat22", "sbm", "poisson"])
@pytest.mark.parametrize("V,SG", [(1, 4), (2, 16), (1, 0)])
def test_column_ordered_schedule_host(name, V, SG):
    g = synth.workload(name, "small")
    h = pc.pcsr_build(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals,
                      pc.make_params(V=V, S=1, SG=SG, flags=HOST | pc.PCSR_FLAG_COLUMN_ORDER))
    e = pc.pcsr_export(h)
    got = pc.pcsr_export_schedule(h)
    sched, xb = column_ordered_schedule(e["rowptr"], e["colidx"], e["trow"], e["P"])
    assert np.array_equal(got["xcd_bounds"], xb)
    assert np.array_equal(got["sched"], sched)
    # a permutation of the items: every vector range appears exactly once
    assert np.array_equal(np.sort(got["sched"][:, 0] * 1), np.sort(e["rowptr"][:-1]))
    h.close()
    h = pc.pcsr_build(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, pc.make_params(V=V, S=1, SG=SG, flags=HOST))
    assert pc.pcsr_export_schedule(h)["sched"] is None
    h.close()
    with pytest.raises(pc.PcsrError):                       # needs balancing
        pc.pcsr_build(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals,
                      pc.make_params(V=V, S=0, flags=HOST | pc.PCSR_FLAG_COLUMN_ORDER))


def test_reorder_by_degree():
    g = synth.workload("rmat20", "small")
    perm = pc.pcsr_reorder_by_degree(g.n_rows, g.rowptr, g.colidx)
    assert np.array_equal(np.sort(perm), np.arange(g.n_rows))
    indeg = np.bincount(g.colidx, minlength=g.n_cols)
    # new id = rank by descending in-degree, ties in original order
    expect = np.empty(g.n_rows, np.int32)
    expect[np.argsort(-indeg, kind="stable")] = np.arange(g.n_rows)
    assert np.array_equal(perm, expect)
    rp, ci, va = pc.pcsr_permute_csr(g.n_rows, g.rowptr, g.colidx, g.vals, perm)
    indeg2 = np.bincount(ci, minlength=g.n_cols)
    assert np.all(np.diff(indeg2) <= 0)                      # hubs first
    with pytest.raises(pc.PcsrError):
        pc.pcsr_reorder_by_degree(2, np.array([0, 1, 2], np.int32), np.array([0, 5], np.int32))
    assert pc.pcsr_reorder_by_degree(0, np.zeros(1, np.int32), np.zeros(0, np.int32)).size == 0


def test_selector_pairs_short_rows_unless_their_rows_of_c_are_part_lines():
    g = synth.workload("road", "small")
    f = np.array(pc.pcsr_features(g.n_rows, g.n_cols, g.rowptr, g.colidx))
    assert f[5] < 6.0 and 0.2 <= f[15]
    for n, single in ((2_000_000, (12, 16)), (167_000, (12, 16)), (166_000, (16,)), (125_000, (16,)), (124_000, ())):
        f[0] = n
        for K in (8, 9, 10, 12, 13, 16, 17, 20, 24, 32, 64):
            assert pc.pcsr_select(f, K).V == (1 if K in single else 2), (n, K)
    f[0], f[15] = 2_000_000, 0.1  # neighbouring rows that share their columns stay paired
    assert pc.pcsr_select(f, 16).V == 2


def test_selector_proposes_the_window_only_where_the_build_keeps_it():
    g = synth.workload("sbm", "small")                       # 24 communities of 500 consecutive ids
    f = np.array(pc.pcsr_features(g.n_rows, g.n_cols, g.rowptr, g.colidx), dtype=np.float64)
    # 12,000 rows give 24 window blocks: far too few for 256 compute units, so no window
    small = pc.pcsr_select(f, 128)
    assert small.col_window == 0 and small.S == 0 and small.V == 1
    f[0] = f[1] = 250_000                                    # the same structure at the full size
    assert pc.pcsr_select(f, 32).col_window == 0            # narrow B rows: the plain kernel ties
    assert pc.pcsr_select(f, 64).col_window == 512
    f[0] = f[1] = 150_000
    assert pc.pcsr_select(f, 64).col_window == 0            # 150,000 rows x 1 slice: too few blocks
    f[0] = f[1] = 250_000
    sel = pc.pcsr_select(f, 128)
    assert sel.col_window == 512 and sel.S == 0 and sel.flags & pc.PCSR_FLAG_WINDOW_IF_USEFUL
    sel.flags |= HOST
    h = pc.pcsr_build(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, sel)
    st = pc.pcsr_window_stats(h)
    assert st["col_window"] == 512 and st["hit_fraction"] > 0.85 and 400 <= st["items_per_block"] <= 500
    assert pc.pcsr_query_launch(h, 128)["lds_bytes"] > 0
    h.close()
    # the same request on the shuffled graph: the build finds no blocks and drops the window
    gs = synth.workload("sbm_shuffled", "small")
    fs = np.array(pc.pcsr_features(gs.n_rows, gs.n_cols, gs.rowptr, gs.colidx), dtype=np.float64)
    shuffled = pc.pcsr_select(fs, 128)
    # long rows, scattered columns: items of 32 in column order from K = 64, paired rows below
    assert shuffled.col_window == 0 and shuffled.S == 1 and shuffled.SG == 32
    assert shuffled.flags & pc.PCSR_FLAG_COLUMN_ORDER and shuffled.lanes_per_row == 16
    narrow = pc.pcsr_select(fs, 32)                           # too few rows to pair them
    assert narrow.S == 0 and narrow.V == 1 and narrow.col_window == 0
    fs[0] = fs[1] = 250_000
    fs[16] = 0.002                                            # near-diagonal share of uniform columns at that size
    assert pc.pcsr_select(fs, 128).col_window == 0
    narrow = pc.pcsr_select(fs, 32)                           # B = 32 MB, scattered: a dword per lane
    assert (narrow.S, narrow.V, narrow.lanes_per_row, narrow.vec, narrow.rep) == (0, 1, 32, 1, 1)
    fs[0] = fs[1] = 100_000                                   # B = 12.8 MB: rows paired instead
    fs[16] = 0.005
    narrow = pc.pcsr_select(fs, 32)
    assert narrow.S == 0 and narrow.V == 2 and narrow.waves_per_wg == 2 and narrow.vec == 4
    k16 = pc.pcsr_select(fs, 16)                              # K = 16: 16 lanes of one dword
    assert (k16.lanes_per_row, k16.vec, k16.rep) == (16, 1, 1)
    road = synth.workload("road", "small")
    fr = pc.pcsr_features(road.n_rows, road.n_cols, road.rowptr, road.colidx)
    r16 = pc.pcsr_select(fr, 16)                              # rows of 3: many rows per wavefront
    assert (r16.V, r16.lanes_per_row, r16.vec) == (2, 4, 4)
    h = pc.pcsr_build(gs.n_rows, gs.n_cols, gs.rowptr, gs.colidx, gs.vals, sel)
    assert pc.pcsr_window_stats(h)["col_window"] == 0
    q = pc.pcsr_query_launch(h, 128)
    assert q["lds_bytes"] == 0 and q["waves_per_wg"] <= 8
    h.close()
    # without the flag the window blocks are kept whatever they look like
    h = pc.pcsr_build(gs.n_rows, gs.n_cols, gs.rowptr, gs.colidx, gs.vals, pc.make_params(col_window=512, flags=HOST))
    assert pc.pcsr_window_stats(h)["col_window"] == 512
    h.close()


def test_selector_walks_scattered_rows_in_bands():
    """Where a B of scattered rows outgrows L2 and the product saves what the table costs; never for rows that are split or local."""
    g = synth.workload("sbm_shuffled", "small")
    f = np.array(pc.pcsr_features(g.n_rows, g.n_cols, g.rowptr, g.colidx), dtype=np.float64)

    def pick(n, deg, K, near=0.0, cv=0.1, d_max=None):
        x = f.copy()
        x[0] = x[1] = n
        x[2], x[4], x[5], x[6], x[7], x[8], x[15], x[16] = n * deg, deg / n, deg, d_max or 2 * deg, cv, cv, 0.5, near
        return pc.pcsr_select(x, K)

    for n, deg, K, bands, shape in ((300_000, 134, 16, True, (16, 1, 1)), (300_000, 134, 32, True, (32, 1, 1)), (300_000, 134, 48, True, (16, 4, 1)),
                                    (100_000, 90, 128, True, (16, 4, 1)), (60_000, 90, 16, False, (16, 1, 1)), (400_000, 9, 16, False, (16, 1, 1)),
                                    (1_000_000, 30, 64, False, (32, 2, 1)), (1_000_000, 44, 128, True, (32, 2, 1))):
        p = pick(n, deg, K)
        assert (p.V, p.S, p.lanes_per_row, p.vec, p.rep) == (1, 0, *shape), (n, deg, K)
        assert bool(p.flags & pc.PCSR_FLAG_COLUMN_BANDS) == bands, (n, deg, K)
    for p in (pick(300_000, 134, 16, near=0.9), pick(300_000, 134, 16, cv=4.0, d_max=20_000), pick(40_000, 134, 64),
              pick(300_000, 134, 128, d_max=2000), pick(300_000, 134, 300)):
        assert not p.flags & pc.PCSR_FLAG_COLUMN_BANDS
    # none of them asks for more alignment or a workspace where it did not, and none splits rows that were not
    assert pick(300_000, 134, 62).vec == 2 and pick(300_000, 134, 63).vec == 1


def test_selector_gives_narrow_rows_more_lanes_than_columns():
    """Up to 8 columns: 16 lanes of one dword for long rows, 8 for items of split ones; short local rows and odd widths keep their shape."""
    g = synth.workload("sbm", "small")
    f = np.array(pc.pcsr_features(g.n_rows, g.n_cols, g.rowptr, g.colidx), dtype=np.float64)

    def pick(deg, K, near=0.9, cv=0.1, d_max=100):
        x = f.copy()
        x[0] = x[1] = 200_000
        x[2], x[4], x[5], x[6], x[7], x[8], x[15], x[16] = x[0] * deg, deg / x[0], deg, d_max, cv, cv, 0.5, near
        p = pc.pcsr_select(x, K)
        return p.S, p.lanes_per_row, p.vec, p.rep

    for K in (2, 4, 6, 8):
        assert pick(16, K) == (0, 16, 1, 1) and pick(9, K, near=0.0) == (0, 16, 1, 1)
        assert pick(40, K, cv=4.0, d_max=20_000) == (1, 8, 1, 1)
        assert pick(15, K)[1:] == (4, 4 if K % 4 == 0 else 2, 1) and pick(7, K, near=0.0)[2] > 1
    for K, lanes in ((1, 4), (3, 4), (5, 8), (7, 8)):
        assert pick(19, K) == (0, lanes, 1, 1) and pick(40, K) == (0, 16, 1, 1)
        assert pick(40, K, cv=4.0, d_max=20_000) == (1, lanes, 1, 1)


def test_query_kernel_reports_what_is_launched():
    """The shape that stands in where the one asked for reads rows badly; elsewhere the two queries agree."""
    shape = lambda q: (q["lanes_per_row"], q["vec"], q["rep"])  # noqa: E731
    g = synth.workload("sbm_shuffled", "small")
    plain = pc.pcsr_build(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, pc.make_params(flags=HOST))
    assert shape(pc.pcsr_query_launch(plain, 75)) == (64, 1, 2)
    q = pc.pcsr_query_kernel(plain, 75)
    assert shape(q) == (32, 4, 1) and q["grid_y"] == 1 and q["grid_x"] > 0
    for K in (8, 16, 32, 64, 128, 512):
        assert pc.pcsr_query_launch(plain, K) == pc.pcsr_query_kernel(plain, K)
    pc.pcsr_set_kernel_params(plain, 8, 1, 2)                # a shape asked for is the shape launched
    assert shape(pc.pcsr_query_kernel(plain, 75)) == (8, 1, 2)
    plain.close()
    p = pc.pcsr_select(pc.pcsr_features(g.n_rows, g.n_cols, g.rowptr, g.colidx), 75)
    p.flags |= HOST
    h = pc.pcsr_build(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, p)
    assert shape(pc.pcsr_query_launch(h, 75)) == (p.lanes_per_row, p.vec, p.rep)
    q = pc.pcsr_query_kernel(h, 75)
    assert q["vec"] == 4 and q["lanes_per_row"] * 4 * q["rep"] * q["grid_y"] >= 75
    h.close()


def test_shapes_passed_in_flags_hold_only_for_the_shape_they_came_with():
    g = synth.workload("sbm_shuffled", "small")
    args = (g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals)
    f = pc.pcsr_features(g.n_rows, g.n_cols, g.rowptr, g.colidx)
    launched = lambda p, K: (lambda q: (q["lanes_per_row"], q["vec"], q["rep"]))(  # noqa: E731
        pc.pcsr_query_kernel(pc.pcsr_build(*args, p), K))
    carried = 0
    for K in (18, 27, 33, 40, 75, 100, 130, 300, 515):
        p = pc.pcsr_select(f, K)
        p.flags |= HOST
        own, taken = (p.lanes_per_row, p.vec, p.rep), launched(p, K)
        carried += taken != own
        for field, value in (("lanes_per_row", 8), ("vec", 2 if p.vec == 1 and K % 2 == 0 else 1), ("rep", 4)):
            changed = type(p).from_buffer_copy(p)
            if getattr(changed, field) == value:
                continue
            setattr(changed, field, value)
            assert launched(changed, K) == (changed.lanes_per_row, changed.vec, changed.rep), (K, field)
    assert carried >= 5
    # bits that pcsr_select never sets, among them codes for 128 and 256 lanes per row
    for bits in [code << 16 for code in range(8)] + [0xfff << 16, 24 << 16, 0xfe0 << 16]:
        p = pc.make_params(lanes_per_row=8, vec=1, rep=1, flags=HOST | bits)
        assert launched(p, 33) == (8, 1, 1), hex(bits)


def _features(name, **fields):
    g = synth.workload(name, "small")
    f = np.array(pc.pcsr_features(g.n_rows, g.n_cols, g.rowptr, g.colidx), dtype=np.float64)
    for k, v in fields.items():
        f[pc.FEATURE_NAMES.index(k)] = v
    return f


def test_item_size_of_power_law_inputs():
    near = 16 / (1 << 19)                                    # permuted ids
    small = _features("rmat20", n=1 << 19, nnz=14e6, d_max=30_000, CV=8.0, near_512=near)
    large = _features("rmat20", n=1 << 20, nnz=16e6, d_max=30_000, CV=8.0, near_512=near)
    for K in (8, 16, 32, 48):
        assert pc.pcsr_select(small, K).SG == 32 and pc.pcsr_select(large, K).SG == 64
    for K in (64, 75, 100, 300):
        assert pc.pcsr_select(small, K).SG == 64 and pc.pcsr_select(large, K).SG == 64
    natural = _features("rmat22", n=1 << 22, nnz=128e6, d_max=100_000, CV=10.0, near_512=0.1)
    assert pc.pcsr_select(natural, 32).SG == 64 and pc.pcsr_select(natural, 64).SG == 32


def test_half_a_wavefront_per_row_only_where_b_is_gathered_from_memory():
    launched = lambda n, d, K: (lambda p: p.flags >> 16 & 7)(pc.pcsr_select(  # noqa: E731
        _features("poisson", n=n, nnz=n * d, d=d, d_hat=d, d_max=2 * d, CV=0.2, PR_2=0.49, near_512=1000 / n), K))
    for K in (40, 52, 60):
        assert launched(30_000, 20.0, K) == launched(90_000, 72.0, K) == 0     # the shape asked for: 16 lanes of 4
        assert launched(250_000, 20.0, K) == launched(500_000, 9.0, K) == 4    # 32 lanes
    assert launched(30_000, 20.0, 33) == 3 and launched(250_000, 20.0, 33) == 4


def test_no_search_for_communities_where_it_would_split_a_row_that_is_whole():
    """A product on a handle with S = 0 needs no workspace; in the order by community rows of over 1024 are split."""
    def picked(d, d_max):
        return pc.pcsr_select(_features("poisson", n=250_000, nnz=250_000 * d, d=d, d_hat=d, d_max=d_max, CV=0.4, PR_2=0.5,
                                        near_512=1000 / 250_000), 512)

    flag = pc.PCSR_FLAG_CLUSTER_IF_USEFUL
    for d_max in (40, 1024):
        assert picked(20.0, d_max).S == 0 and picked(20.0, d_max).flags & flag
    assert picked(20.0, 1025).S == 0 and not picked(20.0, 1025).flags & flag
    assert picked(48.0, 1025).S == 1 and picked(48.0, 1025).flags & flag   # split as it is


def _uniform(n, deg, **fields):
    """Features of rows of about deg scattered columns."""
    return _features("poisson", **{**dict(n=n, n_hat=n, nnz=n * deg, d=deg / n, d_hat=deg, d_max=2 * deg, CV=0.2, CV_hat=0.2, PR_2=0.5,
                                         near_512=1000 / n), **fields})


def _small():
    g = synth.workload("poisson", "small")
    return g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals


def _chosen_for(f, K):
    """pcsr_select's parameters and a (small) handle that has them."""
    p = pc.pcsr_select(f, K)
    p.flags |= HOST
    return p, pc.pcsr_build(*_small(), p)


def _kernel(h, K):
    q = pc.pcsr_query_kernel(h, K)
    return q["lanes_per_row"], q["vec"], q["rep"]


# a B that L2 holds; one that is walked in bands; one of neither
@pytest.mark.parametrize("n,deg,hint,launched", [(8_000, 22, 128, (16, 4, 1)), (20_000, 12, 192, (16, 4, 1)), (60_000, 36, 256, (16, 4, 1)),
                                                 (400_000, 20, 128, (32, 2, 1))])
def test_a_handle_takes_every_even_width_whatever_its_shape_gains(n, deg, hint, launched):
    """Rows of 8 to 40 scattered columns, from K = 64 on: two floats a lane are what widths and operands are held against."""
    p, h = _chosen_for(_uniform(n, deg), hint)
    assert (p.S, p.lanes_per_row, p.vec, p.rep) == (0, 32, 2, 1) and _kernel(h, hint) == launched
    for K in (34, 62, 66, 70, 130, 194, 258):
        assert pc.pcsr_query_launch(h, K)["vec"] == 2
    auto = pc.pcsr_build(*_small(), pc.make_params(V=p.V, flags=HOST))
    for K in (2, 6, 16, 24, 30):                             # few columns: left to the library where another shape stands in
        assert _kernel(h, K) == ((32, 2, 1) if launched == (32, 2, 1) else _kernel(auto, K))
    auto.close()
    h.close()


def test_shapes_of_narrow_rows_are_for_narrow_rows():
    """A dword a lane gains at the widths it was chosen for; at others the handle runs the wide loads that it had."""
    skewed = _uniform(1 << 20, 16, d_hat=25.0, CV=8.0, CV_hat=8.0, d_max=30_000)
    for hint in (4, 8):
        p, h = _chosen_for(skewed, hint)
        assert (p.S, p.lanes_per_row, p.vec, p.rep) == (1, 8, 1, 1)
        assert [_kernel(h, K) for K in (4, 8, 12, 16, 64, 75, 256)] == [(8, 1, 1)] * 2 + [(4, 4, 1)] * 5
        q = pc.pcsr_query_kernel(h, 75)
        assert q["grid_y"] == 5 and q["grid_x"] < pc.pcsr_query_launch(h, 75)["grid_x"]
        h.close()
        p.rep = 2                                            # the caller's shape is the caller's at every width
        assert _kernel(pc.pcsr_build(*_small(), p), 64) == (8, 1, 2)
    for hint, beyond in ((24, (8, 4, 1)), (30, (16, 2, 1))):
        p, h = _chosen_for(_uniform(20_000, 22), hint)
        assert (p.S, p.lanes_per_row, p.vec, p.rep) == (0, 32, 1, 1)
        assert [_kernel(h, K) for K in (8, 17, hint, 32, 33, 128, 256)] == [(32, 1, 1)] * 4 + [beyond] * 3
        h.close()


def test_few_columns_of_rows_that_are_not_split_for_many():
    """Handles for 64 and more columns of long scattered rows: up to 32 they run what is left to the library, unless the caller sets a shape."""
    auto = pc.pcsr_build(*_small(), pc.make_params(flags=HOST))
    for hint in (64, 75, 100, 128, 130, 256):
        f = _uniform(150_000, 60)
        p, h = _chosen_for(f, hint)
        own = p.lanes_per_row, p.vec, p.rep
        assert (p.S, p.V) == (0, 1) and p.flags & pc.PCSR_FLAG_COLUMN_BANDS
        assert [_kernel(h, K) for K in (1, 4, 7, 16, 17, 24, 32)] == [_kernel(auto, K) for K in (1, 4, 7, 16, 17, 24, 32)]
        assert (_kernel(h, 64) == own or hint % 32) and pc.pcsr_query_launch(h, 64)["vec"] == own[1]
        h.close()
        for field, value in (("lanes_per_row", 8), ("vec", 1 if p.vec > 1 else 2), ("rep", 4)):
            changed = type(p).from_buffer_copy(p)
            setattr(changed, field, value)
            h = pc.pcsr_build(*_small(), changed)
            assert _kernel(h, 16) == (changed.lanes_per_row, changed.vec, changed.rep)
            h.close()
        h = pc.pcsr_build(*_small(), p)
        pc.pcsr_set_kernel_params(h, *own, p.waves_per_wg)
        assert _kernel(h, 16) == own
        h.close()
    p, _ = _chosen_for(_uniform(60_000, 60), 64)             # split as before
    assert p.S == 1 and not p.flags >> 29
    auto.close()


def test_few_columns_of_short_scattered_rows():
    """16 lanes where B is beyond what L2 holds or rows are of 12 and more; between them the shapes that they had."""
    shape = lambda n, deg, K: (lambda p: (p.lanes_per_row, p.vec, p.rep))(pc.pcsr_select(_uniform(n, deg), K))  # noqa: E731
    for n, deg in ((300_000, 9), (300_000, 8.5), (400_000, 8.5), (300_000, 11)):
        assert shape(n, deg, 2) == (4, 2, 1) and shape(n, deg, 3) == (4, 1, 1)
        assert shape(n, deg, 6) == shape(n, deg, 8) == (16, 1, 1)
        assert shape(n, deg, 4) == ((16, 1, 1) if deg >= 9 or n > 312_500 else (4, 4, 1))
        assert shape(n, deg, 5) == (16, 1, 1)
    for n, deg in ((1_000_000, 9), (300_000, 12), (60_000, 9)):
        assert shape(n, deg, 2) == shape(n, deg, 3) == shape(n, deg, 4) == shape(n, deg, 5) == (16, 1, 1)
