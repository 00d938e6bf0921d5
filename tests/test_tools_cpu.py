"""CPU checks of the measurement helpers: shape enumeration of the sweep, the report."""
import io
import json
from contextlib import redirect_stdout

from paper_2605_15695_amd import report, sweep


def test_kernel_shapes_cover_k_without_idle_repeats():
    for K in (16, 32, 48, 64, 96, 128, 160, 256, 512, 33):
        shapes = sweep.kernel_shapes(K, quick=False)
        assert shapes
        for lpr, vec, rep in shapes:
            assert K % vec == 0
            tile = lpr * vec * rep
            assert tile * 8 >= K                       # at most 8 grid.y slices
            assert lpr * vec * (rep - 1) < K           # no repeat entirely past K
    quick = sweep.kernel_shapes(128, quick=True)
    # the widest load, plus the two 64-column slices made of narrow loads
    assert quick and all(v == 4 or (l, v, r) in ((32, 2, 1), (64, 1, 1)) for l, v, r in quick)
    assert (32, 2, 1) in quick and (64, 1, 1) in quick
    assert {v for _, v, _ in sweep.kernel_shapes(32, quick=True)} == {1, 2, 4}


def test_report_table_and_geomean(tmp_path):
    base = dict(workload="w", size="full", K=64, nnz=1000, n=100, bytes_min=10_000)
    recs = [
        dict(base, kind="pcsr", V=1, S=0, SG=0, lanes_per_row=16, vec=4, rep=1, waves_per_wg=4,
             items_per_group=1, ms_median=0.5, gflops=256.0, roofline_frac=0.25),
        dict(base, kind="pcsr", V=2, S=0, SG=0, lanes_per_row=16, vec=4, rep=1, waves_per_wg=4,
             items_per_group=1, ms_median=1.0, gflops=128.0, roofline_frac=0.125),
        dict(base, kind="hipsparse", alg="default", ms_median=2.0),
        dict(base, kind="selected", ms_median=0.625),
    ]
    p = tmp_path / "s.jsonl"
    p.write_text("\n".join(json.dumps(r) for r in recs) + "\n")
    out = io.StringIO()
    with redirect_stdout(out):
        assert report.main([str(p)]) == 0
    text = out.getvalue()
    assert "| w | 64 | 100 | 1000 | 1,0,0 / 16,4,1,4,1 | 0.5000 |" in text and text.count("| - |") == 1
    assert "4.00x" in text and "**4.00x**" in text and "80.0 %" in text


def test_rule_alternatives_and_their_table():
    import numpy as np

    import paper_2605_15695_amd as pc
    import synth

    g = synth.workload("sbm_shuffled", "small")
    f = np.array(pc.pcsr_features(g.n_rows, g.n_cols, g.rowptr, g.colidx))
    recs = []
    for K, names in ((75, {"pick", "own shape", "items of 64"}),
                     (96, {"pick", "row tile", "64-column slices", "items of 64"}),
                     (100, {"pick", "own shape", "row tile", "64-column slices", "items of 64"})):
        alt = sweep.rule_alternatives(pc.pcsr_select(f, K), K)
        assert alt[0][0] == "pick" and {a[0] for a in alt} == names
        for i, (name, p, shape) in enumerate(alt):
            p = type(p).from_buffer_copy(p)
            p.flags |= pc.PCSR_FLAG_HOST_ONLY
            h = pc.pcsr_build(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, p)
            if shape:
                pc.pcsr_set_kernel_params(h, *shape, p.waves_per_wg)
            q = pc.pcsr_query_kernel(h, K)
            assert not shape or (q["lanes_per_row"], q["vec"], q["rep"]) == shape
            recs.append(dict(kind="rule", workload="w", K=K, what=name, V=p.V, S=p.S, SG=p.SG, ms=1.0 + i, **q))
    out = io.StringIO()
    with redirect_stdout(out):
        report.rules_table(recs)
    assert "| w | 100 | 1, 1, 32 / 32x4x1 | 1.0000 | 2.00 (" in out.getvalue()


def test_windows_of_communities_are_no_stand_in_shape():
    import numpy as np

    import paper_2605_15695_amd as pc

    f = np.zeros(len(pc.FEATURE_NAMES))
    f[0] = f[1] = 250_000
    f[2], f[4], f[5], f[6], f[7], f[15], f[16] = 12e6, 48.0, 48.0, 80.0, 0.15, 0.5, 0.004
    alt = sweep.rule_alternatives(pc.pcsr_select(f, 256), 256)
    assert "own shape" not in {a[0] for a in alt} and all(a[1].flags & pc.PCSR_FLAG_CLUSTER_WINDOWS for a in alt)
