"""Widths that are no multiple of a vector, in the shapes pcsr_select and the auto launch serve them
with: the moved-back last vector, tiles wider than a row, two loads per lane, split rows with both
write-backs, and the long-row reduction."""
import numpy as np
import pytest

import oracle
import paper_2605_15695_amd as pc
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [17, 18, 19, 31, 33, 36, 63, 65, 66, 100, 129, 255, 257, 258, 300, 501, 513, 515])
@pytest.mark.parametrize("name", ["rmat20", "sbm_shuffled", "road", "sbm", "poisson"])
def test_every_column_is_written_once_and_right(name, K):
    g = synth.workload(name, "small")
    B = synth.dense_operand(g.n_cols, K, "normal", K)
    ref, bound = oracle.spmm(g.rowptr, g.colidx, g.vals, B)
    f = np.array(pc.pcsr_features(g.n_rows, g.n_cols, g.rowptr, g.colidx))
    big = f.copy()
    big[0] = big[1] = 250_000                     # what the rule picks for a matrix of that kind and size
    picks = [pc.pcsr_select(f, K), pc.pcsr_select(big, K)]
    auto = pc.make_params(V=picks[0].V, S=picks[0].S, SG=picks[0].SG)
    atomic = pc.make_params(V=1, S=1, SG=8, flags=pc.PCSR_FLAG_ATOMIC_SPLIT)
    two = pc.make_params(V=2, S=1, SG=8)
    Bd = torch.empty(g.n_cols * K + 1, device="cuda")[1:]   # no better than 4-byte aligned
    Bd.copy_(torch.from_numpy(B).reshape(-1))
    for what, p in (("pick", picks[0]), ("pick big", picks[1]), ("auto", auto), ("atomic", atomic), ("V2", two)):
        if K % 4 == 0 or p.vec in (2, 4) or p.col_window:
            src = torch.from_numpy(B).cuda()
        else:
            src = Bd.reshape(g.n_cols, K)
        h = pc.pcsr_build(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, p)
        Cd = torch.full((g.n_rows + 1, K), float("nan"), device="cuda")
        if K % 2 == 0:
            src = torch.from_numpy(B).cuda()
        pc.pcsr_spmm(h, src, Cd[:-1], K)
        ok, worst = oracle.within_tolerance(Cd[:-1].cpu().numpy(), ref, bound)
        assert ok, (name, K, what, worst)
        assert bool(torch.isnan(Cd[-1]).all()), "wrote past the end"
        h.close()
