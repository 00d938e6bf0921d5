"""Times one GCN / GIN training step (forward, backward, Adam update) with every sparse
product going through pcsr_spmm, beside the same model on torch.sparse (rocSPARSE CSR).
Shape follows the paper's Section 6.5: 5 layers, 16 input and output features, hidden
size 32 / 64 / 128.  Synthetic graphs and random features stand in for the OGB graphs.

    python -m paper_2605_15695_amd.gnn_bench --workload road --model gcn --hidden 64

--dense times the layers' dense kernels on their own, the calls of a backward or a GIN layer both
in one pass and one after the other, beside the torch operations they stand for.

    python -m paper_2605_15695_amd.gnn_bench --dense 2000000
"""
from __future__ import annotations

import argparse
import json
import statistics
import sys
import time


def dense(n: int, widths=((64, 64), (16, 64), (64, 16), (96, 96), (128, 128))) -> None:
    """One JSON line per call and pair of widths: microseconds (median of 20) and TB/s of the arrays
    it reads and writes, each once."""
    import torch
    import torch.nn.functional as F

    from .gnn import _Dense

    def timed(fn):
        since = time.perf_counter()
        while time.perf_counter() - since < 0.05:  # 3 calls leave the clocks where they were: the first figures were 15-25 % high
            for _ in range(3):
                fn()
            torch.cuda.synchronize()
        ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(20)]
        torch.cuda.synchronize()
        for a, b in ev:
            a.record()
            fn()
            b.record()
        torch.cuda.synchronize()
        return statistics.median(a.elapsed_time(b) for a, b in ev) * 1e3

    torch.backends.cuda.matmul.allow_tf32 = False
    for a, b in widths:
        d = _Dense(torch.empty(1, device="cuda"), [(a, b), (b, a), (b, b)])
        X, H = torch.randn(n, a, device="cuda"), torch.randn(n, a, device="cuda")
        G, W, W2 = torch.randn(n, b, device="cuda"), torch.randn(b, a, device="cuda"), torch.randn(b, b, device="cuda")
        b1, b2, Z = torch.randn(b, device="cuda"), torch.randn(b, device="cuda"), torch.randn(n, b, device="cuda")
        cs, dot = torch.empty(a, device="cuda"), torch.empty((), device="cuda")

        def back_apart():
            d.wgrad(G, X, bias=True)
            d.linear(G, W, transposed=True, mask=X, colsum=cs)

        def mlp_apart():
            d.linear(d.linear(X, W, bias=b1, relu=True), W2, bias=b2, relu=True)

        def mlp_back_apart():
            d.wgrad(G, Z, bias=True)
            G1 = d.linear(G, W2, transposed=True, mask=Z)
            d.wgrad(G1, X, bias=True)
            d.linear(G1, W, transposed=True, aux=H, dot=dot)

        calls = [  # name, arrays of a and of b columns it has to read or write, call
            ("X W^T", 1, 1, lambda: d.linear(X, W)),
            ("relu(X W^T + bias)", 1, 1, lambda: d.linear(X, W, bias=b1, relu=True)),
            ("torch: relu(X W^T + bias)", 1, 1, lambda: torch.relu_(F.linear(X, W, b1))),
            ("G W masked by X > 0", 2, 1, lambda: d.linear(G, W, transposed=True, mask=X)),
            ("G^T X, sums of G", 1, 1, lambda: d.wgrad(G, X, bias=True)),
            ("torch: G^T X", 1, 1, lambda: G.t() @ X),
            ("backward of one layer", 2, 1, lambda: d.linear_backward(G, X, W, bias=True, mask=True, colsum=cs)),
            ("the same, call by call", 2, 1, back_apart),
            ("both layers of a GIN layer", 1, 2, lambda: d.mlp(X, W, b1, W2, b2, True)),
            ("the same, call by call ", 1, 2, mlp_apart),
            ("their backward", 3, 2, lambda: d.mlp_backward(G, Z, X, H, W, W2, True)),
            ("the same, call by call  ", 3, 2, mlp_back_apart),
        ]
        for name, na, nb, fn in calls:
            us = timed(fn)
            print(json.dumps({"rows": n, "a": a, "b": b, "call": name.strip(), "us": round(us, 1),
                              "TB_s": round(n * 4.0 * (na * a + nb * b) / us / 1e6, 2)}), flush=True)


def main(argv=None) -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--workload", default="road")
    ap.add_argument("--size", default="full")
    ap.add_argument("--model", default="gcn", choices=["gcn", "gin"])
    ap.add_argument("--hidden", type=int, default=64)
    ap.add_argument("--layers", type=int, default=5)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--no-torch-sparse", action="store_true")
    ap.add_argument("--dense", type=int, default=0, metavar="ROWS")
    args = ap.parse_args(argv)

    import torch

    import synth
    from .gnn import PcsrOperator, make_model

    if not torch.cuda.is_available():
        print("gnn_bench: no GPU visible", file=sys.stderr)
        return 2
    torch.cuda.set_device(0)
    if args.dense:
        dense(args.dense)
        return 0
    g = synth.workload(args.workload, args.size)
    symmetric = args.workload in ("road", "rmat22")
    X = torch.from_numpy(synth.dense_operand(g.n_rows, 16, "normal", 5)).cuda()
    Y = torch.from_numpy(synth.dense_operand(g.n_rows, 16, "normal", 6)).cuda()

    def run(op, label):
        torch.manual_seed(0)
        model = make_model(args.model, op, 16, args.hidden, 16, args.layers).cuda()
        opt = torch.optim.Adam(model.parameters(), lr=1e-3)

        def step():
            opt.zero_grad(set_to_none=True)
            loss = torch.nn.functional.mse_loss(model(X), Y)
            loss.backward()
            opt.step()
            return loss

        for _ in range(args.warmup):
            step()
        torch.cuda.synchronize()
        ts = []
        for _ in range(args.steps):
            t0 = time.perf_counter()
            loss = step()
            torch.cuda.synchronize()
            ts.append((time.perf_counter() - t0) * 1e3)
        return {"impl": label, "ms_per_step_median": statistics.median(ts), "ms_per_step_min": min(ts),
                "final_loss": float(loss)}

    t0 = time.time()
    op = PcsrOperator(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, symmetric=symmetric, K_hint=args.hidden)
    build_s = time.time() - t0
    res = [run(op, "pcsr")]
    if not args.no_torch_sparse:
        A = torch.sparse_csr_tensor(torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.colidx).cuda(),
                                    torch.from_numpy(g.vals).cuda(), size=(g.n_rows, g.n_cols))

        class TorchSparseOp:
            def __call__(self, H):
                return torch.sparse.mm(A, H)

        try:
            res.append(run(TorchSparseOp(), "torch.sparse"))
        except Exception as e:  # noqa: BLE001
            res.append({"impl": "torch.sparse", "error": repr(e)[:200]})
    out = {"workload": f"{args.workload}-{args.size}", "n": g.n_rows, "nnz": g.nnz, "model": args.model,
           "layers": args.layers, "hidden": args.hidden, "operator_build_s": build_s, "results": res}
    if len(res) == 2 and "ms_per_step_median" in res[1]:
        out["speedup_vs_torch_sparse"] = res[1]["ms_per_step_median"] / res[0]["ms_per_step_median"]
    print(json.dumps(out))
    return 0


if __name__ == "__main__":
    sys.exit(main())
