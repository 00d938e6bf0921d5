"""pcsr_spmm's fast marshalling: every way to pass the arguments, and the errors of those that do not fit."""
import numpy as np
import pytest

import paper_2605_15695_amd as pc
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_arguments_and_errors():
    g = synth.workload("poisson", "small")
    K = 24
    h = pc.pcsr_build(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals)
    B = torch.from_numpy(synth.dense_operand(g.n_cols, K, "normal", 3)).cuda()
    out = []
    side = torch.cuda.Stream()
    for call in (lambda C: pc.pcsr_spmm(h, B, C, K), lambda C: pc.pcsr_spmm(h, B=B, C=C, K=K, stream=None),
                 lambda C: pc.pcsr_spmm(h, B, C, K, side), lambda C: pc.pcsr_spmm(h, B, C, K, side.cuda_stream),
                 lambda C: pc.pcsr_spmm(h, B, C, np.int64(K), 0),
                 lambda C: pc.pcsr_spmm(h, torch.nn.Parameter(B), C, K, torch.cuda.current_stream())):
        C = torch.full((g.n_rows, K), float("nan"), device="cuda")
        torch.cuda.synchronize()
        assert call(C) is None
        torch.cuda.synchronize()
        out.append(C)
    assert all(torch.equal(out[0], o) for o in out) and bool(torch.isfinite(out[0]).all())
    C = out[0]
    for bad in ((B.cpu(), C), (B, C.cpu()), (B.double(), C), (B[:, :8], C), (B.t(), C), (B[:-1], C), (B, C[1:]),
                (B.cpu().numpy(), C)):
        with pytest.raises(ValueError):
            pc.pcsr_spmm(h, *bad, K)
    with pytest.raises(pc.PcsrError):
        pc.pcsr_spmm(h, B, B.reshape(g.n_rows, K), K)      # B and C overlap
    h.close()
    with pytest.raises(pc.PcsrError):
        pc.pcsr_spmm(h, B, C, K)


def test_memory_kept_for_reuse_goes_back():
    import ctypes
    import importlib.util

    from paper_2605_15695_amd import binding

    g = synth.workload("sbm", "small")
    B = torch.from_numpy(synth.dense_operand(g.n_cols, 16, "normal", 3)).cuda()
    C = torch.empty(g.n_rows, 16, device="cuda")
    h = pc.pcsr_build(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals)
    pc.pcsr_spmm(h, B, C, 16)
    h.close()
    before = torch.cuda.mem_get_info()[0]
    released = pc.pcsr_release_cached()
    assert released >= g.nnz * 8 and torch.cuda.mem_get_info()[0] >= before
    assert pc.pcsr_release_cached() == 0
    # torch asks before it takes more from the driver
    spec = importlib.util.spec_from_file_location("_pcsr_py", binding.PY_PATH)
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    asked = []
    ask = ctypes.CFUNCTYPE(ctypes.c_int64, ctypes.c_void_p)(lambda stream: asked.append(stream) or 0)
    lib = binding._lib()
    mod.init(*(ctypes.cast(f, ctypes.c_void_p).value for f in (lib.pcsr_spmm, ask)))
    try:
        torch.cuda.empty_cache()
        torch.empty(100 << 20, device="cuda")
        assert asked
    finally:
        mod.init(*(ctypes.cast(f, ctypes.c_void_p).value for f in (lib.pcsr_spmm, lib.pcsr_release_cached_if_low)))


# missing, no library at all, and made for another torch: the call goes through ctypes, with the same checks
@pytest.mark.parametrize("what", ["missing", "broken", "other torch"])
def test_products_without_the_call_module(what, tmp_path, monkeypatch):
    from paper_2605_15695_amd import binding

    g = synth.workload("poisson", "small")
    K = 24
    h = pc.pcsr_build(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals)
    B = torch.from_numpy(synth.dense_operand(g.n_cols, K, "normal", 3)).cuda()
    ref, C = torch.empty(g.n_rows, K, device="cuda"), torch.empty(g.n_rows, K, device="cuda")
    pc.pcsr_spmm(h, B, ref, K)
    monkeypatch.setattr(binding, "_spmm", binding._first_spmm)  # as before the first call
    if what == "other torch":
        monkeypatch.setattr(torch, "__version__", "1.0.0+rocm0")
    else:
        path = tmp_path / "_pcsr_py.so"
        if what == "broken":
            path.write_bytes(b"no library")
        monkeypatch.setattr(binding, "PY_PATH", path)
    with pytest.warns(RuntimeWarning, match="ctypes"):
        pc.pcsr_spmm(h, B, C, K)
    pc.pcsr_spmm(h, B, C, K, torch.cuda.current_stream())
    assert torch.equal(C, ref)
    with pytest.raises(ValueError):
        pc.pcsr_spmm(h, B[:-1], C, K)


def test_an_operator_loads_the_call_module(monkeypatch):
    from paper_2605_15695_amd import binding, gnn

    g = synth.workload("poisson", "small")
    monkeypatch.setattr(binding, "_spmm", binding._first_spmm)
    gnn.PcsrOperator(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, K_hint=32)
    assert binding._spmm not in (binding._first_spmm, binding._spmm_checked)
