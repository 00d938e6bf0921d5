"""Which layers FusedLayers takes: its kernels read raw pointers, so whatever torch's own modules would
broadcast, refuse or hand to a hook has to run module by module.  No GPU calls."""
import pytest

import paper_2605_15695_amd as pc
import synth

torch = pytest.importorskip("torch")

from paper_2605_15695_amd import gnn  # noqa: E402


@pytest.fixture(scope="module")
def op():
    g = synth.workload("poisson", "small")
    return gnn.PcsrOperator(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals,
                            params=pc.make_params(flags=pc.PCSR_FLAG_HOST_ONLY))


def _param(*shape):
    return torch.nn.Parameter(torch.zeros(shape))


def test_plain_layers_are_taken(op):
    assert len(gnn._params(gnn.GCNLayer(op, 16, 64))) == 2
    assert len(gnn._params(gnn.GCNLayer(op, 7, 5, bias=False))) == 1
    assert len(gnn._params(gnn.GINLayer(op, 128, 33))) == 5


def _gin_second(layer):
    layer.mlp[2] = torch.nn.Linear(64, 32)


def _gin_second_wider(layer):
    layer.mlp[2] = torch.nn.Linear(64, 100)


def _gin_mlp_module(layer):
    layer.mlp = torch.nn.Linear(16, 64)


def _gin_weight(layer):
    layer.mlp[2].weight = _param(32, 64)


@pytest.mark.parametrize("change", [_gin_second, _gin_second_wider, _gin_mlp_module, _gin_weight])
def test_gin_layers_of_another_form_are_not(op, change):
    layer = gnn.GINLayer(op, 16, 64)
    change(layer)
    assert gnn._params(layer) is None


def _gcn_module(layer):
    layer.lin = torch.nn.Sequential(torch.nn.Linear(16, 64, bias=False))


def _gcn_weight(layer):
    layer.lin.weight = _param(32, 16)


@pytest.mark.parametrize("change", [_gcn_module, _gcn_weight])
def test_gcn_layers_of_another_form_are_not(op, change):
    layer = gnn.GCNLayer(op, 16, 64)
    change(layer)
    assert gnn._params(layer) is None


def _gcn_one_bias(layer):
    layer.bias = _param(1)


def _gcn_row_bias(layer):
    layer.bias = _param(1, 64)


def _gcn_scalar_bias(layer):
    layer.bias = _param()


@pytest.mark.parametrize("change", [_gcn_one_bias, _gcn_row_bias, _gcn_scalar_bias])
def test_biases_that_broadcast_are_not(op, change):
    layer = gnn.GCNLayer(op, 16, 64)
    change(layer)
    assert gnn._params(layer) is None


@pytest.mark.parametrize("which", [0, 2])
def test_gin_biases_that_broadcast_are_not(op, which):
    layer = gnn.GINLayer(op, 16, 64)
    layer.mlp[which].bias = _param(1)
    assert gnn._params(layer) is None


@pytest.mark.parametrize("eps", [torch.full((64,), 0.5), torch.full((3, 1), 0.5), 0.5, torch.full((1, 1, 1), 0.5)])
def test_eps_other_than_one_value_is_not(op, eps):
    layer = gnn.GINLayer(op, 64, 64)
    del layer.eps
    layer.eps = eps
    assert gnn._params(layer) is None


def test_one_eps_of_any_rank_the_result_keeps_is(op):
    layer = gnn.GINLayer(op, 64, 64)
    for shape in ((), (1,), (1, 1)):
        layer.eps = _param(*shape)
        assert gnn._params(layer) is not None


def test_operators_with_a_product_of_their_own_are_not(op):
    class Dropping(gnn.PcsrOperator):
        def _run(self, handle, n_out, X):
            return 0.5 * super()._run(handle, n_out, X)

    sub = Dropping.__new__(Dropping)
    sub.__dict__.update(op.__dict__)
    assert gnn._params(gnn.GCNLayer(sub, 16, 64)) is None
    own = gnn.PcsrOperator.__new__(gnn.PcsrOperator)
    own.__dict__.update(op.__dict__)
    assert gnn._params(gnn.GINLayer(own, 16, 64)) is not None
    own._run = lambda handle, n_out, X: X
    assert gnn._params(gnn.GINLayer(own, 16, 64)) is None


def test_modules_that_are_watched_or_changed_are_not(op):
    layer = gnn.GINLayer(op, 16, 64)
    from torch.nn.modules.module import (register_module_forward_hook, register_module_forward_pre_hook,
                                         register_module_full_backward_hook, register_module_full_backward_pre_hook)
    for register in (register_module_forward_hook, register_module_forward_pre_hook,
                     register_module_full_backward_hook, register_module_full_backward_pre_hook):
        handle = register(lambda *a: None)
        try:
            assert gnn._params(layer) is None, register
        finally:
            handle.remove()
        assert gnn._params(layer) is not None
    layer.mlp[0].forward = lambda H: H
    assert gnn._params(layer) is None


def test_tensors_of_another_type_are_not(op):
    class Watched(torch.Tensor):
        pass

    layer = gnn.GCNLayer(op, 16, 64, bias=False)
    layer.bias = 0.5
    assert gnn._params(layer) is None
    layer.bias = torch.zeros(64).as_subclass(Watched)
    assert gnn._params(layer) is None
    layer.bias = torch.zeros(64)
    assert gnn._params(layer) is not None


def test_a_copied_model_shares_its_matrix(op):
    import copy

    model = gnn.make_model("gcn", op, 16, 32, 16, 2)
    other = copy.deepcopy(model)
    assert other[0].op.fwd is op.fwd and copy.copy(op.fwd) is op.fwd
    del other
    assert op.fwd.raw and pc.pcsr_query_launch(op.fwd, 16)["vec"] > 0
