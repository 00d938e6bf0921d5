"""GNN integration of the PCSR SpMM (the paper embeds its kernel in GCN / GIN training,
Section 6.5): an autograd function whose forward is C = A*B and whose backward is
dB = A^T * dC, both through pcsr_spmm, plus minimal GCN / GIN layers built on it.

torch supplies tensors, streams, the loss and the optimiser; every sparse product runs in the
library's kernels, and so do the dense products of layers up to MAX_WIDTH features wide with
what surrounds them (bias, ReLU, its backward, the gradient sums): see FusedLayers.
"""
from __future__ import annotations

import ctypes
from typing import NamedTuple

import torch
from torch.nn.modules import module as _all_modules

from . import binding as pc


class PcsrOperator:
    """A fixed sparse matrix A ready for forward (A*B) and backward (A^T*dC) products.

    ``symmetric=True`` states that A equals its transpose (GCN-normalised undirected
    graphs), so one handle serves both directions.  Otherwise the transpose is built once.  Parameters are picked by pcsr_select for width ``K_hint``
    unless ``params`` is given.
    """

    def __init__(self, n_rows, n_cols, rowptr, colidx, vals, symmetric=False, K_hint=64, params=None):
        self.n_rows, self.n_cols = int(n_rows), int(n_cols)

        if symmetric and n_rows != n_cols:
            raise ValueError("a symmetric operator must be square")
        if params is not None:
            params = pc.make_params(**{f: getattr(params, f) for f, _ in pc.pcsr_params_t._fields_ if f != "reserved"})
        if params is not None and params.flags & pc.PCSR_FLAG_HOST_ONLY:
            self.fwd = self.bwd = pc.pcsr_build(self.n_rows, self.n_cols, rowptr, colidx, vals, params)
            if not symmetric:
                self.bwd = pc.pcsr_build(self.n_cols, self.n_rows,
                                         *pc.pcsr_transpose_csr(self.n_rows, self.n_cols, rowptr, colidx, vals), params)
            return
        pc.load_call_module()
        # one upload; check, features, selection, transpose and PCSR generation on the GPU
        self.fwd, self.bwd = pc.pcsr_operator_build(self.n_rows, self.n_cols, rowptr, colidx, vals, params, K_hint,
                                                    not symmetric)
        if symmetric:
            self.bwd = self.fwd

    def apply(self, B: torch.Tensor) -> torch.Tensor:
        return SpMMFunction.apply(B, self)

    __call__ = apply

    def _run(self, handle, n_out, X: torch.Tensor) -> torch.Tensor:
        if X.dtype != torch.float32 or not X.is_cuda or X.dim() != 2:
            raise ValueError("operand must be a 2-D float32 CUDA tensor")
        X = X.contiguous()
        K = X.shape[1]
        out = torch.empty((n_out, K), dtype=torch.float32, device=X.device)
        pc.pcsr_spmm(handle, X, out, K, torch.cuda.current_stream(X.device))
        return out


class SpMMFunction(torch.autograd.Function):
    @staticmethod
    def forward(ctx, B, op: PcsrOperator):
        ctx.op = op
        return op._run(op.fwd, op.n_rows, B)

    @staticmethod
    def backward(ctx, dC):
        op = ctx.op
        return op._run(op.bwd, op.n_cols, dC), None


# widest layer side the library's dense kernels take
MAX_WIDTH = 128


class _Dense:
    """The library's dense kernels on one device and stream, with a workspace for their sums."""

    def __init__(self, X: torch.Tensor, widths):
        self.lib = pc._lib()
        self.stream = torch.cuda.current_stream(X.device).cuda_stream
        self.device = X.device
        floats = max(self.lib.pcsr_gnn_workspace_floats(a, b) for a, b in widths)
        self.ws_floats, self._ws = floats, None

    @property
    def ws(self):
        if self._ws is None:
            self._ws = torch.empty(self.ws_floats, dtype=torch.float32, device=self.device)
        return self._ws.data_ptr()

    def new(self, *shape):
        return torch.empty(shape, dtype=torch.float32, device=self.device)

    @staticmethod
    def _check(rc, where):
        if rc != pc.PCSR_OK:
            raise pc.PcsrError(rc, where)

    def linear(self, X, W, transposed=False, bias=None, relu=False, mask=None, aux=None, dot=None, colsum=None,
               store=True):
        """X * W^T (transposed: X * W) + bias, ReLU, sum(. * aux) into dot, mask, column sums."""
        n, a = X.shape
        b = W.shape[1] if transposed else W.shape[0]
        Y = self.new(n, b) if store else None
        self._check(self.lib.pcsr_gnn_linear(
            n, a, b, X.data_ptr(), W.data_ptr(), int(transposed), _p(bias), int(relu), _p(mask), _p(aux), _p(Y),
            _p(colsum), _p(dot), self.ws if colsum is not None or dot is not None else None, self.stream),
            "pcsr_gnn_linear")
        return Y

    def mlp(self, X, W1, b1, W2, b2, relu):
        """Z = relu(X W1^T + b1), Z W2^T + b2 (ReLU): both, in one pass where the widths allow it"""
        n, (m, a) = X.shape[0], W1.shape
        if _pieces(a, m):
            Z, Y = self.new(n, m), self.new(n, m)
            rc = self.lib.pcsr_gnn_mlp(n, a, m, X.data_ptr(), W1.data_ptr(), b1.data_ptr(), W2.data_ptr(),
                                       b2.data_ptr(), int(relu), Z.data_ptr(), Y.data_ptr(), self.stream)
            if rc != pc.PCSR_E_UNSUPPORTED:
                self._check(rc, "pcsr_gnn_mlp")
                return Z, Y
        Z = self.linear(X, W1, bias=b1, relu=True)
        return Z, self.linear(Z, W2, bias=b2, relu=relu)

    def mlp_backward(self, G, Z, A, H, W1, W2, store):
        """(dA or None, sum(dA * H), dW1, db1, dW2, db2) of mlp(A, ...), in one pass where the widths allow it"""
        n, (m, a) = G.shape[0], W1.shape
        dot = self.new()
        if _pieces(a, m):
            dA = self.new(n, a) if store else None
            dW1, db1, dW2, db2 = self.new(m, a), self.new(m), self.new(m, m), self.new(m)
            rc = self.lib.pcsr_gnn_mlp_backward(
                n, a, m, G.data_ptr(), Z.data_ptr(), A.data_ptr(), H.data_ptr(), W1.data_ptr(), W2.data_ptr(), _p(dA),
                dW1.data_ptr(), db1.data_ptr(), dW2.data_ptr(), db2.data_ptr(), dot.data_ptr(), self.ws, self.stream)
            if rc != pc.PCSR_E_UNSUPPORTED:
                self._check(rc, "pcsr_gnn_mlp_backward")
                return dA, dot, dW1, db1, dW2, db2
        dW2, db2 = self.wgrad(G, Z, bias=True)
        G1 = self.linear(G, W2, transposed=True, mask=Z)
        dW1, db1 = self.wgrad(G1, A, bias=True)
        dA = self.linear(G1, W1, transposed=True, aux=H, dot=dot, store=store)
        return dA, dot, dW1, db1, dW2, db2

    def linear_backward(self, G, X, W, bias=False, mask=False, colsum=None):
        """(dX, dW, column sums of G or None) of Y = X W^T; dX masked by X > 0 if asked, its column
        sums into colsum"""
        n, (b, a) = G.shape[0], W.shape
        if _pieces(a, b):
            dX, dW, db = self.new(n, a), self.new(b, a), self.new(b) if bias else None
            rc = self.lib.pcsr_gnn_linear_backward(n, a, b, G.data_ptr(), X.data_ptr(), W.data_ptr(), int(mask),
                                                   dX.data_ptr(), dW.data_ptr(), _p(db), _p(colsum), self.ws,
                                                   self.stream)
            if rc != pc.PCSR_E_UNSUPPORTED:
                self._check(rc, "pcsr_gnn_linear_backward")
                return dX, dW, db
        dW, db = self.wgrad(G, X, bias=bias)
        return self.linear(G, W, transposed=True, mask=X if mask else None, colsum=colsum), dW, db

    def wgrad(self, G, X, bias=False):
        """(G^T X, column sums of G or None)"""
        dW = self.new(G.shape[1], X.shape[1])
        db = self.new(G.shape[1]) if bias else None
        self._check(self.lib.pcsr_gnn_wgrad(G.shape[0], X.shape[1], G.shape[1], G.data_ptr(), X.data_ptr(),
                                            dW.data_ptr(), _p(db), self.ws, self.stream), "pcsr_gnn_wgrad")
        return dW, db

    def colsum(self, G):
        out = self.new(G.shape[1])
        self._check(self.lib.pcsr_gnn_colsum(G.shape[0], G.shape[1], G.data_ptr(), out.data_ptr(), self.ws,
                                             self.stream), "pcsr_gnn_colsum")
        return out

    def spmm(self, handle, n_out, X, bias=None, relu=False, self_term=None, eps=None, mask=None):
        # an operator's handles can be exchanged, and the library sees only pointers
        if X.shape[0] != handle.n_cols or n_out != handle.n_rows:
            raise ValueError("B must be n_cols x K and C n_rows x K")
        out = self.new(n_out, X.shape[1])
        if bias is not None or self_term is not None or mask is not None or relu:
            epi = pc.pcsr_epilogue_t(_p(bias), _p(self_term), _p(eps), _p(mask), int(relu), 0)
            rc = self.lib.pcsr_spmm_epilogue(handle.raw, X.data_ptr(), out.data_ptr(), X.shape[1], ctypes.byref(epi),
                                             self.stream)
            if rc != pc.PCSR_E_UNSUPPORTED:
                self._check(rc, "pcsr_spmm_epilogue")
                return out
        self._check(self.lib.pcsr_spmm(handle.raw, X.data_ptr(), out.data_ptr(), X.shape[1], self.stream), "pcsr_spmm")
        # handles whose product takes no epilogue: PCSR_FLAG_ATOMIC_SPLIT, where partial sums meet in C
        if self_term is not None:
            out.add_(self_term if eps is None else (1.0 + eps.reshape(())) * self_term)
        if bias is not None:
            out.add_(bias)
        if relu:
            out.relu_()
        return out if mask is None else out.masked_fill_(mask <= 0.0, 0.0)


def _pieces(a, b):
    """Whether the one-pass kernels for two products take these widths."""
    return a % 16 == 0 and b % 16 == 0 and a <= 64 and b <= 64


def _p(t):
    return None if t is None else t.data_ptr()


class FusedLayers(torch.autograd.Function):
    """Forward and backward of a chain of GCN / GIN layers with ReLU between them as one autograd
    node.  Knowing the neighbours of an operation saves the passes that the one-by-one form
    spends on elementwise work: bias and ReLU are applied where the product is stored, the
    backward ReLU mask where the gradient is, (1 + eps) H is added in the aggregation, and
    the bias gradients are summed by the kernel that has the gradient in registers.

    ``steps``: a ``_Step`` per layer; what the modules hold may change before the backward pass.
    ``keeps``: whether a backward pass can follow, for which each layer's arrays are kept.
    ``params``: the layers' parameters in the order of ``_params``."""

    @staticmethod
    def forward(ctx, steps, keeps, X, *params):
        d = _Dense(X, [(1, 1)])
        H, keep, at = X.contiguous(), [], 0
        for step in steps:
            H, *saved = _layer_forward(d, step, H, params[at:at + step.n_params])
            at += step.n_params
            if keeps:
                keep += saved
            del saved  # without a gradient each layer's arrays go before the next layer's are made
        ctx.steps = steps
        ctx.n_params = len(params)
        if keeps:
            ctx.save_for_backward(*params, *keep)
        return H

    @staticmethod
    @torch.autograd.function.once_differentiable
    def backward(ctx, dOut):
        saved = ctx.saved_tensors
        params, keep = saved[:ctx.n_params], list(saved[ctx.n_params:])
        d = _Dense(dOut, [tuple(p.shape) for p in params if p.dim() == 2])
        grads = [None] * ctx.n_params
        need = ctx.needs_input_grad[3:]
        G, db = dOut.contiguous(), None  # gradient at the layer's output, its column sums if known
        at = ctx.n_params
        for i in range(len(ctx.steps) - 1, -1, -1):
            step = ctx.steps[i]
            op = step.op
            need_dH = i > 0 or ctx.needs_input_grad[2]
            masked = i > 0 and ctx.steps[i - 1].relu
            # the layer before wants the column sums of its output gradient for its bias, unless
            # its weight gradient reads that gradient anyway
            sums = i > 0 and ctx.steps[i - 1].linear_first and ctx.steps[i - 1].bias
            at -= step.n_params
            if step.gcn:
                has_b = step.bias
                W = params[at]
                if step.linear_first:
                    H = keep.pop()
                    if has_b and need[at + 1]:
                        grads[at + 1] = db if db is not None else d.colsum(G)
                    db = None
                    if need[at] or need_dH:
                        U = d.spmm(op.bwd, op.n_cols, G)
                        db = d.new(W.shape[1]) if sums and need_dH else None
                        if need[at] and need_dH:
                            G, grads[at], _ = d.linear_backward(U, H, W, mask=masked, colsum=db)
                        elif need[at]:
                            grads[at] = d.wgrad(U, H)[0]
                        else:
                            G = d.linear(U, W, transposed=True, mask=H if masked else None, colsum=db)
                else:
                    A, H = keep.pop(), keep.pop()
                    need_W, dA, s, db = need[at] or (has_b and need[at + 1]), None, None, None
                    if need_W and need_dH:
                        dA, grads[at], s = d.linear_backward(G, A, W, bias=has_b)
                    elif need_W:
                        grads[at], s = d.wgrad(G, A, bias=has_b)
                    elif need_dH:
                        dA = d.linear(G, W, transposed=True)
                    if has_b:
                        grads[at + 1] = s
                    if need_dH:
                        G = d.spmm(op.bwd, op.n_cols, dA, mask=H if masked else None)
            else:
                eps, W1, b1, W2, b2 = params[at:at + 5]
                Z, A, H = keep.pop(), keep.pop(), keep.pop()
                db = dA = None
                if all(need[at:at + 5]):
                    dA, *grads[at:at + 5] = d.mlp_backward(G, Z, A, H, W1, W2, store=need_dH)
                    grads[at] = grads[at].view_as(eps)
                else:
                    if need[at + 3] or need[at + 4]:
                        grads[at + 3], grads[at + 4] = d.wgrad(G, Z, bias=True)
                    G1 = d.linear(G, W2, transposed=True, mask=Z)
                    if need[at + 1] or need[at + 2]:
                        grads[at + 1], grads[at + 2] = d.wgrad(G1, A, bias=True)
                    if need[at]:
                        grads[at] = torch.empty_like(eps)
                    if need[at] or need_dH:
                        dA = d.linear(G1, W1, transposed=True, aux=H if need[at] else None, dot=grads[at],
                                      store=need_dH)
                if need_dH:
                    G = d.spmm(op.bwd, op.n_cols, dA, self_term=dA, eps=eps, mask=H if masked else None)
        return (None, None, G if ctx.needs_input_grad[2] else None,
                *(g if n else None for g, n in zip(grads, need)))


class _Step(NamedTuple):
    """One layer of a chain as the forward pass found it."""
    gcn: bool
    op: PcsrOperator
    n_params: int
    bias: bool          # GCN: added to the layer's output
    linear_first: bool  # GCN: multiplied by the weights before the aggregation
    relu: bool


def _layer_forward(d, step, H, params):
    """(output, then what the layer's backward pass reads) of one layer of a chain"""
    op = step.op
    if step.gcn:
        W, b = params[0], params[1] if step.bias else None
        if step.linear_first:
            return d.spmm(op.fwd, op.n_rows, d.linear(H, W), bias=b, relu=step.relu), H
        A = d.spmm(op.fwd, op.n_rows, H)
        return d.linear(A, W, bias=b, relu=step.relu), H, A
    eps, W1, b1, W2, b2 = params
    A = d.spmm(op.fwd, op.n_rows, H, self_term=H, eps=eps)
    Z, Y = d.mlp(A, W1, b1, W2, b2, step.relu)
    return Y, H, A, Z


def _params(layer):
    """Parameters of a layer in the order FusedLayers takes them, None if they are not what it
    knows (modules exchanged or hooked, other types or shapes, too wide)."""
    linear = torch.nn.Linear
    if type(layer) is GCNLayer:
        lins, own = [layer.lin], [layer.lin]
        if type(layer.lin) is not linear or layer.lin.bias is not None:
            return None
        ps = [layer.lin.weight] if layer.bias is None else [layer.lin.weight, layer.bias]
    elif type(layer) is GINLayer:
        mlp = layer.mlp
        if type(mlp) is not torch.nn.Sequential or [type(m) for m in mlp] != [linear, torch.nn.ReLU, linear]:
            return None
        lins, own = [mlp[0], mlp[2]], [mlp, *mlp]
        if any(m.bias is None for m in lins):
            return None
        # the second layer's weights are read as m x m: both kernels and workspaces rely on it
        if mlp[2].out_features != mlp[0].out_features:
            return None
        ps = [layer.eps, mlp[0].weight, mlp[0].bias, mlp[2].weight, mlp[2].bias]
    else:
        return None
    # a product of the operator's own (edge dropout, scaling, counting) would be passed by
    if type(layer.op) is not PcsrOperator or "_run" in vars(layer.op):
        return None
    if any(_hooked(m) for m in own):
        return None
    for i, m in enumerate(lins):
        if m.in_features > MAX_WIDTH or m.out_features > MAX_WIDTH or m.in_features < 1 or m.out_features < 1:
            return None
        if m.weight.shape != (m.out_features, m.in_features) or (i and m.in_features != lins[i - 1].out_features):
            return None
    if any(type(p) not in _PLAIN for p in ps):
        return None
    # a bias that torch would broadcast is one value, not one per output
    for m, b in zip(lins, [layer.bias] if type(layer) is GCNLayer else [m.bias for m in lins]):
        if b is not None and b.shape != (m.out_features,):
            return None
    # one eps, in device memory; of more than two dimensions it would add one to the result
    if type(layer) is GINLayer and (layer.eps.numel() != 1 or layer.eps.dim() > 2):
        return None
    for p in ps:
        if p.dtype != torch.float32 or not p.is_contiguous():
            return None
    return ps


# tensors without behaviour of their own
_PLAIN = (torch.Tensor, torch.nn.Parameter)


def _hooked(m):
    """Whether somebody watches the module's calls, or its forward is not its class's."""
    return bool(m._forward_hooks or m._forward_pre_hooks or m._backward_hooks or m._backward_pre_hooks
                or "forward" in vars(m) or _all_modules._has_any_global_hook())


def _run_fused(chain, X):
    """The chain through FusedLayers, or None where that does not apply."""
    if type(X) not in _PLAIN or X.dim() != 2 or X.dtype != torch.float32 or not X.is_cuda:
        return None
    # kernels are launched on the current device; torch's own products follow their operands
    if torch.is_autocast_enabled() or X.device.index != torch.cuda.current_device():
        return None
    steps, params, n, width = [], [], X.shape[0], X.shape[1]
    for layer, relu in chain:
        ps = _params(layer)
        if ps is None:
            return None
        gcn = type(layer) is GCNLayer
        first, last = (layer.lin, layer.lin) if gcn else (layer.mlp[0], layer.mlp[2])
        if n != layer.op.n_cols or width != first.in_features or any(p.device != X.device for p in ps):
            return None
        if not gcn and layer.op.n_rows != n:
            return None
        steps.append(_Step(gcn, layer.op, len(ps), gcn and layer.bias is not None,
                           gcn and first.in_features >= first.out_features, relu))
        n, width = layer.op.n_rows, last.out_features
        params += ps
    if n == 0 or X.shape[0] == 0:
        return None
    keeps = torch.is_grad_enabled() and any(t.requires_grad for t in (X, *params))
    return FusedLayers.apply(steps, keeps, X, *params)


class GCNLayer(torch.nn.Module):
    """H' = A_hat (H W) + b, the graph convolution of Kipf & Welling with a pre-normalised
    adjacency operator; the dense product comes first when it narrows the features."""

    def __init__(self, op: PcsrOperator, d_in: int, d_out: int, bias: bool = True):
        super().__init__()
        self.op = op
        self.lin = torch.nn.Linear(d_in, d_out, bias=False)
        self.bias = torch.nn.Parameter(torch.zeros(d_out)) if bias else None

    def forward(self, H):
        out = _run_fused([(self, False)], H)
        if out is not None:
            return out
        if self.lin.in_features >= self.lin.out_features:
            out = self.op(self.lin(H))
        else:
            out = self.lin(self.op(H))
        return out if self.bias is None else out + self.bias


class GINLayer(torch.nn.Module):
    """H' = MLP((1 + eps) H + A H), sum aggregation (Xu et al.)."""

    def __init__(self, op: PcsrOperator, d_in: int, d_out: int, eps: float = 0.0):
        super().__init__()
        self.op = op
        self.eps = torch.nn.Parameter(torch.tensor(float(eps)))
        self.mlp = torch.nn.Sequential(torch.nn.Linear(d_in, d_out), torch.nn.ReLU(),
                                       torch.nn.Linear(d_out, d_out))

    def forward(self, H):
        out = _run_fused([(self, False)], H)
        return out if out is not None else self.mlp((1.0 + self.eps) * H + self.op(H))


class LayerChain(torch.nn.Sequential):
    """Graph layers with ReLU between them, run as one chain where FusedLayers applies and module
    by module otherwise (other operators, data types or devices, hooks, wide layers)."""

    def forward(self, X):
        mods = list(self)
        chain = []
        for i, m in enumerate(mods):
            if type(m) is torch.nn.ReLU and chain and not chain[-1][1] and i + 1 < len(mods):
                chain[-1] = (chain[-1][0], True)
            else:
                chain.append((m, False))
            if _hooked(m):
                chain = []
                break
        out = _run_fused(chain, X) if chain else None
        return out if out is not None else super().forward(X)


def make_model(kind: str, op: PcsrOperator, d_in: int, hidden: int, d_out: int, n_layers: int = 5):
    """n_layers graph layers with ReLU between them (the paper trains 5-layer GCN / GIN
    models with hidden sizes 32, 64, 128 and 16 input / output features)."""
    dims = [d_in] + [hidden] * (n_layers - 1) + [d_out]
    layer = {"gcn": GCNLayer, "gin": GINLayer}[kind]
    mods = []
    for i in range(n_layers):
        mods.append(layer(op, dims[i], dims[i + 1]))
        if i + 1 < n_layers:
            mods.append(torch.nn.ReLU())
    return LayerChain(*mods)
