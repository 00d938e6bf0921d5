"""The fused GNN layers on the GPU: each dense kernel and the SpMM epilogue against fp64 torch at
the edges of their tiles, and whole models against the same model on a dense adjacency."""
import numpy as np
import pytest

import paper_2605_15695_amd as pc
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _close(got, ref, tol=1e-5):
    err = float((got.double() - ref).norm() / ref.norm().clamp_min(1e-30))
    assert err < tol, err


def _dense(a, b):
    from paper_2605_15695_amd.gnn import _Dense
    return _Dense(torch.empty(1, device="cuda"), [(a, b)])


# widths: whole tiles, part tiles, odd (no vector loads), one column, the widest
@pytest.mark.parametrize("a,b", [(16, 64), (64, 64), (64, 16), (24, 48), (96, 32), (128, 128), (33, 7), (1, 1), (47, 65),
                                 (128, 20), (6, 100)])
@pytest.mark.parametrize("n", [1, 31, 257, 70001])
def test_dense_kernels(a, b, n):
    g = torch.Generator(device="cuda").manual_seed(a * 1000 + b)
    X, G, aux = (torch.randn(n, w, generator=g, device="cuda") for w in (a, b, b))
    W, bias = torch.randn(b, a, generator=g, device="cuda"), torch.randn(b, generator=g, device="cuda")
    mask = torch.where(torch.rand(n, b, generator=g, device="cuda") < 0.5, 0.0, 1.0)
    d = _dense(a, b)
    Xd, Wd = X.double(), W.double()
    lin = Xd @ Wd.t()
    _close(d.linear(X, W), lin)
    _close(d.linear(X, W, bias=bias, relu=True), torch.relu(lin + bias.double()))
    csum, dot = torch.empty(b, device="cuda"), torch.empty((), device="cuda")
    Wt = W.t().contiguous()
    Y = d.linear(X, Wt, transposed=True, mask=mask, aux=aux, dot=dot, colsum=csum)
    _close(Y, lin * mask.double())
    size = Xd.abs() @ Wd.abs().t()                  # what the rounding errors scale with
    scale = size.sum(0)
    assert bool(((csum.double() - (lin * mask.double()).sum(0)).abs() <= 1e-6 * scale + 1e-30).all())
    total = (size * aux.double().abs()).sum()
    assert abs(float(dot.double() - (lin * aux.double()).sum())) <= 1e-6 * float(total)
    dW, db = d.wgrad(G, X, bias=True)
    ref = G.double().t() @ Xd
    bound = G.double().abs().t() @ Xd.abs()
    assert bool(((dW.double() - ref).abs() <= 1e-6 * bound).all())
    gb = G.double().abs().sum(0)
    assert bool(((db.double() - G.double().sum(0)).abs() <= 1e-6 * gb).all())
    assert bool(((d.colsum(G).double() - G.double().sum(0)).abs() <= 1e-6 * gb).all())


# weight gradients: one, two and four squares, widths short of a tile, rows short of a step, rows at no multiple of 16 bytes.
# Lanes past the end of a row read the next one: an infinite column there reaches no other column's sum.
# A sum of n terms is off by at most n * 2^-24 of the sum of their magnitudes, 1e-6 up to n = 16; beyond that rounding errors
# of the chains add up like sqrt(n), and a wavefront's chain is 64 terms up to n = 131,072 (one square) or 32,768 (four), and n / 2048
# or n / 512 above.
@pytest.mark.parametrize("a,b", [(1, 128), (2, 40), (17, 33), (48, 48), (49, 96), (65, 64), (80, 97), (96, 96), (127, 5),
                                 (128, 65)])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 64 * 16 + 3, 40009])
@pytest.mark.parametrize("skew", [0, 1])
def test_weight_gradient(a, b, n, skew):
    g = torch.Generator(device="cuda").manual_seed(a * 1000 + b + n)
    X, G = (torch.randn(n * w + skew, generator=g, device="cuda")[skew:].view(n, w) for w in (a, b))
    d = _dense(a, b)
    dW, db = d.wgrad(G, X, bias=True)
    bound = G.double().abs().t() @ X.double().abs()
    assert bool(((dW.double() - G.double().t() @ X.double()).abs() <= 1e-6 * bound).all())
    assert bool(((db.double() - G.double().sum(0)).abs() <= 1e-6 * G.double().abs().sum(0)).all())
    first, sums = dW.clone(), db.clone()
    X[:, 0] = float("inf")
    G[:, 0] = float("inf")
    dW, db = d.wgrad(G, X, bias=True)
    assert torch.equal(dW[1:, 1:], first[1:, 1:]) and torch.equal(db[1:], sums[1:])
    assert bool(torch.isinf(db[0])) and not bool(torch.isfinite(dW[0]).any() or torch.isfinite(dW[:, 0]).any())


# both sides of the lines between its forms: squares in workgroups of their own and together, arrays that the memory-side cache holds
# and larger ones (256 MB), whose rows are read past it on the sides that are read once; tolerances as above
@pytest.mark.parametrize("a,b,n", [(96, 96, 131072), (96, 96, 131073), (128, 100, 131089), (47, 65, 131073), (128, 64, 131100),
                                   (16, 16, (1 << 21) + 5), (128, 16, 500003), (16, 128, 500003), (40, 64, 700001)])
def test_weight_gradient_of_many_rows(a, b, n):
    g = torch.Generator(device="cuda").manual_seed(n + a)
    X, G = (torch.randn(n, w, generator=g, device="cuda") for w in (a, b))
    dW, db = _dense(a, b).wgrad(G, X, bias=True)
    Xd, Gd = X.double(), G.double()
    assert bool(((dW.double() - Gd.t() @ Xd).abs() <= 1e-6 * (Gd.abs().t() @ Xd.abs())).all())
    assert bool(((db.double() - Gd.sum(0)).abs() <= 1e-6 * Gd.abs().sum(0)).all())


# what is left for the second pass: one partial dW for 256 rows at most where dW is cut, or short inputs spend their time on it
@pytest.mark.parametrize("a,b", [(64, 128), (128, 64), (128, 128), (96, 96)])
@pytest.mark.parametrize("n", [5000, 32768])
def test_weight_gradient_leaves_few_partial_sums(a, b, n):
    d = _dense(a, b)
    ws = d._ws = torch.full((d.ws_floats,), float("nan"), device="cuda")
    d.wgrad(torch.randn(n, b, device="cuda"), torch.randn(n, a, device="cuda"), bias=True)
    assert int((~torch.isnan(ws)).sum()) == -(-n // 256) * (a * b + b)


# exact widths: each set of arrays beside X has a loop of its own, and sums of eight groups of rows are put apart (of 16 rows: from
# 131,072 or 262,144 rows on, with one and two workgroups to a compute unit)
@pytest.mark.parametrize("a,b", [(16, 16), (64, 64), (16, 128), (128, 48), (128, 128)])
@pytest.mark.parametrize("n", [15, 300007])
@pytest.mark.parametrize("aux,mask,store,sums", [(0, 0, 1, 0), (0, 1, 1, 0), (1, 0, 1, 1), (0, 1, 1, 1), (1, 0, 0, 1), (0, 0, 1, 1), (1, 1, 1, 1)])
def test_arrays_beside_the_rows(a, b, n, aux, mask, store, sums):
    g = torch.Generator(device="cuda").manual_seed(a + b + n)
    X, A, M = (torch.randn(n, w, generator=g, device="cuda") for w in (a, b, b))
    W = torch.randn(a, b, generator=g, device="cuda")
    dot, csum = torch.empty((), device="cuda"), torch.empty(b, device="cuda")
    Y = _dense(a, b).linear(X, W, transposed=True, mask=M if mask else None, aux=A if aux else None, dot=dot if aux else None,
                            colsum=csum if sums else None, store=bool(store))
    lin, size = X.double() @ W.double(), X.double().abs() @ W.double().abs()
    if aux:
        assert abs(float(dot.double() - (lin * A.double()).sum())) <= 1e-6 * float((size * A.double().abs()).sum())
    if mask:
        lin = lin * (M > 0)
    if store:
        _close(Y, lin)
    else:
        assert Y is None
    if sums:
        assert bool(((csum.double() - lin.sum(0)).abs() <= 1e-6 * size.sum(0)).all())


# rows short of a piece: the bias of rows that are not there is in no sum
@pytest.mark.parametrize("a,b", [(16, 16), (64, 64), (128, 128), (96, 32), (24, 48), (33, 7)])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 1000 * 16 + 5])
@pytest.mark.parametrize("relu", [False, True])
def test_column_sums_with_a_bias(a, b, n, relu):
    g = torch.Generator(device="cuda").manual_seed(a * 1000 + b)
    X = torch.randn(n, a, generator=g, device="cuda")
    W, bias = torch.randn(b, a, generator=g, device="cuda"), 3.0 + torch.rand(b, generator=g, device="cuda")
    csum = torch.empty(b, device="cuda")
    Y = _dense(a, b).linear(X, W, bias=bias, relu=relu, colsum=csum)
    ref = X.double() @ W.double().t() + bias.double()
    if relu:
        ref = torch.relu(ref)
    _close(Y, ref)
    # fp32 sums of n terms in short chains: 1e-6 of the sum of the magnitudes, as above
    scale = (X.double().abs() @ W.double().abs().t() + bias.double()).sum(0)
    assert bool(((csum.double() - ref.sum(0)).abs() <= 1e-6 * scale).all())


# one pass for two products: each width of the 16-row pieces, rows short of a piece, a misaligned input
@pytest.mark.parametrize("a,m", [(16, 16), (32, 48), (48, 32), (64, 64), (16, 64)])
@pytest.mark.parametrize("n,skew", [(1, 0), (15, 0), (17, 1), (70001, 0)])
def test_two_products_in_one_pass(a, m, n, skew):
    g = torch.Generator(device="cuda").manual_seed(a * 100 + m)
    A, H = (torch.randn(n * a + 1, generator=g, device="cuda")[skew:skew + n * a].view(n, a) for _ in range(2))
    G = torch.randn(n, m, generator=g, device="cuda")
    W1, W2 = torch.randn(m, a, generator=g, device="cuda"), torch.randn(m, m, generator=g, device="cuda")
    b1, b2 = torch.randn(m, generator=g, device="cuda"), torch.randn(m, generator=g, device="cuda")
    d = _dense(a, m)
    d.ws_floats = max(d.ws_floats, d.lib.pcsr_gnn_workspace_floats(m, m))
    Ad, Hd, Gd, W1d, W2d = (t.double() for t in (A, H, G, W1, W2))
    Z, Y = d.mlp(A, W1, b1, W2, b2, True)
    _close(Z, torch.relu(Ad @ W1d.t() + b1.double()))
    _close(Y, torch.relu(Z.double() @ W2d.t() + b2.double()))
    dA, dot, dW1, db1, dW2, db2 = d.mlp_backward(G, Z, A, H, W1, W2, True)
    G1 = (Gd @ W2d) * (Z > 0)
    _close(dA, G1 @ W1d)
    _close(dW2, Gd.t() @ Z.double())
    _close(dW1, G1.t() @ Ad)
    _close(db2, Gd.sum(0))
    _close(db1, G1.sum(0))
    total = ((Gd.abs() @ W2d.abs()) @ W1d.abs() * Hd.abs()).sum()
    assert abs(float(dot.double() - ((G1 @ W1d) * Hd).sum())) <= 1e-6 * float(total)
    cs = torch.empty(a, device="cuda")
    for mask in (False, True):
        dX, dW, db = d.linear_backward(G, A, W1, bias=True, mask=mask, colsum=cs)
        ref = (Gd @ W1d) * ((Ad > 0) if mask else 1.0)
        _close(dX, ref)
        _close(dW, Gd.t() @ Ad)
        _close(db, Gd.sum(0))
        _close(cs, ref.sum(0))


# rows past the end are zeros, and zeros times an infinite weight are not: sums stay infinite, not NaN
@pytest.mark.parametrize("n", [1, 17, 32, 4097])
def test_sums_over_rows_with_an_infinite_weight(n):
    g = torch.Generator(device="cuda").manual_seed(n)
    A, H, G = (0.5 + torch.rand(n, 32, generator=g, device="cuda") for _ in range(3))
    W1, W2 = (0.5 + torch.rand(32, 32, generator=g, device="cuda") for _ in range(2))
    W1[3, 5] = float("inf")
    d = _dense(32, 32)
    cs = torch.empty(32, device="cuda")
    d.linear_backward(G, A, W1, bias=True, colsum=cs)
    assert bool(torch.isinf(cs[5])) and bool(torch.isfinite(cs[:5]).all())
    dA, dot, *_ = d.mlp_backward(G, A, A, H, W1, W2, True)
    assert bool(torch.isinf(dA[:, 5]).all()) and bool(torch.isinf(dot))


def _matches(got, ref, size, terms):
    """Infinite and no number where ref is; elsewhere within the bound of a chain of so many fp32 sums, one rounding each."""
    got, ref = got.double(), torch.where(ref.abs() > 3.4028235e38, ref * float("inf"), ref)
    finite = torch.isfinite(ref)
    assert bool((torch.isnan(got) == torch.isnan(ref)).all()) and bool((torch.isinf(got) == torch.isinf(ref)).all())
    assert bool((got == ref)[torch.isinf(ref)].all())
    assert bool(((got - ref).abs() <= terms * 2.0 ** -24 * size + 1e-30)[finite].all())


# products in pieces: rows, weights and biases that have no pieces (from 2^50 and 2^16 on, and infinities), in the first rows, among those of
# a loop that has begun, in a group that is not whole.  One number of a product may be all of its size, so that every sum after it is
# rounded at that size: the bound is that of the whole chain, of as many terms as the product has and, for sums over rows, as a wavefront has
# rows (40009 / 2048 groups of 16, or steps of 16 rows in four parts) and a column has partial sums (512, 16 of them in a chain).
@pytest.mark.parametrize("a,b", [(16, 64), (32, 64), (64, 64), (48, 64), (64, 96), (96, 96), (64, 128), (128, 128)])
@pytest.mark.parametrize("n,row", [(5, 0), (40009, 39000), (40009, 40008)])
@pytest.mark.parametrize("value,where", [(float("inf"), "row"), (-3e30, "row"), (2.0 ** 60, "row"), (float("inf"), "weight"),
                                         (2.0 ** 20, "weight"), (1e30, "weight"), (float("inf"), "bias"), (1e30, "bias"),
                                         (2.0 ** 50, "row"), (1.1e15, "row"), (2.0 ** 16, "weight"), (65535.0, "weight"), (1.1e15, "bias"),
                                         (2.0 ** 50, "bias")])
def test_numbers_without_pieces(a, b, n, row, value, where):
    g = torch.Generator(device="cuda").manual_seed(a * 100 + b)
    X, H = (torch.randn(n, a, generator=g, device="cuda") for _ in range(2))
    G = torch.randn(n, b, generator=g, device="cuda")
    W1, W2 = torch.randn(b, a, generator=g, device="cuda"), torch.randn(b, b, generator=g, device="cuda")
    b1, b2 = torch.randn(b, generator=g, device="cuda"), torch.randn(b, generator=g, device="cuda")
    if where == "row":
        X[row, 7] = value
        G[row, 9] = value
    elif where == "weight":
        W1[5, 3] = value
    else:
        b1[5] = value
    d = _dense(a, b)
    d.ws_floats = max(d.ws_floats, d.lib.pcsr_gnn_workspace_floats(b, b))
    Xd, Gd, Hd, W1d, W2d, b1d, b2d = (t.double() for t in (X, G, H, W1, W2, b1, b2))
    size1 = Xd.abs() @ W1d.abs().t() + b1d.abs()
    _matches(d.linear(X, W1, bias=b1, relu=True), torch.relu(Xd @ W1d.t() + b1d), size1, a + 2)
    cs = torch.empty(a, device="cuda")
    back, size = Gd @ W1d, Gd.abs() @ W1d.abs()
    _matches(d.linear(G, W1, transposed=True, colsum=cs), back, size, b + 2)
    _matches(cs, back.sum(0), size.sum(0), b + 400)
    Z, Y = d.mlp(X, W1, b1, W2, b2, True)
    _matches(Z, torch.relu(Xd @ W1d.t() + b1d), size1, a + 2)
    _matches(Y, torch.relu(Z.double() @ W2d.t() + b2d), Z.double().abs() @ W2d.abs().t() + b2d.abs(), b + 2)
    dX, dW, db = d.linear_backward(G, X, W1, bias=True, colsum=cs)
    _matches(dX, back, size, b + 2)
    _matches(dW, Gd.t() @ Xd, Gd.abs().t() @ Xd.abs(), 400)
    Z = torch.relu(torch.randn(n, b, generator=g, device="cuda"))
    dA, dot, dW1, db1, dW2, db2 = d.mlp_backward(G, Z, X, H, W1, W2, True)
    G1 = torch.where(Z > 0, Gd @ W2d, 0.0)
    size2 = torch.where(Z > 0, Gd.abs() @ W2d.abs(), 0.0)
    _matches(dA, G1 @ W1d, size2 @ W1d.abs(), 2 * b + 4)
    _matches(dW1, G1.t() @ Xd, size2.t() @ Xd.abs(), b + 400)
    _matches(dW2, Gd.t() @ Z.double(), Gd.abs().t() @ Z.double(), 400)
    _matches(db1, G1.sum(0), size2.sum(0), b + 400)


def _in_pieces(a, b, seed, scale_rows=1.0, scale_weights=1.0, n=20011):
    """(name, got, 64 bits, magnitudes) of the layers' products of normal numbers, whatever form the widths take them in"""
    g = torch.Generator(device="cuda").manual_seed(seed)
    X, H = (torch.randn(n, a, generator=g, device="cuda") * scale_rows for _ in range(2))
    G = torch.randn(n, b, generator=g, device="cuda") * scale_rows
    W1 = torch.randn(b, a, generator=g, device="cuda") * scale_weights
    W2 = torch.randn(b, b, generator=g, device="cuda")
    zero = torch.zeros(b, device="cuda")
    d = _dense(a, b)
    d.ws_floats = max(d.ws_floats, d.lib.pcsr_gnn_workspace_floats(b, b))
    Xd, Gd, W1d, W2d = (t.double() for t in (X, G, W1, W2))
    fwd, back = (Xd @ W1d.t(), Xd.abs() @ W1d.abs().t()), (Gd @ W1d, Gd.abs() @ W1d.abs())
    yield "linear", d.linear(X, W1), *fwd
    yield "turned", d.linear(G, W1, transposed=True), *back
    Z, Y = d.mlp(X, W1, zero, W2, zero, False)
    yield "first", Z, torch.relu(fwd[0]), fwd[1]
    yield "second", Y, Z.double() @ W2d.t(), Z.double().abs() @ W2d.abs().t()
    yield "back", d.linear_backward(G, X, W1)[0], *back
    Z = torch.relu(torch.randn(n, b, generator=g, device="cuda"))
    on = (Z > 0).double()
    dA = d.mlp_backward(G, Z, X, H, W1, W2, True)[0]
    yield "both", dA, (Gd @ W2d * on) @ W1d, (Gd.abs() @ W2d.abs() * on) @ W1d.abs()


# Against 64 bits: the fp32 instructions are off by 1.45e-7 over 64 terms and 2.03e-7 over 128 (2-norm), pieces by 0.50 and 0.65e-7; with
# all six products in one accumulator it is 0.93 and 1.53e-7, to one side, and without the two smallest 34e-7.  The mean difference is
# 0.4e-10 of the magnitudes at most, where that of one accumulator is ten times as much.
@pytest.mark.parametrize("a,b,pieces", [(64, 64, ("first", "second", "back")), (32, 64, ("first", "second", "both")), (64, 96, ("linear", "turned")),
                                        (64, 128, ("linear", "turned")), (96, 96, ("linear", "turned")), (96, 128, ("linear", "turned")),
                                        (128, 128, ("linear", "turned"))])
def test_products_in_pieces_are_more_exact_than_fp32_ones(a, b, pieces):
    most = {32: 0.65e-7, 64: 0.75e-7, 96: 0.85e-7, 128: 0.95e-7}
    seen = []
    for name, got, ref, size in _in_pieces(a, b, a * 100 + b):
        off = got.double() - ref
        seen.append((name, float(off.norm() / ref.norm()), float((off / size.clamp_min(1e-30)).mean())))
    for name, norm, mean in seen:
        if name in pieces:
            terms = a if name in ("linear", "first") else b
            assert norm < (1.1e-7 if name == "both" else most[terms]), seen
            assert abs(mean) < 1.5e-10, seen


# Numbers near the least that a float can be: bf16 does not reach as low, so the pieces are of numbers 2^16 times as large.  The
# bound is that of a chain of fp32 sums, each off by half of the last bit or of the least number.
@pytest.mark.parametrize("a,b", [(32, 64), (64, 64), (64, 96), (96, 96), (64, 128), (128, 128)])
@pytest.mark.parametrize("rows,weights", [(-105, 0), (-115, 0), (-124, 0), (-130, 0), (-146, 0), (0, -115), (0, -130), (0, -146), (-60, -60),
                                          (40, -130), (-130, 12)])
def test_small_numbers_have_pieces(a, b, rows, weights):
    for name, got, ref, size in _in_pieces(a, b, a * 100 + b, 2.0 ** rows, 2.0 ** weights, n=4099):
        terms = 2 * b + 4 if name == "both" else b + 2 if name in ("turned", "back", "second") else a + 2
        off = (got.double() - ref).abs()
        # (the products of two layers round twice: the second takes the least number of the first by its weights)
        least = terms * 2.0 ** -150 * (1.0 + 4.0 * b * max(2.0 ** weights, 1.0) * (name == "both"))
        assert bool((off <= terms * 2.0 ** -24 * size + least).all()), (name, float((off / (size + 1e-300)).max()))
        # no sum is near the least number (of two layers, nor the first one's): the fp32 instructions' 2-norm over 128 terms, and over two layers
        if min(rows + weights, rows if name == "both" else 0) >= -120:
            assert float(off.norm() / ref.norm()) < 2.5e-7, name


# one large number whose weight is zero beside small ones: these are the result
def test_small_numbers_beside_large_ones():
    n, a, b = 1000, 96, 128
    g = torch.Generator(device="cuda").manual_seed(1)
    X, W = torch.randn(n, a, generator=g, device="cuda") * 2.0 ** -118, torch.randn(b, a, generator=g, device="cuda")
    X[:, 5], W[:, 5] = 3.0, 0.0
    ref, size = X.double() @ W.double().t(), X.double().abs() @ W.double().abs().t()
    _matches(_dense(a, b).linear(X, W) * 2.0 ** 100, ref * 2.0 ** 100, size * 2.0 ** 100, a + 2)


@pytest.mark.parametrize("a,b", [(64, 64), (64, 96), (64, 128), (128, 128)])
@pytest.mark.parametrize("n,row", [(5, 0), (4099, 3000), (4099, 4098)])
@pytest.mark.parametrize("where", ["row", "weight"])
def test_no_number_shows_where_it_belongs(a, b, n, row, where):
    g = torch.Generator(device="cuda").manual_seed(a * 100 + b)
    X, G = torch.randn(n, a, generator=g, device="cuda"), torch.randn(n, b, generator=g, device="cuda")
    W = torch.randn(b, a, generator=g, device="cuda")
    if where == "row":
        X[row, 7] = G[row, 9] = float("nan")
    else:
        W[5, 3] = float("nan")
    d = _dense(a, b)
    Xd, Gd, Wd = X.double(), G.double(), W.double()
    _matches(d.linear(X, W), Xd @ Wd.t(), Xd.abs() @ Wd.abs().t(), a + 2)
    for got in (d.linear(G, W, transposed=True), d.linear_backward(G, X, W)[0]):
        _matches(got, Gd @ Wd, Gd.abs() @ Wd.abs(), b + 2)


@pytest.mark.parametrize("name,kw", [("rmat20", dict(V=1, S=1, SG=4)), ("rmat20", dict(V=2, S=0)),
                                     ("sbm", dict(V=1, col_window=512)), ("road", dict(V=2, items_per_group=2)),
                                     ("rmat22", dict(V=2, S=1, SG=2))])
@pytest.mark.parametrize("K", [16, 33])
def test_spmm_epilogue(name, kw, K):
    g = synth.workload(name, "small")
    h = pc.pcsr_build(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, pc.make_params(**kw))
    B = torch.from_numpy(synth.dense_operand(g.n_cols, K, "normal", 3)).cuda()
    own = torch.from_numpy(synth.dense_operand(g.n_rows, K, "normal", 4)).cuda()
    mask = torch.from_numpy(synth.dense_operand(g.n_rows, K, "normal", 5)).cuda()
    bias = torch.from_numpy(synth.dense_operand(1, K, "normal", 6)).cuda().reshape(-1)
    eps = torch.tensor(0.25, device="cuda")
    d = _dense(1, 1)
    plain = d.spmm(h, g.n_rows, B)
    _close(d.spmm(h, g.n_rows, B, bias=bias, relu=True), torch.relu(plain.double() + bias.double()), 1e-6)
    _close(d.spmm(h, g.n_rows, B, self_term=own, eps=eps, mask=mask),
           torch.where(mask <= 0, 0.0, plain.double() + 1.25 * own.double()), 1e-6)


@pytest.mark.parametrize("kind", ["gcn", "gin"])
@pytest.mark.parametrize("dims", [(16, 32, 16, 5), (8, 20, 24, 3), (64, 64, 16, 2), (7, 33, 5, 3), (16, 16, 16, 1)])
@pytest.mark.parametrize("x_grad", [False, True])
def test_models_match_dense_adjacency(kind, dims, x_grad):
    import scipy.sparse as sp

    from paper_2605_15695_amd import gnn

    d_in, hidden, d_out, layers = dims
    g = synth.workload("poisson", "small")
    op = gnn.PcsrOperator(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, K_hint=hidden)
    torch.manual_seed(1)
    model = gnn.make_model(kind, op, d_in, hidden, d_out, layers).cuda()
    X = torch.from_numpy(synth.dense_operand(g.n_rows, d_in, "normal", 9)).cuda().requires_grad_(x_grad)
    calls = []
    out = model(X)
    assert type(out.grad_fn).__name__ == "FusedLayersBackward"
    out.square().mean().backward()
    A = torch.from_numpy(sp.csr_matrix((g.vals, g.colidx, g.rowptr), shape=(g.n_rows, g.n_cols)).toarray()
                         .astype(np.float64))

    class DenseOp:
        def __call__(self, H):
            calls.append(1)
            return A @ H

    ref = gnn.make_model(kind, DenseOp(), d_in, hidden, d_out, layers).double()
    ref.load_state_dict({k: v.double().cpu() for k, v in model.state_dict().items()})
    Xr = X.detach().double().cpu().requires_grad_(x_grad)
    r = ref(Xr)
    r.square().mean().backward()
    assert len(calls) == layers
    _close(out.cpu(), r.detach(), 1e-4)
    for p, q in zip(model.parameters(), ref.parameters()):
        _close(p.grad.cpu(), q.grad, 1e-3)
    if x_grad:
        _close(X.grad.cpu(), Xr.grad, 1e-3)


def test_hooked_or_wide_models_run_module_by_module():
    from paper_2605_15695_amd import gnn

    g = synth.workload("poisson", "small")
    op = gnn.PcsrOperator(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, K_hint=32)
    X = torch.from_numpy(synth.dense_operand(g.n_rows, 16, "normal", 9)).cuda()
    model = gnn.make_model("gcn", op, 16, 32, 16, 3).cuda()
    plain = model(X)
    seen = []
    model[1].register_forward_hook(lambda m, i, o: seen.append(o.shape))
    out = model(X)
    assert seen == [(g.n_rows, 32)]
    _close(out.detach(), plain.detach().double(), 1e-5)
    wide = gnn.make_model("gin", op, 16, 160, 16, 2).cuda()
    wide(X).sum().backward()
    assert all(p.grad is not None for p in wide.parameters())


def test_epilogue_on_a_handle_with_a_shape_of_its_own():
    g = synth.workload("sbm", "small")
    h = pc.pcsr_build(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, pc.make_params(lanes_per_row=16, vec=1, rep=2))
    B = torch.from_numpy(synth.dense_operand(g.n_cols, 32, "normal", 3)).cuda()
    d = _dense(1, 1)
    _close(d.spmm(h, g.n_rows, B, relu=True), torch.relu(d.spmm(h, g.n_rows, B).double()), 1e-6)


def _narrower_second(layer):
    layer.mlp[2] = torch.nn.Linear(64, 32)


def _one_bias(layer):
    layer.bias = torch.nn.Parameter(torch.full((1,), 0.5))


def _one_inner_bias(layer):
    layer.mlp[0].bias = torch.nn.Parameter(torch.full((1,), 0.5))


def _eps_vector(layer):
    layer.eps = torch.nn.Parameter(torch.linspace(0.0, 1.0, 16))


def _eps_number(layer):
    del layer.eps
    layer.eps = 0.25


# layers that the fused node does not take give what torch's own modules give
@pytest.mark.parametrize("kind,change", [("gin", _narrower_second), ("gcn", _one_bias), ("gin", _one_inner_bias),
                                         ("gin", _eps_vector), ("gin", _eps_number)])
def test_changed_layers_match_torch(kind, change):
    from paper_2605_15695_amd import gnn

    g = synth.workload("poisson", "small")
    op = gnn.PcsrOperator(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, K_hint=64)
    torch.manual_seed(2)
    layer = {"gcn": gnn.GCNLayer, "gin": gnn.GINLayer}[kind](op, 16, 64)
    change(layer)
    layer = layer.cuda()
    X = torch.from_numpy(synth.dense_operand(g.n_rows, 16, "normal", 9)).cuda()
    out = layer(X)
    out.square().mean().backward()
    assert type(out.grad_fn).__name__ != "FusedLayersBackward"
    grads = [p.grad.clone() for p in layer.parameters()]
    layer.zero_grad()
    if kind == "gcn":
        ref = op(layer.lin(X)) if layer.lin.in_features >= layer.lin.out_features else layer.lin(op(X))
        ref = ref + layer.bias
    else:
        ref = layer.mlp((1.0 + layer.eps) * X + op(X))
    ref.square().mean().backward()
    assert out.shape == ref.shape and torch.equal(out, ref)
    for a, p in zip(grads, layer.parameters()):
        _close(a, p.grad.double(), 1e-6)


def test_an_operator_with_its_own_product_is_asked():
    from paper_2605_15695_amd import gnn

    class Scaled(gnn.PcsrOperator):
        def _run(self, handle, n_out, X):
            return 0.5 * super()._run(handle, n_out, X)

    g = synth.workload("poisson", "small")
    args = (g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals)
    X = torch.from_numpy(synth.dense_operand(g.n_rows, 16, "normal", 9)).cuda()
    for kind in ("gcn", "gin"):
        torch.manual_seed(3)
        model = gnn.make_model(kind, gnn.PcsrOperator(*args, K_hint=32), 16, 32, 16, 1).cuda()
        torch.manual_seed(3)
        scaled = gnn.make_model(kind, Scaled(*args, K_hint=32), 16, 32, 16, 1).cuda()
        half = gnn.PcsrOperator(*args[:4], g.vals * np.float32(0.5), K_hint=32)
        model[0].op = half
        _close(scaled(X).detach(), model(X).detach().double(), 1e-5)


def test_operands_on_another_device_than_the_current_one_are_left_to_torch(monkeypatch):
    from paper_2605_15695_amd import gnn

    g = synth.workload("poisson", "small")
    op = gnn.PcsrOperator(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, K_hint=32)
    layer = gnn.GCNLayer(op, 16, 16).cuda()
    X = torch.from_numpy(synth.dense_operand(g.n_rows, 16, "normal", 9)).cuda()
    assert gnn._run_fused([(layer, False)], X) is not None
    monkeypatch.setattr(torch.cuda, "current_device", lambda: X.device.index + 1)
    assert gnn._run_fused([(layer, False)], X) is None


# split panels whose partial sums meet in C take no epilogue: the elementwise tail follows the product
@pytest.mark.parametrize("kind", ["gcn", "gin"])
@pytest.mark.parametrize("features", [16, 48])
def test_layers_on_an_operator_with_atomic_sums(kind, features):
    from paper_2605_15695_amd import gnn

    g = synth.workload("rmat20", "small")
    args = (g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals)
    X = torch.from_numpy(synth.dense_operand(g.n_rows, features, "normal", 9)).cuda()
    results = []
    for flags in (0, pc.PCSR_FLAG_ATOMIC_SPLIT):
        op = gnn.PcsrOperator(*args, params=pc.make_params(V=1, S=1, SG=8, flags=flags))
        torch.manual_seed(4)
        model = gnn.make_model(kind, op, features, 32, 16, 3).cuda()
        for p in model.parameters():                   # biases and eps that matter
            if p.dim() < 2:
                torch.nn.init.constant_(p, 0.25)
        out = model(X)
        out.square().mean().backward()
        results.append([out.detach(), *(p.grad for p in model.parameters())])
    for a, b in zip(*results):
        _close(b, a.double(), 1e-4)


@pytest.mark.parametrize("kind", ["gcn", "gin"])
def test_forward_alone_keeps_no_layer_but_the_current_one(kind):
    from paper_2605_15695_amd import gnn

    g = synth.workload("road", "small")
    op = gnn.PcsrOperator(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, symmetric=True, K_hint=128)
    model = gnn.make_model(kind, op, 128, 128, 128, 8).cuda()
    X = torch.randn(g.n_rows, 128, device="cuda")
    array = X.numel() * 4

    def peak():
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_allocated()
        out = model(X)
        torch.cuda.synchronize()
        return (torch.cuda.max_memory_allocated() - before) / array, out

    with torch.no_grad():
        model(X)                                       # the handle's own first call
        few, out = peak()
    most, ref = peak()
    assert torch.equal(out, ref) and ref.requires_grad and not out.requires_grad
    # input, aggregate, hidden and output rows of one layer; a graph keeps two to three of each of the eight
    assert few <= 4.5 and most > 8, (few, most)
    frozen = [p.requires_grad_(False) for p in model.parameters()]
    assert frozen and peak()[0] <= 4.5


def test_backward_uses_the_operator_of_its_forward():
    from paper_2605_15695_amd import gnn

    g = synth.workload("poisson", "small")
    args = (g.n_rows, g.n_cols, g.rowptr, g.colidx)
    one = gnn.PcsrOperator(*args, g.vals, K_hint=32)
    other = gnn.PcsrOperator(*args, g.vals * np.float32(3.0), K_hint=32)
    X = torch.from_numpy(synth.dense_operand(g.n_rows, 16, "normal", 9)).cuda()
    for kind in ("gcn", "gin"):
        model = gnn.make_model(kind, one, 16, 32, 16, 2).cuda()
        want = torch.autograd.grad(model(X).square().mean(), list(model.parameters()))
        loss = model(X).square().mean()
        for layer in (model[0], model[2]):             # the next batch's graph
            layer.op = other
            if kind == "gcn":
                layer.bias = None
        got = torch.autograd.grad(loss, [p for p in model.parameters()])
        want = want if kind == "gin" else [w for w in want if w.dim() == 2]
        for a, b in zip(got, want):
            assert torch.equal(a, b)


def test_a_handle_of_another_size_is_refused():
    from paper_2605_15695_amd import gnn

    g, small = synth.workload("poisson", "small"), synth.workload("sbm", "small")
    op = gnn.PcsrOperator(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, K_hint=32)
    X = torch.from_numpy(synth.dense_operand(g.n_rows, 16, "normal", 9)).cuda()
    wrong = pc.pcsr_build(small.n_rows, small.n_cols, small.rowptr, small.colidx, small.vals)
    assert small.n_rows != g.n_rows
    layer = gnn.GCNLayer(op, 16, 32).cuda()
    out = layer(X)
    op.bwd = wrong
    with pytest.raises(ValueError):
        layer(X.requires_grad_(True)).sum().backward()
    op.fwd = wrong
    with pytest.raises(ValueError):
        layer(X)
    assert out.shape == (g.n_rows, 32)


@pytest.mark.parametrize("V", [1, 2])
@pytest.mark.parametrize("K", [16, 33, 128, 512])
def test_every_part_of_the_tail_alone_and_with_the_others(V, K):
    """Tails with a self term or a mask run other instances than those without."""
    g = synth.workload("poisson", "small")
    h = pc.pcsr_build(g.n_rows, g.n_cols, g.rowptr, g.colidx, g.vals, pc.make_params(V=V))
    B, own, mask, bias = (torch.from_numpy(synth.dense_operand(n, K, "normal", 3 + i)).cuda()
                          for i, n in enumerate((g.n_cols, g.n_rows, g.n_rows, 1)))
    d = _dense(1, 1)
    plain = d.spmm(h, g.n_rows, B).double()
    for parts in range(1, 16):
        kw = dict(self_term=own if parts & 1 else None, bias=bias.reshape(-1) if parts & 2 else None, relu=bool(parts & 4),
                  mask=mask if parts & 8 else None)
        want = plain + (own.double() if parts & 1 else 0.0) + (bias.double() if parts & 2 else 0.0)
        want = torch.relu(want) if parts & 4 else want
        want = torch.where(mask <= 0, 0.0, want) if parts & 8 else want
        _close(d.spmm(h, g.n_rows, B, **kw), want, 1e-6)
    h.close()
