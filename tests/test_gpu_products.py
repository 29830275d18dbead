"""The dense products of a layer (H W, dZ W^T, A^T dZ) at the edges of their tiles, against fp64.

The graph has a self-loop per node and nothing else, so the GCN layer's aggregate is its input bit for bit
and the mean aggregator's is zero: what comes out of the layer calls is the product alone."""
import types

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (63, 17, 15), (64, 32, 16), (65, 33, 129), (130, 602, 41), (1000, 127, 130), (517, 66, 9),
          (4099, 128, 172), (40000, 100, 47), (70001, 128, 128)]
# one depth step, forward (d_in <= 32) or backward (d_out <= 32): weights that stay in LDS, a workgroup per row tile or a walk
SHAPES += [(130001, 16, 172), (30001, 9, 47), (50000, 32, 128), (129, 31, 33), (100001, 602, 9), (50001, 100, 16), (33000, 16, 16),
           (200000, 128, 32)]


def _loops(n):
    ptr, col = np.arange(n + 1, dtype=np.int32), np.arange(n, dtype=np.int32)
    none = np.zeros(0, np.int32)
    return types.SimpleNamespace(part_id=0, n_in=n, n_halo=0, nnz0=n, e_in=n, e_bd=0, row_ptr0=ptr, col0=col, t_in_ptr=ptr.copy(),
                                 t_in_col=col.copy(), halo_ptr=np.zeros(1, np.int32), halo_col=none, halo_gid=np.zeros(0, np.int64),
                                 deg_in=np.ones(n, np.int32), deg_halo=none)


@pytest.mark.parametrize("kind", [0, 1], ids=["gcn", "sage"])
@pytest.mark.parametrize("n,d_in,d_out", SHAPES, ids=[f"{a}x{b}x{c}" for a, b, c in SHAPES])
def test_products(n, d_in, d_out, kind):
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(n + 7 * d_in + 13 * d_out)
    f32 = lambda *s: torch.randn(*s, device=dev, generator=gen)  # noqa: E731
    i32 = lambda k: torch.zeros(k, dtype=torch.int32, device=dev)  # noqa: E731
    ctx = pkg.Context(_loops(n), [d_in, d_out], 0, device=dev, layer_kind=kind)
    kept, remap, n_kept, nnz = i32(1), i32(1), i32(1), i32(1)
    ctx.sample_boundary(1, 0, 0.5, kept, remap, n_kept)
    csr = i32(n + 1), i32(n), i32(n + 1), i32(n)    # must outlive the layer calls
    ctx.build_sampled_csr(remap, kept, n_kept, *csr, nnz)
    # a factor of 2^-20 .. 2^20 per element: no piece of a split value may get lost
    X = f32(n, d_in) * torch.exp2(torch.randint(-20, 21, (n, d_in), device=dev, generator=gen).float())
    W, dH = f32((1 + kind) * d_in, d_out), f32(n, d_out)
    A, H = torch.full((n, d_in), 7.0, device=dev), torch.full((n, d_out), 7.0, device=dev)
    dW, dX = torch.full_like(W, 7.0), torch.full_like(X, 7.0)
    ctx.gcn_layer_fwd(1, 0.5, X, None, W, A, H, False)
    ctx.gcn_layer_bwd(1, 0.5, dH, None, A, X, W, dW, dX, None)
    torch.cuda.synchronize()
    Ad = torch.zeros_like(X) if kind else X
    assert torch.equal(A, Ad)
    Z = torch.cat([Ad, X], 1).double() if kind else X.double()
    Wd = W.double()

    def check(name, got, a, b):
        ref, size = a @ b, a.abs() @ b.abs()
        over = (got.double() - ref).abs() / (4.0 * 2.0 ** -24 * (1 + a.shape[1] ** 0.5) * size + 1e-300)
        assert over.max() <= 1.0, f"{name}: {over.max().item():.3g} of the allowance"

    check("H W", H, Z, Wd)
    check("A^T dZ", dW, Z.t().contiguous(), dH.double())
    check("dZ W^T", dX, dH.double(), Wd[d_in * kind:].t().contiguous())
    ctx.close()


@pytest.mark.parametrize("kind", [0, 1], ids=["gcn", "sage"])
@pytest.mark.parametrize("n,d_in,d_out", [(512, 17, 33), (513, 33, 9), (1536, 66, 47), (1537, 66, 47), (400, 602, 256), (512, 300, 509)], ids=lambda v: str(v))
def test_products_of_few_rows(n, d_in, d_out, kind):
    """On either side of the lines up to which A^T dZ is a single launch: 512 rows, three times as many, 512 tiles."""
    test_products(n, d_in, d_out, kind)


@pytest.mark.parametrize("half_zero", [False, True], ids=["normal", "masked"])
@pytest.mark.parametrize("n,d_in,d_out", [(2000, 96, 128), (2000, 64, 512), (4000, 512, 512), (4099, 128, 172), (60000, 128, 128)],
                         ids=lambda v: str(v))
def test_backward_products_round_once_a_step(n, d_in, d_out, half_zero):
    """The error of dZ W^T and A^T dZ over the whole result, which the element-wise allowance above is too wide for.

    A 32-deep step is rounded once at its own size and once where it joins the running sum.  The rounding of a sum x to the
    nearest has a standard deviation of 0.42 * 2^-24 |x| on average, and the running sum of n steps of random terms has at
    step i the size sqrt(i / n) of the whole: 0.42 * 2^-24 sqrt(n / 2) for all n, and once more that of one step, 2^-24 at
    most.  Taken with a factor 1.7: 2^-24 (1 + 0.5 sqrt(n)).  A^T dZ is cut into splits of at most 1024 rows here."""
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(n + d_out)
    f32 = lambda *s: torch.randn(*s, device=dev, generator=gen)  # noqa: E731
    i32 = lambda k: torch.zeros(k, dtype=torch.int32, device=dev)  # noqa: E731
    ctx = pkg.Context(_loops(n), [d_in, d_out], 0, device=dev)
    kept, remap, n_kept, nnz = i32(1), i32(1), i32(1), i32(1)
    ctx.sample_boundary(1, 0, 0.5, kept, remap, n_kept)
    csr = i32(n + 1), i32(n), i32(n + 1), i32(n)
    ctx.build_sampled_csr(remap, kept, n_kept, *csr, nnz)
    A, W, dZ = f32(n, d_in), f32(d_in, d_out), f32(n, d_out)
    if half_zero:
        dZ *= f32(n, d_out) > 0
    dW, dX = torch.zeros_like(W), torch.zeros_like(A)
    ctx.gcn_layer_bwd(1, 0.5, dZ, None, A, None, W, dW, dX, None)
    torch.cuda.synchronize()
    for name, got, a, b, depth in (("dZ W^T", dX, dZ, W.t().contiguous(), d_out), ("A^T dZ", dW, A.t().contiguous(), dZ, min(n, 1024))):
        ref = a.double() @ b.double()
        err = ((got.double() - ref).norm() / ref.norm()).item()
        assert err <= 2.0 ** -24 * (1 + 0.5 * (depth / 32) ** 0.5), f"{name}: {err:.3g}"
    ctx.close()


def _layer(n, d_in, d_out, kind, part=None):
    import torch
    import paper_2203_10983_amd as pkg
    i32 = lambda k: torch.zeros(k, dtype=torch.int32, device="cuda:0")  # noqa: E731
    ctx = pkg.Context(part or _loops(n), [d_in, d_out], 0, device=torch.device("cuda:0"), layer_kind=kind)
    kept, remap, n_kept, nnz = i32(1), i32(1), i32(1), i32(1)
    ctx.sample_boundary(1, 0, 0.5, kept, remap, n_kept)
    csr = i32(n + 1), i32(n), i32(n + 1), i32(n)
    ctx.build_sampled_csr(remap, kept, n_kept, *csr, nnz)
    return ctx, (kept, remap, n_kept, nnz, csr)


# the split forward products of a last layer: one product of both halves (144, 160), two added (130, 301), odd depths, every
# number of column tiles from 1 to 8, few rows and many
@pytest.mark.parametrize("kind", [0, 1], ids=["gcn", "sage"])
@pytest.mark.parametrize("n,d_in,d_out", [(1, 129, 1), (9000, 66, 17), (200, 144, 33), (517, 301, 50), (1000, 131, 79), (2000, 160, 96), (3000, 602, 112),
                                          (4099, 512, 128), (20001, 65, 130), (40000, 256, 172), (30000, 128, 64)], ids=lambda v: str(v))
def test_forward_products_of_last_layers(n, d_in, d_out, kind):
    """Each element within the allowance, the whole as close as sums that round once a 32-deep step at the size of the running one
    (2^-24 (1 + 0.5 sqrt(steps)), derived in test_backward_products_round_once_a_step), and once more where two products are added;
    few rows give the bits that many give."""
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(n + d_out)
    f32 = lambda *s: torch.randn(*s, device="cuda:0", generator=gen)  # noqa: E731
    X, W = f32(n, d_in), f32((1 + kind) * d_in, d_out)
    got = {}
    for m in (n, (n + 2) // 3):
        ctx, keep = _layer(m, d_in, d_out, kind)
        A, H = torch.empty(m, d_in, device="cuda:0"), torch.full((m, d_out), 7.0, device="cuda:0")
        ctx.gcn_layer_fwd(1, 0.5, X[:m], None, W, A, H, False)
        R = torch.full_like(H, 7.0)
        ctx.gcn_layer_fwd(1, 0.5, X[:m], None, W, A, R, True)
        torch.cuda.synchronize()
        assert torch.equal(R, H.clamp(min=0))
        got[m] = H
        ctx.close()
    assert torch.equal(got[(n + 2) // 3], got[n][:(n + 2) // 3])
    Z, Wd = X.double(), W[kind * d_in:].double()
    ref, size = Z @ Wd, Z.abs() @ Wd.abs()
    assert ((got[n].double() - ref).abs() <= 4.0 * 2.0 ** -24 * (1 + d_in ** 0.5) * size).all()
    if n * d_out >= 1000:  # (a handful of elements has no typical error)
        err = ((got[n].double() - ref).norm() / ref.norm()).item()
        assert err <= 2.0 ** -24 * (1 + 0.5 * (((1 + kind) * d_in + 31) // 32) ** 0.5), err


@pytest.mark.parametrize("relu", [False, True], ids=["last", "relu"])
@pytest.mark.parametrize("kind", [0, 1], ids=["gcn", "sage"])
@pytest.mark.parametrize("d_in,d_out", [(144, 20), (130, 49), (301, 172)], ids=lambda v: str(v))
def test_infinities_and_nan_in_forward_products(d_in, d_out, kind, relu):
    """As test_infinities_and_nan_in_backward_products; max(NaN, 0) of a hidden unit is 0, as it is for the narrower layers."""
    import torch
    n = 300
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(d_in)
    f32 = lambda *s: torch.rand(*s, device="cuda:0", generator=gen) + 0.5  # noqa: E731  (one sign: no infinities cancel by chance)
    X, W = f32(n, d_in), f32((1 + kind) * d_in, d_out)
    inf, half, top = float("inf"), kind * d_in, 3.40e38  # top: rounds to an infinite bf16
    W[half + 7] *= 0.1
    X[5, 3], X[n - 1, d_in - 1], X[17, 0], X[33, 7], X[60, 1] = inf, -inf, float("nan"), top, top
    W[half + 1, 2], W[half + d_in - 1, 7] = inf, -inf
    X[40, 1] = 0.0                                       # 0 * inf
    ctx, keep = _layer(n, d_in, d_out, kind)
    A, H = torch.empty(n, d_in, device="cuda:0"), torch.full((n, d_out), 7.0, device="cuda:0")
    ctx.gcn_layer_fwd(1, 0.5, X, None, W, A, H, relu)
    torch.cuda.synchronize()
    Z = torch.cat([A, X], 1) if kind else X  # (the mean over no neighbours: zero, or NaN where zero times infinity is)
    ref = torch.stack([(row[:, None] * W.cpu()).double().sum(0) for row in Z.cpu()]).float()  # products that overflow do so in fp32
    if relu:
        ref = torch.where(ref.isnan(), 0.0, ref).clamp(min=0)
    got = H.cpu()
    assert torch.equal(got.isnan(), ref.isnan())
    assert torch.equal(got.isinf(), ref.isinf()) and torch.equal(got[got.isinf()], ref[ref.isinf()])
    ok = ref.isfinite()
    assert 0 < int(ok.sum()) < ok.numel() and torch.allclose(got[ok], ref[ok], rtol=1e-5, atol=0)
    ctx.close()


@pytest.mark.parametrize("x,w", [(1e-33, 1.0), (1e-36, 1.0), (1.0, 1e-36), (1e-38, 1e4), (1e-30, 1e-4)])
@pytest.mark.parametrize("kind", [0, 1], ids=["gcn", "sage"])
@pytest.mark.parametrize("d_in,d_out", [(144, 20), (130, 49), (301, 172)], ids=lambda v: str(v))
def test_forward_products_of_small_operands(d_in, d_out, kind, x, w):
    """Operands whose last bits lie below the range of bf16 give what sums in fp32 give: each element within a rounding of its terms'
    size at every step, and of the smallest number there is."""
    import torch
    n = 300
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(d_in)
    X, W = x * torch.randn(n, d_in, device="cuda:0", generator=gen), w * torch.randn((1 + kind) * d_in, d_out, device="cuda:0", generator=gen)
    X[7], W[:, 3] = 0.0, 0.0
    ctx, keep = _layer(n, d_in, d_out, kind)
    A, H = torch.empty(n, d_in, device="cuda:0"), torch.full((n, d_out), 7.0, device="cuda:0")
    ctx.gcn_layer_fwd(1, 0.5, X, None, W, A, H, False)
    torch.cuda.synchronize()
    Z = torch.cat([A, X], 1) if kind else A
    ref, size = Z.double() @ W.double(), Z.double().abs() @ W.double().abs()
    k = Z.shape[1]
    assert ((H.double() - ref).abs() <= 4.0 * (2.0 ** -24 * (1 + k ** 0.5) * size + 2.0 ** -149 * k)).all()
    assert bool((H[7] == 0).all()) and bool((H[:, 3] == 0).all()) and int((H != 0).sum()) == (n - 1) * (d_out - 1)
    ctx.close()


def test_infinities_in_a_product_before_the_aggregate():
    """A layer that multiplies first reads kept boundary rows by record, scaled on their way in, and pads its odd width."""
    import torch
    import paper_2203_10983_amd as pkg
    n, nb, d_in, d_out = 150000, 300, 160, 41
    P = _loops(n)
    P.n_halo = P.e_bd = nb  # boundary node u is a neighbour of node u
    P.nnz0 = n + nb
    P.row_ptr0 = (np.arange(n + 1) + np.minimum(np.arange(n + 1), nb)).astype(np.int32)
    P.col0 = np.concatenate([np.stack([np.arange(nb), n + np.arange(nb)], 1).ravel(), np.arange(nb, n)]).astype(np.int32)
    P.halo_ptr, P.halo_col = np.arange(nb + 1, dtype=np.int32), np.arange(nb, dtype=np.int32)
    P.halo_gid, P.deg_halo = n + np.arange(nb, dtype=np.int64), np.full(nb, 2, np.int32)
    P.deg_in = np.diff(P.row_ptr0).astype(np.int32)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(1)
    f32 = lambda *s: torch.rand(*s, device="cuda:0", generator=gen) + 0.5  # noqa: E731
    X, halo, W = f32(n, d_in), f32(nb, d_in), f32(d_in, d_out)
    inf, top = float("inf"), 3.40e38
    W[7] *= 0.1
    X[400, 3], X[n - 1, d_in - 1], X[70001, 5], X[501, 7] = inf, -inf, float("nan"), top
    halo[3, 4], halo[nb - 1, 0], halo[100, 159], halo[200, 7] = inf, float("nan"), -inf, top
    ctx = pkg.Context(P, [d_in, d_out], 0, device=torch.device("cuda:0"))
    assert ctx.layer_plan(1) == pkg.LAYER_UPDATE_FIRST
    dW, loss = torch.zeros_like(W), torch.zeros(1, device="cuda:0")
    ctx.train_step(1, 0, 1.0, X, [halo], torch.zeros(n, dtype=torch.int32, device="cuda:0"), [W], [dW], [None], loss, 0.0)
    torch.cuda.synchronize()
    got = ctx.ws_tensor(pkg.VIEW_H, 1, torch.float32).view(n, d_out).cpu().double()
    d = torch.from_numpy(P.deg_in).double()
    S = X.cpu().double() / d[:, None]
    S[:nb] += halo.cpu().double() / 2
    ref = S @ W.cpu().double()
    assert torch.equal(got.isfinite(), ref.isfinite()) and int((~ref.isfinite()).sum()) == 6 * d_out
    assert torch.equal(got.isnan(), ref.isnan()) and torch.equal(got[got.isinf()], ref[ref.isinf()])
    ok = ref.isfinite()
    assert torch.allclose(got[ok], ref[ok], rtol=1e-5, atol=0)
    ctx.close()


@pytest.mark.parametrize("kind", [0, 1], ids=["gcn", "sage"])
@pytest.mark.parametrize("n,d_in,d_out", [(70, 16, 16), (300, 50, 20), (300, 20, 52), (4000, 128, 130)], ids=lambda v: str(v))
def test_infinities_and_nan_in_backward_products(n, d_in, d_out, kind):
    """A result is infinite or NaN where the sum of the operands' products is, and nowhere else."""
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(n + d_out)
    f32 = lambda *s: torch.rand(*s, device=dev, generator=gen) + 0.5  # noqa: E731  (one sign: no infinities cancel by chance)
    i32 = lambda k: torch.zeros(k, dtype=torch.int32, device=dev)  # noqa: E731
    ctx = pkg.Context(_loops(n), [d_in, d_out], 0, device=dev, layer_kind=kind)
    kept, remap, n_kept, nnz = i32(1), i32(1), i32(1), i32(1)
    ctx.sample_boundary(1, 0, 0.5, kept, remap, n_kept)
    csr = i32(n + 1), i32(n), i32(n + 1), i32(n)
    ctx.build_sampled_csr(remap, kept, n_kept, *csr, nnz)
    A, H, W, dZ = f32(n, d_in), f32(n, d_in), f32((1 + kind) * d_in, d_out), f32(n, d_out)
    inf, top = float("inf"), 3.40e38                        # top: rounds to an infinite bf16
    dZ[5, 3], dZ[n - 1, d_out - 1], dZ[17, 0], dZ[33, 1] = inf, -inf, float("nan"), top
    A[9, 2], A[n - 2, d_in - 1], A[41, 1] = inf, -inf, top
    H[11, 3], H[n - 3, d_in - 2] = inf, top
    W[kind * d_in + 1, 2], W[kind * d_in + d_in - 1, 7] = inf, -inf
    A[50, 4], dZ[50, 4] = inf, 0.0                          # inf * 0
    dW, dX = torch.zeros_like(W), torch.zeros(n, d_in, device=dev)
    ctx.gcn_layer_bwd(1, 0.5, dZ, None, A, H, W, dW, dX, None)
    torch.cuda.synchronize()
    pairs = [("A^T dZ", dW, (torch.cat([A, H], 1) if kind else A).t(), dZ)]
    if kind == 0:  # the mean aggregator's dH_in gathers with a weight of zero, and zero times infinity is NaN
        pairs.append(("dZ W^T", dX, dZ, W.t()))
    for name, got, a, b in pairs:
        a, b, got = a.cpu(), b.cpu(), got.cpu()
        ref = torch.stack([(row[:, None] * b).double().sum(0) for row in a]).float()  # products that overflow do so in fp32
        assert torch.equal(got.isnan(), ref.isnan()), name
        assert torch.equal(got.isinf(), ref.isinf()) and torch.equal(got[got.isinf()], ref[ref.isinf()]), name
        ok = ref.isfinite()
        assert 0 < int(ok.sum()) and torch.allclose(got[ok], ref[ok], rtol=1e-5, atol=0), name
    ctx.close()


@pytest.mark.parametrize("kind,shared,d_out", [(0, "dH_out", 48), (0, "A_saved", 48), (0, "H_out", 48), (0, "A_saved", 20),
                                               (1, "dH_out", 48), (1, "A_saved", 48), (1, "H_in", 48), (1, "H_in", 20)])
def test_input_gradient_may_overwrite_what_it_came_from(kind, shared, d_out):
    """dH_in in the place of an operand of the same call (bns_gcn_layer_bwd) changes neither gradient."""
    import torch
    import paper_2203_10983_amd as pkg
    n, d_in, dev = 1000, 48, torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(n + d_out)
    f32 = lambda *s: torch.randn(*s, device=dev, generator=gen)  # noqa: E731
    i32 = lambda k: torch.zeros(k, dtype=torch.int32, device=dev)  # noqa: E731
    ctx = pkg.Context(_loops(n), [d_in, d_out], 0, device=dev, layer_kind=kind)
    kept, remap, n_kept, nnz = i32(1), i32(1), i32(1), i32(1)
    ctx.sample_boundary(1, 0, 0.5, kept, remap, n_kept)
    csr = i32(n + 1), i32(n), i32(n + 1), i32(n)
    ctx.build_sampled_csr(remap, kept, n_kept, *csr, nnz)
    W = f32((1 + kind) * d_in, d_out)
    ops = dict(dH_out=f32(n, d_out), H_out=f32(n, d_out) if shared == "H_out" else None, A_saved=f32(n, d_in), H_in=f32(n, d_in))

    def bwd(o, dX):
        dW = torch.zeros_like(W)
        ctx.gcn_layer_bwd(1, 0.5, o["dH_out"], o["H_out"], o["A_saved"], o["H_in"], W, dW, dX, None)
        torch.cuda.synchronize()
        return dW, dX

    dW, dX = bwd(ops, torch.zeros(n, d_in, device=dev))
    copies = {k: v if v is None else v.clone() for k, v in ops.items()}
    dW2, dX2 = bwd(copies, copies[shared])
    assert torch.equal(dX, dX2) and torch.equal(dW, dW2)
    ctx.close()


@pytest.mark.parametrize("kind", [0, 1], ids=["gcn", "sage"])
@pytest.mark.parametrize("d_in,d_out", [(64, 33), (64, 66), (36, 98), (64, 129), (16, 1), (130, 33), (144, 47), (144, 172), (301, 9)])
def test_dropout_of_few_rows_is_that_of_many(d_in, d_out, kind):
    """An element's draw depends on its row, column, layer and epoch alone, and its sum on nothing but its terms: the same
    rows give the same bits whatever tiles the number of rows leads to."""
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(d_in + 13 * d_out)
    X = torch.randn(70001, d_in, device=dev, generator=gen)
    W = torch.randn((1 + kind) * d_in, d_out, device=dev, generator=gen)
    i32 = lambda k: torch.zeros(k, dtype=torch.int32, device=dev)  # noqa: E731
    got = {}
    for n in (1, 500, 70001):
        for q in (0.0, 0.5):
            ctx = pkg.Context(_loops(n), [d_in, d_out], 0, device=dev, layer_kind=kind)
            ctx.set_dropout(q)
            kept, remap, n_kept, nnz = i32(1), i32(1), i32(1), i32(1)
            ctx.sample_boundary(1, 3, 0.5, kept, remap, n_kept)
            csr = i32(n + 1), i32(n), i32(n + 1), i32(n)
            ctx.build_sampled_csr(remap, kept, n_kept, *csr, nnz)
            H = torch.full((n, d_out), 7.0, device=dev)
            ctx.gcn_layer_fwd(1, 0.5, X[:n], None, W, torch.empty(n, d_in, device=dev), H, True)
            torch.cuda.synchronize()
            got[n, q] = H
            ctx.close()
    for q in (0.0, 0.5):
        assert torch.equal(got[1, q], got[70001, q][:1]) and torch.equal(got[500, q], got[70001, q][:500])
    dropped = got[70001, 0.5] == 0
    assert torch.equal(got[70001, 0.5], torch.where(dropped, 0.0, 2.0 * got[70001, 0.0]))
    on = got[70001, 0.0] > 0
    k, m = int((on & dropped).sum()), int(on.sum())
    assert abs(k - m / 2) <= 5 * (m / 4) ** 0.5


@pytest.mark.parametrize("n,d_in,d_out", [(17000, 300, 130), (17409, 602, 130), (40000, 130, 130), (20011, 602, 130), (30011, 66, 290)], ids=lambda v: str(v))
def test_forward_products_however_their_columns_are_dealt(n, d_in, d_out):
    """A hidden layer's product, whose columns go to workgroups by how many tiles the fullest compute unit gets: each element within
    the allowance, and the bits of the same rows in a product that deals them otherwise."""
    import torch
    import paper_2203_10983_amd as pkg
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(n)
    f32 = lambda *s: torch.randn(*s, device="cuda:0", generator=gen)  # noqa: E731
    i32 = lambda k: torch.zeros(k, dtype=torch.int32, device="cuda:0")  # noqa: E731
    X, W = f32(n, d_in), f32(d_in, d_out)
    got = []
    for m in (n, 9100):
        ctx = pkg.Context(_loops(m), [d_in, d_out, 8], 0, device=torch.device("cuda:0"))
        kept, remap, n_kept, nnz = i32(1), i32(1), i32(1), i32(1)
        ctx.sample_boundary(1, 0, 0.5, kept, remap, n_kept)
        csr = i32(m + 1), i32(m), i32(m + 1), i32(m)
        ctx.build_sampled_csr(remap, kept, n_kept, *csr, nnz)
        A, H = torch.empty(m, d_in, device="cuda:0"), torch.full((m + 1, d_out), 7.0, device="cuda:0")
        ctx.gcn_layer_fwd(1, 0.5, X[:m], None, W, A, H[:m], True)
        torch.cuda.synchronize()
        assert bool((H[m] == 7.0).all())
        got.append(H[:m])
        ctx.close()
    assert torch.equal(got[1], got[0][:9100])
    ref, size = (X.double() @ W.double()).clamp(min=0), X.double().abs() @ W.double().abs()
    assert ((got[0].double() - ref).abs() <= 4.0 * 2.0 ** -24 * (1 + d_in ** 0.5) * size).all()
