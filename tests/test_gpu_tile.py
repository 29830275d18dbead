"""Layers of small partitions, aggregate and product in one launch, against the two launches that run while their phases are
timed.  Forward, and backward where the output is the narrower side, the same sums in the same order, so the same bits; else the
transposed aggregate has changed places with the product, and both results lie within a few roundings (2^-24) of the exact one.
Random graphs with hubs of up to eight segments of 256 entries; on either side of each limit, and which form runs is
counted in launches.  And the subgraph of
such a step, whose launch the stand-alone calls do not take, at that launch's limits."""
import ctypes as C
import types

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TIMED = (1 << 3) | (1 << 4) | (1 << 5) | (1 << 7) | (1 << 8)  # aggregate, update, loss, and the backward passes of the first two


def _partition(n, deg, hub, n_halo, rng, lists=4):
    """n rows of about deg entries, row n // 2 with hub; symmetric inner part with self-loops, boundary nodes next to 1 to `lists` rows."""
    pairs = {(v, v) for v in range(n)}
    for _ in range(int(n * deg / 2)):
        a, b = (int(x) for x in rng.integers(0, n, 2))
        pairs |= {(a, b), (b, a)}
    for b in rng.choice(n, size=min(n, hub), replace=False):
        pairs |= {(n // 2, int(b)), (int(b), n // 2)}
    inner = np.array(sorted(pairs), dtype=np.int64)
    halo = np.array(sorted({(b, int(v)) for b in range(n_halo) for v in rng.integers(0, n, 1 + b % lists)}), dtype=np.int64).reshape(-1, 2)
    both = np.concatenate([inner, np.stack([halo[:, 1], n + halo[:, 0]], 1)])
    both = both[np.lexsort((both[:, 1], both[:, 0]))]
    ptr = lambda of, m: np.concatenate([[0], np.cumsum(np.bincount(of, minlength=m))])  # noqa: E731
    i32 = lambda x: np.ascontiguousarray(x, dtype=np.int32)  # noqa: E731
    return types.SimpleNamespace(
        part_id=0, n_in=n, n_halo=n_halo, nnz0=len(both), e_in=len(inner), e_bd=len(halo), row_ptr0=i32(ptr(both[:, 0], n)), col0=i32(both[:, 1]),
        t_in_ptr=i32(ptr(inner[:, 0], n)), t_in_col=i32(inner[:, 1]), halo_ptr=i32(ptr(halo[:, 0], n_halo)), halo_col=i32(halo[:, 1]),
        halo_gid=np.arange(n, n + n_halo, dtype=np.int64), deg_in=i32(np.bincount(both[:, 0], minlength=n)),
        deg_halo=i32(np.bincount(halo[:, 0], minlength=n_halo) + 1))


def _launches(call):
    """Kernels that a call puts on its stream: it is recorded, counted and not run."""
    import torch
    import paper_2203_10983_amd as pkg
    hip, graph, nodes = pkg.load_library(), C.c_void_p(), C.c_size_t()
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream()):
        stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
        assert hip.hipStreamBeginCapture(stream, 1) == 0
        try:
            call()
        finally:
            assert hip.hipStreamEndCapture(stream, C.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, C.byref(nodes)) == 0 and hip.hipGraphDestroy(graph) == 0
    return nodes.value


def _one_launch_layers(ctx, P, dims, layer_kind, cached_X):
    """Per layer call: does it run as one launch, forward (beside the records of the kept rows) and backward (beside what a call
    without an input gradient launches)?  By the rules that a step goes by."""
    import torch
    i32 = lambda k: torch.zeros(k, dtype=torch.int32, device="cuda:0")  # noqa: E731
    f32 = lambda *k: torch.zeros(*k, device="cuda:0")  # noqa: E731
    n, nb = P.n_in, P.n_halo
    kept, remap, n_kept = i32(nb), i32(nb), i32(1)
    csr = i32(n + 1), i32(P.nnz0), i32(n + nb + 1), i32(P.nnz0), i32(1)
    ctx.sample_boundary(3, 0, 0.5, kept, remap, n_kept)
    ctx.build_sampled_csr(remap, kept, n_kept, *csr)
    fwd, bwd = [], []
    for l, (a, b) in enumerate(zip(dims, dims[1:]), 1):
        H_in, Hu, W, dW = cached_X if l == 1 and cached_X is not None else f32(n, a), f32(nb, a), f32((1 + layer_kind) * a, b), f32((1 + layer_kind) * a, b)
        A, H, G, dH, dhalo = f32(n, a), f32(n, b), f32(n, b), f32(n, a), f32(nb, a)
        fwd.append(_launches(lambda: ctx.gcn_layer_fwd(l, 0.5, H_in, Hu, W, A, H, False)) == 2)
        with_dH = _launches(lambda: ctx.gcn_layer_bwd(l, 0.5, G, H, A, H_in, W, dW, dH, dhalo))
        bwd.append(with_dH - _launches(lambda: ctx.gcn_layer_bwd(l, 0.5, G, H, A, H_in, W, dW, None, None)) == 1)
    return "".join("21"[x] for x in fwd), "".join("21"[x] for x in bwd[1:])


# segments: of the longest row, forward and transposed.  fwd, bwd (from layer 2 on): launches of aggregate and product, in one (1) or
# each in its own (2 or more).
@pytest.mark.parametrize("n,deg,hub,dims,layer_kind,drop,cached,segments,fwd,bwd", [
    (1, 0, 0, (12, 16, 1), 0, 0.0, False, (1, 1), "11", "2"), (7, 2, 0, (64, 16, 8), 0, 0.0, False, (1, 1), "11", "1"),
    (17, 3, 0, (16, 129, 12, 2), 1, 0.3, False, (1, 1), "121", "22"), (500, 5, 0, (64, 172, 8), 0, 0.5, True, (1, 1), "12", "2"),
    (600, 8, 560, (128, 128, 47), 0, 0.0, False, (3, 3), "11", "1"), (2100, 4, 2000, (100, 128, 17), 1, 0.0, True, (8, 8), "11", "2"),
    (2100, 4, 2048, (100, 128, 17), 1, 0.0, True, (9, 8), "22", "2"), (3584, 20, 300, (32, 256, 16), 1, 0.3, False, (2, 2), "12", "2"),
    (3585, 20, 300, (32, 36, 16), 1, 0.0, False, (2, 2), "22", "2"), (3585, 20, 0, (60, 33, 9), 0, 0.0, False, (1, 1), "12", "2"),
    (8192, 3, 0, (36, 128, 20, 5), 1, 0.0, False, (1, 1), "111", "22"), (8193, 3, 0, (36, 128, 5), 0, 0.0, False, (1, 1), "22", "2"),
    (1, 0, 0, (8, 8, 8), 0, 0.0, False, (1, 1), "22", "1"), (9, 2, 0, (5, 33, 12), 0, 0.0, False, (1, 1), "22", "1"),
    (700, 12, 600, (16, 100, 100, 47), 1, 0.3, False, (3, 3), "111", "11"), (700, 12, 600, (64, 128, 36, 12), 0, 0.3, False, (3, 3), "111", "11"),
    (900, 4, 800, (64, 64, 36), 0, 0.0, True, (4, 4), "11", "2"), (2457, 4, 0, (12, 128, 128, 128), 1, 0.0, False, (1, 1), "111", "11"),
    (2458, 4, 0, (12, 128, 128, 128), 1, 0.0, False, (1, 1), "111", "22"), (2600, 4, 0, (12, 128, 128, 128), 1, 0.0, False, (1, 1), "111", "22")])
def test_one_launch_equals_two(n, deg, hub, dims, layer_kind, drop, cached, segments, fwd, bwd):
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(n)
    n_halo, L = n // 2 + 1, len(dims) - 1
    P = _partition(n, deg, hub, n_halo, np.random.default_rng(n))
    assert segments == tuple(-(-int(np.diff(ptr).max()) // 256) for ptr in (P.row_ptr0, P.t_in_ptr))
    r = lambda *s: torch.randn(*s, device=dev, generator=gen)  # noqa: E731
    X, halo = r(n, dims[0]), [r(n_halo, d) for d in dims[:-1]]
    W = [r((1 + layer_kind) * a, b) / a ** 0.5 for a, b in zip(dims, dims[1:])]
    labels = torch.randint(-1, dims[-1], (n,), device=dev, generator=gen, dtype=torch.int32)  # -1: outside the training set
    out, losses = [], []
    for mask in (TIMED, 0):
        ctx = pkg.Context(P, list(dims), 0, layer_kind=layer_kind, device=dev)
        ctx.set_dropout(drop)
        if cached:
            ctx.cache_input_aggregate(X)
        if mask:
            ctx.profile_enable(mask, 512)
        dW, loss = [torch.zeros_like(w) for w in W], torch.zeros(1, device=dev)
        dhalo = [None] + [torch.zeros(n_halo, d, device=dev) for d in dims[1:-1]]
        for epoch in range(2):
            ctx.train_step(3, epoch, 0.5, X, halo, labels, W, dW, dhalo, loss, 0.0)
        torch.cuda.synchronize()
        if mask:
            assert ctx.profile_read()["gemm_fwd"][1] >= 2 * L  # two launches
        else:
            assert _one_launch_layers(ctx, P, dims, layer_kind, X if cached else None) == (fwd, bwd)
            # (a step on arrays of the workspace again, as the views below are)
            ctx.train_step(3, 1, 0.5, X, halo, labels, W, dW, dhalo, loss, 0.0)
            torch.cuda.synchronize()
        A = [ctx.ws_tensor(pkg.VIEW_A, l, torch.float32).clone() for l in range(1, L + 1)] + [ctx.ws_tensor(pkg.VIEW_DZ, L, torch.float32).clone()]
        losses.append(loss.double())
        dZ = [ctx.ws_tensor(pkg.VIEW_DZ, l, torch.float32).clone() for l in range(1, L)]
        out.append((A + [ctx.ws_tensor(pkg.VIEW_H, l, torch.float32).clone() for l in range(1, L + 1)], dZ + dhalo[1:]))
        ctx.close()
    for two, one in zip(out[0][0], out[1][0]):
        assert torch.isfinite(two).all() and torch.equal(two, one)
    # positive terms, added in other orders: per node, wavefront, workgroup, then all
    assert (losses[0] - losses[1]).abs() <= 24 * 2.0 ** -24 * losses[0]
    narrowing = layer_kind == 0 and all(b < a for a, b in zip(dims[1:], dims[2:]))
    for two, one in zip(out[0][1], out[1][1]):
        if narrowing:
            assert torch.equal(two, one)
        else:  # six roundings of the split product and two of the aggregate's on either side, through up to two layers
            assert (two.double() - one.double()).norm() <= 32 * 2.0 ** -24 * two.double().norm()


def test_in_place_layer_keeps_two_launches():
    """H_out on top of H_in: every row is gathered before one is overwritten."""
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    n, d = 700, 64
    P = _partition(n, 6, 0, 50, np.random.default_rng(5))
    ctx = pkg.Context(P, [d, d], 0, device=dev)
    i32 = lambda k: torch.zeros(k, dtype=torch.int32, device=dev)  # noqa: E731
    kept, remap, n_kept, nnz = i32(50), i32(50), i32(1), i32(1)
    ctx.sample_boundary(1, 0, 0.5, kept, remap, n_kept)
    csr = i32(n + 1), i32(P.nnz0), i32(n + 51), i32(P.nnz0)
    ctx.build_sampled_csr(remap, kept, n_kept, *csr, nnz)
    X, Xb, W = (torch.randn(k, d, device=dev) for k in (n, 50, d))
    A, H = torch.zeros(n, d, device=dev), torch.zeros(n, d, device=dev)
    ctx.gcn_layer_fwd(1, 0.5, X, Xb, W, A, H, True)
    ctx.gcn_layer_fwd(1, 0.5, X, Xb, W, A, X, True)
    assert torch.equal(X, H)
    ctx.close()


def test_backward_with_infinite_gradients():
    """Products that are not finite are formed again as plain sums, in one launch as in two."""
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    n, d_in, d_out, nb = 300, 64, 16, 40
    P = _partition(n, 6, 0, nb, np.random.default_rng(6))
    i32 = lambda k: torch.zeros(k, dtype=torch.int32, device=dev)  # noqa: E731
    gen = torch.Generator(device=dev)
    gen.manual_seed(6)
    dZ, A, X, W = (torch.randn(*s, device=dev, generator=gen) for s in ((n, d_out), (n, d_in), (n, d_in), (d_in, d_out)))
    dZ[3, 2], dZ[7, 5], dZ[11, 0] = float("inf"), float("-inf"), float("nan")
    out = []
    for mask in (TIMED, 0):
        ctx = pkg.Context(P, [d_in, d_in, d_out], 0, device=dev)
        ctx.profile_enable(mask, 16)
        kept, remap, n_kept, nnz = i32(nb), i32(nb), i32(1), i32(1)
        ctx.sample_boundary(1, 0, 0.5, kept, remap, n_kept)
        csr = i32(n + 1), i32(P.nnz0), i32(n + nb + 1), i32(P.nnz0)
        ctx.build_sampled_csr(remap, kept, n_kept, *csr, nnz)
        dH, dhalo, dW = torch.zeros(n, d_in, device=dev), torch.zeros(nb, d_in, device=dev), torch.zeros_like(W)
        ctx.gcn_layer_bwd(2, 0.5, dZ, None, A, X, W, dW, dH, dhalo)
        out.append((dH, dhalo))
        torch.cuda.synchronize()
        ctx.close()
    for two, one in zip(*out):
        torch.testing.assert_close(one, two, rtol=0, atol=0, equal_nan=True)
    assert torch.isinf(out[1][0]).any() and torch.isnan(out[1][0]).any() and torch.isfinite(out[1][0]).any()


@pytest.mark.parametrize("n,deg,n_halo,lists,p,one", [(3, 1, 1, 1, 1.0, True), (1023, 4, 1025, 2, 0.5, True), (300, 3, 8192, 1, 0.0, True),
                                                      (300, 3, 8193, 1, 0.0, False), (900, 3, 2900, 4, 1.0, True), (900, 3, 3400, 4, 0.1, False),
                                                      (2000, 3, 2850, 1, 1.0, True), (2000, 3, 2870, 1, 1.0, False),
                                                      (1150, 40, 100, 3, 1.0, True), (1158, 40, 100, 3, 1.0, False)])
def test_subgraph_of_a_step_at_the_limits(n, deg, n_halo, lists, p, one):
    """Sampling and subgraph of a step in one launch or three, on either side of each limit, as its launches and its timers say; the same arrays."""
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    P = _partition(n, deg, 0, n_halo, np.random.default_rng(n_halo), lists)
    assert one == (max(n_halo, P.e_bd) <= 8192 and P.e_in + 3 * n + n_halo + 12 * np.ceil(p * n_halo) <= 51200)
    launches = []
    for Q in (P, _partition(n, deg, 0, 8193, np.random.default_rng(n_halo), 1)):  # (too many boundary nodes for one launch)
        f32 = lambda *s: torch.zeros(*s, device=dev)  # noqa: E731
        args = (p, f32(n, 8), [f32(Q.n_halo, 8)], torch.zeros(n, dtype=torch.int32, device=dev), [f32(8, 8)], [f32(8, 8)], [None], f32(1), 0.0)
        ctx = pkg.Context(Q, [8, 8], 0, device=dev)
        launches.append(_launches(lambda: ctx.train_step(11, 2, *args)))
        ctx.close()
    assert n == 3 or launches[0] == launches[1] - (2 if one else 0)  # (8193 boundary nodes make long rows of three)
    ctx = pkg.Context(P, [8, 8], 0, device=dev)
    i32 = lambda k: torch.zeros(k, dtype=torch.int32, device=dev)  # noqa: E731
    f32 = lambda *s: torch.zeros(*s, device=dev)  # noqa: E731
    ctx.profile_enable(3, 16)
    W = [torch.randn(8, 8, device=dev)]
    ctx.train_step(11, 2, p, f32(n, 8), [f32(n_halo, 8)], i32(n), W, [f32(8, 8)], [None], f32(1), 0.0)
    torch.cuda.synchronize()
    assert (ctx.profile_read()["build"][1] == 0) == one
    view = lambda w: ctx.ws_tensor(w, 0, torch.int32).clone()  # noqa: E731
    got = [view(v) for v in (pkg.VIEW_KEPT_IDS, pkg.VIEW_REMAP, pkg.VIEW_ROW_PTR, pkg.VIEW_COL_IDX, pkg.VIEW_T_ROW_PTR, pkg.VIEW_T_COL_IDX)]
    counts = int(view(pkg.VIEW_N_KEPT)[0]), int(view(pkg.VIEW_NNZ)[0])
    kept, remap, n_kept, nnz = i32(n_halo), i32(n_halo), i32(1), i32(1)
    ctx.sample_boundary(11, 2, p, kept, remap, n_kept)
    csr = i32(n + 1), i32(P.nnz0), i32(n + n_halo + 1), i32(P.nnz0)
    ctx.build_sampled_csr(remap, kept, n_kept, *csr, nnz)
    K, m = int(n_kept), int(nnz)
    assert counts == (K, m)
    for a, b, k in zip(got, (kept, remap) + csr, (K, n_halo, n + 1, m, n + K + 1, m)):
        assert torch.equal(a[:k], b[:k])
    ctx.close()


@pytest.mark.parametrize("n", [500, 5003])
@pytest.mark.parametrize("d_in,d_out", [(130, 66), (100, 47), (64, 64), (20, 17), (9, 3)])
def test_backward_masks_and_pads_in_one_pass(n, d_in, d_out):
    """A layer's gradient masked by the call equals the same gradient masked before it: dense and, where it is gathered in padded rows, there."""
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    nb = 60
    P = _partition(n, 4, 0, nb, np.random.default_rng(n))
    i32 = lambda k: torch.zeros(k, dtype=torch.int32, device=dev)  # noqa: E731
    gen = torch.Generator(device=dev)
    gen.manual_seed(d_in)
    G, H, A, W = (torch.randn(*s, device=dev, generator=gen) for s in ((n, d_out), (n, d_out), (n, d_in), (d_in, d_out)))
    H.clamp_(min=0)
    out = []
    for dZ, mask in ((G, H), (torch.where(H > 0, G, torch.zeros_like(G)), None)):
        ctx = pkg.Context(P, [d_in, d_in, d_out], 0, device=dev)
        kept, remap, n_kept, nnz = i32(nb), i32(nb), i32(1), i32(1)
        ctx.sample_boundary(1, 0, 0.5, kept, remap, n_kept)
        csr = i32(n + 1), i32(P.nnz0), i32(n + nb + 1), i32(P.nnz0)
        ctx.build_sampled_csr(remap, kept, n_kept, *csr, nnz)
        dH, dhalo, dW = torch.zeros(n, d_in, device=dev), torch.zeros(nb, d_in, device=dev), torch.zeros_like(W)
        ctx.gcn_layer_bwd(2, 0.5, dZ, mask, A, A, W, dW, dH, dhalo)
        out.append((dH, dhalo, dW))
        torch.cuda.synchronize()
        ctx.close()
    for a, b in zip(*out):
        assert torch.equal(a, b) and a.abs().sum() > 0
