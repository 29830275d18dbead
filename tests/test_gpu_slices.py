"""Aggregates whose XCDs take the feature slices in turn, with the kept boundary rows dealt among the inner ones (one, two or
four to a wavefront, or none kept at all), against fp64.

Cliques with self-loops, large and many enough for the launch to take turns (1 250 000 entries), each boundary node next to a
few inner ones; degrees count the entries, so that the inner part of A H0 is a clique sum."""
import types

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _partition(cliques, size, n_halo, rng):
    n = cliques * size
    first = np.repeat(np.arange(cliques) * size, size)
    lists = [np.sort(rng.choice(n, size=1 + b % 5, replace=False)) for b in range(n_halo)]  # inner neighbours per boundary node
    halo_ptr = np.concatenate([[0], np.cumsum([len(x) for x in lists])])
    halo_col = np.concatenate(lists)
    row, col = np.repeat(np.arange(n), size), (first[:, None] + np.arange(size)).reshape(-1)
    row = np.concatenate([row, halo_col])
    col = np.concatenate([col, n + np.repeat(np.arange(n_halo), np.diff(halo_ptr))])
    order = np.lexsort((col, row))
    ptr = np.concatenate([[0], np.cumsum(np.bincount(row, minlength=n))])
    i32 = lambda x: np.ascontiguousarray(x, dtype=np.int32)  # noqa: E731
    return types.SimpleNamespace(
        part_id=0, n_in=n, n_halo=n_halo, nnz0=len(col), e_in=n * size, e_bd=len(halo_col), row_ptr0=i32(ptr), col0=i32(col[order]),
        t_in_ptr=i32(np.arange(n + 1) * size), t_in_col=i32((first[:, None] + np.arange(size)).reshape(-1)), halo_ptr=i32(halo_ptr),
        halo_col=i32(halo_col), halo_gid=np.arange(n, n + n_halo, dtype=np.int64), deg_in=i32(np.diff(ptr)), deg_halo=i32(np.diff(halo_ptr) + 1))


@pytest.mark.parametrize("cliques,size,d,n_halo,p", [(20, 257, 256, 1, 1.0), (20, 257, 512, 3001, 0.5), (79, 128, 128, 5000, 0.3),
                                                     (79, 128, 200, 700, 1.0), (5, 515, 256, 16000, 1.0), (79, 128, 128, 300, 0.0), (6300, 16, 128, 20000, 0.5),
                                                     # widths that are no multiple of 4, dealt (16384 wavefronts, 13 entries a row): in slices and whole
                                                     (20, 257, 130, 3001, 0.3), (20, 257, 258, 1, 1.0), (20, 257, 602, 3001, 0.5), (600, 48, 47, 5000, 0.5),
                                                     # 32 floats and less: dealt beside fewer short rows than segments, not beside more
                                                     (600, 48, 32, 5000, 0.5), (600, 48, 30, 5000, 0.5), (600, 48, 32, 40000, 1.0),
                                                     # no kept row; two and four rows to a wavefront
                                                     (79, 128, 263, 300, 0.0), (6300, 16, 66, 20000, 0.5), (20, 257, 602, 24000, 1.0), (20, 257, 511, 24000, 1.0)])
def test_aggregate_in_turns(cliques, size, d, n_halo, p):
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(d + n_halo)
    P = _partition(cliques, size, n_halo, np.random.default_rng(size))
    assert P.e_in >= 1250000
    n = P.n_in
    i32 = lambda k: torch.zeros(k, dtype=torch.int32, device=dev)  # noqa: E731
    ctx = pkg.Context(P, [d, d], 0, device=dev)
    kept, remap, n_kept, nnz = i32(n_halo), i32(n_halo), i32(1), i32(1)
    ctx.sample_boundary(1, 0, p, kept, remap, n_kept)
    csr = i32(n + 1), i32(P.nnz0), i32(n + n_halo + 1), i32(P.nnz0)  # must outlive the layer calls
    ctx.build_sampled_csr(remap, kept, n_kept, *csr, nnz)
    X, Xb, dH = (torch.randn(k, d, device=dev, generator=gen) for k in (n, n_halo, n))
    A, H, dX = (torch.full((n, d), 7.0, device=dev) for _ in range(3))
    dW, dhalo = torch.zeros(d, d, device=dev), torch.full((n_halo, d), 7.0, device=dev)
    ctx.gcn_layer_fwd(1, p, X, Xb, torch.eye(d, device=dev), A, H, False)
    ctx.gcn_layer_bwd(1, p, dH, None, A, X, torch.eye(d, device=dev), dW, dX, dhalo)
    torch.cuda.synchronize()
    K = int(n_kept)
    kept = kept[:K].long()
    s_in = torch.from_numpy(P.deg_in).to(dev).double().rsqrt()[:, None]
    s_bd = torch.from_numpy(P.deg_halo).to(dev).double().rsqrt()[:, None] / max(p, 1e-3)
    clique = torch.arange(n, device=dev) // size

    def inner(x):
        return torch.zeros(cliques, d, device=dev, dtype=torch.float64).index_add_(0, clique, x)[clique]

    node = torch.repeat_interleave(torch.arange(n_halo, device=dev), torch.from_numpy(np.diff(P.halo_ptr)).to(dev))
    of = torch.from_numpy(P.halo_col).long().to(dev)
    is_kept = (remap >= 0)[node]
    node, of = node[is_kept], of[is_kept]
    ref_A = s_in * inner(s_in * X).index_add_(0, of, (s_bd * Xb)[node])
    ref_dhalo = torch.zeros(n_halo, d, device=dev, dtype=torch.float64).index_add_(0, node, (s_in * dH)[of]) * s_bd
    # sums of up to 600 terms of size 1 with weights of about 1 / 300: a rounding is 2^-24 of a running sum below 1
    tol = dict(rtol=1e-5, atol=1e-5)
    torch.testing.assert_close(A.double(), ref_A, **tol)
    torch.testing.assert_close(dX.double(), s_in * inner(s_in * dH), **tol)
    torch.testing.assert_close(dhalo[:K].double(), ref_dhalo[kept], **tol)
    assert bool((dhalo[K:] == 7.0).all())
    ctx.close()


@pytest.mark.parametrize("d", [2, 3, 5, 6, 7, 18, 33, 65, 66, 129, 130, 258, 263, 510, 602, 770, 1022])
@pytest.mark.parametrize("cliques,size,n_halo", [(40, 23, 90), (2, 300, 70), (1, 2305, 50), (4, 512, 90)])
def test_rows_of_any_width(d, cliques, size, n_halo):
    """Widths that are no multiple of four: the last four columns of a row overlap those before them.  Rows of one segment, of
    two (a workgroup each) and of ten (partial sums), and 4096 segments, which are taken by column; nothing is written past the last row."""
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(d)
    P = _partition(cliques, size, n_halo, np.random.default_rng(size))
    n, e = P.n_in, d
    i32 = lambda k: torch.zeros(k, dtype=torch.int32, device=dev)  # noqa: E731
    ctx = pkg.Context(P, [d, e], 1, device=dev)
    kept, remap, n_kept, nnz = i32(n_halo), i32(n_halo), i32(1), i32(1)
    ctx.sample_boundary(1, 0, 1.0, kept, remap, n_kept)
    csr = i32(n + 1), i32(P.nnz0), i32(n + n_halo + 1), i32(P.nnz0)  # must outlive the layer calls
    ctx.build_sampled_csr(remap, kept, n_kept, *csr, nnz)
    X, Xb, W, dH = (torch.randn(*k, device=dev, generator=gen) for k in ((n, d), (n_halo, d), (d, e), (n, e)))
    W /= d ** 0.5
    A, dX, dhalo = (torch.full((k + 1, d), 7.0, device=dev) for k in (n, n, n_halo))  # one row more than there is
    H, dW = torch.zeros(n, e, device=dev), torch.zeros(d, e, device=dev)
    ctx.gcn_layer_fwd(1, 1.0, X, Xb, W, A[:n], H, False)
    ctx.gcn_layer_bwd(1, 1.0, dH, None, A[:n], X, W, dW, dX[:n], dhalo[:n_halo])
    torch.cuda.synchronize()
    s_in, s_bd = (torch.from_numpy(x).to(dev).double().rsqrt()[:, None] for x in (P.deg_in, P.deg_halo))
    clique = torch.arange(n, device=dev) // size

    def inner(x):
        return torch.zeros(cliques, x.shape[1], device=dev, dtype=torch.float64).index_add_(0, clique, x)[clique]

    node = torch.repeat_interleave(torch.arange(n_halo, device=dev), torch.from_numpy(np.diff(P.halo_ptr)).to(dev))
    of = torch.from_numpy(P.halo_col).long().to(dev)
    G = dH.double() @ W.double().T
    ref_A = s_in * inner(s_in * X).index_add_(0, of, (s_bd * Xb)[node])
    ref_dhalo = torch.zeros(n_halo, d, device=dev, dtype=torch.float64).index_add_(0, node, (s_in * G)[of]) * s_bd
    # a sum of k terms in chains of at most 256 per partial sum; elements of G are sums of d products, together of size 1
    for x, ref in ((A, ref_A), (dX, s_in * inner(s_in * G)), (dhalo, ref_dhalo)):
        torch.testing.assert_close(x[:-1].double(), ref, rtol=1e-5, atol=3e-5)
        assert bool((x[-1] == 7.0).all())
    ctx.close()


@pytest.mark.parametrize("d,e,p", [(12, 12, 1.0), (33, 33, 0.97), (64, 47, 0.97), (64, 64, 1.0), (66, 66, 1.0), (128, 128, 0.97), (130, 130, 1.0), (200, 256, 1.0), (256, 256, 0.97),
                                   (512, 512, 1.0)])
def test_many_short_rows(d, e, p):
    """Kept boundary rows that a wavefront takes eight at a time: rows of one to three entries, groups of more than
    64 entries, a last group that is not whole."""
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(d)
    n, nb = 3000, 70003
    rng = np.random.default_rng(d)
    count = 1 + np.arange(nb) % 3
    count[3::500] = 80
    node = np.repeat(np.arange(nb), count)
    k = np.arange(len(node)) - np.repeat(np.cumsum(count) - count, count)
    of = (rng.integers(0, n, nb)[node] + 31 * k) % n
    by_node = np.lexsort((of, node))
    node, of = node[by_node], of[by_node]
    row, col = np.concatenate([np.arange(n), of]), np.concatenate([np.arange(n), n + node])
    order = np.lexsort((col, row))
    ptr = lambda x, m: np.concatenate([[0], np.cumsum(np.bincount(x, minlength=m))])  # noqa: E731
    i32 = lambda x: np.ascontiguousarray(x, dtype=np.int32)  # noqa: E731
    P = types.SimpleNamespace(
        part_id=0, n_in=n, n_halo=nb, nnz0=len(col), e_in=n, e_bd=len(node), row_ptr0=i32(ptr(row, n)), col0=i32(col[order]), t_in_ptr=i32(np.arange(n + 1)),
        t_in_col=i32(np.arange(n)), halo_ptr=i32(ptr(node, nb)), halo_col=i32(of), halo_gid=np.arange(n, n + nb, dtype=np.int64),
        deg_in=i32(np.bincount(row, minlength=n)), deg_halo=i32(count + 1))
    z32 = lambda m: torch.zeros(m, dtype=torch.int32, device=dev)  # noqa: E731
    ctx = pkg.Context(P, [d, e], 1, device=dev)
    kept, remap, n_kept, nnz = z32(nb), z32(nb), z32(1), z32(1)
    ctx.sample_boundary(1, 0, p, kept, remap, n_kept)
    csr = z32(n + 1), z32(P.nnz0), z32(n + nb + 1), z32(P.nnz0)  # must outlive the layer calls
    ctx.build_sampled_csr(remap, kept, n_kept, *csr, nnz)
    X, Xb, W, dZ = (torch.randn(*s, device=dev, generator=gen) for s in ((n, d), (nb, d), (d, e), (n, e)))
    W /= d ** 0.5
    A, dX, dhalo, dW = torch.zeros(n, d, device=dev), torch.zeros(n, d, device=dev), torch.full((nb + 1, d), 7.0, device=dev), torch.zeros(d, e, device=dev)
    ctx.gcn_layer_bwd(1, p, dZ, None, A, X, W, dW, dX, dhalo[:nb])
    torch.cuda.synchronize()
    K = int(n_kept)
    assert K >= 65536 and (p == 1.0 or K % 8)
    s_in, s_bd = (torch.from_numpy(x).to(dev).double().rsqrt()[:, None] for x in (P.deg_in, P.deg_halo))
    G = s_in * (dZ.double() @ W.double().T)
    node, of = torch.from_numpy(node).to(dev), torch.from_numpy(of).to(dev)
    ref = torch.zeros(nb, d, device=dev, dtype=torch.float64).index_add_(0, node, G[of]) * s_bd / p
    # sums of at most 80 elements, each a sum of e products that is of size 1
    torch.testing.assert_close(dhalo[:K].double(), ref[kept[:K].long()], rtol=1e-5, atol=3e-5)
    torch.testing.assert_close(dX.double(), s_in * G, rtol=1e-5, atol=3e-5)
    assert bool((dhalo[K:] == 7.0).all())
    ctx.close()


def _long_row_sums(rows, X, Xb, kept, n, w_halo, nseg):
    """Sums of rows of several segments, rounding by rounding: a segment's entries go in turn to two running sums (32 lanes to an entry,
    half a wavefront), which are added; the segments are added in ascending order.  All weights are 0, 1 or w_halo, a power of two."""
    out = []
    for (v, cols), k in zip(rows, nseg):
        x = np.stack([X[c] * np.float32(c != v) if c < n else Xb[kept[c - n]] * np.float32(w_halo) for c in cols])
        chunk, total = max(1, -(-len(cols) // k)), np.zeros(X.shape[1], np.float32)
        for s in range(0, len(cols), chunk):
            acc = np.zeros((2, X.shape[1]), np.float32)
            for e, row in enumerate(x[s:s + chunk]):
                acc[e % 2] += row
            total += acc[0] + acc[1]
        out.append(total)
    return np.stack(out)


@pytest.mark.parametrize("cached", [False, True])
@pytest.mark.parametrize("n", [3000, 20000, 98304])  # layers of one launch, of two, and of one after the long rows
@pytest.mark.parametrize("d,bd", [(128, 20), (128, 200), (100, 20), (68, 200)])
def test_order_of_the_sums_of_long_rows(d, bd, n, cached):
    """Which hidden units a ReLU switches on hangs on the last bit of a forward sum: its order is that of the width alone, whatever the
    share of the boundary entries, the route of the layer and the slices of a launch."""
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(d + bd + n)
    nb, p = 2000, 0.5
    long = np.sort(rng.choice(n, size=24, replace=False))
    deg = np.full(n, 4)
    deg[long] = rng.integers(257, 1300, long.size)
    n_bd = np.zeros(n, dtype=np.int64)
    n_bd[long] = bd
    lists = [np.unique(np.append(rng.integers(0, n, deg[v]), v)) for v in range(n)]
    bds = [np.sort(rng.choice(nb, size=k, replace=False)) for k in n_bd]
    bds[0] = np.arange(nb)  # (every boundary node has a neighbour)
    cols = [np.concatenate([a, n + b]) for a, b in zip(lists, bds)]
    row, col = np.repeat(np.arange(n), [len(c) for c in cols]), np.concatenate(cols)
    inner = col < n
    t, h = np.lexsort((row[inner], col[inner])), np.lexsort((row[~inner], col[~inner]))
    i32 = lambda x: np.ascontiguousarray(x, dtype=np.int32)  # noqa: E731
    ptr = lambda of, m: i32(np.concatenate([[0], np.cumsum(np.bincount(of, minlength=m))]))  # noqa: E731
    P = types.SimpleNamespace(
        part_id=0, n_in=n, n_halo=nb, nnz0=len(col), e_in=int(inner.sum()), e_bd=int((~inner).sum()), row_ptr0=ptr(row, n), col0=i32(col),
        t_in_ptr=ptr(col[inner], n), t_in_col=i32(row[inner][t]), halo_ptr=ptr(col[~inner] - n, nb), halo_col=i32(row[~inner][h]),
        halo_gid=np.arange(n, n + nb, dtype=np.int64), deg_in=i32(np.full(n, 1025)), deg_halo=i32(np.full(nb, 1025)))
    z32 = lambda m: torch.zeros(m, dtype=torch.int32, device=dev)  # noqa: E731
    ctx = pkg.Context(P, [d, 8], 0, device=dev, layer_kind=1)
    kept, remap, n_kept, nnz = z32(nb), z32(nb), z32(1), z32(1)
    ctx.sample_boundary(3, 0, p, kept, remap, n_kept)
    csr = z32(n + 1), z32(P.nnz0), z32(n + nb + 1), z32(P.nnz0)
    ctx.build_sampled_csr(remap, kept, n_kept, *csr, nnz)
    gen = torch.Generator(device=dev)
    gen.manual_seed(d)
    X, Xb, W = (torch.randn(*s, device=dev, generator=gen) for s in ((n, d), (nb, d), (2 * d, 8)))
    A, H = torch.zeros(n, d, device=dev), torch.zeros(n, 8, device=dev)
    if cached:
        ctx.cache_input_aggregate(X)
    ctx.gcn_layer_fwd(1, p, X, Xb, W, A, H, False)
    torch.cuda.synchronize()
    rp, ci, of = csr[0].cpu().numpy(), csr[1].cpu().numpy(), kept.cpu().numpy()
    rows = [(v, ci[rp[v]:rp[v + 1]]) for v in long]
    parts = [[(v, c[c < n]) for v, c in rows], [(v, c[c >= n]) for v, c in rows]] if cached else [rows]
    nseg = [-(-len(cols[v]) // 256) for v in long]
    sums = [_long_row_sums(r, X.cpu().numpy(), Xb.cpu().numpy(), of, n, 1 / p, nseg) for r in parts]
    want = (sums[1] + sums[0] if cached else sums[0]) * np.float32(1.0 / 1024)
    got = A.cpu().numpy()[long]
    assert np.allclose(got, want, rtol=1e-4, atol=1e-5)  # (or the weights are not those of the docstring)
    assert np.array_equal(got, want)
    ctx.close()
