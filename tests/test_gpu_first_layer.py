"""The first layer's forward pass in the launch that draws the subgraph of a small partition: everything that a step leaves has the bits of the launches that a
timed step makes (one for the subgraph, one or two for the layer), and which form ran is counted."""
import types

import numpy as np
import pytest

from test_gpu_tile import _launches

pytestmark = pytest.mark.gpu


def _partition(n, deg, n_halo, bd_most, rng):
    """Rows of 0 to 2 deg inner neighbours and 0 to bd_most boundary ones, every boundary node with one inner neighbour at least."""
    rows, cols = [], []
    for v in range(n):
        inner = np.union1d(rng.choice(n, size=rng.integers(0, 2 * deg + 1), replace=False), [v])
        rows.append(np.full(len(inner), v)); cols.append(inner)
        bd = n + rng.choice(n_halo, size=rng.integers(0, bd_most + 1), replace=False) if n_halo else np.zeros(0, int)
        rows.append(np.full(len(bd), v)); cols.append(bd)
    rows.append(rng.integers(0, n, size=n_halo)); cols.append(n + np.arange(n_halo))
    key = np.unique(np.concatenate(rows).astype(np.int64) * (n + n_halo) + np.concatenate(cols))
    row, col = key // (n + n_halo), key % (n + n_halo)
    i32 = lambda x: np.ascontiguousarray(x, dtype=np.int32)  # noqa: E731
    ptr = lambda of, m: i32(np.concatenate([[0], np.cumsum(np.bincount(of, minlength=m))]))  # noqa: E731
    inner = col < n
    t = np.sort(col[inner] * n + row[inner])
    h = np.sort((col[~inner] - n) * n + row[~inner])
    return types.SimpleNamespace(part_id=3, n_in=n, n_halo=n_halo, nnz0=len(key), e_in=int(inner.sum()), e_bd=len(h), row_ptr0=ptr(row, n), col0=i32(col),
                                 t_in_ptr=ptr(t // n, n), t_in_col=i32(t % n), halo_ptr=ptr(h // n, n_halo) if n_halo else np.zeros(1, np.int32), halo_col=i32(h % n) if n_halo else np.zeros(0, np.int32),
                                 halo_gid=np.arange(n_halo, dtype=np.int64) * 7 + (1 << 33), deg_in=i32(np.bincount(row, minlength=n)),
                                 deg_halo=i32(np.bincount(col[~inner] - n, minlength=n_halo) + 2 if n_halo else np.zeros(0)))


def _fits(P, p):
    """The host's conditions for one launch of the subgraph, and for a first layer without rows of several segments."""
    return (max(P.n_halo, P.e_bd) <= 8192 and P.e_in + 3 * P.n_in + P.n_halo + 12 * np.ceil(p * P.n_halo) <= 51200 and P.n_in <= 8192 and
            np.diff(P.row_ptr0).max() <= 256)


def _launches_saved(ctx, P, dims, kind, p):
    """Launches that a step has less than the same step with the subgraph, the first layer's aggregate and its one product apart: 2 where all are one launch, 1 where
    the first layer is one beside the subgraph's.  (Features on top of the saved aggregate keep them apart; such a step is recorded and never run.)"""
    import torch
    import paper_2203_10983_amd as pkg
    f32 = lambda *s: torch.zeros(*s, device="cuda:0")  # noqa: E731
    n, nb = P.n_in, P.n_halo
    W = [f32((1 + kind) * a, b) for a, b in zip(dims, dims[1:])]
    rest = ([f32(nb, a) for a in dims[:-1]], torch.zeros(n, dtype=torch.int32, device="cuda:0"), W, [f32(*w.shape) for w in W],
            [None] + [f32(nb, a) for a in dims[1:-1]], f32(1), 0.0)
    apart, now = (_launches(lambda: ctx.train_step(11, 0, p, X, *rest)) for X in (ctx.ws_tensor(pkg.VIEW_A, 1, torch.float32), f32(n, dims[0])))
    return apart - now - (kind == 1 and dims[0] % 16 != 0)  # (a mean aggregator of such a width has two products)


@pytest.mark.parametrize("kind", [0, 1], ids=["gcn", "sage"])
@pytest.mark.parametrize("n,deg,n_halo,bd_most,dims,p,q,cached", [
    (1, 0, 2, 1, [64, 16, 8], 0.5, 0.0, False), (9, 1, 40, 20, [12, 7, 3], 0.5, 0.0, False), (500, 2, 330, 2, [64, 16, 8], 0.1, 0.0, False),
    # rows of more than 64 inner entries and of more than 64 boundary ones, kept or not; 128 floats; tiles of 16 rows
    (150, 60, 600, 50, [36, 130, 5], 0.5, 0.3, False), (90, 18, 450, 70, [128, 128, 128, 9], 0.9, 0.0, False), (65, 32, 2000, 120, [16, 33, 4], 1.0, 0.5, True),
    (90, 30, 900, 80, [100, 66, 9], 0.0, 0.0, False), (333, 8, 1500, 24, [20, 256, 47], 0.5, 0.0, True), (700, 3, 0, 0, [68, 16, 8], 0.5, 0.0, False),
    (3585, 2, 8192, 0, [64, 30, 8], 0.1, 0.1, False), (8192, 1, 300, 1, [36, 140, 8], 0.1, 0.0, False)], ids=lambda v: "x".join(map(str, v)) if isinstance(v, list) else str(v))
def test_bits_of_two_launches(n, deg, n_halo, bd_most, dims, p, q, cached, kind):
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(n + dims[0])
    P = _partition(n, deg, n_halo, bd_most, np.random.default_rng(n))
    assert _fits(P, p) and (dims[0] < 128 or P.nnz0 < 64 * n)
    L = len(dims) - 1
    f32 = lambda *s: torch.randn(*s, device=dev, generator=gen)  # noqa: E731
    X, halo_h = f32(n, dims[0]), [f32(n_halo, d).clamp_(min=0) for d in dims[:-1]]
    labels = torch.randint(0, dims[-1], (n,), device=dev, dtype=torch.int32, generator=gen)
    W = [f32((1 + kind) * a, b) / a ** 0.5 for a, b in zip(dims, dims[1:])]
    ctx = pkg.Context(P, dims, 0, device=dev, layer_kind=kind)
    ctx.set_dropout(q)
    if cached:
        ctx.cache_input_aggregate(X)

    def step(mask, epoch):
        ctx.profile_enable(mask, 64)
        dW, loss = [torch.zeros_like(w) for w in W], torch.zeros(1, device=dev)
        dhalo = [None] + [torch.zeros(n_halo, d, device=dev) for d in dims[1:-1]]
        ctx.train_step(11, epoch, p, X, halo_h, labels, W, dW, dhalo, loss, 0.0)
        torch.cuda.synchronize()
        ctx.profile_enable(0, 0)
        f = [ctx.ws_tensor(v, l, torch.float32).clone() for v in (pkg.VIEW_A, pkg.VIEW_H) for l in range(1, L + 1)]
        k, m = int(ctx.ws_tensor(pkg.VIEW_N_KEPT)[0]), int(ctx.ws_tensor(pkg.VIEW_NNZ)[0])
        i = [ctx.ws_tensor(pkg.VIEW_REMAP), ctx.ws_tensor(pkg.VIEW_ROW_PTR), ctx.ws_tensor(pkg.VIEW_KEPT_IDS)[:k], ctx.ws_tensor(pkg.VIEW_COL_IDX)[:m],
             ctx.ws_tensor(pkg.VIEW_T_ROW_PTR)[:n + k + 1], ctx.ws_tensor(pkg.VIEW_T_COL_IDX)[:m]]
        return f + [t.clone() for t in i], dW + dhalo[1:], loss, (k, m)

    for epoch in range(2):
        steps = []
        # untimed; the selection and subgraph steps timed, so that the first layer alone moves to a launch of its own; every phase timed.  (The untimed
        # step is the first of its epoch: what it leaves unwritten is that of another sample.)
        for fill, mask in ((7.0, 0), (8.0, 3), (9.0, 0xFFFFFFFF)):
            for t in ctx.ws_tensor(pkg.VIEW_H, 1, torch.float32), ctx.ws_tensor(pkg.VIEW_A, 1, torch.float32):
                t.fill_(fill)
            steps.append(step(mask, epoch))
        (one, grads, loss, counts), (two, two_grads, two_loss, two_counts), (timed, _, timed_loss, timed_counts) = steps
        assert counts == two_counts == timed_counts
        for a, b, c in zip(one, two, timed):
            assert torch.equal(a, b) and torch.equal(a, c)
        for a, b in zip(grads + [loss], two_grads + [two_loss]):
            assert torch.isfinite(a).all() and torch.equal(a, b)
        assert torch.allclose(loss, timed_loss, rtol=1e-6)  # partial sums of other rows
    assert _launches_saved(ctx, P, dims, kind, p) == 2  # it was one launch
    ctx.close()


@pytest.mark.parametrize("kind", [0, 1], ids=["gcn", "sage"])
@pytest.mark.parametrize("n,d,one", [(3584, 128, True), (3585, 128, False), (3585, 100, False), (3585, 64, True)])
def test_wide_rows_of_many_tiles_have_a_launch_of_their_own(n, d, one, kind):
    """Counted beside the same step on features that share memory with the layer's results, which has the subgraph, the aggregate and the update
    apart (recorded, not run)."""
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    P = _partition(n, 2, 700, 1, np.random.default_rng(n))
    dims = [d, 40, 8]
    assert _fits(P, 0.1)
    ctx = pkg.Context(P, dims, 0, device=dev, layer_kind=kind)
    assert _launches_saved(ctx, P, dims, kind, 0.1) == (2 if one else 1)
    ctx.close()
