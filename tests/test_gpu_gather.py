"""The aggregate at the edges of its batches (64 entries), load groups (8 steps) and segments (256), against fp64.

The graph is a set of cliques with self-loops, so that A H0 is the clique's mean on every row, and every row of
a clique of k nodes gathers k entries, forward and in the transposed pass."""
import types

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CLIQUES = [1, 2, 3, 4, 5, 15, 16, 17, 31, 32, 33, 35, 36, 37, 60, 63, 64, 65, 96, 97, 127, 128, 129, 255, 256, 257, 515]


def _cliques():
    size = np.repeat(CLIQUES, CLIQUES).astype(np.int32)
    first = np.repeat(np.cumsum(CLIQUES) - CLIQUES, CLIQUES).astype(np.int32)
    ptr = np.concatenate([[0], np.cumsum(size)]).astype(np.int32)
    col = np.concatenate([np.arange(f, f + k, dtype=np.int32) for f, k in zip(first, size)])
    none = np.zeros(0, np.int32)
    n = len(size)
    return types.SimpleNamespace(part_id=0, n_in=n, n_halo=0, nnz0=len(col), e_in=len(col), e_bd=0, row_ptr0=ptr, col0=col,
                                 t_in_ptr=ptr.copy(), t_in_col=col.copy(), halo_ptr=np.zeros(1, np.int32), halo_col=none,
                                 halo_gid=np.zeros(0, np.int64), deg_in=size, deg_halo=none), first


@pytest.mark.parametrize("d", [3, 16, 33, 36, 41, 47, 61, 64, 68, 100, 128, 129, 200, 602])
def test_aggregate(d):
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(d)
    part, first = _cliques()
    n = part.n_in
    which = torch.unique(torch.from_numpy(first.astype(np.int64)).to(dev), return_inverse=True)[1]
    count = torch.tensor(CLIQUES, device=dev, dtype=torch.float64)

    def clique_mean(x):
        s = torch.zeros(len(CLIQUES), x.shape[1], device=dev, dtype=torch.float64).index_add_(0, which, x.double())
        return (s / count[:, None])[which]

    i32 = lambda k: torch.zeros(k, dtype=torch.int32, device=dev)  # noqa: E731
    ctx = pkg.Context(part, [d, d], 0, device=dev)
    kept, remap, n_kept, nnz = i32(1), i32(1), i32(1), i32(1)
    ctx.sample_boundary(1, 0, 0.5, kept, remap, n_kept)
    csr = i32(n + 1), i32(part.nnz0), i32(n + 1), i32(part.nnz0)    # must outlive the layer calls
    ctx.build_sampled_csr(remap, kept, n_kept, *csr, nnz)
    X, dH = torch.randn(n, d, device=dev, generator=gen), torch.randn(n, d, device=dev, generator=gen)
    W = torch.eye(d, device=dev)
    A, H, dW, dX = (torch.full((k, d), 7.0, device=dev) for k in (n, n, d, n))
    ctx.gcn_layer_fwd(1, 0.5, X, None, W, A, H, False)
    ctx.gcn_layer_bwd(1, 0.5, dH, None, A, X, W, dW, dX, None)
    torch.cuda.synchronize()
    torch.testing.assert_close(A.double(), clique_mean(X), rtol=0, atol=2e-6)
    torch.testing.assert_close(dX.double(), clique_mean(dH), rtol=0, atol=2e-6)
    ctx.close()
