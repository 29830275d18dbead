"""Rows of several segments: added up by the wavefront that is the last to finish one (up to 65536 segments and slices, more than eight to the
longest row) or by a launch behind, call after call."""
import numpy as np
import pytest

from test_gpu_slices import _partition

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [3, 6, 64, 130, 256, 300])
@pytest.mark.parametrize("cliques,size", [(1, 2305), (2, 2600), (12, 513)])  # 23050, 57200 and (three to a row) 18468 segments
def test_call_after_call(cliques, size, d):
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(d)
    P = _partition(cliques, size, 20, np.random.default_rng(size))
    n, n_halo = P.n_in, P.n_halo
    i32 = lambda k: torch.zeros(k, dtype=torch.int32, device=dev)  # noqa: E731
    ctx = pkg.Context(P, [d, d], 0, device=dev)
    s_in, s_bd = (torch.from_numpy(x).to(dev).double().rsqrt()[:, None] for x in (P.deg_in, P.deg_halo))
    clique = torch.arange(n, device=dev) // size
    node = torch.repeat_interleave(torch.arange(n_halo, device=dev), torch.from_numpy(np.diff(P.halo_ptr)).to(dev))
    of = torch.from_numpy(P.halo_col).long().to(dev)
    kept, remap, n_kept, nnz = i32(n_halo), i32(n_halo), i32(1), i32(1)
    csr = i32(n + 1), i32(P.nnz0), i32(n + n_halo + 1), i32(P.nnz0)
    ctx.sample_boundary(1, 0, 1.0, kept, remap, n_kept)
    ctx.build_sampled_csr(remap, kept, n_kept, *csr, nnz)

    def inner(x):
        return torch.zeros(cliques, d, device=dev, dtype=torch.float64).index_add_(0, clique, x)[clique]

    for _ in range(3):
        X, Xb, dH = (torch.randn(k, d, device=dev, generator=gen) for k in (n, n_halo, n))
        A, H, dX = (torch.full((n, d), 7.0, device=dev) for _ in range(3))
        dW, dhalo, eye = torch.zeros(d, d, device=dev), torch.zeros(n_halo, d, device=dev), torch.eye(d, device=dev)
        ctx.gcn_layer_fwd(1, 1.0, X, Xb, eye, A, H, False)
        ctx.gcn_layer_bwd(1, 1.0, dH, None, A, X, eye, dW, dX, dhalo)
        torch.cuda.synchronize()
        # sums of up to 2600 terms of size 1 with weights of about 1 / 2600, and those of the boundary: a rounding is 2^-24 of a sum of size 1
        tol = dict(rtol=1e-5, atol=1e-5)
        torch.testing.assert_close(A.double(), s_in * inner(s_in * X).index_add_(0, of, (s_bd * Xb)[node]), **tol)
        torch.testing.assert_close(dX.double(), s_in * inner(s_in * dH), **tol)
    ctx.close()
