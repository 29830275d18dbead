"""Rows of several segments: added up by the wavefront that is the last to finish one (up to 45056 segments and slices, 9 to 64 to the longest
row, or more beside many short rows) or by a launch behind, call after call, with the same bits."""
import types

import numpy as np
import pytest

from test_gpu_slices import _partition
from test_gpu_tile import _launches

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


def _hubs(segments, n, n_filled, fill):
    """n inner nodes with a self-loop.  Row j < len(segments) has an entry in each of the first columns, one more than segments[j] - 1 segments hold;
    rows 100 .. 100 + n_filled have `fill` entries, from their own column on; node n - 1 has a boundary neighbour.  The degrees (the weights) do not
    depend on any of it."""
    row = [np.full(256 * (k - 1) + 1, j) for j, k in enumerate(segments)] + [np.repeat(np.arange(100, 100 + n_filled), fill), np.arange(n)]
    col = [np.arange(len(r)) for r in row[:len(segments)]] + [(np.arange(100, 100 + n_filled)[:, None] + np.arange(fill)).reshape(-1) % n, np.arange(n)]
    key = np.unique(np.concatenate(row).astype(np.int64) * n + np.concatenate(col))
    row, col = key // n, key % n
    t = np.sort(col * n + row)
    i32 = lambda x: np.ascontiguousarray(x, dtype=np.int32)  # noqa: E731
    ptr = lambda of: np.concatenate([[0], np.cumsum(np.bincount(of, minlength=n))])  # noqa: E731
    row_ptr = ptr(row)
    row_ptr[n] += 1
    return types.SimpleNamespace(
        part_id=0, n_in=n, n_halo=1, nnz0=len(key) + 1, e_in=len(key), e_bd=1, row_ptr0=i32(row_ptr), col0=i32(np.append(col, n)), t_in_ptr=i32(ptr(t // n)),
        t_in_col=i32(t % n), halo_ptr=i32([0, 1]), halo_col=i32([n - 1]), halo_gid=np.array([n], dtype=np.int64), deg_in=i32(np.arange(n) % 7 + 2), deg_halo=i32([2]))


@pytest.mark.parametrize("d", [6, 64, 130, 256, 300])  # 256: in two slices, 300: two pieces to a lane
@pytest.mark.parametrize("segments,n_filled,by_last", [((9, 17, 64), 22528, True), ((17, 100), 22528, True), ((65, 2000), 32768, False)],
                         ids=["up-to-64", "longer-aside", "longer"])
def test_rows_of_many_segments(segments, n_filled, by_last, d):
    """The same rows beside n_filled others of one segment, and of two, which are too many segments for the wavefronts to add up: the second takes one launch
    more where the first has none for the sums, and the bits are the same."""
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(d)
    n = max(131072, 256 * max(segments))
    X, Xb, W = (torch.randn(*s, device=dev, generator=gen) for s in ((n, d), (1, d), (d, 4)))
    sums, launches = [], []
    for fill in (256, 257):
        P = _hubs(segments, n, n_filled, fill)
        per_row = -(-np.diff(P.row_ptr0) // 256)
        n_part = int(per_row[per_row > 1].sum())
        assert by_last == (max(segments) <= 64 or n - len(segments) >= 1024 * max(segments))
        assert per_row.max() == max(segments) and P.nnz0 < 64 * n and n_part == sum(segments) + (2 * n_filled if fill == 257 else 0)
        i32 = lambda k: torch.zeros(k, dtype=torch.int32, device=dev)  # noqa: E731
        ctx = pkg.Context(P, [d, 4], 0, device=dev)
        kept, remap, n_kept, nnz = i32(1), i32(1), i32(1), i32(1)
        ctx.sample_boundary(1, 0, 1.0, kept, remap, n_kept)
        csr = i32(n + 1), i32(P.nnz0), i32(n + 2), i32(P.nnz0)
        ctx.build_sampled_csr(remap, kept, n_kept, *csr, nnz)
        A, H = torch.full((n, d), 7.0, device=dev), torch.zeros(n, 4, device=dev)
        call = lambda: ctx.gcn_layer_fwd(1, 1.0, X, Xb, W, A, H, False)  # noqa: E731
        launches.append(_launches(call))
        for _ in range(3):
            A.fill_(7.0)
            call()
            torch.cuda.synchronize()
            s_in = torch.from_numpy(P.deg_in).to(dev).double().rsqrt()[:, None]
            for row in (*range(len(segments)), 100, 100 + n_filled - 1):
                cols = torch.from_numpy(P.col0[P.row_ptr0[row]:P.row_ptr0[row + 1]]).to(dev).long()
                terms = s_in[row] * s_in[cols] * X[cols].double()
                allowance = 4.0 * 2.0 ** -24 * len(cols) ** 0.5 * terms.abs().sum(0)
                assert ((A[row].double() - terms.sum(0)).abs() <= allowance).all(), row
        sums.append(A[:len(segments)].clone())
        ctx.close()
    assert launches[1] - launches[0] == (1 if by_last else 0)
    assert torch.equal(*sums)
