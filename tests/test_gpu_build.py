"""Subgraph step: rows whose boundary entries end around the words and tiles (64 and 2048 entries) that the places are counted by, and rows of
several tiles, against the static CSR filtered on the host."""
import types

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _partition(per_row, n_halo, rng):
    """Inner nodes with a self-loop each, row v with per_row[v] boundary nodes; every boundary node has a neighbour."""
    n = len(per_row)
    lists = [np.sort(rng.choice(n_halo, size=k, replace=False)) for k in per_row]
    lists[-1] = np.arange(n_halo)
    row = np.concatenate([np.arange(n), np.repeat(np.arange(n), [len(x) for x in lists])])
    col = np.concatenate([np.arange(n), n + np.concatenate(lists)])
    order = np.lexsort((col, row))
    row, col = row[order], col[order]
    bd = col >= n
    by_node = np.lexsort((row[bd], col[bd]))
    ptr = lambda of, m: np.concatenate([[0], np.cumsum(np.bincount(of, minlength=m))])  # noqa: E731
    i32 = lambda x: np.ascontiguousarray(x, dtype=np.int32)  # noqa: E731
    return types.SimpleNamespace(
        part_id=0, n_in=n, n_halo=n_halo, nnz0=len(col), e_in=n, e_bd=int(bd.sum()), row_ptr0=i32(ptr(row, n)), col0=i32(col),
        t_in_ptr=i32(np.arange(n + 1)), t_in_col=i32(np.arange(n)), halo_ptr=i32(ptr(col[bd] - n, n_halo)), halo_col=i32(row[bd][by_node]),
        halo_gid=np.arange(n, n + n_halo, dtype=np.int64), deg_in=i32(np.bincount(row, minlength=n)),
        deg_halo=i32(np.bincount(col[bd] - n, minlength=n_halo) + 1))


@pytest.mark.parametrize("p", [0.0, 0.37, 1.0])
@pytest.mark.parametrize("per_row", [(0, 0), (63, 1, 0, 64, 65), (2047, 1, 2048, 2049, 0), (3, 9000, 2, 0, 0, 8200, 1), (1,) * 5000, (0,) * 2047 + (9000,), (0,) * 2048 + (3, 1)])
def test_rows_around_words_and_tiles(per_row, p):
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    nb = 9000
    P = _partition(per_row, nb, np.random.default_rng(len(per_row)))
    n = P.n_in
    i32 = lambda k: torch.full((k,), -7, dtype=torch.int32, device=dev)  # noqa: E731
    ctx = pkg.Context(P, [4, 4], 0, device=dev)
    kept, remap, n_kept, nnz = i32(nb), i32(nb), i32(1), i32(1)
    ctx.sample_boundary(5, 1, p, kept, remap, n_kept)
    row_ptr, col, t_row_ptr, t_col = i32(n + 1), i32(P.nnz0), i32(n + nb + 1), i32(P.nnz0)
    ctx.build_sampled_csr(remap, kept, n_kept, row_ptr, col, t_row_ptr, t_col, nnz)
    torch.cuda.synchronize()
    remap = remap.cpu().numpy()
    K = int(n_kept[0])
    assert K == (remap >= 0).sum() and (p != 1.0 or K == nb) and (p != 0.0 or K == 0)
    row0 = np.repeat(np.arange(n), np.diff(P.row_ptr0))
    new = np.where(P.col0 < n, P.col0, n + remap[np.maximum(P.col0 - n, 0)])
    stay = (P.col0 < n) | (new >= n)
    row, new = row0[stay], new[stay]
    assert int(nnz[0]) == len(new)
    assert np.array_equal(row_ptr.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(row, minlength=n))]))
    assert np.array_equal(col.cpu().numpy()[:len(new)], new)
    order = np.lexsort((row, new))
    assert np.array_equal(t_row_ptr.cpu().numpy()[:n + K + 1], np.concatenate([[0], np.cumsum(np.bincount(new, minlength=n + K))]))
    assert np.array_equal(t_col.cpu().numpy()[:len(new)], row[order])
    ctx.close()


def _few_long_rows(n, per_row, n_halo):
    """n inner nodes with a self-loop and per_row boundary nodes each: those whose number is that of the row up to multiples of n_halo / per_row."""
    step = n_halo // per_row
    v = np.arange(n)
    col = np.concatenate([v[:, None], n + np.arange(per_row) * step + (v % step)[:, None]], 1)
    rows = [np.arange(r, n, step) for r in range(step)]
    ptr = lambda count: np.concatenate([[0], np.cumsum(count)])  # noqa: E731
    i32 = lambda x: np.ascontiguousarray(x.reshape(-1), dtype=np.int32)  # noqa: E731
    count = np.tile([len(x) for x in rows], per_row)
    return types.SimpleNamespace(
        part_id=0, n_in=n, n_halo=n_halo, nnz0=col.size, e_in=n, e_bd=n * per_row, row_ptr0=i32(np.arange(n + 1) * (per_row + 1)), col0=i32(col),
        t_in_ptr=i32(np.arange(n + 1)), t_in_col=i32(v), halo_ptr=i32(ptr(count)), halo_col=i32(np.tile(np.concatenate(rows), per_row)),
        halo_gid=np.arange(n, n + n_halo, dtype=np.int64), deg_in=i32(np.full(n, per_row + 1)), deg_halo=i32(count + 1))


def test_rows_of_thousands_of_tiles_take_no_longer():
    """Eight million boundary entries in 2000 rows, which one workgroup places, and in 200000: the places of both, and about the same time."""
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    best = []
    for n, per_row in ((2000, 4000), (200000, 40)):
        nb = 40000
        P = _few_long_rows(n, per_row, nb)
        i32 = lambda k: torch.full((k,), -7, dtype=torch.int32, device=dev)  # noqa: E731
        ctx = pkg.Context(P, [4, 4], 0, device=dev)
        kept, remap, n_kept, nnz = i32(nb), i32(nb), i32(1), i32(1)
        ctx.sample_boundary(5, 1, 0.1, kept, remap, n_kept)
        row_ptr, col, t_row_ptr, t_col = i32(n + 1), i32(P.nnz0), i32(n + nb + 1), i32(P.nnz0)
        times = []
        for _ in range(6):
            begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            torch.cuda.synchronize()
            torch.cuda._sleep(200000)  # (the launches are queued behind it: their time is the GPU's)
            begin.record()
            ctx.build_sampled_csr(remap, kept, n_kept, row_ptr, col, t_row_ptr, t_col, nnz)
            end.record()
            end.synchronize()
            times.append(begin.elapsed_time(end))
        best.append(min(times[1:]))
        static = torch.from_numpy(P.col0).to(dev).view(n, per_row + 1).long()
        stay = torch.cat([torch.ones(n, 1, dtype=torch.bool, device=dev), (remap >= 0)[static[:, 1:] - n]], 1)
        assert torch.equal(row_ptr[1:].long(), stay.sum(1).cumsum(0)) and int(row_ptr[0]) == 0 and int(nnz[0]) == int(stay.sum())
        new = torch.cat([static[:, :1], n + remap.long()[static[:, 1:] - n]], 1)[stay]
        assert torch.equal(col[:new.numel()].long(), new)
        ctx.close()
    assert best[0] <= 2 * best[1], best
