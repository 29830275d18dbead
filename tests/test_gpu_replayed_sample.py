"""The stand-alone calls after a captured step: what its replays leave in the workspace is the latest sample."""
import numpy as np
import pytest

from bns_inputs import SAMPLING_SEED
from oracle import bns_oracle as orc
from test_gpu_tile import _partition

pytestmark = pytest.mark.gpu


class _Program:
    """A context on a partition whose subgraph is one launch of a step at p = 0.1 and several at p = 1, inputs, a stream for captures."""

    def __init__(self):
        import torch
        import paper_2203_10983_amd as pkg
        self.torch, self.pkg = torch, pkg
        dev = torch.device("cuda:0")
        n, n_halo, d = 600, 7000, 8
        self.P = _partition(n, 3, 0, n_halo, np.random.default_rng(n), lists=1)
        self.ctx = pkg.Context(self.P, [d, d], 0, device=dev)
        f32 = lambda *k: torch.ones(*k, device=dev)  # noqa: E731
        W = [f32(d, d)]
        self.args = (f32(n, d), [f32(n_halo, d)], torch.zeros(n, dtype=torch.int32, device=dev), W, [f32(d, d)], None, f32(1))
        self.stream = torch.cuda.Stream()
        i32 = lambda n: torch.zeros(n, dtype=torch.int32, device=dev)  # noqa: E731
        self.csr = [i32(self.P.n_in + 1), i32(self.P.nnz0), i32(self.P.n_in + self.P.n_halo + 1), i32(self.P.nnz0), i32(1)]
        self.own = i32(self.P.n_halo), i32(self.P.n_halo), i32(1)  # remap, kept_ids, n_kept
        view = lambda v, n: self.ctx.ws_tensor(v)[:n]  # noqa: E731
        self.in_workspace = view(pkg.VIEW_REMAP, self.P.n_halo), view(pkg.VIEW_KEPT_IDS, self.P.n_halo), view(pkg.VIEW_N_KEPT, 1)

    def sample(self, into, epoch, p):
        self.ctx.sample_boundary(SAMPLING_SEED, epoch, p, into[1], into[0], into[2])

    def capture(self, epoch, p):
        self.torch.cuda.synchronize()
        with self.torch.cuda.stream(self.stream):
            self.ctx.graph_capture(SAMPLING_SEED, epoch, p, *self.args)
        self.torch.cuda.synchronize()

    def replay(self, n):
        with self.torch.cuda.stream(self.stream):
            self.ctx.graph_replay(n)
        self.torch.cuda.synchronize()

    def check(self, epoch, p):
        """The subgraph just built is that of this draw."""
        self.torch.cuda.synchronize()
        sub = orc.sample_and_build(self.P, SAMPLING_SEED, epoch, p)
        nnz = int(self.csr[4][0])
        assert nnz == sub["col_idx"].size
        assert np.array_equal(self.csr[0].cpu().numpy(), sub["row_ptr"])
        assert np.array_equal(self.csr[1][:nnz].cpu().numpy(), sub["col_idx"])


def test_which_steps_count_the_boundary_entries():
    """What the other tests of this file rest on."""
    g = _Program()
    for p, build in ((0.1, 0), (1.0, 1)):
        g.ctx.profile_enable(3, 16)
        g.ctx.train_step(SAMPLING_SEED, 0, p, *g.args)
        g.torch.cuda.synchronize()
        assert g.ctx.profile_read()["build"][1] == build
    g.ctx.close()


def test_build_on_the_sample_of_a_replay():
    """A sample into the workspace arrays, a replay of one launch that draws another one there, and a stand-alone build on them:
    its keep flags are those of the replay."""
    g = _Program()
    g.capture(7, 0.1)
    g.sample(g.in_workspace, 3, 0.9)
    g.replay(1)
    g.ctx.build_sampled_csr(*g.in_workspace, *g.csr)
    g.check(7, 0.1)
    g.ctx.close()


def test_build_after_a_capture_on_the_sample_before_it():
    """A capture runs nothing: the boundary entries of the one-launch step before it are still to be counted."""
    g = _Program()
    g.ctx.train_step(SAMPLING_SEED, 5, 0.1, *g.args)
    g.capture(6, 1.0)
    g.ctx.build_sampled_csr(*g.in_workspace, *g.csr)
    g.check(5, 0.1)
    g.ctx.close()


def test_build_refuses_a_sample_that_a_replay_has_replaced():
    """The row starts in the workspace are those of the replay's kept nodes: with the lists of other nodes a build could write past
    the end of the transposed columns.  So is one on a captured step that has not run.  A new sample is accepted again."""
    g = _Program()
    g.capture(7, 0.1)
    refused = "do not hold the latest sample"
    with pytest.raises(g.pkg.BnsError, match=refused):
        g.ctx.build_sampled_csr(*g.in_workspace, *g.csr)
    g.sample(g.own, 3, 0.9)
    g.replay(0)
    g.ctx.build_sampled_csr(*g.own, *g.csr)
    g.check(3, 0.9)
    g.replay(2)
    with pytest.raises(g.pkg.BnsError, match=refused) as e:
        g.ctx.build_sampled_csr(*g.own, *g.csr)
    assert e.value.status == 1
    g.sample(g.own, 4, 0.5)
    g.ctx.build_sampled_csr(*g.own, *g.csr)
    g.check(4, 0.5)
    g.ctx.close()


def test_layers_are_refused_while_a_captured_step_has_not_run():
    """A capture makes the workspace arrays current; until a step has run they hold nothing to gather by."""
    g = _Program()
    g.sample(g.own, 3, 0.5)
    g.ctx.build_sampled_csr(*g.own, *g.csr)
    g.capture(7, 0.1)
    X, (Xb,), _, (W,), (dW,) = g.args[:5]
    A, H = g.torch.zeros_like(X), g.torch.zeros_like(X)
    fwd = lambda: g.ctx.gcn_layer_fwd(1, 0.1, X, Xb, W, A, H, False)  # noqa: E731
    for call in (fwd, lambda: g.ctx.gcn_layer_bwd(1, 0.1, X, None, X, None, W, dW, A, None)):
        with pytest.raises(g.pkg.BnsError, match="has not run") as e:
            call()
        assert e.value.status == 1
    g.replay(1)
    fwd()
    g.torch.cuda.synchronize()
    assert g.torch.equal(A, g.ctx.ws_tensor(g.pkg.VIEW_A, 1, g.torch.float32).view_as(A))
    g.ctx.close()
