"""Mean-aggregator layers that shrink: their backward pass gathers the gradient at the output width and multiplies
[mean^T dZ | dZ] by [W_n ; W_s]^T afterwards (from 3073 rows and the second layer on)."""
import pytest

import test_gpu_parity as parity
from test_gpu_products import _loops

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [0.5, 1.0, 0.0])
@pytest.mark.parametrize("graph", ["e-narrow", "e-narrow2"], ids=["101-7", "512-101"])
def test_against_oracle(graph, p):
    """The last layer on 20000 rows with a hub of 600 entries: dZ in rows padded to 8 and 104 floats, products of one depth step and of several, with
    the boundary rows' behind them."""
    case = parity._Case.get(graph, 1, 1), p, 7
    d_in, d_out = case[0].w.dims[-2:]
    assert 8 * d_out <= 7 * d_in and case[0].w.part.n_in > 3072
    parity.test_layers_with_oracle_activations(case)
    parity.test_train_step_end_to_end(case)


@pytest.mark.parametrize("huge", [False, True], ids=["normal", "huge"])
@pytest.mark.parametrize("n,d_in,d_out", [(3073, 130, 66), (3137, 9, 3), (4000, 33, 32), (4000, 33, 28), (5000, 64, 47), (20001, 128, 96), (3200, 301, 100)],
                         ids=lambda v: str(v))
def test_products(n, d_in, d_out, huge):
    """Without neighbours only dZ W_s^T is left: every element against fp64, into a buffer of its own and over dZ; huge: a value that
    the split cannot hold.  (33 -> 32 shrinks by less than an eighth and multiplies first, as an output over dZ does.)"""
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(n + d_in)
    f32 = lambda *s: torch.randn(*s, device=dev, generator=gen)  # noqa: E731
    i32 = lambda k: torch.zeros(k, dtype=torch.int32, device=dev)  # noqa: E731
    ctx = pkg.Context(_loops(n), [8, d_in, d_out], 0, device=dev, layer_kind=1)
    kept, remap, n_kept, nnz = i32(1), i32(1), i32(1), i32(1)
    ctx.sample_boundary(1, 0, 0.5, kept, remap, n_kept)
    csr = i32(n + 1), i32(n), i32(n + 1), i32(n)
    ctx.build_sampled_csr(remap, kept, n_kept, *csr, nnz)
    W, X, A = f32(2 * d_in, d_out), f32(n, d_in), f32(n, d_in)
    shared = torch.zeros(n * d_in, device=dev)
    dZ = shared[:n * d_out].view(n, d_out).copy_(f32(n, d_out))
    W.clamp_(-0.9, 0.9)
    if huge:
        dZ[n // 2] = 0.0
        dZ[n // 2, d_out - 1] = 3.4e38
    ref, size = dZ.double() @ W[d_in:].double().t(), dZ.double().abs() @ W[d_in:].double().abs().t()
    dW, dX = torch.zeros_like(W), torch.full((n, d_in), 7.0, device=dev)
    for out in (dX, shared.view(n, d_in)):    # the second in the place of dZ
        ctx.gcn_layer_bwd(2, 0.5, dZ, None, A, X, W, dW, out, None)
        torch.cuda.synchronize()
        over = (out.double() - ref).abs() / (4.0 * 2.0 ** -24 * (1 + d_out ** 0.5) * size + 1e-300)
        assert over.max() <= 1.0, f"{over.max().item():.3g} of the allowance"
    ctx.close()
