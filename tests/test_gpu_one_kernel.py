"""Layers that aggregate and update in one kernel, at the sizes from which a step runs them so, and one row below."""
import pytest

import test_gpu_parity as parity
from edge_workloads import star_wide
from test_gpu_products import _loops

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,kind,layers", [("e-starw-large", 0, [1, 2]), ("e-dense-large", 0, [1]), ("e-dense-large", 1, [1, 3])],
                         ids=["star-gcn", "dense-gcn", "dense-sage"])
def test_one_kernel_layers_against_oracle(name, kind, layers):
    c = parity._Case.get(name, 1, kind)
    plans = [c.ctx.layer_plan(l) for l in range(1, c.w.n_layers + 1)]
    assert [l for l, k in enumerate(plans, 1) if k == c.pkg.LAYER_ONE_KERNEL] == layers, plans
    parity.test_layers_with_oracle_activations((c, 0.5, 4))
    parity.test_train_step_end_to_end((c, 0.5, 4))
    parity.test_train_step_with_cached_input_aggregate((c, 0.5, 4))


def test_one_kernel_layer_with_dropout():
    parity.test_dropout_against_oracle("e-dense-large", 1, 0, 0.3)


@pytest.mark.parametrize("make,first", [(_loops, 32768), (lambda n: star_wide(n).part, 98304)], ids=["short-rows", "long-rows"])
def test_rows_from_which_a_layer_is_one_kernel(make, first):
    import torch
    import paper_2203_10983_amd as pkg
    dev = torch.device("cuda:0")
    for n, plan in ((first - 1, pkg.LAYER_TWO_KERNELS), (first, pkg.LAYER_ONE_KERNEL)):
        part = make(n)
        ctx = pkg.Context(part, [100, 128, 5], 0, device=dev)
        assert ctx.layer_plan(1) == plan, n
        ctx.close()
