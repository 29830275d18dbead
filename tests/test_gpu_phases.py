"""Phase timers (bns_profile_enable): every phase of a step is recorded, and timing changes no result."""
import pytest

from bns_inputs import SAMPLING_SEED, make_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg,scale", [(1, 1), (3, 32)], ids=["tiny", "cfg3-s32"])
def test_timed_step_equals_untimed_step(cfg, scale):
    import torch
    import paper_2203_10983_amd as pkg
    w, dev = make_workload(cfg, scale=scale), torch.device("cuda:0")
    ctx = pkg.Context(w.part, w.dims, w.loss_kind, device=dev)
    put = lambda a: torch.from_numpy(a.copy()).to(dev)  # noqa: E731
    X, halo_h, labels = put(w.X), [put(h) for h in w.halo_h], put(w.labels)

    def step(mask):
        W = [put(x) for x in w.W]
        dW, loss = [torch.empty_like(x) for x in W], torch.zeros(1, device=dev)
        ctx.profile_enable(mask, 256)
        for epoch in range(2):
            ctx.train_step(SAMPLING_SEED, epoch, 0.5, X, halo_h, labels, W, dW, None, loss, 1e-3)
        torch.cuda.synchronize()
        phases = ctx.profile_read()
        ctx.profile_enable(0, 0)
        return W + dW + [loss], phases

    plain, none = step(0)
    timed, phases = step(0xFFFFFFFF)
    assert all(torch.equal(a, b) for a, b in zip(plain, timed))
    assert all(n == 0 for _, n in none.values())
    for name in ("sample", "spmm_fwd", "loss", "gemm_dw", "gemm_da", "spmm_bwd", "sgd"):
        assert phases[name][1] >= 2 and phases[name][0] > 0.0, name
    assert phases["sgd"][1] == 2 and phases["sample"][1] == 2
    ctx.close()
