"""What a program that trains with this framework has it do, as cases to be timed.

A case is one partition (a power-law graph's share, or an even one), a model on it, and how the
program drives the library:

  mode "step"    one training iteration: bns_train_step, with its own SGD update (optim "sgd") or
                 followed by Adam on every weight (optim "adam")
  mode "replay"  the epoch loop as a captured HIP graph, `epochs` iterations in one call
  mode "layers"  a program with a loop of its own: sample, induced subgraph, every layer forward,
                 every layer backward through the separate entry points

Every pass is the next epoch, so it draws another boundary sample.  Sizes and widths are those of
the five configurations of bns_inputs/workloads.py, of the scaled copies and of the odd widths that
the tests run.
"""
import functools
import math
import types

import numpy as np
import torch

import paper_2203_10983_amd as bns

SEED = 2203
SGD_PER_NODE = 0.01     # the loss is a sum over the nodes: the rate is divided by their number
ADAM_RATE = 1e-3

# ------------------------------------------------------------------------------------------------
# n_in inner nodes with deg_in inner neighbours each on average, n_halo boundary nodes, deg_bd
# boundary entries per inner node, tail exponent of the degree distribution (0: all nodes alike).
TINY = dict(n_in=500, n_halo=330, deg_in=2.5, deg_bd=0.75, exponent=0.0)
SMALL = dict(n_in=9570, n_halo=23300, deg_in=45.0, deg_bd=4.8, exponent=2.3)
DENSE = dict(n_in=29125, n_halo=197758, deg_in=416.0, deg_bd=73.0, exponent=2.1)
MEDIUM = dict(n_in=306250, n_halo=746157, deg_in=45.0, deg_bd=4.8, exponent=2.3)
WIDE = dict(n_in=89625, n_halo=211570, deg_in=16.0, deg_bd=4.0, exponent=2.5)
LARGE = dict(n_in=578125, n_halo=3080688, deg_in=21.0, deg_bd=7.3, exponent=2.2)
ODD = dict(n_in=20011, n_halo=30011, deg_in=14.0, deg_bd=4.0, exponent=2.5)


def _case(name, part, dims, layer="gcn", loss="ce", p=0.1, dropout=0.0, optim="sgd", mode="step", epochs=1, cached=False):
    c = dict(part, dims=dims, layer=layer, loss=loss, p=p, dropout=dropout, optim=optim, mode=mode, epochs=epochs, cached=cached)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest configuration, one call per epoch: latency and launches
        _case("tiny-step", TINY, "64,16,8"),
        # the same as a program runs many epochs of it: the captured loop
        _case("tiny-replay10", TINY, "64,16,8", mode="replay", epochs=10),
        # a partition of a small graph, as the quick parity runs have it
        _case("small-step", SMALL, "100,128,128,47"),
        # a program's own loop over the layer entry points, widths that are no multiple of 4
        _case("odd-layers", ODD, "602,130,66,9", p=0.5, optim="none", mode="layers"),
        # long rows (hundreds of neighbours), wide first layer, at the usual sampling rate
        _case("dense-p01", DENSE, "602,256,256,256,41"),
        # the same without sampling: the baseline that every user of the method runs beside it
        _case("dense-p1", DENSE, "602,256,256,256,41", p=1.0),
        # medium rows, narrow odd output
        _case("medium-gcn", MEDIUM, "100,128,128,47"),
        # the paper's own model and training set-up: mean aggregator, dropout, Adam
        _case("medium-sage-adam", MEDIUM, "100,128,128,47", layer="sage", dropout=0.3, optim="adam"),
        # many labels per node, wide layers: the dense products weigh most
        _case("wide-bce", WIDE, "300,512,512,512,100", loss="bce"),
        # the same with the concatenated update (products of twice the depth)
        _case("wide-sage-bce", WIDE, "300,512,512,512,100", layer="sage", loss="bce", dropout=0.1),
        # the largest share: what the benchmark's headline runs
        _case("large-gcn", LARGE, "128,128,128,172"),
        # the largest share with the mean aggregator and the input aggregate kept between epochs
        _case("large-sage-cached", LARGE, "128,128,128,172", layer="sage", p=0.1, cached=True),
    ]


def _between(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    top = max(_cost(c) for c in listed())
    while True:
        n_in = int(round(_between(rng, 400, 580000)))
        deg_in = round(min(_between(rng, 2.5, 420), n_in / 16), 2)
        deg_bd = round(deg_in * _between(rng, 0.1, 0.4), 3)
        part = dict(n_in=n_in, n_halo=max(1, int(n_in * deg_bd * _between(rng, 0.1, 0.75))), deg_in=deg_in, deg_bd=deg_bd,
                    exponent=rng.choice((0.0, 2.1, 2.2, 2.3, 2.5)))
        loss = rng.choice(("ce", "ce", "bce"))
        hidden = rng.choice((16, 66, 100, 128, 130, 256, 512))
        dims = [rng.choice((64, 100, 128, 300, 602))] + [hidden] * rng.randint(1, 3) + [rng.choice((8, 9, 41, 47, 100, 172))]
        mode = rng.choice(("step", "step", "step", "replay", "layers"))
        c = _case(None, part, ",".join(map(str, dims)), layer=rng.choice(("gcn", "gcn", "sage")), loss=loss,
                  p=rng.choice((0.01, 0.1, 0.1, 0.5, 1.0)), mode=mode,
                  dropout=0.0 if mode == "layers" else rng.choice((0.0, 0.0, 0.3, 0.5)),
                  optim="none" if mode == "layers" else "sgd" if mode == "replay" else rng.choice(("sgd", "adam")),
                  epochs=rng.randint(2, 10) if mode == "replay" and n_in < 20000 else 1,
                  cached=mode != "layers" and rng.random() < 0.25)
        if _cost(c) <= top and sum(_entries(c)) <= sum(_entries(LARGE)):
            return c


# ------------------------------------------------------------------------------------------------
def _dims(case):
    return [int(x) for x in case["dims"].split(",")]


def _entries(case):
    """(inner entries with the self-loops, boundary entries) as drawn: repeated edges of the hubs collapse."""
    n = case["n_in"]
    return n * (1 + case["deg_in"]), max(case["n_halo"], n * case["deg_bd"])


def _cost(case):
    """Of one pass, in floats moved per row and entry: keeps a drawn case within the largest listed one."""
    d, (e_in, e_bd) = _dims(case), _entries(case)
    wide = 2 if case["layer"] == "sage" else 1
    nnz = e_in + case["p"] * e_bd
    agg = nnz * (2 * sum(d) - d[0] - d[-1])
    prod = sum(3 * wide * case["n_in"] * a * b for a, b in zip(d, d[1:])) / 12
    held = case["n_halo"] * 8 * sum(d[:-1])  # features and gradients of all boundary nodes
    return case["epochs"] * (agg + prod) + held


def work(case):
    d, (e_in, e_bd) = _dims(case), _entries(case)
    n, kept, L = case["n_in"], case["p"] * case["n_halo"], len(d) - 1
    nnz = e_in + case["p"] * e_bd
    wide = 2 if case["layer"] == "sage" else 1
    weights = sum(wide * a * b for a, b in zip(d, d[1:]))
    # inputs: graph, gids, degrees, features, the kept boundary rows, labels, weights
    b = 4 * (e_in + 2 * e_bd + 3 * n) + 16 * case["n_halo"] + 4 * n * d[0] + 4 * kept * sum(d[:-1])
    b += n * (d[-1] if case["loss"] == "bce" else 4) + 4 * weights
    # outputs: the subgraph and its transpose, logits, weight gradients, gradients of the boundary rows, weights
    b += 8 * nnz + 4 * n * d[-1] + 4 * weights + 4 * kept * sum(d[1:-1])
    b += {"sgd": 4, "adam": 20, "none": 0}[case["optim"]] * weights
    # products: forward, weight gradient, input gradient (not of the first layer); aggregates both ways
    f = sum((3 if l else 2) * 2 * wide * n * d[l] * d[l + 1] for l in range(L))
    f += sum((2 if l else 1) * 2 * nnz * min(d[l], d[l + 1]) for l in range(L))
    return {"bytes": case["epochs"] * b, "flops": case["epochs"] * f}


def tolerance(case):
    # Everything is fp32.  A chain of two layers or more has hidden units whose pre-activation lies within rounding of
    # zero, about one in ten million: another order of summation switches them, and with each the gradient of that unit.
    # Of n such units k switched ones change a gradient by about sqrt(k / n).  One whole unit of one node shows in the
    # few boundary rows next to it.  Adam divides a gradient by its own size: an element that cancels to rounding may
    # step the other way.
    return {"rel": 1e-3, "max": 0.5}


# ------------------------------------------------------------------------------------------------
def _weights(gen, n, exponent, mean):
    """Node weights of a Chung-Lu graph: a Pareto tail cut at sqrt(total), scaled to `mean`."""
    if exponent == 0.0:
        return torch.full((n,), mean, dtype=torch.float64, device="cuda")
    w = (1.0 - torch.rand(n, generator=gen, dtype=torch.float64, device="cuda")) ** (-1.0 / (exponent - 1.0))
    for _ in range(4):
        w = (w * (mean / w.mean())).clamp_(max=max(mean, math.sqrt(n * mean) * 4))
    return w


def _partition(case, gen):
    """The arrays of one partition as a partitioner hands them over (host arrays), drawn on the GPU."""
    n, nb = case["n_in"], case["n_halo"]
    rand = lambda m: torch.rand(m, generator=gen, dtype=torch.float64, device="cuda")  # noqa: E731
    cdf = torch.cumsum(_weights(gen, n, case["exponent"], case["deg_in"]), 0)
    node = lambda m: torch.searchsorted(cdf, rand(m) * cdf[-1], right=True).clamp_(max=n - 1)  # noqa: E731
    a, b = node(int(n * case["deg_in"] / 2)), node(int(n * case["deg_in"] / 2))
    # boundary entries: every boundary node has one, the rest fall on them by weight
    m_bd = max(nb, int(n * case["deg_bd"]))
    bw = _weights(gen, nb, case["exponent"], m_bd / nb)
    bcdf = torch.cumsum(bw, 0)
    bd = torch.cat([torch.arange(nb, device="cuda"), torch.searchsorted(bcdf, rand(m_bd - nb) * bcdf[-1], right=True).clamp_(max=nb - 1)])
    rows_bd = node(m_bd)
    cols = n + nb
    loop = torch.arange(n, device="cuda")
    key = torch.unique(torch.cat([a * cols + b, b * cols + a, loop * (cols + 1), rows_bd * cols + n + bd]))
    row, col = key // cols, key % cols

    def ptr(of, m):
        return torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), torch.cumsum(torch.bincount(of, minlength=m), 0)])

    def host(t, dtype=np.int32):
        return np.ascontiguousarray(t.to(torch.int64 if dtype is np.int64 else torch.int32).cpu().numpy())

    inner = col < n
    t_in = torch.sort(col[inner] * n + row[inner]).values
    h = torch.sort((col[~inner] - n) * n + row[~inner]).values
    inc = torch.bincount(h // n, minlength=nb)
    rp = ptr(row, n)
    gid = n + torch.cumsum(1 + torch.randint(0, 37, (nb,), generator=gen, device="cuda"), 0)
    full = torch.maximum((bw * (case["deg_in"] + case["deg_bd"]) * nb / m_bd).round().to(torch.int64), inc)
    P = types.SimpleNamespace(
        part_id=0, n_in=n, n_halo=nb, row_ptr0=host(rp), col0=host(col), t_in_ptr=host(ptr(t_in // n, n)), t_in_col=host(t_in % n),
        halo_ptr=host(ptr(h // n, nb)), halo_col=host(h % n), halo_gid=host(gid, np.int64), deg_in=host(rp[1:] - rp[:-1]), deg_halo=host(full + 1))
    P.nnz0, P.e_in, P.e_bd = int(P.col0.size), int(P.t_in_col.size), int(P.halo_col.size)
    return P


@functools.lru_cache(maxsize=None)
def _loop_stream():
    """The stream of the program's captured epoch loops (a capture needs a created one)."""
    return torch.cuda.Stream()


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    P, d = _partition(case, gen), _dims(case)
    n, nb, L, sage = P.n_in, P.n_halo, len(d) - 1, case["layer"] == "sage"
    f32 = dict(dtype=torch.float32, device="cuda")
    normal = lambda *shape: torch.randn(*shape, generator=gen, **f32)  # noqa: E731
    s = types.SimpleNamespace(case=case, P=P, dims=d, L=L, sage=sage, epoch=0)
    s.lr = SGD_PER_NODE / n if case["optim"] == "sgd" else 0.0
    s.X = normal(n, d[0])
    # boundary features as other partitions would send them: inputs for layer 1, activations after that
    s.halo_h = [normal(nb, d[0])] + [normal(nb, d[l]).clamp_(min=0) for l in range(1, L)]
    if case["loss"] == "bce":
        s.labels = (torch.rand(n, d[-1], generator=gen, device="cuda") < 0.05).to(torch.uint8)
    else:  # classes of falling size; a tenth of the nodes is outside the training set
        pr = torch.cumsum(1.0 / torch.arange(1, d[-1] + 1, device="cuda", dtype=torch.float64), 0)
        s.labels = torch.searchsorted(pr, torch.rand(n, generator=gen, device="cuda", dtype=torch.float64) * pr[-1]).clamp_(max=d[-1] - 1).to(torch.int32)
        s.labels[torch.rand(n, generator=gen, device="cuda") < 0.1] = -1
    s.W = []
    for a, b in zip(d, d[1:]):
        a = 2 * a if sage else a
        s.W.append((torch.rand(a, b, generator=gen, **f32) * 2 - 1) * math.sqrt(6.0 / (a + b)))
    s.dW = [torch.zeros_like(w) for w in s.W]
    s.dhalo = [None] + [torch.zeros(nb, d[l], **f32) for l in range(1, L)]
    s.loss = torch.zeros(1, **f32)
    s.ctx = bns.Context(P, d, 1 if case["loss"] == "bce" else 0, layer_kind=1 if sage else 0)
    s.ctx.set_dropout(case["dropout"])
    if case["cached"]:
        s.ctx.cache_input_aggregate(s.X)
    if case["mode"] == "layers":
        i32 = dict(dtype=torch.int32, device="cuda")
        s.kept, s.remap, s.n_kept, s.nnz = torch.zeros(nb, **i32), torch.zeros(nb, **i32), torch.zeros(1, **i32), torch.zeros(1, **i32)
        room = math.ceil(sum(_entries(case))) + 1  # entries before repeated edges collapse
        s.row_ptr, s.col = torch.zeros(n + 1, **i32), torch.zeros(room, **i32)
        s.t_row_ptr, s.t_col = torch.zeros(n + nb + 1, **i32), torch.zeros(room, **i32)
        s.A = [torch.zeros(n, d[l], **f32) for l in range(L)]
        s.H = [torch.zeros(n, d[l + 1], **f32) for l in range(L)]
        s.G = [torch.zeros(n, d[l], **f32) for l in range(L)] + [normal(n, d[L])]  # G[L]: gradient from the program's own loss
        s.out = dict(kept=s.kept, remap=s.remap, n_kept=s.n_kept, nnz=s.nnz, row_ptr=s.row_ptr, col=s.col, t_row_ptr=s.t_row_ptr,
                     t_col=s.t_col, A=s.A, H=s.H, dH=s.G[1:L], dW=s.dW, dhalo=s.dhalo[1:])
        return s
    if case["optim"] == "adam":
        s.m, s.v = [torch.zeros_like(w) for w in s.W], [torch.zeros_like(w) for w in s.W]
    view = s.ctx.ws_tensor
    s.out = dict(loss=s.loss, W=s.W, dW=s.dW, dhalo=s.dhalo[1:], remap=view(bns.VIEW_REMAP), n_kept=view(bns.VIEW_N_KEPT),
                 row_ptr=view(bns.VIEW_ROW_PTR), logits=view(bns.VIEW_H, L, torch.float32))
    if case["optim"] == "adam":
        s.out.update(m=s.m, v=s.v)
    if case["mode"] == "replay":
        s.stream = _loop_stream()
        s.stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s.stream):
            s.ctx.graph_capture(SEED, 1, case["p"], s.X, s.halo_h, s.labels, s.W, s.dW, s.dhalo, s.loss, s.lr)
        s.stream.synchronize()
    return s


def run(s):
    c, p = s.case, s.case["p"]
    s.epoch += 1
    if c["mode"] == "replay":
        with torch.cuda.stream(s.stream):
            s.ctx.graph_replay(c["epochs"])
        return s.out
    if c["mode"] == "step":
        s.ctx.train_step(SEED, s.epoch, p, s.X, s.halo_h, s.labels, s.W, s.dW, s.dhalo, s.loss, s.lr)
        if c["optim"] == "adam":
            for W, dW, m, v in zip(s.W, s.dW, s.m, s.v):
                bns.adam_update(W, dW, m, v, ADAM_RATE, t=s.epoch)
        return s.out
    s.ctx.sample_boundary(SEED, s.epoch, p, s.kept, s.remap, s.n_kept)
    s.ctx.build_sampled_csr(s.remap, s.kept, s.n_kept, s.row_ptr, s.col, s.t_row_ptr, s.t_col, s.nnz)
    for l in range(1, s.L + 1):
        H_in = s.X if l == 1 else s.H[l - 2]
        s.ctx.gcn_layer_fwd(l, p, H_in, s.halo_h[l - 1], s.W[l - 1], s.A[l - 1], s.H[l - 1], l < s.L)
    for l in range(s.L, 0, -1):
        H_in = s.X if l == 1 else s.H[l - 2]
        s.ctx.gcn_layer_bwd(l, p, s.G[l], s.H[l - 1] if l < s.L else None, s.A[l - 1], H_in, s.W[l - 1], s.dW[l - 1],
                            s.G[l - 1] if l > 1 else None, s.dhalo[l - 1])
    return s.out
