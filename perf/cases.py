"""The work whose speed matters to a user of this package, as cases that can be timed.

A case is a table (node factors n1..n3, dimension factors d1..d3, TT rank r), a minibatch (its size
and how its ids are distributed), and what is done with it (`mode`):

  train       forward + backward_update, every step doing its own index work
  lookahead   the training loop with look-ahead: forward of batch k, prepare of batch k+2,
              backward_update of batch k, over three rotating batches
  eval        forward_eval: lookup only
  static      tt_emb_lookup_static: lookup without a handle or a workspace (serving loops)
  table       materialize: consecutive rows of the dense table

Table shapes, ranks, batch sizes and id distributions are those of `workloads.CONFIGS` and of the
rank sweep measured beside them, ranks 4 to 128, tables of 1,000 to 120 million nodes, batches of
one to 500,000 ids.

Cores are i.i.d. N(0, 1/r) (0.1^2 for the smallest table); upstream gradients are normal, scaled so
that the first step moves the cores by a few per cent.  The learning rate decays with the square of
the step number: the same gradients are applied thousands of times when a case is timed, and this
keeps the cores finite while every step runs the same instructions.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2206_10581_amd as tt

FLAG_IDS_READY = 4          # the ids are complete in device memory when prepare is called


def _case(name, mode, n, d, r, batch, ids, s=0.0, opt="sgd", reindex=False, max_batch=0, first=0):
    c = {"mode": mode, "n1": n[0], "n2": n[1], "n3": n[2], "d1": d[0], "d2": d[1], "d3": d[2], "r": r,
         "batch": batch, "ids": ids, "s": s, "opt": opt, "reindex": reindex,
         "max_batch": max_batch or batch, "first": first}
    return dict(c, name=name) if name else c


def listed():
    return [
        # a toy table (the first configuration): launches and host time count, nothing else
        _case("tiny_step", "train", (10, 10, 10), (2, 2, 2), 4, 256, "uniform"),
        # a serving request of a thousand ids against a mid-sized table: latency
        _case("serve_static", "static", (136, 136, 136), (4, 4, 8), 32, 1025, "zipf", 1.1),
        # ogbn-arxiv's own factorisation (d1 = 8), a sampled-neighbourhood minibatch
        _case("arxiv_step", "train", (55, 55, 56), (8, 4, 4), 16, 50_000, "uniform"),
        # a 175k-node graph, width 64, trained with Adam
        _case("small_adam", "train", (56, 56, 56), (4, 4, 4), 16, 50_000, "uniform", opt="adam"),
        # the default benchmark: 2.5M nodes, rank 32, degree-skewed minibatch of 200,000 ids
        _case("zipf_step", "train", (136, 136, 136), (4, 4, 8), 32, 200_000, "zipf", 1.1),
        # the same as the look-ahead loop the benchmark leads with
        _case("zipf_lookahead", "lookahead", (136, 136, 136), (4, 4, 8), 32, 200_000, "zipf", 1.1),
        # a 111M-node graph at rank 16, half a million ids, trained with Adagrad
        _case("large_adagrad", "train", (480, 480, 482), (4, 4, 8), 16, 500_000, "zipf", 1.0,
              opt="adagrad"),
        # the same graph in partition order at rank 64: 500 blocks of 1,000 neighbouring ids
        _case("clusters_step", "train", (480, 480, 482), (4, 4, 8), 64, 500_000, "clusters"),
        # ogbn-products' own factorisation: dimension factors that are not multiples of four
        _case("products_step", "train", (125, 140, 140), (4, 5, 5), 32, 200_000, "zipf", 1.1),
        # inference over ogbn-papers100M's factorisation with renumbered nodes, an odd batch
        _case("papers_eval", "eval", (480, 500, 500), (8, 4, 4), 16, 499_999, "zipf", 1.0,
              reindex=True),
        # evaluation over all nodes: a long run of table rows, produced 200,000 at a time
        _case("table_rows", "table", (136, 136, 136), (4, 4, 8), 32, 600_001, "rows",
              max_batch=200_000, first=12_345),
        # the top of the rank sweep on ogbn-papers100M's factorisation
        _case("papers_rank128", "train", (480, 500, 500), (8, 4, 4), 128, 500_000, "zipf", 1.0),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


# what a drawn case may cost at most (flops of a step if every id and prefix were distinct): below
# the largest listed case; shapes that are not multiples of four run at a lower rate
_FLOPS_MOST, _FLOPS_MOST_RAGGED = 450e9, 50e9


def draw(rng):
    mode = rng.choices(["train", "lookahead", "eval", "static", "table"], [9, 3, 4, 2, 2])[0]
    d = rng.choice([(4, 4, 8), (4, 4, 8), (4, 4, 4), (8, 4, 4), (8, 4, 4), (4, 5, 5), (2, 2, 2)])
    if d == (2, 2, 2):
        r, N = 4, _log_uniform(rng, 1e3, 1e5)
    else:
        r, N = rng.choice([8, 16, 16, 32, 32, 64, 128]), _log_uniform(rng, 1e4, 1.2e8)
    root = N ** (1 / 3)
    n = [max(4, min(600, round(root * rng.uniform(0.85, 1.15)))) for _ in range(3)]
    n12, total = n[0] * n[1], n[0] * n[1] * n[2]
    ids, s = rng.choice([("uniform", 0.0), ("zipf", round(rng.uniform(0.8, 1.2), 2)),
                         ("zipf", round(rng.uniform(0.8, 1.2), 2)), ("clusters", 0.0)])
    opt = rng.choice(["sgd", "sgd", "sgd", "adagrad", "adam"]) if mode in ("train", "lookahead") else "sgd"
    reindex = mode in ("train", "eval") and rng.random() < 0.25
    batch, max_batch, first = int(_log_uniform(rng, 200, 500_000)), 0, 0
    if mode == "static":                      # the request has to fit the library's 64 MiB scratch
        per_id = 200 * max(1, d[0] // 4) + 4 * d[0] * d[1] * r
        batch = int(_log_uniform(rng, 1, min(50_000, (40 << 20) // per_id)))
        max_batch = 1 << 20
    elif mode == "table":
        ids, s = "rows", 0.0
        batch = int(_log_uniform(rng, 500, min(total, 1_000_000)))
        max_batch = max(500, int(batch * rng.uniform(0.2, 1.2)))
        first = rng.randrange(0, total - batch + 1)
    f1, f2 = 2 * d[0] * r * d[1] * r, 2 * d[0] * d[1] * r * d[2]
    most = _FLOPS_MOST if d[1] % 4 == 0 else _FLOPS_MOST_RAGGED
    while 3 * (min(batch, n12) * f1 + batch * f2) > most:
        batch = batch * 3 // 4
    return _case(None, mode, n, d, r, batch, ids, s, opt, reindex, max_batch, first)


# ---- inputs

def _ids(case, seed):
    """int64 ids of one minibatch, made on the host (they are small)."""
    N, B = case["n1"] * case["n2"] * case["n3"], case["batch"]
    rng = np.random.default_rng(seed)
    if case["ids"] == "rows":
        return np.arange(case["first"], case["first"] + B, dtype=np.int64)
    if case["ids"] == "uniform":
        return rng.integers(0, N, size=B, dtype=np.int64)
    if case["ids"] == "zipf":
        # bounded power law: the inverse of the continuous distribution function, rounded down,
        # ranks scattered over the table by an affine bijection
        s, u = case["s"], rng.random(B)
        if abs(s - 1.0) < 1e-9:
            k = np.exp(u * math.log(N + 1.0))
        else:
            k = np.power(1.0 + u * (math.pow(N + 1.0, 1.0 - s) - 1.0), 1.0 / (1.0 - s))
        rank = np.clip(k.astype(np.int64) - 1, 0, N - 1)
        a = int(rng.integers(N // 3, N // 2))
        while math.gcd(a, N) != 1:
            a += 1
        return (rank * a + int(rng.integers(0, N))) % N
    # clusters: runs of a thousand draws from blocks of a thousand neighbouring ids
    length = min(1000, N)
    blocks = -(-B // 1000)
    starts = rng.integers(0, N - length + 1, size=blocks, dtype=np.int64)
    return (np.repeat(starts, 1000)[:B] + rng.integers(0, length, size=B, dtype=np.int64))


def prepare(case, seed):
    dev = torch.device("cuda:0")
    n = (case["n1"], case["n2"], case["n3"])
    d = (case["d1"], case["d2"], case["d3"])
    r, B, mode = case["r"], case["batch"], case["mode"]
    D, N = d[0] * d[1] * d[2], n[0] * n[1] * n[2]
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed * 2 + 1)
    std = 0.1 if r == 4 else 1 / math.sqrt(r)
    cores = [torch.randn(shape, generator=gen, device=dev) * std
             for shape in ((n[0], d[0], r), (n[1], r, d[1], r), (n[2], r, d[2]))]
    batches = 3 if mode == "lookahead" else 1
    ids = [torch.from_numpy(_ids(case, [seed, j])).to(dev) for j in range(batches)]
    out = [torch.empty((B, D), dtype=torch.float32, device=dev) for _ in range(batches)]
    state = {"mode": mode, "ids": ids, "out": out, "step": 0, "first": case["first"], "batch": B}
    if mode == "static":
        # a serving program keeps the configuration and the cores, nothing else
        state["cfg"] = tt.binding.make_config(n, d, (r, r), case["max_batch"])
        state["cores"] = cores
        rc = tt.tt_emb_lookup_static(state["cfg"], *(c.data_ptr() for c in cores), 0, 0, 0,
                                     torch.cuda.current_stream().cuda_stream)
        if rc:
            raise tt.TTEmbError(rc, "tt_emb_lookup_static")
        return state
    emb = tt.TTEmbedding(n, d, (r, r), case["max_batch"], cores, device=dev,
                         flags=FLAG_IDS_READY if mode == "lookahead" else 0)
    state["emb"] = emb
    if case["reindex"]:
        # nodes renumbered over the whole table by a bijection
        a = N // 2 + 1 + seed % 1000
        while math.gcd(a, N) != 1:
            a += 1
        table = torch.arange(N, device=dev, dtype=torch.int64)
        emb.set_reindex(table.mul_(a).remainder_(N).to(torch.int32))
    if mode in ("train", "lookahead"):
        if case["opt"] == "adam":
            emb.set_adam()
        elif case["opt"] == "adagrad":
            emb.set_adagrad()
        scale = math.sqrt(min(1.0, n[2] / B))
        state["grad"] = [torch.randn((B, D), generator=gen, device=dev) * scale for _ in range(batches)]
    if mode == "lookahead":
        torch.cuda.synchronize()
        emb.prepare(ids[0])
        emb.prepare(ids[1])
    return state


def _trained(state, k):
    emb = state["emb"]
    got = {"rows": state["out"][k], "cores": emb.cores}
    if getattr(emb, "adagrad_state", None):
        got["sums"] = emb.adagrad_state
    if getattr(emb, "adam_state", None):
        got["moments"] = emb.adam_state
    return got


def run(state):
    mode, step = state["mode"], state["step"]
    ids, out = state["ids"], state["out"]
    if mode == "static":
        cores = state["cores"]
        rc = tt.tt_emb_lookup_static(state["cfg"], cores[0].data_ptr(), cores[1].data_ptr(),
                                     cores[2].data_ptr(), ids[0].data_ptr(), state["batch"],
                                     out[0].data_ptr(), torch.cuda.current_stream().cuda_stream)
        if rc:
            raise tt.TTEmbError(rc, "tt_emb_lookup_static")
        return out[0]
    emb = state["emb"]
    if mode == "eval":
        return emb.forward_eval(ids[0], out[0])
    if mode == "table":
        return emb.materialize(state["first"], state["batch"], out[0])
    state["step"] = step + 1
    lr = 0.01 / (1 + step) ** 2
    if mode == "lookahead":
        k = step % 3
        emb.wait_backward(1)
        emb.forward(ids[k], out[k])
        emb.prepare(ids[(k + 2) % 3])
        emb.backward_update(state["grad"][k], lr)
        return _trained(state, k)
    emb.forward(ids[0], out[0])
    emb.backward_update(state["grad"][0], lr)
    return _trained(state, 0)


def work(case):
    """Ids in, rows out (and gradients in); the touched core slices and their optimiser state once
    each way; one prefix product per distinct (i1,i2), one row product per distinct id, and twice
    those in the backward pass."""
    n1, n2, n3 = case["n1"], case["n2"], case["n3"]
    d1, d2, d3, r, B = case["d1"], case["d2"], case["d3"], case["r"], case["batch"]
    D = d1 * d2 * d3
    u = np.unique(_ids(case, [0, 0]))
    if case["reindex"]:                    # distinct prefixes are counted on the renumbered rows
        N = n1 * n2 * n3
        a = N // 2 + 1
        while math.gcd(a, N) != 1:
            a += 1
        u = np.unique(u * a % N)
    q = np.unique(u // n3)
    touched = 4 * (np.unique(q // n2).size * d1 * r + np.unique(q % n2).size * r * d2 * r
                   + np.unique(u % n3).size * r * d3)
    once = int(q.size) * 2 * d1 * r * d2 * r + int(u.size) * 2 * d1 * d2 * r * d3
    ids_bytes = 0 if case["mode"] == "table" else (12 if case["reindex"] else 8) * B
    if case["mode"] not in ("train", "lookahead"):
        return {"bytes": ids_bytes + 4 * D * B + touched, "flops": once}
    state = {"sgd": 0, "adagrad": 1, "adam": 2}[case["opt"]]
    return {"bytes": ids_bytes + 8 * D * B + (2 + 2 * state) * touched,
            "flops": 3 * once + (B - int(u.size)) * D}


def tolerance(case):
    # fp32 products and sums in another order.  The first step of an adaptive rule moves an entry by
    # the learning rate times the sign of its gradient: an entry whose gradient cancels to nothing
    # may move either way (2 * 0.01 over cores of 1/sqrt(r)), which only the largest difference sees.
    if case["opt"] in ("adam", "adagrad"):
        return {"rel": 1e-5, "max": 0.3}
    return {"rel": 1e-5, "max": 2e-4}
