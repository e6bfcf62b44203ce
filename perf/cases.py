"""Performance cases: the work a user of this framework has it do, through its public entry points.

A case names a kind of work, the sizes of a synthetic hypergraph (sizes by a truncated power law or uniform,
members uniform or by a node popularity, as in ``synth``) and the options of the call:

* ``refine``    a multi-level refinement on a plan that is kept;
* ``stop``      the same with the early stop decided on the device;
* ``train``     forward and backward of one level's sweeps with learnable log-weights and coarse embedding;
* ``train_all`` forward and backward through a whole hierarchy;
* ``coarsen``   the coarsening of a hypergraph resident in device memory, every step;
* ``features``  the same driven by bag-of-words node features;
* ``pipeline``  the whole method from a hypergraph in device memory: coarsening, plan, refinement;
* ``score``     hyperedge-prediction features of candidate node sets on a plan that is kept.

Inputs are drawn on the GPU.  A case's sizes fix the hypergraph, its weights and its word counts up to the numbering
of the nodes, which the seed draws, like the embeddings: inputs of different seeds differ in every array, and their
coarse levels have the same sizes (which hyperedge a node joins does not depend on the nodes' numbers).  ``exact``
restates each computation in plain torch in 64 bits.
"""
import math

import torch

import paper_2103_09660_amd as H

OMEGA = 0.5


def listed():
    return [
        # a citation-sized hypergraph refined again and again (parameter studies): latency and launches count
        {"name": "refine-tiny-f32", "kind": "refine", "nodes": 2000, "edges": 1000, "zipf": 0.0, "cap": 8, "skew": 0.0,
         "weighted": False, "d": 32, "dtype": "f32", "order": "jacobi", "steps": 3, "sweeps": 10, "residuals": True},
        # the same size until it has converged, instead of a fixed number of sweeps
        {"name": "stop-tiny-f32", "kind": "stop", "nodes": 2000, "edges": 1000, "zipf": 0.0, "cap": 8, "skew": 0.0,
         "weighted": False, "d": 32, "dtype": "f32", "order": "jacobi", "steps": 3, "sweeps": 100, "tol": 2e-3},
        # a co-authorship-sized hypergraph with hub nodes and weights
        {"name": "refine-hub-200k-f32", "kind": "refine", "nodes": 200000, "edges": 100000, "zipf": 2.1, "cap": 500,
         "skew": 1.5, "weighted": True, "d": 64, "dtype": "f32", "order": "jacobi", "steps": 5, "sweeps": 20,
         "residuals": False},
        # odd sizes, a width that is no power of two, the edge-first order, 16-bit storage
        {"name": "refine-odd-150k-bf16", "kind": "refine", "nodes": 150001, "edges": 90007, "zipf": 2.1, "cap": 700,
         "skew": 0.0, "weighted": False, "d": 72, "dtype": "bf16", "order": "edge_first", "steps": 4, "sweeps": 15,
         "residuals": False},
        # the large refinement: millions of rows in 16-bit storage
        {"name": "refine-zipf-2m-bf16", "kind": "refine", "nodes": 2000000, "edges": 1500000, "zipf": 2.1, "cap": 2000,
         "skew": 0.0, "weighted": False, "d": 128, "dtype": "bf16", "order": "jacobi", "steps": 8, "sweeps": 20,
         "residuals": False},
        # one training step: a level's sweeps forward and backward, checkpointed
        {"name": "train-500k-f32", "kind": "train", "nodes": 500000, "edges": 300000, "zipf": 2.1, "cap": 1000,
         "skew": 0.0, "weighted": False, "d": 128, "dtype": "f32", "order": "jacobi", "steps": 1, "sweeps": 10,
         "ckpt": 5},
        # one training step through every level of a citation-sized hierarchy
        {"name": "train-all-20k-f32", "kind": "train_all", "nodes": 19717, "edges": 7963, "zipf": 2.1, "cap": 171,
         "skew": 0.0, "weighted": False, "d": 64, "dtype": "f32", "order": "jacobi", "steps": 4, "sweeps": 10,
         "ckpt": 5},
        # coarsening a large hypergraph, every step
        {"name": "coarsen-zipf-2m", "kind": "coarsen", "nodes": 2000000, "edges": 1500000, "zipf": 2.1, "cap": 2000,
         "skew": 0.0, "weighted": False, "steps": 8},
        # coarsening by word counts, a million documents
        {"name": "features-bow-1m", "kind": "features", "nodes": 1000000, "edges": 600000, "zipf": 2.1, "cap": 500,
         "skew": 0.0, "weighted": False, "steps": 6, "k": 512, "words_lo": 5, "words_hi": 40},
        # the whole method on a citation-sized hypergraph that arrives new
        {"name": "pipeline-20k-f32", "kind": "pipeline", "nodes": 19717, "edges": 7963, "zipf": 2.1, "cap": 171,
         "skew": 0.0, "weighted": False, "d": 64, "dtype": "f32", "order": "jacobi", "steps": 4, "sweeps": 10},
        # the whole method on a large weighted hypergraph that arrives new
        {"name": "pipeline-700k-bf16", "kind": "pipeline", "nodes": 700001, "edges": 450000, "zipf": 2.1, "cap": 1000,
         "skew": 0.0, "weighted": True, "d": 64, "dtype": "bf16", "order": "jacobi", "steps": 5, "sweeps": 10},
        # hyperedge-prediction features of a million and a half candidate sets
        {"name": "score-zipf-2m-bf16", "kind": "score", "nodes": 2000000, "edges": 1500000, "zipf": 2.1, "cap": 2000,
         "skew": 0.0, "weighted": False, "d": 128, "dtype": "bf16", "op": "variance"},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["refine", "refine", "stop", "train", "train_all", "coarsen", "features", "pipeline", "score"])
    # the largest hypergraph of each kind (the listed cases hold the larger ones)
    most = {"refine": 1000000, "stop": 100000, "train": 500000, "train_all": 100000, "coarsen": 2000000,
            "features": 400000, "pipeline": 1000000, "score": 2000000}[kind]
    nodes = _log_uniform(rng, 1500, most)
    case = {"kind": kind, "nodes": nodes, "edges": int(nodes * rng.uniform(0.35, 0.8)) | 1}
    if nodes < 5000 and rng.random() < 0.5:
        case.update(zipf=0.0, cap=rng.randint(5, 20), skew=0.0)
    else:
        case.update(zipf=rng.choice([2.0, 2.1, 2.3]), cap=min(nodes // 8, rng.randint(100, 2000)),
                    skew=rng.choice([0.0, 0.0, 0.6, 1.5]))
    case["weighted"] = rng.random() < 0.4
    if kind in ("refine", "stop", "train", "train_all", "pipeline", "score"):
        case["d"] = rng.choice([16, 32, 40, 64, 72, 96, 128] + ([200, 256] if nodes < 300000 else []))
        case["dtype"] = "f32" if kind in ("train", "train_all") else rng.choice(["f32", "bf16"])
        case["order"] = rng.choice(["jacobi", "jacobi", "edge_first"])
    if kind != "score":
        case["steps"] = 1 if kind == "train" else rng.randint(2, 6)
    if kind == "refine":
        case.update(sweeps=rng.choice([5, 10, 20]), residuals=rng.random() < 0.3)
    elif kind == "stop":
        case.update(sweeps=rng.choice([50, 80]), tol=rng.choice([1e-2, 3e-3]))
    elif kind in ("train", "train_all"):
        case.update(sweeps=rng.choice([4, 7, 10]), ckpt=rng.choice([1, 3, 5]))
    elif kind == "pipeline":
        case["sweeps"] = rng.choice([5, 10])
    elif kind == "features":
        case.update(k=rng.choice([128, 300, 500, 512]), words_lo=5, words_hi=rng.choice([20, 50]))
    elif kind == "score":
        case["op"] = rng.choice(["variance", "variance", "mean", "min", "max"])
    return case


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------

def _cdf(n, exponent, first):
    c = torch.arange(first, first + n, dtype=torch.float64, device="cuda").pow(-exponent).cumsum(0)
    return c / c[-1]


def _hypergraph(case, g, number):
    """(offsets int32, members int32, weights float32 or None), node v numbered number[v]; a member drawn twice counts
    once."""
    n, m, cap = case["nodes"], case["edges"], case["cap"]
    if case["zipf"]:
        u = torch.rand(m, generator=g, device="cuda", dtype=torch.float64)
        sizes = 2 + torch.searchsorted(_cdf(cap - 1, case["zipf"], 2), u).clamp_(max=cap - 2)
    else:
        sizes = torch.randint(2, cap + 1, (m,), generator=g, device="cuda")
    row = torch.repeat_interleave(torch.arange(m, device="cuda"), sizes)
    if case["skew"]:
        perm = torch.randperm(n, generator=g, device="cuda")
        u = torch.rand(row.numel(), generator=g, device="cuda", dtype=torch.float64)
        node = perm[torch.searchsorted(_cdf(n, case["skew"], 1), u).clamp_(max=n - 1)]
    else:
        node = torch.randint(0, n, (row.numel(),), generator=g, device="cuda")
    key = (row * n + number[node]).sort().values
    key = key[torch.cat([torch.ones(1, dtype=torch.bool, device="cuda"), key[1:] != key[:-1]])]
    row = key // n
    ptr = torch.zeros(m + 1, dtype=torch.int64, device="cuda")
    ptr[1:] = torch.bincount(row, minlength=m).cumsum(0)
    w = torch.rand(m, generator=g, device="cuda") * 1.5 + 0.5 if case["weighted"] else None
    return ptr.int(), (key - row * n).int(), w


def _words(case, g, number):
    """Bag-of-words counts: a few distinct words a document by a Zipf word popularity, each 1 to 3 times, 2% empty
    documents and 5% copies of another document."""
    n, k = case["nodes"], case["k"]
    words = torch.randint(case["words_lo"], case["words_hi"] + 1, (n,), generator=g, device="cuda")
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), words)
    u = torch.rand(row.numel(), generator=g, device="cuda", dtype=torch.float64)
    perm = torch.randperm(k, generator=g, device="cuda")
    slot = row * k + perm[torch.searchsorted(_cdf(k, 1.1, 1), u).clamp_(max=k - 1)]
    counts = 1 + slot * 2654435761 % 2147483647 % 3     # by the slot, so that a word drawn twice has one count
    x = torch.zeros(n * k, dtype=torch.int32, device="cuda")
    x[slot] = counts.int()
    x = x.view(n, k)
    x[torch.rand(n, generator=g, device="cuda") < 0.02] = 0
    copies = (torch.rand(n, generator=g, device="cuda") < 0.05).nonzero().squeeze(1)
    x[copies] = x[torch.randint(0, n, (copies.numel(),), generator=g, device="cuda")]
    return torch.empty_like(x).index_copy_(0, number, x)


def _inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    number = torch.randperm(case["nodes"], generator=g, device="cuda")
    return (g, number) + _hypergraph(case, _of_sizes(case), number)


def _of_sizes(case):
    return torch.Generator(device="cuda").manual_seed(case["nodes"] * 1000003 + case["edges"])


def _normal(g, rows, d, dtype):
    z = torch.randn(rows, d, generator=g, device="cuda")
    return z.to(torch.bfloat16) if dtype == "bf16" else z


def _options(case):
    return {"order": case["order"]} if case["order"] != "jacobi" else None


def _rows(level):
    return level.n_nodes + level.n_edges


def prepare(case, seed):
    g, number, ptr, idx, w = _inputs(case, seed)
    kind = case["kind"]
    if kind == "score":
        plan = H.ScorePlan.from_device(ptr, idx, case["nodes"], case["d"], case["dtype"])
        return {"case": case, "plan": plan, "z": _normal(g, case["nodes"], case["d"], case["dtype"])}
    level = H.DeviceLevel(case["nodes"], case["edges"], idx.numel(), ptr, idx, w)
    state = {"case": case, "level": level}
    if kind == "features":
        state["x"] = _words(case, _of_sizes(case), number)
        return state
    if kind == "coarsen":
        return state
    levels, maps = H.coarsen_hierarchy_device(level, case["steps"])
    state["z"] = _normal(g, _rows(levels[-1]), case["d"], case["dtype"])
    state["sweeps"] = [case["sweeps"]] * len(levels)
    if kind == "pipeline":
        return state        # its levels and plan are part of the pass
    state["plan"] = H.Plan.from_device(levels, maps, case["d"], case["dtype"], _options(case))
    if kind == "stop":
        state["tol"] = case["tol"] * math.sqrt(_rows(level) * case["d"])
    if kind in ("train", "train_all"):
        state["z"].requires_grad_(True)
        state["thetas"] = _thetas(g, levels if kind == "train_all" else levels[:1])
        state["g"] = torch.randn(_rows(level), case["d"], generator=g, device="cuda")
    return state


def _thetas(g, levels):
    return [(0.2 * torch.randn(lv.n_edges, generator=g, device="cuda")).requires_grad_(True) for lv in levels]


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "refine":
        z, res, _ = state["plan"].refine(state["z"], state["sweeps"], OMEGA, residuals=case["residuals"])
        return (z, res) if case["residuals"] else z
    if kind == "stop":
        z, _, done = state["plan"].refine(state["z"], state["sweeps"], OMEGA, tol=state["tol"])
        return z, done
    if kind == "train":
        theta = state["thetas"][0]
        out = H.refine_level(state["z"], theta, state["plan"], 0, case["sweeps"], OMEGA, from_coarse=True,
                             ckpt_every=case["ckpt"])
        return [out] + list(torch.autograd.grad(out, [state["z"], theta], state["g"]))
    if kind == "train_all":
        out = H.refine_hierarchy(state["z"], state["thetas"], state["plan"], state["sweeps"], OMEGA,
                                 ckpt_every=case["ckpt"])
        return [out] + list(torch.autograd.grad(out, [state["z"]] + state["thetas"], state["g"]))
    if kind == "coarsen":
        levels, maps = H.coarsen_hierarchy_device(state["level"], case["steps"])
        return [[lv.edge_ptr, lv.edge_idx] + ([] if lv.edge_w is None else [lv.edge_w]) for lv in levels[1:]], maps
    if kind == "features":
        levels, maps, feats = H.coarsen_hierarchy_features_device(state["level"], state["x"], case["steps"])
        return [[lv.edge_ptr, lv.edge_idx] for lv in levels[1:]], maps, feats[1:]
    if kind == "pipeline":
        levels, maps = H.coarsen_hierarchy_device(state["level"], case["steps"])
        plan = H.Plan.from_device(levels, maps, case["d"], case["dtype"], _options(case))
        z, _, _ = plan.refine(state["z"], state["sweeps"], OMEGA)
        return z, maps
    return state["plan"].score(state["z"], case["op"])


# ----------------------------------------------------------------------------
# the work of a pass
# ----------------------------------------------------------------------------

def work(case):
    """Each sweep reads the level's matrix and adjacency once and writes the matrix once; each coarsening step reads
    a level once and writes the next.  Level sizes are estimates (a step keeps about three quarters of the rows and
    nine tenths of the incidences); a member drawn twice is not taken off."""
    n, m, cap = case["nodes"], case["edges"], case["cap"]
    if case["zipf"]:
        p = [k ** -case["zipf"] for k in range(2, cap + 1)]
        mean = sum(k * q for k, q in enumerate(p, 2)) / sum(p)
    else:
        mean = (2 + cap) / 2
    kind, steps = case["kind"], case.get("steps", 0)
    size = [((n + m) * 0.75 ** i, m * mean * 0.9 ** i) for i in range(steps + 1)]
    e = 2 if case.get("dtype") == "bf16" else 4
    d = case.get("d", 0)

    def sweep(rows, nnz):
        return rows * 2 * d * e + 8 * nnz, 4 * nnz * d

    coarsening = sum(8 * rows + 4 * nnz for rows, nnz in size[:-1]) + sum(4 * nnz + 8 * rows for rows, nnz in size[1:])
    if kind == "score":
        return {"bytes": n * d * e + 4 * m * mean + 4 * m * d, "flops": 4 * m * mean * d}
    if kind == "coarsen":
        return {"bytes": coarsening, "flops": 0}
    if kind == "features":
        # every count read for the hyperedge sums and again for the coarse rows, which are written
        feats = sum(3 * 4 * case["k"] * n * 0.75 ** i for i in range(steps))
        return {"bytes": coarsening + feats, "flops": sum(4 * nnz * case["k"] for _, nnz in size[:-1])}
    if kind == "train":
        k = case["sweeps"]
        b, f = sweep(*size[0])
        return {"bytes": 3 * k * b, "flops": 3 * k * f}
    passes = {"refine": case.get("sweeps"), "stop": min(10, case.get("sweeps", 0)), "pipeline": case.get("sweeps"),
              "train_all": 3 * case.get("sweeps", 0)}[kind]
    total = [passes * sum(x) for x in zip(*(sweep(*s) for s in size))]
    return {"bytes": total[0] + (coarsening if kind == "pipeline" else 0), "flops": total[1]}


# ----------------------------------------------------------------------------
# the same in plain torch, 64 bits
# ----------------------------------------------------------------------------

def _coarsen(n, ptr, idx, w):
    """One featureless coarsening step: each node joins its hyperedge of largest weight, then fewest members, then
    lowest id; groups are numbered by their smallest node; a hyperedge whose members all chose it goes."""
    m = ptr.numel() - 1
    sizes = ptr[1:] - ptr[:-1]
    inc = torch.repeat_interleave(torch.arange(m, device="cuda"), sizes)
    order = torch.sort(sizes, stable=True).indices
    if w is not None:
        order = order[torch.sort(w[order], stable=True, descending=True).indices]
    rank = torch.empty_like(order)
    rank[order] = torch.arange(m, device="cuda")
    best = torch.full((n,), m, device="cuda").scatter_reduce(0, idx, rank[inc], "amin")
    nodes = torch.arange(n, device="cuda")
    group = torch.where(best < m, best, m + nodes)
    first = torch.full((m + n,), n, device="cuda").scatter_reduce(0, group, nodes, "amin")[group]
    rep = (torch.cumsum(first == nodes, 0) - 1)[first]
    mine = torch.zeros(m, dtype=torch.int64, device="cuda").scatter_add(0, inc, (best[idx] == rank[inc]).long())
    kept = mine != sizes
    edge_rep = torch.where(kept, torch.cumsum(kept, 0) - 1, -1)
    nc, mc = int(rep.max()) + 1, int(kept.sum())
    on = kept[inc]
    key = torch.unique(edge_rep[inc[on]] * nc + rep[idx[on]])
    c_ptr = torch.zeros(mc + 1, dtype=torch.int64, device="cuda")
    c_ptr[1:] = torch.bincount(key // nc, minlength=mc).cumsum(0)
    rowmap = torch.cat([rep, torch.where(kept, nc + edge_rep, rep[idx[ptr[:-1]]])])
    return rowmap, (nc, c_ptr, key % nc, None if w is None else w[kept])


class _Level:
    """One level's sweep in 64 bits; `log_w` takes the place of the weights where they are learnt."""

    def __init__(self, n, ptr, idx, w, log_w=None):
        self.n, self.m = n, ptr.numel() - 1
        self.sizes = (ptr[1:] - ptr[:-1]).double().unsqueeze(1)
        self.idx = idx
        self.inc = torch.repeat_interleave(torch.arange(self.m, device="cuda"), ptr[1:] - ptr[:-1])
        self.w = log_w.exp() if log_w is not None else w.double() if w is not None else \
            torch.ones(self.m, dtype=torch.float64, device="cuda")
        self.total = torch.zeros(n, dtype=torch.float64, device="cuda").index_add(0, idx, self.w[self.inc]).unsqueeze(1)
        self.matrices = None
        if log_w is None and idx.numel() > 200000:      # long sums: a sparse product instead of atomic sums
            order = torch.sort(idx, stable=True).indices
            n_ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
            n_ptr[1:] = torch.bincount(idx, minlength=n).cumsum(0)
            one = torch.ones(idx.numel(), dtype=torch.float64, device="cuda")
            self.matrices = (torch.sparse_csr_tensor(ptr.int(), idx.int(), one, (self.m, n)),
                             torch.sparse_csr_tensor(n_ptr.int(), self.inc[order].int(), one, (n, self.m)))

    def members(self, zn):
        if self.matrices:
            return self.matrices[0] @ zn
        return torch.zeros(self.m, zn.shape[1], dtype=zn.dtype, device="cuda").index_add(0, self.inc, zn[self.idx])

    def incident(self, ze):
        zw = ze * self.w.unsqueeze(1)
        if self.matrices:
            return self.matrices[1] @ zw
        return torch.zeros(self.n, zw.shape[1], dtype=zw.dtype, device="cuda").index_add(0, self.idx, zw[self.inc])

    def sweep(self, z, order):
        zn, ze = z[:self.n], z[self.n:]
        new_e = (1 - OMEGA) * ze + OMEGA * self.members(zn) / self.sizes
        mean = self.incident(new_e if order == "edge_first" else ze) / torch.where(self.total > 0, self.total, 1.0)
        new_n = torch.where(self.total > 0, (1 - OMEGA) * zn + OMEGA * mean, zn)
        return torch.cat([new_n, new_e])


def _hierarchy(case, ptr, idx, w):
    levels, rowmaps = [(case["nodes"], ptr.long(), idx.long(), w)], []
    for _ in range(case["steps"]):
        rowmap, coarse = _coarsen(*levels[-1])
        rowmaps.append(rowmap)
        levels.append(coarse)
    return levels, rowmaps


def _score(case, ptr, idx, z):
    sizes = (ptr[1:] - ptr[:-1]).long()
    inc = torch.repeat_interleave(torch.arange(sizes.numel(), device="cuda"), sizes)
    count, out = sizes.double().unsqueeze(1), []
    for c in range(0, case["d"], 16):
        x = z[:, c:c + 16].double()[idx.long()]
        zero = torch.zeros(sizes.numel(), x.shape[1], dtype=torch.float64, device="cuda")
        if case["op"] in ("min", "max"):
            at = inc.unsqueeze(1).expand_as(x)
            out.append(zero.scatter_reduce(0, at, x, "a" + case["op"], include_self=False))
            continue
        mean = zero.index_add(0, inc, x) / count
        out.append(mean if case["op"] == "mean" else zero.index_add(0, inc, (x - mean[inc]).square()) / count)
    return torch.cat(out, 1)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("coarsen", "features"):
        return None         # whole numbers (a coarse weight is a copy)
    g, _, ptr, idx, w = _inputs(case, seed)
    if kind == "score":
        return _score(case, ptr, idx, _normal(g, case["nodes"], case["d"], case["dtype"]))
    levels, rowmaps = _hierarchy(case, ptr, idx, w)
    top = levels[-1]
    z = _normal(g, top[0] + top[1].numel() - 1, case["d"], case["dtype"]).double()
    if kind in ("train", "train_all"):
        return _exact_train(case, g, levels, rowmaps, z)
    tol = case["tol"] * math.sqrt((case["nodes"] + case["edges"]) * case["d"]) if kind == "stop" else 0.0
    residuals, done = [], [0] * len(levels)
    for i in range(len(levels) - 1, -1, -1):
        level = _Level(*levels[i])
        if i < len(levels) - 1:
            z = z[rowmaps[i]]
        for _ in range(case["sweeps"]):
            new = level.sweep(z, case["order"])
            done[i] += 1
            if kind == "stop" or case.get("residuals"):
                residuals.append((new - z).norm())
            z = new
            if kind == "stop" and float(residuals[-1]) <= tol:
                break
    if kind == "stop":
        return z, torch.tensor(done, dtype=torch.int32)
    if kind == "pipeline":
        return z, None
    return (z, torch.stack(residuals)) if case["residuals"] else z


def _exact_train(case, g, levels, rowmaps, z):
    learnt = levels if case["kind"] == "train_all" else levels[:1]
    thetas = [(0.2 * torch.randn(lv[1].numel() - 1, generator=g, device="cuda")).double().requires_grad_(True)
              for lv in learnt]
    cot = torch.randn(case["nodes"] + case["edges"], case["d"], generator=g, device="cuda").double()
    outs, grads = [], []
    for c in range(0, case["d"], 32):                   # columns are independent; the weights' gradients add up
        zc = z[:, c:c + 32].clone().requires_grad_(True)
        x = zc
        for i in range(len(learnt) - 1, -1, -1):
            level = _Level(*levels[i], log_w=thetas[i])
            if i < len(levels) - 1:
                x = x[rowmaps[i]]
            for _ in range(case["sweeps"]):
                x = level.sweep(x, case["order"])
        grads.append(torch.autograd.grad(x, [zc] + thetas, cot[:, c:c + 32]))
        outs.append(x.detach())
    return [torch.cat(outs, 1), torch.cat([q[0] for q in grads], 1)] + \
        [sum(t) for t in zip(*(q[1:] for q in grads))]
