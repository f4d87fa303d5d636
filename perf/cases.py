"""What a user of this library has it do, as measurable cases.

A case is one verification block (or a batch of them) through one MoE layer,
route -> select -> grouped expert FFN, by way of `ops.VerifyLayer.step`, or
through a chain of layers by way of `ops.VerifyStack.step`.  The fields:

  kind      "step" (one layer) or "stack" (`layers` chained layers)
  trees     trees per call (requests verified together)
  nodes     nodes per tree, the root included (1: plain decoding, no draft)
  draft     "tree" (breadth-first draft tree) or "chain" (parent = NULL)
  depth     depth limit of a tree
  hidden, inner, experts, top_k, dtype   the layer
  mode      selection rule: "self" (self-sizing), "all" (natural routing),
            "fixed" / "moespec" / "count" (fixed budget `budget`)
  resident  share of experts in the residency mask (0: no mask)
  rho       correlation of a node's hidden state with its parent's

Inputs come from the seed alone: trees, hidden states and probabilities from
the package's workload generator on the host, expert weights on the GPU.
"""
import numpy as np
import torch

from paper_2608_02989_amd import _lib, ops
from paper_2608_02989_amd import workload as W

MODES = {"self": _lib.MODE_SELF_SIZING, "all": _lib.MODE_ALL_EXPERTS, "fixed": _lib.MODE_FIXED_BUDGET,
         "moespec": _lib.MODE_MOESPEC, "count": _lib.MODE_COUNT}
BETA = 0.5


def _case(name, **kw):
    c = {"kind": "step", "trees": 1, "nodes": 32, "draft": "tree", "depth": 6, "hidden": 2048, "inner": 768,
         "experts": 128, "top_k": 8, "dtype": "bf16", "mode": "self", "budget": 0, "resident": 0.0, "rho": 0.9,
         "layers": 1}
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest layer of the test suite: all latency and launches, fp32
        _case("small_fp32_8", nodes=8, hidden=256, inner=128, experts=16, top_k=2, dtype="f32", depth=3),
        # plain autoregressive decoding: a root alone, its natural top-8
        _case("decode_1", nodes=1),
        # a draft chain, the usual non-tree drafter's block (ragged: 6 nodes)
        _case("chain_6", nodes=6, draft="chain"),
        # one request's draft tree on the Qwen3-30B-A3B-shaped layer
        _case("qwen3_30b_a3b_32", nodes=32),
        # the same layer in a pass over consecutive layers, 60-node trees
        _case("stack_4x60", kind="stack", layers=4, nodes=60, depth=8),
        # fp32 experts (a checkpoint served without rounding), ragged block
        _case("fp32_37", nodes=37, depth=8, experts=64, dtype="f32"),
        # the wide layer under a residency mask, one request
        _case("wide_64_masked", nodes=64, depth=8, hidden=4096, inner=1536, resident=0.25),
        # one GPU's share of the wide layer under 8-way tensor parallelism
        _case("wide_tp8_share_64", nodes=64, depth=8, hidden=4096, inner=192),
        # many small experts, top-10, standard speculative decoding (natural routing)
        _case("natural_512e_64", nodes=64, depth=8, inner=512, experts=512, top_k=10, mode="all"),
        # four requests together on the Qwen3-30B-A3B-shaped layer
        _case("batch_4x60", trees=4, nodes=60, depth=8),
        # eight requests on the wide layer
        _case("wide_batch_8x64", trees=8, nodes=64, depth=8, hidden=4096, inner=1536),
        # a full server: 32 requests on the Qwen3-30B-A3B-shaped layer
        _case("batch_32x60", trees=32, nodes=60, depth=8),
    ]


def _log_uniform(rng, lo, hi):
    return lo * (hi / lo) ** rng.random()


def draw(rng):
    """A case between the listed ones in every size, with no more expert bytes
    than the wide layer and no more arithmetic than its batch of eight."""
    while True:
        c = _case(None)
        c["trees"] = 1 if rng.random() < 0.6 else int(round(_log_uniform(rng, 2, 32)))
        c["nodes"] = int(round(_log_uniform(rng, 1, 64)))
        c["draft"] = "chain" if c["nodes"] <= 16 and rng.random() < 0.3 else "tree"
        c["depth"] = rng.randint(4, 8)
        c["hidden"] = 32 * int(round(_log_uniform(rng, 8, 128)))
        c["inner"] = 32 * int(round(_log_uniform(rng, 4, 64)))
        c["experts"] = rng.choice([16, 32, 60, 64, 96, 128, 160, 256, 512])
        c["top_k"] = min(c["experts"], rng.choice([1, 2, 4, 6, 8, 8, 8, 10]))
        c["dtype"] = "f32" if rng.random() < 0.2 else "bf16"
        c["mode"] = rng.choice(["self", "self", "self", "all", "fixed", "moespec", "count"])
        if c["mode"] in ("fixed", "moespec", "count"):
            c["budget"] = min(c["experts"], c["top_k"] + rng.randint(1, 32))
        elif c["mode"] == "self" and rng.random() < 0.25:
            c["resident"] = 0.25
        c["rho"] = rng.choice([0.9, 0.9, 0.9, 0.0])
        if c["trees"] == 1 and rng.random() < 0.15:
            c["kind"], c["layers"] = "stack", rng.randint(2, 4)
        eb = 4 if c["dtype"] == "f32" else 2
        weights = c["layers"] * c["experts"] * 3 * c["hidden"] * c["inner"] * eb
        flops = c["trees"] * c["nodes"] * c["top_k"] * 6 * c["hidden"] * c["inner"] * c["layers"]
        # fp32 products run on the fp32 matrix instructions, at a sixteenth of the rate
        if 1 << 22 <= weights <= 128 * 3 * 4096 * 1536 * 2 and flops * (16 if eb == 4 else 1) <= 512 * 8 * 6 * 4096 * 1536:
            return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _rng(seed, *stream):
    return np.random.default_rng(np.random.SeedSequence([seed, *stream]))


def _trees(case, seed):
    """Host arrays of the block: parent (None for chains), depth, prob, offsets."""
    parents, depths, probs, offsets = [], [], [], [0]
    for b in range(case["trees"]):
        if case["draft"] == "chain":
            par, dep, sib = W.chain(case["nodes"])
        else:
            # a tree of `nodes` nodes needs the depth: 1..4 children per node
            par, dep, sib = W.make_tree(_rng(seed, 1, b), case["nodes"], case["depth"])
        parents.append(np.where(par < 0, -1, par + offsets[-1]).astype(np.int32))
        depths.append(dep.astype(np.int32))
        probs.append(W.commit_probs(_rng(seed, 2, b), "depth_sibling", dep, sib))
        offsets.append(offsets[-1] + case["nodes"])
    return np.concatenate(parents), np.concatenate(depths), np.concatenate(probs), np.asarray(offsets, np.int32)


def _hidden(case, seed, parent, offsets):
    """Hidden states, rounded to the layer's type (a CPU tensor)."""
    rows = []
    for b in range(case["trees"]):
        par = parent[offsets[b]:offsets[b + 1]]
        rows.append(W.correlated_hidden(_rng(seed, 3, b), np.where(par < 0, -1, par - offsets[b]), case["hidden"], 1.0,
                                        case["rho"]))
    h = torch.from_numpy(np.concatenate(rows))
    return h if case["dtype"] == "f32" else h.to(torch.bfloat16)


def _mask(case, seed):
    if case["resident"] <= 0.0:
        return None
    m = np.zeros(case["experts"], np.uint8)
    m[_rng(seed, 4).choice(case["experts"], size=int(round(case["resident"] * case["experts"])), replace=False)] = 1
    return m


def _router(case, seed, layer):
    return (_rng(seed, 5, layer).standard_normal((case["experts"], case["hidden"])) * 0.02).astype(np.float32)


def _experts(case, seed, layer):
    """w_gate, w_up [E, I, H], w_down [E, H, I] on the GPU."""
    E, I, H = case["experts"], case["inner"], case["hidden"]
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * (seed + 1) + layer)
    return tuple(torch.randn(shape, dtype=dt, device="cuda", generator=g).mul_(0.02)
                 for shape in ((E, I, H), (E, I, H), (E, H, I)))


def _layer(case, seed, layer):
    wg, wu, wd = _experts(case, seed, layer)
    return ops.VerifyLayer(torch.from_numpy(_router(case, seed, layer)).cuda(), wg, wu, wd, case["top_k"],
                           max_tokens=case["trees"] * case["nodes"], max_trees=case["trees"], beta=BETA,
                           mode=MODES[case["mode"]], budget=case["budget"])


def prepare(case, seed):
    parent, depth, prob, offsets = _trees(case, seed)
    mask = _mask(case, seed)
    layers = [_layer(case, seed, n) for n in range(case["layers"])]
    return {
        "layer": layers[0],
        "stack": ops.VerifyStack(layers, case["nodes"]) if case["kind"] == "stack" else None,
        "hidden": _hidden(case, seed, parent, offsets).cuda(),
        "parent": None if case["draft"] == "chain" else torch.from_numpy(parent).cuda(),
        "depth": torch.from_numpy(depth).cuda(),
        "prob": torch.from_numpy(prob).cuda(),
        "offsets": offsets if case["trees"] > 1 else None,
        "resident": None if mask is None else torch.from_numpy(mask).cuda(),
    }


def run(state):
    if state["stack"] is not None:
        state["stack"].step(state["hidden"], state["parent"], state["depth"], state["prob"], state["offsets"])
        T = state["hidden"].shape[0]
        return {"h%d" % (n + 1): h[:T] for n, h in enumerate(state["stack"].h[1:])}
    logits, sel, out = state["layer"].step(state["hidden"], state["parent"], state["depth"], state["prob"],
                                           state["offsets"], state["resident"])
    return {"logits": logits, "eligible": sel["eligible"], "idx": sel["idx"], "gate": sel["gate"],
            "stats": sel["stats"], "out": out}


# ---------------------------------------------------------------------------
# the same in 64 bits, in plain numpy and torch
# ---------------------------------------------------------------------------
def _top(z, k):
    """The k largest of each row of z, ties to the lower index: [T, k]."""
    return np.argsort(-z, axis=1, kind="stable")[:, :k]


def _selection(case, z, parent, depth, prob, offsets, mask):
    """Eligible sets [B, E], routed experts [T, k], gates [T, k] from 64-bit logits."""
    E, k = case["experts"], case["top_k"]
    kmin = min(k, E)
    rank_z = z.astype(np.float32)  # experts are ranked by their fp32 logits
    p = np.exp(z - z.max(axis=1, keepdims=True))
    p /= p.sum(axis=1, keepdims=True)
    natural = _top(rank_z, k)
    eligible = np.zeros((case["trees"], E), np.uint8)
    idx, gate = np.zeros((len(z), k), np.int32), np.zeros((len(z), k))
    for b in range(case["trees"]):
        rows = np.arange(offsets[b], offsets[b + 1])
        n_d = np.bincount(depth[rows])
        alpha = prob[rows].astype(np.float64) ** BETA / np.sqrt(n_d[depth[rows]])
        u, votes = np.zeros(E), np.zeros(E, np.int64)
        for a, t in zip(alpha, rows):
            u[natural[t]] += a * p[t, natural[t]]
            votes[natural[t]] += 1
        inside = np.zeros(E, bool)
        if case["mode"] == "all":
            inside[:] = True
        elif case["mode"] in ("moespec", "count"):
            score = p[rows].sum(axis=0) if case["mode"] == "moespec" else votes.astype(np.float64)
            inside[np.argsort(-score, kind="stable")[:max(kmin, min(case["budget"], E))]] = True
        else:
            inside[natural[rows[0]]] = True
            rest = np.flatnonzero(~inside)
            if case["mode"] == "self":
                q = u[rest][u[rest] > 0]
                take = 0
                if q.size:
                    q = q / q.sum()
                    take = min(max(int(np.ceil(np.exp(-(q * np.log(q)).sum()) - 1e-9)), 1), q.size)
                take = min(max(take, kmin - k), rest.size)
            else:
                take = min(max(max(kmin, min(case["budget"], E)) - k, 0), rest.size)
            inside[rest[np.argsort(-u[rest], kind="stable")[:take]]] = True
            if mask is not None:
                spare = votes[~inside].sum()
                gone = np.flatnonzero(inside & (mask == 0))
                gone = gone[np.argsort(u[gone], kind="stable")]
                limit = min(gone.size, inside.sum() - k)
                m = int((np.cumsum(votes[gone[:max(limit, 0)]]) <= spare).sum())
                inside[gone[:m]] = False
        eligible[b] = inside
        idx[rows] = _top(np.where(inside[None, :], rank_z[rows], -np.inf), k)
    sel = np.take_along_axis(z, idx, axis=1)
    gate = np.exp(sel - sel.max(axis=1, keepdims=True))
    return eligible, idx, gate / gate.sum(axis=1, keepdims=True)


def exact(case, seed):
    if case["kind"] == "stack":
        return None  # states are rounded to bf16 between layers and routing follows them: no 64-bit value
    parent, depth, prob, offsets = _trees(case, seed)
    x = _hidden(case, seed, parent, offsets).double()
    z = (x.numpy() @ _router(case, seed, 0).astype(np.float64).T)
    _, idx, gate = _selection(case, z, parent, depth, prob, offsets, _mask(case, seed))
    wg, wu, wd = _experts(case, seed, 0)
    x, idx_t, gate_t = x.cuda(), torch.from_numpy(idx).cuda(), torch.from_numpy(gate).cuda()
    out = torch.zeros_like(x)
    for e in np.unique(idx):
        t, j = torch.nonzero(idx_t == int(e), as_tuple=True)
        g, up = x[t] @ wg[e].double().T, x[t] @ wu[e].double().T
        out[t] += gate_t[t, j][:, None] * ((g * torch.sigmoid(g) * up) @ wd[e].double().T)
    return {"logits": torch.from_numpy(z), "eligible": None, "idx": None, "gate": gate_t, "stats": None, "out": out}


# ---------------------------------------------------------------------------
# what a pass cannot do without, and how far outputs may be apart
# ---------------------------------------------------------------------------
def work(case):
    """Weights of the experts that one block of this case routes to (seed 0),
    the router, hidden states, routing and outputs, each once."""
    parent, depth, prob, offsets = _trees(case, 0)
    x = _hidden(case, 0, parent, offsets).double().numpy()
    T, H, I, E, k = len(x), case["hidden"], case["inner"], case["experts"], case["top_k"]
    _, idx, _ = _selection(case, x @ _router(case, 0, 0).astype(np.float64).T, parent, depth, prob, offsets,
                           _mask(case, 0))
    eb = 4 if case["dtype"] == "f32" else 2
    layer_bytes = (len(np.unique(idx)) * 3 * H * I * eb + E * H * 4 + T * E * 4 + T * k * 8 + T * H * (eb + 4)
                   + T * 12 + case["trees"] * E)
    layer_flops = T * k * 6 * H * I + 2 * T * E * H
    return {"bytes": float(layer_bytes * case["layers"]), "flops": float(layer_flops * case["layers"])}


def tolerance(case):
    # bf16: activations are rounded to bf16 once (2^-9 each; 1.7e-3 from the
    # 64-bit result measured); fp32: sums of up to a few thousand fp32 products
    # (7e-7 measured); four times these.  A stack's states are rounded to bf16
    # between layers and routing follows them.
    if case["kind"] == "stack":
        return {"rel": 1e-2, "max": 0.5}
    if case["dtype"] == "f32":
        return {"rel": 3e-6, "max": 1e-4, "differ": 0.002}
    return {"rel": 7e-3, "max": 0.1, "differ": 0.002}
