"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the
same seeded inputs.

* route: normwise max-relative error <= 1e-5 against the fp64 product
* select: given the same fp32 logits, eligible sets, restricted indices and
  statistics bit-exact; gates within one fp32 rounding
* forward: normwise max-relative error <= 1e-4 (fp32) / 2e-2 (bf16) and the
  same per output row (1e-4 / 1e-2) against the fp64 grouped oracle on full
  outputs at every workload shape; the elementwise figure is reported beside
  them; the lowest-gate slot's contribution is checked on its own
* end to end (route -> select -> forward): as above, with the oracle routing
  its own fp64 logits, at every workload shape
"""
import numpy as np
import pytest
import torch

from oracle import acceptmoe_oracle as O
from paper_2608_02989_amd import _lib as L
from paper_2608_02989_amd import ops
from paper_2608_02989_amd import workload as W

from _util import (FWD_TOL, GATE_RTOL, LOGIT_TOL, HostExperts, check_forward, hidden_for, normwise_rel,
                   oracle_logits32)

pytestmark = pytest.mark.gpu

DEV = "cuda"


def say(*a):
    print(*a, flush=True)


def to_dev_hidden(cfg, arr):
    if cfg.dtype == "bf16":
        return torch.from_numpy(arr.view(np.int16)).view(torch.bfloat16).to(DEV)
    return torch.from_numpy(np.ascontiguousarray(arr, np.float32)).to(DEV)


def normwise_l2(got, ref):
    return float(np.linalg.norm(np.asarray(got, np.float64) - ref) / np.linalg.norm(ref))


def i32(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.int32)).to(DEV)


def f32(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(DEV)


def u8(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a, np.uint8)).to(DEV)


# ---------------------------------------------------------------------------
# route
# ---------------------------------------------------------------------------
ROUTE_CASES = [("fp32_small", None, None, None), ("qwen3_30b_a3b", None, None, None),
               ("wide_offload", None, None, None), ("batched_8x64", None, None, None),
               ("qwen3_30b_a3b", 37, 100, None), ("batched_8x64", None, 100, None),
               # H % 32 == 16: the last packed chunk is half padding; with these H the
               # hidden state is staged in two blocks, the second holding that one chunk
               ("fp32_small", None, None, 1040), ("qwen3_30b_a3b", 21, 40, 2064),
               ("fp32_small", None, 24, 48), ("qwen3_30b_a3b", 1, None, None)]


@pytest.mark.parametrize("name,T,E,H", ROUTE_CASES)
def test_route_parity(gpu, name, T, E, H):
    cfg = W.CONFIGS[name]
    if E is not None:
        cfg = W.LayerConfig(**{**cfg.__dict__, "E": E})
    if H is not None:
        cfg = W.LayerConfig(**{**cfg.__dict__, "H": H})
    blk = W.make_block(cfg, block=3, T=T if T else None, B=1 if T else None)
    hdev, h64 = hidden_for(cfg, blk.hidden)
    rw = W.router_weights(cfg)
    say(f"route {name} T={len(h64)} E={cfg.E} H={cfg.H}")
    rp = ops.pack_router_weights(f32(rw))
    z = ops.route(to_dev_hidden(cfg, hdev), rp).cpu().numpy()
    ref = O.route(h64, rw.astype(np.float64))
    err = normwise_rel(z, ref)
    assert err <= LOGIT_TOL, err
    # fixed reduction order: identical on a second call
    z2 = ops.route(to_dev_hidden(cfg, hdev), rp).cpu().numpy()
    assert np.array_equal(z.view(np.uint32), z2.view(np.uint32))


# ---------------------------------------------------------------------------
# select (bit-exact given the same fp32 logits)
# ---------------------------------------------------------------------------
def run_select_both(z32, parent, depth, prob, offs, k, beta=0.5, mode=0, budget=0, cap=-1, resident=None,
                    parent_none=False):
    par_dev = None if parent_none else i32(parent)
    got = ops.select(f32(z32), par_dev, i32(depth), f32(prob), offs, k, beta, mode, budget, cap, u8(resident))
    torch.cuda.synchronize()
    got = {kk: v.cpu().numpy() for kk, v in got.items()}
    ref = O.select(z32, None if parent_none else parent, depth, prob, offs, k, beta, mode, resident,
                   None if cap < 0 else cap, budget)
    return got, ref


def assert_select_equal(got, ref, context=""):
    amb = ref["ambiguous"]
    assert not amb.any(), f"oracle reports near-tie decisions {amb} {context}"
    assert np.array_equal(got["eligible"], ref["eligible"]), context
    assert np.array_equal(got["idx"], ref["idx"]), context
    assert np.array_equal(got["stats"].astype(np.int64), ref["stats"]), (got["stats"], ref["stats"], context)
    np.testing.assert_allclose(got["gate"], ref["gate"], rtol=GATE_RTOL, atol=0, err_msg=context)


def block_inputs(cfg, block=0, layer=0, rho=0.9, T=None, B=None):
    blk = W.make_block(cfg, block=block, layer=layer, rho=rho, T=T, B=B)
    _, h64 = hidden_for(cfg, blk.hidden)
    z32 = oracle_logits32(h64, W.router_weights(cfg, layer))
    return blk, z32


SEL_CONFIGS = [
    ("fp32_small", 0.9, 0), ("fp32_small", 0.0, 1), ("qwen3_30b_a3b", 0.9, 0), ("qwen3_30b_a3b", 0.0, 2),
    ("qwen3_30b_a3b_x48", 0.9, 5), ("wide_offload", 0.9, 0), ("wide_offload", 0.0, 3),
    ("batched_8x64", 0.9, 0), ("batched_8x64", 0.0, 4),
]


@pytest.mark.parametrize("name,rho,seed", SEL_CONFIGS)
def test_select_parity_configs(gpu, name, rho, seed):
    cfg = W.CONFIGS[name]
    blk, z32 = block_inputs(cfg, block=seed, rho=rho)
    say(f"select {name} rho={rho} seed={seed} T={len(z32)} B={len(blk.offsets) - 1}")
    got, ref = run_select_both(z32, blk.parent, blk.depth, blk.prob, blk.offsets, cfg.k,
                               resident=blk.resident)
    assert_select_equal(got, ref, name)


@pytest.mark.parametrize("E,k,T", [(48, 3, 23), (200, 6, 40), (512, 32, 33), (16, 16, 9), (64, 1, 17),
                                   (100, 8, 130), (128, 8, 1024), (128, 8, 64), (128, 8, 65),
                                   (256, 8, 64), (257, 8, 20)])
def test_select_parity_shapes(gpu, E, k, T):
    rng = np.random.default_rng(E * 1000 + k)
    par, dep, sib = W.make_tree(rng, T, 10)
    prob = (0.75 ** dep * 0.6 ** sib).astype(np.float32)
    z32 = (rng.standard_normal((T, E)) * 2).astype(np.float32)
    res = (rng.random(E) < 0.4).astype(np.uint8)
    say(f"select shape E={E} k={k} T={T}")
    for resident in (None, res):
        got, ref = run_select_both(z32, par, dep, prob, None, k, resident=resident)
        assert_select_equal(got, ref, f"E={E} k={k} T={T} mask={resident is not None}")


@pytest.mark.parametrize("mode,budget", [(L.MODE_ALL_EXPERTS, 0), (L.MODE_FIXED_BUDGET, 24),
                                         (L.MODE_FIXED_BUDGET, 3), (L.MODE_MOESPEC, 24), (L.MODE_COUNT, 24),
                                         (L.MODE_COUNT, 200)])
def test_select_parity_modes(gpu, mode, budget):
    cfg = W.CONFIGS["wide_offload"]
    blk, z32 = block_inputs(cfg, block=7, rho=0.5)
    say(f"select mode={mode} budget={budget}")
    for resident in (None, blk.resident):
        got, ref = run_select_both(z32, blk.parent, blk.depth, blk.prob, blk.offsets, cfg.k, mode=mode,
                                   budget=budget, resident=resident)
        assert_select_equal(got, ref, f"mode={mode}")


def test_select_parity_masks_and_caps(gpu):
    cfg = W.CONFIGS["qwen3_30b_a3b"]
    blk, z32 = block_inputs(cfg, block=11, rho=0.9)
    E = cfg.E
    say("select masks and caps")
    for resident, cap in ((np.ones(E, np.uint8), -1), (np.zeros(E, np.uint8), -1), (np.zeros(E, np.uint8), 2),
                          (np.zeros(E, np.uint8), 0), (blk.resident, -1)):
        got, ref = run_select_both(z32, blk.parent, blk.depth, blk.prob, None, cfg.k, resident=resident, cap=cap)
        assert_select_equal(got, ref, f"cap={cap}")


def test_select_parity_beta_and_chain(gpu):
    rng = np.random.default_rng(5)
    E, k, T = 64, 4, 20
    par, dep, _ = W.chain(T)
    prob = (0.8 ** dep).astype(np.float32)
    z32 = rng.standard_normal((T, E)).astype(np.float32)
    say("select chain / beta / no parent")
    for beta in (0.5, 0.0, 1.0, 2.0):
        got, ref = run_select_both(z32, par, dep, prob, None, k, beta=beta)
        assert_select_equal(got, ref, f"beta={beta}")
    got, ref = run_select_both(z32, par, dep, prob, None, k, parent_none=True)
    assert_select_equal(got, ref, "parent=None")


def test_select_parity_root_only_and_ties(gpu):
    say("select root-only and all-tie logits")
    z = np.random.default_rng(0).standard_normal((1, 128)).astype(np.float32)
    got, ref = run_select_both(z, np.array([-1]), np.array([0]), np.array([0.9], np.float32), None, 8)
    assert_select_equal(got, ref, "root only")
    assert got["eligible"].sum() == 8
    # every logit equal: lowest indices win everywhere
    T = 12
    rng = np.random.default_rng(1)
    par, dep, sib = W.make_tree(rng, T, 4)
    z = np.zeros((T, 40), np.float32)
    got, ref = run_select_both(z, par, dep, np.ones(T, np.float32), None, 5)
    assert_select_equal(got, ref, "ties")
    assert (got["idx"] == np.arange(5)).all()
    # signed zeros and repeated values
    z = rng.integers(-3, 3, size=(T, 40)).astype(np.float32)
    z[z == 0] = -0.0
    z[::2, ::3] = 0.0
    got, ref = run_select_both(z, par, dep, (0.7 ** dep).astype(np.float32), None, 5)
    assert_select_equal(got, ref, "repeated")


# a batch of small, empty and invalid trees, with and without a tree of more
# than 64 nodes
@pytest.mark.parametrize("sizes", [[64, 1, 0, 17, 64, 5, 33], [100, 1, 0, 17, 64, 5, 33]])
def test_select_parity_batch_with_invalid_trees(gpu, sizes):
    rng = np.random.default_rng(9)
    E, k = 128, 8
    pars, deps, probs = [], [], []
    offs = [0]
    for s in sizes:
        par, dep, sib = W.make_tree(rng, s, 8) if s else (np.zeros(0, np.int32),) * 3
        pars.append(np.where(par < 0, -1, par + offs[-1]))
        deps.append(dep)
        probs.append((0.75 ** dep * 0.6 ** sib).astype(np.float32))
        offs.append(offs[-1] + s)
    par = np.concatenate(pars).astype(np.int32)
    dep = np.concatenate(deps).astype(np.int32)
    prob = np.concatenate(probs).astype(np.float32)
    T = offs[-1]
    z32 = rng.standard_normal((T, E)).astype(np.float32)
    # corrupt: tree 3 bad depth, tree 5 parent into tree 4, tree 6 negative prob
    dep[offs[3] + 4] += 1
    par[offs[5] + 2] = offs[4]
    prob[offs[6] + 7] = -0.5
    say(f"select batch with invalid trees offs={offs}")
    got, ref = run_select_both(z32, par, dep, prob, offs, k)
    codes = got["stats"][:, L.NUM_STATS - 2]
    assert codes[2] == O.TREE_EMPTY and codes[3] != 0 and codes[5] == O.TREE_BAD_PARENT
    assert codes[6] == O.TREE_BAD_PROB and codes[0] == 0 and codes[1] == 0
    assert_select_equal(got, ref, "batch with invalid trees")


# blocks whose trees all have at most 16 nodes (8 above 256 experts) run in one
# launch: against the oracle, and bit for bit against the three launches, which
# the same trees take when a larger tree follows them
@pytest.mark.parametrize("E,k,sizes", [(128, 8, [16, 1, 0, 7, 16, 2]), (20, 20, [3, 16]), (64, 1, [1]), (256, 10, [9, 16]),
                                       (512, 32, [8, 1, 5]), (300, 6, [8])])
@pytest.mark.parametrize("mode,budget", [(L.MODE_SELF_SIZING, 0), (L.MODE_ALL_EXPERTS, 0), (L.MODE_FIXED_BUDGET, 24),
                                         (L.MODE_MOESPEC, 24), (L.MODE_COUNT, 24)])
def test_select_small_trees_match_general_path(gpu, E, k, sizes, mode, budget):
    rng = np.random.default_rng(E + k)
    budget = min(budget, E)

    def block(sz):
        pars, deps, probs, offs = [], [], [], [0]
        r = np.random.default_rng(E)
        for n in sz:
            par, dep, sib = W.make_tree(r, n, 6) if n else (np.zeros(0, np.int32),) * 3
            pars.append(np.where(par < 0, -1, par + offs[-1]))
            deps.append(dep)
            probs.append((0.75 ** dep * 0.6 ** sib).astype(np.float32))
            offs.append(offs[-1] + n)
        par, dep, prob = (np.concatenate(x) for x in (pars, deps, probs))
        return par.astype(np.int32), dep.astype(np.int32), prob.astype(np.float32), offs

    par, dep, prob, offs = block(sizes + [17])
    z32 = rng.standard_normal((offs[-1], E)).astype(np.float32)
    z32[0, : E // 2] = 0.25                       # ties at the root
    if len(sizes) > 3:
        par[offs[3] + 2] = offs[0]                # a parent in another tree
    T, B = offs[-2], len(sizes)
    for resident, beta in ((None, 0.5), ((rng.random(E) < 0.3).astype(np.uint8), 1.5)):
        say(f"select small trees E={E} k={k} sizes={sizes} mode={mode} mask={resident is not None}")
        got, ref = run_select_both(z32[:T], par[:T], dep[:T], prob[:T], offs[:-1], k, beta, mode, budget,
                                   resident=resident)
        big, _ = run_select_both(z32, par, dep, prob, offs, k, beta, mode, budget, resident=resident)
        assert_select_equal(got, ref, "small trees")
        for key, n in (("eligible", B), ("idx", T), ("gate", T), ("stats", B)):
            assert np.array_equal(got[key][:n].view(np.uint8), big[key][:n].view(np.uint8)), key
    if len(sizes) == 1:                            # chain, no parents; no statistics asked for
        n = sizes[0]
        got, ref = run_select_both(z32[:n], None, np.arange(n), prob[:n], None, k, 0.5, mode, budget, parent_none=True)
        assert_select_equal(got, ref, "small chain")


# the largest batch of trees: ACCEPTMOE_MAX_TREES ragged trees (empty ones
# included), with a residency mask and in the fixed-budget mode
@pytest.mark.parametrize("mode,budget", [(L.MODE_SELF_SIZING, 0), (L.MODE_FIXED_BUDGET, 12)])
def test_select_parity_max_trees(gpu, mode, budget):
    rng = np.random.default_rng(21)
    E, k = 64, 4
    sizes = rng.integers(0, 10, size=L.MAX_TREES)
    sizes[0], sizes[-1] = 0, 9
    pars, deps, probs = [], [], []
    offs = [0]
    for s_ in sizes:
        s_ = int(s_)
        par, dep, sib = W.make_tree(rng, s_, 4) if s_ else (np.zeros(0, np.int32),) * 3
        pars.append(np.where(par < 0, -1, par + offs[-1]))
        deps.append(dep)
        probs.append((0.75 ** dep * 0.6 ** sib).astype(np.float32))
        offs.append(offs[-1] + s_)
    par = np.concatenate(pars).astype(np.int32)
    dep = np.concatenate(deps).astype(np.int32)
    prob = np.concatenate(probs).astype(np.float32)
    z32 = rng.standard_normal((offs[-1], E)).astype(np.float32)
    resident = (rng.random(E) < 0.3).astype(np.uint8)
    say(f"select {L.MAX_TREES} trees T={offs[-1]} mode={mode}")
    got, ref = run_select_both(z32, par, dep, prob, offs, k, mode=mode, budget=budget, resident=resident)
    codes = got["stats"][:, L.NUM_STATS - 2]
    assert (codes[sizes == 0] == O.TREE_EMPTY).all() and (codes[sizes > 0] == 0).all()
    assert_select_equal(got, ref, f"{L.MAX_TREES} trees")


# ---------------------------------------------------------------------------
# forward
# ---------------------------------------------------------------------------
def forward_case(cfg, idx, gate, blk_hidden, layer=0, E=None):
    hdev, h64 = hidden_for(cfg, blk_hidden)
    wg, wu, wd = W.expert_weights_torch(cfg, layer, DEV, E=E)
    got = ops.moe_forward(to_dev_hidden(cfg, hdev), ops.pack_gate_up_weights(wg, wu), ops.pack_expert_weights(wd),
                          i32(idx), f32(gate))
    torch.cuda.synchronize()
    return got.cpu().numpy(), h64, (HostExperts(wg), HostExperts(wu), HostExperts(wd))


FWD_CONFIGS = [("fp32_small", 0), ("qwen3_30b_a3b", 0), ("qwen3_30b_a3b", 1), ("wide_offload", 0),
               ("batched_8x64", 0)]


# every output row at every workload shape, 8 trees x 64 nodes (512 tokens,
# a separate S' per tree) included
@pytest.mark.parametrize("name,seed", FWD_CONFIGS)
def test_forward_parity_full(gpu, name, seed):
    cfg = W.CONFIGS[name]
    blk, z32 = block_inputs(cfg, block=seed)
    sel = O.select(z32, blk.parent, blk.depth, blk.prob, blk.offsets, cfg.k, resident=blk.resident)
    say(f"forward {name} seed={seed} routed={sel['stats'][:, O.ST_ROUTED]}")
    got, h64, (wg, wu, wd) = forward_case(cfg, sel["idx"], sel["gate"], blk.hidden)
    ref = O.moe_forward_grouped(h64, wg, wu, wd, sel["idx"], sel["gate"], cfg.dtype)
    check_forward(got, ref, cfg.dtype, f"forward {name} block {seed}")
    # rows computed one at a time by an independent oracle routine agree with the grouped one
    rows = [0, len(h64) // 2, len(h64) - 1]
    ref_rows = O.moe_forward_rows(h64, wg, wu, wd, sel["idx"], sel["gate"], rows, cfg.dtype)
    assert normwise_rel(ref_rows, ref[rows]) <= 1e-12


# The output is linear in the gates, so doubling the gate of slot j adds that
# slot's own contribution g_tj * FFN_e(x_t): the difference of two GPU calls
# isolates it.  Slot k-1 holds each node's lowest gate (slots are in logit-
# descending order), the contribution a tensor-wide error figure could hide.
@pytest.mark.parametrize("name", ["qwen3_30b_a3b", "wide_offload", "batched_8x64"])
def test_forward_lowest_gate_slot(gpu, name):
    cfg = W.CONFIGS[name]
    blk, z32 = block_inputs(cfg, block=3)
    sel = O.select(z32, blk.parent, blk.depth, blk.prob, blk.offsets, cfg.k, resident=blk.resident)
    idx, gate = sel["idx"], sel["gate"]
    j = cfg.k - 1
    gate2 = gate.copy()
    gate2[:, j] *= 2.0
    hdev, h64 = hidden_for(cfg, blk.hidden)
    wg, wu, wd = W.expert_weights_torch(cfg, 0, DEV)
    pgu, pd = ops.pack_gate_up_weights(wg, wu), ops.pack_expert_weights(wd)
    hd = to_dev_hidden(cfg, hdev)
    say(f"forward lowest-gate slot {name}")
    y1 = ops.moe_forward(hd, pgu, pd, i32(idx), f32(gate)).cpu().numpy().astype(np.float64)
    y2 = ops.moe_forward(hd, pgu, pd, i32(idx), f32(gate2)).cpu().numpy().astype(np.float64)
    only_j = np.full_like(idx, -1)
    only_j[:, j] = idx[:, j]
    ref = O.moe_forward_grouped(h64, HostExperts(wg), HostExperts(wu), HostExperts(wd), only_j, gate,
                                cfg.dtype)
    check_forward(y2 - y1, ref, cfg.dtype, f"slot {j} contribution {name}")


# T = 100 takes the column path (I < 256), T = 300 the grouped path
@pytest.mark.parametrize("dtype,T", [("bf16", 100), ("f32", 100), ("bf16", 300), ("f32", 300)])
def test_forward_parity_ragged_and_hot_expert(gpu, dtype, T):
    # T not a multiple of 16, E not a multiple of 64, one expert receiving every token
    cfg = W.LayerConfig("ragged", 90 + (dtype == "f32"), dtype, T=T, B=1, H=256, E=20, k=3, I=96,
                        depth_max=6, commit_rule="depth_sibling", hidden_std=1.0)
    rng = np.random.default_rng(3)
    h32 = rng.standard_normal((T, cfg.H)).astype(np.float32)
    others = np.array([e for e in range(cfg.E) if e != 7])
    # expert 7 gets every token (several passes or items); the rest distinct per row
    idx = np.stack([np.concatenate([[7], rng.permutation(others)[:cfg.k - 1]]) for _ in range(T)])
    idx = idx.astype(np.int32)
    idx[5] = [3, -1, 25]                            # invalid entries are skipped
    idx[6] = [-1, -1, -1]                           # no expert at all -> zero row
    idx[9] = [4, 11, 4]                             # a repeated expert counts once (first slot)
    gate = rng.random((T, cfg.k)).astype(np.float32)
    say(f"forward ragged dtype={dtype} T={T}")
    got, h64, (wg, wu, wd) = forward_case(cfg, idx, gate, h32)
    clean = np.where((idx >= 0) & (idx < cfg.E), idx, -1)
    clean[9, 2] = -1
    ref = O.moe_forward_grouped(h64, wg, wu, wd, clean, gate, cfg.dtype)
    check_forward(got, ref, cfg.dtype, f"ragged hot expert T={T}")
    assert np.all(got[6] == 0.0)


# no token routed at all (every entry invalid): no expert is streamed and the
# output is zero; then a routed call on the same workspace (no stale dispatch)
@pytest.mark.parametrize("T", [32, 300])
def test_forward_no_routed_expert(gpu, T):
    cfg = W.LayerConfig("unrouted", 93 + T, "bf16", T=T, B=1, H=256, E=20, k=4, I=96, depth_max=6,
                        commit_rule="depth_sibling", hidden_std=1.0)
    rng = np.random.default_rng(T + 17)
    h32 = rng.standard_normal((T, cfg.H)).astype(np.float32)
    hdev, h64 = hidden_for(cfg, h32)
    wg, wu, wd = W.expert_weights_torch(cfg, 0, DEV)
    pgu, pd = ops.pack_gate_up_weights(wg, wu), ops.pack_expert_weights(wd)
    ws = ops.forward_workspace(T, cfg.H, cfg.I, cfg.E, cfg.k, torch.bfloat16, DEV)
    out = torch.full((T, cfg.H), 7.0, dtype=torch.float32, device=DEV)
    idx = np.full((T, cfg.k), -1, np.int32)
    idx[::3, 1] = cfg.E + 5                         # out of range: skipped as well
    gate = rng.random((T, cfg.k)).astype(np.float32)
    say(f"forward no routed expert T={T}")
    ops.moe_forward(to_dev_hidden(cfg, hdev), pgu, pd, i32(idx), f32(gate), out=out, workspace=ws)
    torch.cuda.synchronize()
    assert torch.count_nonzero(out).item() == 0
    idx2 = np.stack([rng.permutation(cfg.E)[:cfg.k] for _ in range(T)]).astype(np.int32)
    ops.moe_forward(to_dev_hidden(cfg, hdev), pgu, pd, i32(idx2), f32(gate), out=out, workspace=ws)
    torch.cuda.synchronize()
    ref = O.moe_forward_grouped(h64, HostExperts(wg), HostExperts(wu), HostExperts(wd), idx2, gate, cfg.dtype)
    check_forward(out.cpu().numpy(), ref, cfg.dtype, f"routed after unrouted T={T}")


# more tokens than a grid's y dimension holds (65,535): the grouped path and its
# combine over 65,600 tokens of a small layer.  Above 65,536 tokens a workgroup of
# the dispatch does two chunks of 256; the last one gets 64 tokens, and 256 + 208
# at 66,000
@pytest.mark.parametrize("T", [65_600, 66_000])
def test_forward_parity_many_tokens(gpu, T):
    cfg = W.LayerConfig("many", 99, "bf16", T=T, B=1, H=64, E=6, k=2, I=32, depth_max=6,
                        commit_rule="depth_sibling", hidden_std=1.0)
    rng = np.random.default_rng(65_600)
    h32 = rng.standard_normal((T, cfg.H)).astype(np.float32)
    idx = np.stack([rng.permutation(cfg.E)[:cfg.k] for _ in range(T)]).astype(np.int32)
    gate = rng.random((T, cfg.k)).astype(np.float32)
    say(f"forward many tokens T={T}")
    got, h64, (wg, wu, wd) = forward_case(cfg, idx, gate, h32)
    ref = O.moe_forward_grouped(h64, wg, wu, wd, idx, gate, cfg.dtype)
    check_forward(got, ref, cfg.dtype, f"many tokens T={T}")


# forward path limits: k > 8 in the in-LDS dispatch, exactly 256 tokens / 2048
# slots (the largest block of the column path, which a thin I stays on), 257
# tokens (grouped path), E = 48
@pytest.mark.parametrize("T,k,E,dtype", [(40, 32, 64, "bf16"), (37, 12, 48, "f32"), (256, 8, 64, "bf16"),
                                         (257, 8, 64, "bf16")])
def test_forward_parity_path_limits(gpu, T, k, E, dtype):
    cfg = W.LayerConfig("limits", 95 + T + k, dtype, T=T, B=1, H=256, E=E, k=k, I=128, depth_max=6,
                        commit_rule="depth_sibling", hidden_std=1.0)
    rng = np.random.default_rng(T * 100 + k)
    h32 = rng.standard_normal((T, cfg.H)).astype(np.float32)
    idx = np.stack([rng.permutation(E)[:k] for _ in range(T)]).astype(np.int32)
    gate = rng.random((T, k)).astype(np.float32)
    say(f"forward limits T={T} k={k} E={E} dtype={dtype}")
    got, h64, (wg, wu, wd) = forward_case(cfg, idx, gate, h32)
    ref = O.moe_forward_grouped(h64, wg, wu, wd, idx, gate, cfg.dtype)
    check_forward(got, ref, cfg.dtype, f"limits T={T} k={k} E={E}")


# grouped path, experts of 40, 70, 100, 130 and 260 tokens: bf16 items of 3, 5 and 7
# M-tiles, one of 130 rows in two M groups and two for 260 (144 + 116); fp32 one to
# five items of up to 4 M-tiles each
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_forward_parity_m_groups(gpu, dtype):
    T, k, E = 300, 2, 8
    cfg = W.LayerConfig("mgroups", 171 + (dtype == "f32"), dtype, T=T, B=1, H=256, E=E, k=k, I=128,
                        depth_max=6, commit_rule="depth_sibling", hidden_std=1.0)
    t = np.arange(T)
    slot0 = np.where(t < 70, 0, np.where(t < 170, 1, 2))
    slot1 = np.where(t < 260, 3, 4)
    idx = np.stack([slot0, slot1], axis=1).astype(np.int32)
    assert np.bincount(idx.reshape(-1), minlength=E).tolist() == [70, 100, 130, 260, 40, 0, 0, 0]
    rng = np.random.default_rng(77)
    gate = rng.random((T, k)).astype(np.float32)
    h32 = rng.standard_normal((T, cfg.H)).astype(np.float32)
    say(f"forward M groups T={T} dtype={dtype}")
    got, h64, (wg, wu, wd) = forward_case(cfg, idx, gate, h32)
    ref = O.moe_forward_grouped(h64, wg, wu, wd, idx, gate, cfg.dtype)
    check_forward(got, ref, cfg.dtype, f"M groups {dtype}")


# routing rows of 16 and 17 slots (the kernels hold rows of up to 8, 16 or 32)
# on both FFN paths; one token alone takes workgroups without an item
@pytest.mark.parametrize("T,k", [(1, 16), (20, 16), (20, 17), (300, 16), (300, 17)])
def test_forward_parity_row_sizes(gpu, T, k):
    cfg = W.LayerConfig("rows", 1200 + k, "bf16", T=T, B=1, H=128, E=40, k=k, I=96, depth_max=6,
                        commit_rule="depth_sibling", hidden_std=1.0)
    rng = np.random.default_rng(T + k)
    h32 = rng.standard_normal((T, cfg.H)).astype(np.float32)
    idx = np.stack([rng.permutation(cfg.E)[:k] for _ in range(T)]).astype(np.int32)
    gate = rng.random((T, k)).astype(np.float32)
    got, h64, (wg, wu, wd) = forward_case(cfg, idx, gate, h32)
    ref = O.moe_forward_grouped(h64, wg, wu, wd, idx, gate, cfg.dtype)
    check_forward(got, ref, cfg.dtype, f"row sizes T={T} k={k}")


# Grouped GEMMs (blocks beyond the in-workgroup dispatch): experts at the edges
# of the M-tiles per wave (bf16: 1, 2, 3, 4, 6, 8), of the two M groups
# (10 and 12 M-tiles together; fp32: above 32 rows) and of an item (192 rows;
# fp32: 64), K chunks that do not fill the last LDS stage (H = 160, I = 96:
# 5 and 3 bf16 chunks) and output runs that end inside a workgroup's share.
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,counts", [(400, [1, 16, 17, 48, 49, 64, 96, 97]),
                                      (515, [112, 128, 129, 160, 161, 192, 193, 400, 15, 32, 33, 65])])
def test_forward_parity_grouped_edges(gpu, dtype, T, counts):
    E, k = len(counts) + 1, len(counts)
    cfg = W.LayerConfig("grouped", 960 + T, dtype, T=T, B=1, H=160, E=E, k=k, I=96, depth_max=6,
                        commit_rule="depth_sibling", hidden_std=1.0)
    rng = np.random.default_rng(T)
    h32 = rng.standard_normal((T, cfg.H)).astype(np.float32)
    gate = rng.random((T, k)).astype(np.float32)
    idx = np.full((T, k), -1, np.int32)  # expert 0 stays without tokens
    for j, n in enumerate(counts):
        idx[rng.permutation(T)[:n], j] = j + 1
    got, h64, (wg, wu, wd) = forward_case(cfg, idx, gate, h32)
    ref = O.moe_forward_grouped(h64, wg, wu, wd, idx, np.where(idx < 0, 0.0, gate).astype(np.float32), cfg.dtype)
    check_forward(got, ref, cfg.dtype, f"grouped edges T={T} {dtype}")


# fp32: quarter runs up to 128 items of one run each, half runs from 129, whole runs
# for items before the last 256; experts at the edges of the M-tiles (1 to 4) and of
# the split into 64 rows and a rest, 9 and 7 K chunks, 9 tiles of H and 7 of I, which
# end inside a quarter and a half run
@pytest.mark.parametrize("singles", [105, 106, 300])
def test_forward_parity_fp32_runs(gpu, singles):
    counts = [1, 16, 17, 32, 33, 48, 49, 64, 65, 96, 97, 112, 113, 128, 129] + [1] * singles
    T, k, E = 400, 4, len(counts)
    cfg = W.LayerConfig("fp32runs", 990 + singles, "f32", T=T, B=1, H=144, E=E, k=k, I=112, depth_max=6,
                        commit_rule="depth_sibling", hidden_std=1.0)
    flat = np.full(T * k, -1, np.int32)
    flat[:sum(counts)] = np.repeat(np.arange(E), counts)
    idx = np.ascontiguousarray(flat.reshape(k, T).T)  # an expert's rows follow each other, so no token repeats one
    rng = np.random.default_rng(singles)
    h32 = rng.standard_normal((T, cfg.H)).astype(np.float32)
    gate = rng.random((T, k)).astype(np.float32)
    got, h64, (wg, wu, wd) = forward_case(cfg, idx, gate, h32)
    ref = O.moe_forward_grouped(h64, wg, wu, wd, idx, np.where(idx < 0, 0.0, gate).astype(np.float32), cfg.dtype)
    check_forward(got, ref, cfg.dtype, f"fp32 runs singles={singles}")


# the three kinds of items of the grouped GEMMs in one block: one expert above
# 128 rows (half runs, two M groups), whole runs, and the last items' half runs;
# 18 tiles of I and 34 of H end inside a run and inside a half run
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("H,I", [(544, 288), (288, 96)])
def test_forward_parity_grouped_runs(gpu, dtype, H, I):
    T, E, k = 300, 128, 4
    cfg = W.LayerConfig("runs", 970 + H, dtype, T=T, B=1, H=H, E=E, k=k, I=I, depth_max=6,
                        commit_rule="depth_sibling", hidden_std=1.0)
    rng = np.random.default_rng(H)
    h32 = rng.standard_normal((T, H)).astype(np.float32)
    gate = rng.random((T, k)).astype(np.float32)
    idx = (1 + (k * np.arange(T)[:, None] + np.arange(k)) % (E - 1)).astype(np.int32)
    idx[rng.permutation(T)[:150], 1] = 0
    got, h64, (wg, wu, wd) = forward_case(cfg, idx, gate, h32)
    ref = O.moe_forward_grouped(h64, wg, wu, wd, idx, gate, cfg.dtype)
    check_forward(got, ref, cfg.dtype, f"grouped runs H={H} I={I} {dtype}")


# both sides of every edge between the column and the grouped path: the token
# counts 96 / 97 (fp32 192 / 193), slots x I per down workgroup (1920, and 640 with
# single k-steps: I = 352), 12 rows per expert, I = 256, and the most tokens and
# slots the column path's lists hold.  Up to 256 tokens the dispatch of the
# grouped path is one workgroup.
@pytest.mark.parametrize("dtype,T,H,I,E,k,grouped", [
    ("bf16", 96, 256, 256, 40, 3, False), ("bf16", 97, 256, 256, 40, 3, True),
    ("bf16", 160, 1024, 256, 80, 6, False), ("bf16", 160, 1024, 256, 79, 6, True), ("bf16", 161, 1024, 256, 81, 6, True),
    ("bf16", 116, 1024, 352, 24, 1, False), ("bf16", 117, 1024, 352, 24, 1, True),
    ("bf16", 256, 128, 256, 16, 8, True), ("bf16", 256, 128, 224, 16, 8, False), ("bf16", 70, 128, 256, 40, 32, True),
    ("f32", 192, 256, 256, 20, 3, False), ("f32", 193, 256, 256, 20, 3, True), ("f32", 240, 256, 256, 20, 1, False),
    ("f32", 241, 256, 256, 20, 1, True), ("f32", 193, 256, 352, 20, 1, True), ("f32", 256, 256, 256, 20, 8, True),
    # two column tiles; experts of 60 to 70 rows, two passes of three M-tiles and fewer
    ("f32", 193, 4096, 256, 20, 1, False), ("f32", 200, 256, 256, 3, 1, False), ("f32", 256, 128, 48, 16, 8, False)])
def test_forward_parity_path_edges(gpu, dtype, T, H, I, E, k, grouped):
    cfg = W.LayerConfig("edges", 1400 + T + I + E, dtype, T=T, B=1, H=H, E=E, k=k, I=I, depth_max=6,
                        commit_rule="depth_sibling", hidden_std=1.0)
    ws = L.lib().acceptmoe_moe_forward_workspace_size(T, H, I, E, k, L.BF16 if dtype == "bf16" else L.F32)
    assert (ws >= T * k * (I * cfg.wbytes + H * 4)) == grouped
    rng = np.random.default_rng(T + I + k)
    h32 = rng.standard_normal((T, H)).astype(np.float32)
    idx = np.stack([rng.permutation(E)[:k] for _ in range(T)]).astype(np.int32)
    gate = rng.random((T, k)).astype(np.float32)
    say(f"forward edges {dtype} T={T} H={H} I={I} E={E} k={k}")
    got, h64, (wg, wu, wd) = forward_case(cfg, idx, gate, h32)
    ref = O.moe_forward_grouped(h64, wg, wu, wd, idx, gate, cfg.dtype)
    check_forward(got, ref, cfg.dtype, f"edges {dtype} T={T} H={H} I={I} E={E} k={k}")


# fp32 blocks just above the line between the paths keep the grouped path's error
# on the column path: both add sums of 16 chunks (4.9e-7 to 5.5e-7 measured here and
# on the grouped path); one running sum over all of K gives 6.9e-7 to 1.1e-6
@pytest.mark.parametrize("E,k,H,I", [(128, 1, 2048, 768), (64, 2, 4064, 320), (32, 1, 3424, 1952)])
def test_forward_fp32_column_error(gpu, E, k, H, I):
    T = 200
    assert L.lib().acceptmoe_moe_forward_workspace_size(T, H, I, E, k, L.F32) < T * k * (I * 4 + H * 4)
    cfg = W.LayerConfig("colerr", 1600 + I, "f32", T=T, B=1, H=H, E=E, k=k, I=I, depth_max=6,
                        commit_rule="depth_sibling", hidden_std=1.0)
    rng = np.random.default_rng(I)
    h32 = rng.standard_normal((T, H)).astype(np.float32)
    idx = np.stack([rng.permutation(E)[:k] for _ in range(T)]).astype(np.int32)
    gate = rng.random((T, k)).astype(np.float32)
    got, h64, (wg, wu, wd) = forward_case(cfg, idx, gate, h32)
    err = normwise_l2(got, O.moe_forward_grouped(h64, wg, wu, wd, idx, gate, cfg.dtype))
    say(f"forward fp32 column error E={E} k={k} H={H} I={I}: {err:.3e}")
    assert err <= 6.2e-7, err


# one layer, one workspace: blocks of the grouped path, then of the column path,
# then larger ones again, each as in buffers of its own
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_step_across_paths(gpu, dtype):
    cfg = W.LayerConfig("across", 1500, dtype, T=64, B=5, H=256, E=24, k=4, I=256, depth_max=6,
                        commit_rule="depth_sibling", hidden_std=1.0)
    blk = W.make_block(cfg)
    hdev, _ = hidden_for(cfg, blk.hidden)
    weights = W.expert_weights_torch(cfg, 0, DEV)
    rw = f32(W.router_weights(cfg))
    layer = ops.VerifyLayer(rw, *weights, cfg.k, max_tokens=320, max_trees=5)
    layer.fwd_ws.fill_(0xFF)
    for B in (5, 1, 4, 2, 5):
        T = 64 * B
        args = (to_dev_hidden(cfg, hdev[:T]), i32(blk.parent[:T]), i32(blk.depth[:T]), f32(blk.prob[:T]),
                blk.offsets[:B + 1])
        say(f"step across paths {dtype} T={T}")
        ref = ops.VerifyLayer(rw, *weights, cfg.k, max_tokens=T, max_trees=B).step(*args)
        torch.cuda.synchronize()
        layer.logits.fill_(float("nan"))
        layer.out.fill_(float("nan"))
        got = layer.step(*args)
        torch.cuda.synchronize()
        assert torch.equal(got[0], ref[0]) and torch.equal(got[2], ref[2])
        for key in ref[1]:
            assert torch.equal(got[1][key], ref[1][key]), key


# the most items of two M groups that a block's routing entries allow (experts
# whose rows split into short big items: bf16 257 = 144 + 113): every
# output run has a workgroup.  The workspace starts as NaN, so a run that nobody
# computes shows.
@pytest.mark.parametrize("dtype,T,k,groups", [("f32", 400, 8, [(49, 65), (15, 1)]),
                                              ("bf16", 755, 7, [(20, 257), (1, 129), (16, 1)])])
def test_forward_parity_most_big_items(gpu, dtype, T, k, groups):
    counts = [c for n, c in groups for _ in range(n)]
    E = len(counts)
    cfg = W.LayerConfig("bigitems", 980 + T, dtype, T=T, B=1, H=4096, E=E, k=k, I=64, depth_max=6,
                        commit_rule="depth_sibling", hidden_std=1.0)
    flat = np.full(T * k, -1, np.int32)
    flat[:sum(counts)] = np.repeat(np.arange(E), counts)
    idx = np.ascontiguousarray(flat.reshape(k, T).T)  # an expert's rows follow each other, so no token repeats one
    rng = np.random.default_rng(T)
    h32 = rng.standard_normal((T, cfg.H)).astype(np.float32)
    gate = rng.random((T, k)).astype(np.float32)
    hdev, h64 = hidden_for(cfg, h32)
    wg, wu, wd = W.expert_weights_torch(cfg, 0, DEV)
    ws = ops.forward_workspace(T, cfg.H, cfg.I, E, k, wg.dtype, DEV).fill_(0xFF)
    say(f"forward most big items {dtype}")
    y = ops.moe_forward(to_dev_hidden(cfg, hdev), ops.pack_gate_up_weights(wg, wu), ops.pack_expert_weights(wd),
                        i32(idx), f32(gate), workspace=ws)
    ref = O.moe_forward_grouped(h64, HostExperts(wg), HostExperts(wu), HostExperts(wd), idx, gate, cfg.dtype)
    check_forward(y.cpu().numpy(), ref, cfg.dtype, f"most big items {dtype}")


# one GPU's share of a tensor-parallel split over I: thin I gives the column-tile
# down pass 3-step stages (one column tile at H = 1024, two at H = 4096)
@pytest.mark.parametrize("H,I,T,E", [(1024, 96, 32, 64), (4096, 192, 64, 32)])
def test_forward_parity_thin_shard(gpu, H, I, T, E):
    cfg = W.LayerConfig("thin", 96 + I, "bf16", T=T, B=1, H=H, E=E, k=8, I=I, depth_max=6,
                        commit_rule="depth_sibling", hidden_std=1.0)
    rng = np.random.default_rng(H + I)
    h32 = rng.standard_normal((T, H)).astype(np.float32)
    idx = np.stack([rng.permutation(E)[:cfg.k] for _ in range(T)]).astype(np.int32)
    gate = rng.random((T, cfg.k)).astype(np.float32)
    say(f"forward thin shard H={H} I={I} T={T} E={E}")
    got, h64, (wg, wu, wd) = forward_case(cfg, idx, gate, h32)
    ref = O.moe_forward_grouped(h64, wg, wu, wd, idx, gate, cfg.dtype)
    check_forward(got, ref, cfg.dtype, f"thin shard H={H} I={I}")


# fp32 with I / 16 odd: the last gate/up tile pair is half padding (column and grouped paths)
@pytest.mark.parametrize("T", [37, 300])
def test_forward_parity_odd_tile_count(gpu, T):
    cfg = W.LayerConfig("oddtiles", 97 + T, "f32", T=T, B=1, H=128, E=12, k=3, I=80, depth_max=6,
                        commit_rule="depth_sibling", hidden_std=1.0)
    rng = np.random.default_rng(T + 5)
    h32 = rng.standard_normal((T, cfg.H)).astype(np.float32)
    idx = np.stack([rng.permutation(cfg.E)[:cfg.k] for _ in range(T)]).astype(np.int32)
    gate = rng.random((T, cfg.k)).astype(np.float32)
    say(f"forward odd tile count T={T} I={cfg.I}")
    got, h64, (wg, wu, wd) = forward_case(cfg, idx, gate, h32)
    ref = O.moe_forward_grouped(h64, wg, wu, wd, idx, gate, cfg.dtype)
    check_forward(got, ref, cfg.dtype, f"odd tile count T={T}")


def test_pack_gate_up_layout_documented(gpu):
    # fp32 stacks whose values encode (matrix, e, i, h); I / 16 = 3 -> the last pair's second tiles are zero
    E, I, H = 2, 48, 32
    e_, i_, h_ = np.meshgrid(np.arange(E), np.arange(I), np.arange(H), indexing="ij")
    g = (e_ * 1e6 + i_ * 1e3 + h_ + 1).astype(np.float32)
    u = -g
    pk = ops.pack_gate_up_weights(f32(g), f32(u))
    nbytes = L.lib().acceptmoe_packed_gate_up_bytes(L.F32, E, I, H)
    assert pk.data.numel() * 4 == nbytes == E * 2 * 32 * H * 4 * 2
    frags = pk.data.cpu().numpy().reshape(-1, 64, 4)          # [fragment][lane][4 floats]
    npairs, kc_per_row = 2, H * 4 // 64
    assert frags.shape[0] == E * npairs * kc_per_row * 4
    for fi in range(frags.shape[0]):
        f = fi % 4
        kc = (fi // 4) % kc_per_row
        pair = (fi // 4 // kc_per_row) % npairs
        e = fi // 4 // kc_per_row // npairs
        src = u if f >= 2 else g
        for lane in range(64):
            row = (2 * pair + (f & 1)) * 16 + lane % 16
            col = kc * 16 + (lane // 16) * 4
            want = src[e, row, col:col + 4] if row < I else np.zeros(4, np.float32)
            assert np.array_equal(frags[fi, lane], want), (fi, lane)


def bf16_rne_np(x):
    """fp32 -> nearest-even bf16, returned as fp32 (written from the formats' definitions)."""
    b = np.asarray(x, np.float32).view(np.uint32).astype(np.uint64)
    r = ((b + 0x7FFF + ((b >> 16) & 1)) >> 16).astype(np.uint32)
    return (r << 16).view(np.float32)


@pytest.mark.parametrize("kind", ["index", "normal"])
def test_pack_router_layout_documented(gpu, kind):
    # E = 20 pads rows to 32; H = 48 pads columns to 64 (the second chunk is half padding)
    E, H = 20, 48
    if kind == "index":     # values encode (e, h) and need more than one bf16 plane
        e_, h_ = np.meshgrid(np.arange(E), np.arange(H), indexing="ij")
        src = (e_ * 1000 + h_ + 1 + 1.0 / 3.0).astype(np.float32)
    else:
        src = np.random.default_rng(5).normal(0, 0.02, (E, H)).astype(np.float32)
    rp = ops.pack_router_weights(f32(src))
    raw = rp.data.cpu().numpy().view(np.uint16).astype(np.uint32)
    planes = (raw << 16).view(np.float32).reshape(-1, 3, 64, 8)   # [et*nchunk + c][plane][lane][8]
    nchunk = (H + 31) // 32
    assert planes.shape[0] == ((E + 15) // 16) * nchunk
    seen = np.zeros((E, H), bool)
    for f in range(planes.shape[0]):
        et, c = divmod(f, nchunk)
        for lane in range(64):
            row = et * 16 + lane % 16
            cols = c * 32 + 8 * (lane // 16) + np.arange(8)
            hi, mid, lo = planes[f, 0, lane], planes[f, 1, lane], planes[f, 2, lane]
            if row >= E or cols[0] >= H:
                assert not hi.any() and not mid.any() and not lo.any(), (f, lane)
                continue
            w = src[row, cols]
            assert np.array_equal(hi, bf16_rne_np(w)), (f, lane)
            assert np.array_equal(mid, bf16_rne_np(w - hi)), (f, lane)
            assert np.array_equal(lo, bf16_rne_np((w - hi) - mid)), (f, lane)
            # the three planes rebuild the fp32 weight exactly
            assert np.array_equal((hi.astype(np.float64) + mid + lo).astype(np.float32), w), (f, lane)
            seen[row, cols] = True
    assert seen.all()


def test_pack_layout_documented(gpu):
    # fp32 stack whose values encode (e, n, k): check the documented fragment layout
    E, N, K = 2, 32, 48
    e_, n_, k_ = np.meshgrid(np.arange(E), np.arange(N), np.arange(K), indexing="ij")
    src = (e_ * 1e6 + n_ * 1e3 + k_).astype(np.float32)
    packed = ops.pack_expert_weights(f32(src)).cpu().numpy().reshape(-1, 4)   # 16-B pieces
    kc_per_row = K * 4 // 64
    for piece in range(0, packed.shape[0], 7):
        lane = piece % 64
        frag = piece // 64
        kc = frag % kc_per_row
        nt = (frag // kc_per_row) % (N // 16)
        e = frag // kc_per_row // (N // 16)
        row = nt * 16 + lane % 16
        col = kc * 16 + (lane // 16) * 4
        assert np.array_equal(packed[piece], src[e, row, col:col + 4]), piece


# ---------------------------------------------------------------------------
# end to end through VerifyLayer (route -> select -> forward)
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("name,rho", [("fp32_small", 0.9), ("qwen3_30b_a3b", 0.9), ("qwen3_30b_a3b", 0.0),
                                      ("wide_offload", 0.9), ("batched_8x64", 0.9)])
def test_end_to_end(gpu, name, rho):
    cfg = W.CONFIGS[name]
    blk = W.make_block(cfg, block=2, rho=rho)
    hdev, h64 = hidden_for(cfg, blk.hidden)
    rw = W.router_weights(cfg)
    wg, wu, wd = W.expert_weights_torch(cfg, 0, DEV)
    layer = ops.VerifyLayer(f32(rw), wg, wu, wd, cfg.k, max_tokens=cfg.total_tokens, max_trees=cfg.B)
    say(f"end to end {name} rho={rho}")
    hd = to_dev_hidden(cfg, hdev)
    logits, sel, out = layer.step(hd, i32(blk.parent), i32(blk.depth), f32(blk.prob), blk.offsets.tolist(),
                                  u8(blk.resident))
    torch.cuda.synchronize()
    z_gpu = logits.cpu().numpy()
    z_ref64 = O.route(h64, rw.astype(np.float64))
    assert normwise_rel(z_gpu, z_ref64) <= LOGIT_TOL
    ref = O.select(z_ref64.astype(np.float32), blk.parent, blk.depth, blk.prob, blk.offsets, cfg.k,
                   resident=blk.resident)
    assert not ref["ambiguous"].any()
    got_idx = sel["idx"].cpu().numpy()
    assert np.array_equal(sel["eligible"].cpu().numpy(), ref["eligible"])
    assert np.array_equal(got_idx, ref["idx"])
    y_ref = O.moe_forward_grouped(h64, HostExperts(wg), HostExperts(wu), HostExperts(wd), ref["idx"],
                                  ref["gate"], cfg.dtype)
    y = out.cpu().numpy()
    check_forward(y, y_ref, cfg.dtype, f"end to end {name} rho={rho}")
    if cfg.B > 1:
        # each tree has its own eligible set and statistics
        assert np.array_equal(sel["stats"].cpu().numpy()[:, :L.NUM_STATS - 1], ref["stats"][:, :L.NUM_STATS - 1])
        assert len({tuple(r) for r in ref["eligible"].tolist()}) > 1
    # determinism: a second step gives bit-identical results
    logits2, sel2, out2 = layer.step(hd, i32(blk.parent), i32(blk.depth), f32(blk.prob), blk.offsets.tolist(),
                                     u8(blk.resident))
    torch.cuda.synchronize()
    assert np.array_equal(out2.cpu().numpy().view(np.uint32), y.view(np.uint32))
    assert np.array_equal(sel2["idx"].cpu().numpy(), got_idx)


# ---------------------------------------------------------------------------
# HIP graph capture of a whole step: every replay equals the eager result
# ---------------------------------------------------------------------------
# VerifyLayer.step makes the three calls itself: the same bits as route(),
# select() and moe_forward(), at the layer's full size and below it, on another
# stream, and larger or mistyped blocks refused before anything is launched.
# Each step finds its buffers poisoned, and the other stream's step gets inputs
# that only that stream's own queue has written and is waited for alone.
def test_step_matches_separate_calls(gpu):
    cfg = W.LayerConfig("step", 88, "bf16", T=12, B=3, H=256, E=24, k=4, I=96, depth_max=6,
                        commit_rule="depth_sibling", hidden_std=1.0)
    blk = W.make_block(cfg)
    hdev, _ = hidden_for(cfg, blk.hidden)
    wg, wu, wd = W.expert_weights_torch(cfg, 0, DEV)
    layer = ops.VerifyLayer(f32(W.router_weights(cfg)), wg, wu, wd, cfg.k, max_tokens=36, max_trees=3, budget=9,
                            mode=L.MODE_FIXED_BUDGET)
    side = torch.cuda.Stream()
    busy = torch.randn(2048, 2048, device=DEV)
    for B, stream in ((3, None), (1, None), (2, side), (3, side)):
        T = 12 * B
        hid, par, dep, pr = (to_dev_hidden(cfg, hdev[:T]), i32(blk.parent[:T]), i32(blk.depth[:T]), f32(blk.prob[:T]))
        offs = blk.offsets[:B + 1] if B > 1 else None
        z = ops.route(hid, layer.router)
        sel = ops.select(z, par, dep, pr, offs, cfg.k, 0.5, L.MODE_FIXED_BUDGET, 9)
        y = ops.moe_forward(hid, layer.wgu, layer.wd, sel["idx"], sel["gate"])
        for t in (layer.logits, layer.out, layer.sel_out["gate"]):
            t.fill_(float("nan"))
        for t in (layer.sel_ws, layer.fwd_ws, layer.sel_out["eligible"]):
            t.fill_(0xFF)
        for t in (layer.sel_out["idx"], layer.sel_out["stats"]):
            t.fill_(-7)
        late = torch.zeros_like(hid)
        torch.cuda.synchronize()
        if stream is None:
            logits, outs, out = layer.step(hid, par, dep, pr, offs)
            torch.cuda.synchronize()
        else:
            with torch.cuda.stream(stream):
                for _ in range(40):
                    busy = (busy @ busy).clamp_(-1.0, 1.0)
                late.copy_(hid)
            logits, outs, out = layer.step(late, par, dep, pr, offs, stream=stream)
            stream.synchronize()
        with torch.cuda.stream(stream if stream is not None else torch.cuda.current_stream()):
            got = [t.clone() for t in (logits, out, *(outs[key] for key in sel))]
        torch.cuda.synchronize()
        assert logits.shape == z.shape and out.shape == y.shape
        for name, t, want in zip(("logits", "out", *sel), got, (z, y, *sel.values())):
            assert torch.equal(t, want), (name, B)
    hid, par, dep, pr = (to_dev_hidden(cfg, hdev), i32(blk.parent), i32(blk.depth), f32(blk.prob))
    with pytest.raises(ValueError):
        layer.step(torch.cat([hid, hid]), par, dep, pr)
    with pytest.raises(ValueError):
        layer.step(hid, par, dep, pr, [0, 9, 18, 27, 36])
    with pytest.raises(ValueError):
        layer.step(hid[:, :128].contiguous(), par, dep, pr)
    with pytest.raises(TypeError):
        layer.step(hid.float(), par, dep, pr)
    with pytest.raises(TypeError):
        layer.step(hid, par.long(), dep, pr)


def test_graph_replay_matches_eager(gpu):
    cfg = W.CONFIGS["qwen3_30b_a3b"]
    rw = W.router_weights(cfg)
    wg, wu, wd = W.expert_weights_torch(cfg, 0, DEV)
    layer = ops.VerifyLayer(f32(rw), wg, wu, wd, cfg.k, max_tokens=cfg.T)
    blocks = []
    for b in range(2):
        blk = W.make_block(cfg, block=b)
        hdev, _ = hidden_for(cfg, blk.hidden)
        blocks.append((to_dev_hidden(cfg, hdev), i32(blk.parent), i32(blk.depth), f32(blk.prob)))

    def snap():
        return (layer.out[:cfg.T].clone(), layer.sel_out["idx"][:cfg.T].clone(),
                layer.sel_out["eligible"][:1].clone())

    layer.step(*blocks[0])
    torch.cuda.synchronize()
    ref = snap()
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            layer.step(*blocks[0])
    torch.cuda.synchronize()
    say("graph replay vs eager")
    for rep in range(3):
        layer.step(*blocks[1])          # eager work on other inputs in between
        torch.cuda.synchronize()
        other = snap()
        assert not torch.equal(other[0], ref[0])
        g.replay()
        torch.cuda.synchronize()
        got = snap()
        for a, b in zip(got, ref):
            assert torch.equal(a, b), f"replay {rep} differs"
