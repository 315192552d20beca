"""The workloads this library is timed on, and the inputs they run on.

One decoding iteration of dynamic-width speculative beam decoding calls the library in this order: draft steps and
forest layout, forest attention (once per transformer layer), verification with the selection of the next beams, cache
commit.  The cases take these calls through the public entry points at the sizes of the repository's own
configurations (c1 .. c5 of dsbd_synth) and of shapes between and around them: batches, ragged lengths, both cache
layouts, both head dimensions, odd vocabularies, fixed and dynamic width, with and without warping.

A case is a dict of plain values.  `topo` seeds what a pass's work depends on (trees, prefix lengths, the plan of a
commit); every value in the inputs comes from the seed given to prepare().
"""
import numpy as np
import torch

import paper_2409_16560_amd as dsbd

DEV = "cuda"

BASE = {
    "kind": "step",          # step | attention | verify | draft | commit
    "prompts": 1,
    "beams_lo": 4, "beams_hi": 4,        # input beams per prompt
    "tree": "random",        # chain | fork_chain | binary | random | sampled (layers of draws, as the draft stage lays out)
    "nodes_lo": 8, "nodes_hi": 8,        # nodes per tree (sampled: draws per layer)
    "gamma": 3,              # draft depth (sampled trees and the draft stage)
    "prefix_lo": 512, "prefix_hi": 512,  # prefix tokens per beam (equal within a prompt)
    "shared": 0,             # leading tokens of the prefix that the beams of a prompt share
    "heads": 32, "kv_heads": 32, "dim": 128,
    "head_major": False,     # caches [Hkv, L, D] instead of [L, Hkv, D]
    "vocab": 32000,
    "independent": False,    # draft logits independent of the target's (else: the target's plus noise)
    "t": -1.0,               # threshold of the dynamic width; < 0: fixed width
    "top_k": 0, "top_p": 1.0,
    "keep_one": False,       # one cache survives (Section 3.4)
    "keep_buffers": True,    # the caller keeps outputs and workspaces; else the calls allocate them
    "topo": 1,
}


def _case(name=None, **kw):
    c = dict(BASE, **kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call anybody makes: two three-token chains behind a short prompt, a toy vocabulary (c1); launches
        # and host work are all there is
        _case("step_tiny", beams_lo=2, beams_hi=2, tree="chain", nodes_lo=3, nodes_hi=3, prefix_lo=32, prefix_hi=32,
              heads=4, kv_heads=4, dim=64, vocab=256, independent=True),
        # an early iteration of one interactive request (c2)
        _case("step_small", tree="fork_chain", nodes_lo=7, nodes_hi=7),
        # one request of ordinary length whose beams share the prompt's half of the cache (c3)
        _case("step_shared_prefix", beams_lo=8, beams_hi=8, tree="binary", nodes_lo=15, nodes_hi=15, prefix_lo=2048,
              prefix_hi=2048, shared=1024),
        # a serving batch of unequal requests (c4): the largest amount of data
        _case("step_batch", prompts=16, beams_lo=1, beams_hi=8, nodes_lo=4, nodes_hi=16, prefix_lo=1024, prefix_hi=4096),
        # one long request with grouped heads and the large vocabulary (c5), fixed width
        _case("step_large", beams_lo=8, beams_hi=8, tree="binary", nodes_lo=31, nodes_hi=31, prefix_lo=8192,
              prefix_hi=8192, kv_heads=8, vocab=128256),
        # the same vocabulary in the setting of the paper's experiments: a forest as the draft stage samples it, top-k 10
        # / top-p 0.8 on the joints, dynamic width
        _case("step_warped_dynamic", beams_lo=5, beams_hi=5, tree="sampled", nodes_lo=12, nodes_hi=12, gamma=4,
              prefix_lo=3001, prefix_hi=3001, kv_heads=8, vocab=128256, t=0.9, top_k=10, top_p=0.8),
        # one transformer layer's attention of a small batch: head-major caches, head dimension 64, ragged everything,
        # nothing kept by the caller
        _case("attention_ragged_64", kind="attention", prompts=5, beams_lo=1, beams_hi=6, nodes_lo=2, nodes_hi=13,
              prefix_lo=700, prefix_hi=3000, kv_heads=8, dim=64, head_major=True, keep_buffers=False),
        # ... and of one very long request with few beams, where the cache has to be split to fill the chip
        _case("attention_long", kind="attention", beams_lo=2, beams_hi=2, nodes_lo=23, nodes_hi=23, prefix_lo=49151,
              prefix_hi=49151, kv_heads=8),
        # verification alone with the dynamic width, a vocabulary that no row length divides, one surviving cache
        _case("verify_dynamic_odd", kind="verify", prompts=3, beams_lo=3, beams_hi=6, tree="sampled", nodes_lo=10,
              nodes_hi=10, vocab=50273, t=0.7, keep_one=True),
        # the draft stage of one request: four sampling steps of sixteen draws, warped, and the forest's layout
        _case("draft_warped", kind="draft", beams_lo=8, beams_hi=8, nodes_lo=16, nodes_hi=16, gamma=4, vocab=128256,
              top_k=10, top_p=0.8),
        # the draft stage of a batch without warping
        _case("draft_batch", kind="draft", prompts=8, beams_lo=1, beams_hi=6, nodes_lo=8, nodes_hi=8, gamma=3),
        # the caches following the output beams of the long request: most of them copied whole
        _case("commit_large", kind="commit", beams_lo=8, beams_hi=8, tree="binary", nodes_lo=31, nodes_hi=31,
              prefix_lo=8192, prefix_hi=8192, kv_heads=8),
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over the logarithm."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    # no case above the largest listed one, neither in data nor in arithmetic
    most = max(work(c)["bytes"] for c in listed())
    most_flops = max(work(c)["flops"] for c in listed())
    while True:
        kind = rng.choice(["step"] * 4 + ["attention"] * 2 + ["verify"] * 2 + ["draft"] * 2 + ["commit"])
        vocab = rng.choice([32000, 50273, 128256, _log(rng, 256, 140000)])
        heads, kv_heads = rng.choice([(32, 32), (32, 8), (32, 8), (16, 4), (40, 40), (4, 4)])
        warped = rng.random() < 0.4
        tree = rng.choice(["chain", "fork_chain", "binary", "random", "sampled", "sampled"])
        prompts = rng.choice([1, 1, 1, _log(rng, 1, 16)])
        beams_lo = rng.randint(1, 8)
        prefix = _log(rng, 32, 49151 if kind == "attention" and prompts == 1 else 8192)
        if kind == "draft":
            nodes_lo = nodes_hi = rng.choice([4, 8, 16, rng.randint(2, 16)])
        elif tree == "binary":
            nodes_lo = nodes_hi = rng.choice([3, 7, 15, 31])
        elif tree == "sampled":
            nodes_lo = nodes_hi = rng.randint(3, 15)
        elif tree == "random":
            nodes_lo, nodes_hi = 2, rng.randint(3, 31)
        else:
            nodes_lo = nodes_hi = rng.randint(2, 8)
        c = _case(
            kind=kind, prompts=prompts, beams_lo=beams_lo, beams_hi=rng.randint(beams_lo, 8), tree=tree,
            nodes_lo=nodes_lo, nodes_hi=nodes_hi, gamma=rng.randint(2, 4 if kind != "draft" else 3),
            prefix_lo=max(16, int(prefix * rng.uniform(0.4, 1.0))), prefix_hi=prefix,
            shared=int(prefix * rng.uniform(0.1, 0.4)) if rng.random() < 0.3 else 0,
            heads=heads, kv_heads=kv_heads, dim=rng.choice([128, 128, 64]), head_major=rng.random() < 0.25,
            vocab=vocab, independent=rng.random() < 0.15, t=rng.choice([-1.0, -1.0, 0.9, 0.7]),
            top_k=rng.choice([10, 10, rng.randint(2, 32)]) if warped else 0, top_p=rng.choice([0.8, 0.8, 0.95]) if warped else 1.0,
            keep_one=rng.random() < 0.2, keep_buffers=rng.random() < 0.75, topo=rng.randint(1, 1 << 20))
        w = work(c)
        if w["bytes"] <= most and w["flops"] <= most_flops:
            return c


# ------------------------------------------------------------------------------------------------ shapes

def _tree(kind, n, rng):
    if kind == "chain":
        return [-1] + list(range(n - 1))
    if kind == "fork_chain":
        return ([-1, 0, 0] + [i - 2 for i in range(3, n)])[:n]
    if kind == "binary":                       # complete, depth first
        out = []

        def rec(par, size):
            me = len(out)
            out.append(par)
            if size > 1:
                rec(me, (size - 1) // 2)
                rec(me, (size - 1) // 2)
        rec(-1, n)
        return out
    return [-1] + [int(rng.integers(0, i)) for i in range(1, n)]


class Shape:
    """Trees and lengths of a case: host arrays, a function of the case alone."""

    def __init__(self, c):
        rng = np.random.default_rng(c["topo"])
        self.tree_prompt, self.tree_off, parent, rank, self.length, self.beams = [], [0], [], [], [], []
        for p in range(c["prompts"]):
            W = int(rng.integers(c["beams_lo"], c["beams_hi"] + 1))
            L = int(rng.integers(c["prefix_lo"], c["prefix_hi"] + 1))
            self.beams.append(W)
            if c["tree"] == "sampled":
                # layers of draws: a draw's parent is one of the layer before, some beams far likelier than others;
                # laid out tree by tree, inside a tree by (layer, draw)
                S, trees, last = c["nodes_lo"], [[(-1, 0)] for _ in range(W)], [(b, 0) for b in range(W)]
                for _ in range(c["gamma"]):
                    wt = rng.exponential(1.0, len(last)) ** 1.5
                    src = rng.choice(len(last), S, p=wt / wt.sum())
                    nxt = []
                    for j in range(S):
                        b, par = last[int(src[j])]
                        trees[b].append((par, j))
                        nxt.append((b, len(trees[b]) - 1))
                    last = nxt
            else:
                trees = []
                for _ in range(W):
                    n = int(rng.integers(c["nodes_lo"], c["nodes_hi"] + 1))
                    trees.append([(a, i) for i, a in enumerate(_tree(c["tree"], n, rng))])
            for tr in trees:
                base = self.tree_off[-1]
                parent += [-1 if a < 0 else a + base for a, _ in tr]
                rank += [r for _, r in tr]
                self.tree_off.append(base + len(tr))
                self.tree_prompt.append(p)
                self.length.append(L)
        self.rank = rank if c["tree"] == "sampled" else None
        self.parent = np.asarray(parent, dtype=np.int64)
        self.n_trees, self.n_nodes = len(self.tree_prompt), len(parent)
        depth = np.zeros(self.n_nodes, dtype=np.int64)
        for i, a in enumerate(self.parent):
            depth[i] = 0 if a < 0 else depth[a] + 1
        self.depth, self.max_depth = depth, int(depth.max())
        self.sizes = np.diff(self.tree_off)
        self.shared = [min(c["shared"], L) for L in self.length]
        self.own = [L - s for L, s in zip(self.length, self.shared)]
        self.W_cap = max(16, max(self.beams))
        self.rng = rng

    def unique_tokens(self):
        first = {}
        for t in range(self.n_trees):
            first.setdefault(self.tree_prompt[t], self.shared[t])
        return sum(self.own) + sum(first.values())


def _plan(s):
    """A next-beam plan as the selection writes it: some beams leave no output, others several."""
    rows = []
    for p in range(len(s.beams)):
        trees = [t for t in range(s.n_trees) if s.tree_prompt[t] == p]
        wt = s.rng.exponential(1.0, len(trees)) ** 1.5
        out = []
        for _ in range(len(trees)):
            t = trees[int(s.rng.choice(len(trees), p=wt / wt.sum()))]
            n, path = int(s.rng.integers(s.tree_off[t], s.tree_off[t + 1])), []
            while n >= 0:
                path.append(n)
                n = int(s.parent[n])
            out.append((t, path[::-1]))
        rows.append(out)
    return rows


def work(c):
    """Bytes and operations of a pass: every input read once, every output written once."""
    s = Shape(c)
    tok, V, row = 2 * c["kv_heads"] * c["dim"] * 2, c["vocab"], c["heads"] * c["dim"] * 2
    nbytes = flops = 0.0
    if c["kind"] in ("step", "attention"):
        nbytes += (s.unique_tokens() + s.n_nodes) * tok + s.n_nodes * (2 * row + 4 * c["heads"])
        seen = float(sum(int(s.sizes[t]) * s.length[t] for t in range(s.n_trees)) + int((s.depth + 1).sum()))
        flops += 4.0 * c["heads"] * c["dim"] * seen
    if c["kind"] in ("step", "verify"):
        nbytes += 2.0 * s.n_nodes * V * 4 + s.n_nodes * 24
        flops += 2.0 * s.n_nodes * V * 3
    if c["kind"] == "draft":
        rows = sum(s.beams) + (c["gamma"] - 1) * c["prompts"] * c["nodes_lo"]
        nbytes += 4.0 * rows * V + 24.0 * c["gamma"] * c["prompts"] * c["nodes_lo"]
        flops += 3.0 * rows * V
    if c["kind"] == "commit":
        taken, read, paths = set(), set(), set()
        for out in _plan(s):
            for t, path in out:
                nbytes += len(path) * tok
                paths.update(path)
                if t in taken:
                    nbytes += s.own[t] * tok
                    read.add(t)
                taken.add(t)
        nbytes += sum(s.own[t] for t in read) * tok + len(paths) * tok
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(c):
    # Decisions (tokens, beams, statuses, widths) are taken in fp64 and are whole numbers: none may differ.
    if c["kind"] in ("step", "attention"):
        # bf16 outputs of bf16 products: against the same attention in 64 bits 2.3e-3 (largest 8.6e-3 of the root mean
        # square), most of it the rounding of the output itself
        return {"rel": 1e-2, "max": 0.035}
    if c["kind"] == "verify":
        # log-sum-exps and log-probabilities in 32 bits: 1.2e-7 (largest 2.6e-7) against 64 bits
        return {"rel": 5e-7, "max": 1e-6}
    if c["kind"] == "draft":
        return {"rel": 1e-12, "max": 1e-11}    # fp64 likelihoods: 2e-15 against another order of the sums
    return "exact"


# ------------------------------------------------------------------------------------------------ inputs

class State:
    pass


def _uniform(gen, shape):
    """24-bit uniforms in [0, 1)."""
    return torch.randint(0, 1 << 24, shape, generator=gen, device=DEV, dtype=torch.int32).to(torch.float32) * (1.0 / (1 << 24))


def _caches(c, gen, lens, capacity=None):
    """One cache per entry of lens, as views of one pool."""
    H, D = c["kv_heads"], c["dim"]
    cap = max(max(lens), 1) if capacity is None else capacity
    if c["head_major"] or capacity is not None:
        shape = (len(lens), H, cap, D) if c["head_major"] else (len(lens), cap, H, D)
        pool = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
        pool.normal_(generator=gen)
        return pool, [pool[i, :, :n] if c["head_major"] else pool[i, :n] for i, n in enumerate(lens)]
    pool = torch.empty((sum(lens), H, D), dtype=torch.bfloat16, device=DEV)
    pool.normal_(generator=gen)
    return pool, list(torch.split(pool, lens))


def _forest(c, s, token):
    return dsbd.Forest(np.asarray(s.tree_prompt, dtype=np.int32), np.asarray(s.tree_off, dtype=np.int32),
                       s.parent.astype(np.int32), token, None if s.rank is None else np.asarray(s.rank, dtype=np.int32),
                       n_prompts=c["prompts"], max_tree_nodes=int(s.sizes.max()), max_depth=s.max_depth,
                       max_prompt_trees=max(s.beams), device=DEV)


def _logits(c, gen, n):
    z = torch.empty((n, c["vocab"]), dtype=torch.float32, device=DEV).normal_(generator=gen)
    return z.mul_(2.0 if c["vocab"] < 1000 else 3.0)


def _prepare_attention(c, s, gen, st):
    def tree_rows(heads):
        return torch.empty((s.n_nodes, heads, c["dim"]), dtype=torch.bfloat16, device=DEV).normal_(generator=gen)
    st.q, st.k_tree, st.v_tree = tree_rows(c["heads"]), tree_rows(c["kv_heads"]), tree_rows(c["kv_heads"])
    cap = None
    st.pools, ks, vs, shared = [], None, None, {}
    if max(s.shared) > 0:
        cap = max(s.length)                     # one capacity: the strides are common to all segments
        pk, k = _caches(c, gen, [s.shared[s.tree_prompt.index(p)] for p in range(c["prompts"])], cap if c["head_major"] else None)
        pv, v = _caches(c, gen, [s.shared[s.tree_prompt.index(p)] for p in range(c["prompts"])], cap if c["head_major"] else None)
        st.pools += [pk, pv]
        shared = dict(k_shared=[k[p] for p in s.tree_prompt], v_shared=[v[p] for p in s.tree_prompt])
    pk, ks = _caches(c, gen, s.own, cap if c["head_major"] else None)
    pv, vs = _caches(c, gen, s.own, cap if c["head_major"] else None)
    st.pools += [pk, pv]
    st.kv = dsbd.PrefixKV(ks, vs, head_major=c["head_major"], **shared)
    st.attn = {}
    if c["keep_buffers"]:
        st.attn = {
            "out": torch.empty_like(st.q), "lse": torch.empty((s.n_nodes, c["heads"]), dtype=torch.float32, device=DEV),
            "workspace": torch.empty(dsbd.dsbd_forest_attention_workspace_bytes(st.forest, st.kv, c["heads"], c["kv_heads"], c["dim"]),
                                     dtype=torch.uint8, device=DEV),
            "fault": torch.zeros(1, dtype=torch.int32, device=DEV)}


def _prepare_verify(c, s, gen, st):
    N, T, V = s.n_nodes, s.n_trees, c["vocab"]
    st.zp = _logits(c, gen, N)
    st.zq = _logits(c, gen, N)
    if not c["independent"]:
        st.zq.mul_(0.5 / 3.0).add_(st.zp)
    # a draft token is a draw of the small model at its parent, among its leading entries where that model is cut too
    par = torch.from_numpy(np.maximum(s.parent, 0)).to(DEV)
    if c["top_k"] > 0:
        k = min(c["top_k"], V)
        val, idx = torch.topk(st.zq, k, dim=1)
        val, idx = val[par], idx[par]
        u = torch.rand((N, k), generator=gen, device=DEV).clamp_(1e-7, 1.0 - 1e-7)
        token = idx.gather(1, (val - torch.log(-torch.log(u))).argmax(1, keepdim=True)).squeeze(1)
    else:
        token = torch.empty(N, dtype=torch.int64, device=DEV)
        for i in range(0, N, 64):
            z = st.zq[par[i:i + 64]]
            e = torch.empty_like(z).exponential_(generator=gen)
            token[i:i + 64] = (z - torch.log(e)).argmax(1)
    st.token = token.to(torch.int32)
    st.blp = -3.0 * torch.rand(T, generator=gen, device=DEV, dtype=torch.float64)
    noise = torch.empty(T, dtype=torch.float64, device=DEV).normal_(generator=gen)
    st.blq = st.blp + 0.25 * noise
    st.u_accept = _uniform(gen, (N,))
    st.u_resid = _uniform(gen, (c["prompts"], s.max_depth + 2))
    st.u_fill = _uniform(gen, (c["prompts"], s.max_depth + 2, s.W_cap))


def _zeroed(record):
    """Slots that a call leaves alone hold zeros (only the written ones mean anything)."""
    for v in vars(record).values():
        if isinstance(v, torch.Tensor):
            v.zero_()
    return record


def prepare(case, seed):
    c, s, st = case, Shape(case), State()
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    st.c, st.s = c, s
    if c["kind"] == "draft":
        counts, W_S, P = s.beams, c["nodes_lo"], c["prompts"]
        st.root_off = torch.tensor(np.concatenate([[0], np.cumsum(counts)]), dtype=torch.int32, device=DEV)
        st.layer_off = torch.arange(P + 1, dtype=torch.int32, device=DEV) * W_S
        st.root_token = torch.randint(0, c["vocab"], (sum(counts),), generator=gen, device=DEV, dtype=torch.int32)
        st.z = [_logits(c, gen, sum(counts) if l == 0 else P * W_S) for l in range(c["gamma"])]
        st.cum = -3.0 * torch.rand(sum(counts), generator=gen, device=DEV, dtype=torch.float64)
        st.u = [_uniform(gen, (P, W_S)) for _ in range(c["gamma"])]
        return st
    if c["kind"] == "commit":
        st.forest = _forest(c, s, None)
        _prepare_commit(c, s, gen, st)
        return st
    st.token = None
    if c["kind"] in ("step", "verify"):
        _prepare_verify(c, s, gen, st)
    st.forest = _forest(c, s, st.token)
    if c["kind"] in ("step", "attention"):
        _prepare_attention(c, s, gen, st)
    if c["kind"] in ("step", "verify"):
        st.params = dict(t=c["t"], top_k=c["top_k"], top_p=c["top_p"], W_cap=s.W_cap)
        st.ver = {"result": _zeroed(dsbd.VerifyResult.allocate(st.forest, s.W_cap)),
                  "next_beams": _zeroed(dsbd.NextBeams.allocate(st.forest, s.W_cap))}
        if c["keep_buffers"]:
            n = dsbd.dsbd_verify_forest_workspace_bytes(st.forest, c["vocab"], 0, 1, s.W_cap, c["t"], c["top_k"], c["top_p"])
            st.ver["workspace"] = torch.empty(n, dtype=torch.uint8, device=DEV)
    return st


def _prepare_commit(c, s, gen, st):
    """Source caches with room to grow, a plan, and destinations: the first next beam of a tree continues in its
    buffer, every other one gets a fresh buffer (what the decode loop does)."""
    grow = s.max_depth + 1
    cap = max(s.own) + grow
    st.k_tree = torch.empty((s.n_nodes, c["kv_heads"], c["dim"]), dtype=torch.bfloat16, device=DEV).normal_(generator=gen)
    st.v_tree = torch.empty_like(st.k_tree).normal_(generator=gen)
    st.k_pool, k = _caches(c, gen, s.own, cap)
    st.v_pool, v = _caches(c, gen, s.own, cap)
    st.kv = dsbd.PrefixKV(k, v, head_major=c["head_major"])
    plan, P, W = _plan(s), c["prompts"], s.W_cap
    fresh = sum(len(o) - len({t for t, _ in o}) for o in plan)
    shape = (fresh,) + tuple(st.k_pool.shape[1:])
    st.k_new = torch.zeros(shape, dtype=torch.bfloat16, device=DEV)
    st.v_new = torch.zeros(shape, dtype=torch.bfloat16, device=DEV)
    i32 = lambda *sh: np.full(sh, -1, dtype=np.int32)   # noqa: E731
    n_next, src_tree, src_out, path_len, path = i32(P), i32(P, W), i32(P, W), np.zeros((P, W), dtype=np.int32), i32(P, W, s.max_depth + 1)
    dst_k, dst_v, used = [None] * (P * W), [None] * (P * W), 0
    for p, out in enumerate(plan):
        n_next[p], taken = len(out), set()
        for j, (t, pth) in enumerate(out):
            src_tree[p, j], src_out[p, j], path_len[p, j] = t, j, len(pth)
            path[p, j, :len(pth)] = pth
            if t in taken:
                dst_k[p * W + j], dst_v[p * W + j] = st.k_new[used], st.v_new[used]
                used += 1
            else:
                dst_k[p * W + j], dst_v[p * W + j] = st.k_pool[t], st.v_pool[t]
                taken.add(t)
    d = lambda a: torch.from_numpy(a).to(DEV)            # noqa: E731
    st.plan = dsbd.NextBeams.allocate(st.forest, W)
    st.plan.n_next, st.plan.src_tree, st.plan.src_out, st.plan.path_len, st.plan.path = map(d, (n_next, src_tree, src_out, path_len, path))
    st.dst = dsbd.KVDst(dst_k, dst_v, st.kv, head_major=c["head_major"])
    st.fault = torch.zeros(1, dtype=torch.int32, device=DEV)


# ------------------------------------------------------------------------------------------------ a pass

def _fields(record, skip=()):
    return {k: v for k, v in vars(record).items() if isinstance(v, torch.Tensor) and k not in skip}


def run(st):
    c, out = st.c, {}
    if c["kind"] == "draft":
        off, cum, width, par, tok = st.root_off, st.cum, max(st.s.beams), [], []
        for l in range(c["gamma"]):
            p_, t_, lp, fault = dsbd.dsbd_draft_layer(off, st.z[l], cum, st.u[l], c["nodes_lo"], max_prompt_beams=width,
                                                      top_k=c["top_k"], top_p=c["top_p"])
            par.append(p_.reshape(-1))
            tok.append(t_.reshape(-1))
            cum, off, width = lp.reshape(-1), st.layer_off, c["nodes_lo"]
            out["logp%d" % l], out["fault%d" % l] = lp, fault
        f, nr, no, mx, fault = dsbd.dsbd_build_forest(st.root_off, torch.stack(par), torch.stack(tok), st.root_token,
                                                      n_roots=int(st.root_token.numel()), max_prompt_trees=max(st.s.beams))
        out.update(tree_off=f.tree_off, parent=f.parent, token=f.token, rank=f.draft_rank, tree_prompt=f.tree_prompt,
                   node_of_root=nr, node_of=no, max_tree_nodes=mx, fault=fault)
        return out
    if c["kind"] == "commit":
        length, fault = dsbd.dsbd_commit_kv(st.forest, st.kv, st.k_tree, st.v_tree, st.plan, st.s.W_cap, st.dst, fault=st.fault)
        return {"k": st.k_pool, "v": st.v_pool, "k_new": st.k_new, "v_new": st.v_new, "len": length, "fault": fault}
    if c["kind"] in ("step", "attention"):
        o, lse, fault = dsbd.dsbd_forest_attention(st.forest, st.kv, st.q, st.k_tree, st.v_tree, **st.attn)
        out.update(attn=o, attn_lse=lse, attn_fault=fault)
    if c["kind"] in ("step", "verify"):
        res, nxt = dsbd.dsbd_verify_forest_select(st.forest, st.zp, st.zq, st.blp, st.blq, st.u_accept, st.u_resid,
                                                  st.u_fill, keep_one=c["keep_one"], **st.params, **st.ver)
        out.update(verified=_fields(res), next=_fields(nxt, skip=("fault",)))
    return out
