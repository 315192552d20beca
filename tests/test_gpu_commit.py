"""Cache commit along plans with many destinations per source, against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,trees,W_cap,L,Hkv,D,head_major,per", [
    (1, 1, 64, 33, 1, 8, False, 3),        # one source for every slot; pieces that fill no load round; a chunk of one token
    (1, 8, 16, 256, 8, 128, False, 3),     # whole chunks
    (3, 3, 5, 17, 3, 40, True, 3),         # odd piece counts, a token behind a chunk, several prompts
    (40, 2, 4, 7, 2, 16, False, 3),        # fewer tokens than a chunk
    (2, 2, 3, 0, 2, 16, False, 3),         # empty caches: path rows alone
    (1, 2, 4, 40, 40, 128, True, 3),       # more pieces than one round of loads takes
    (1, 8, 16, 32, 40, 128, False, 64),    # long paths: several units each, fewer and ...
    (3, 2, 64, 5, 3, 40, True, 61),        # ... more of them than a prompt has workgroups; units cut short
    (2, 3, 7, 0, 2, 16, False, 9),         # a unit of one token
])
def test_commit_plans_with_shared_sources(P, trees, W_cap, L, Hkv, D, head_major, per):
    import paper_2409_16560_amd as dsbd
    from oracle import commit as o_commit
    rng = np.random.default_rng(P * 1000 + L)
    T, depth = P * trees, per - 1
    N = T * per
    cap = L + depth + 1
    gen = torch.Generator().manual_seed(7)
    shape = (T, Hkv, cap, D) if head_major else (T, cap, Hkv, D)
    view = lambda pool, i, n: pool[i, :, :n] if head_major else pool[i, :n]      # noqa: E731
    src = [torch.randn(shape, generator=gen).to(torch.bfloat16) for _ in range(2)]
    tree = [torch.randn((N, Hkv, D), generator=gen).to(torch.bfloat16) for _ in range(2)]
    lens = [max(0, L - int(x)) for x in rng.integers(0, 4, T)]
    n_next = rng.integers(0, W_cap + 1, P).astype(np.int32)
    n_next[0] = W_cap
    src_tree = np.full((P, W_cap), -1, dtype=np.int32)
    path_len = np.zeros((P, W_cap), dtype=np.int32)
    path = np.full((P, W_cap, depth + 1), -1, dtype=np.int32)
    for p in range(P):
        for s in range(int(n_next[p])):
            b = p * trees + int(trees * rng.random() ** 3)
            src_tree[p, s], path_len[p, s] = b, int(rng.integers(0, depth + 2))
            path[p, s, :path_len[p, s]] = b * per + np.arange(path_len[p, s])
    bits = lambda t: t.contiguous().view(torch.int16).cpu().numpy()      # noqa: E731
    own = lambda x, i: bits(view(x, i, lens[i]).transpose(0, 1) if head_major else view(x, i, lens[i]))      # noqa: E731
    rk, rv, rlen = o_commit.commit_kv([own(src[0], i) for i in range(T)], [own(src[1], i) for i in range(T)],
                                      bits(tree[0]), bits(tree[1]), n_next, src_tree, path_len, path)
    dev = [x.cuda() for x in src]
    kv = dsbd.PrefixKV([view(dev[0], i, lens[i]) for i in range(T)], [view(dev[1], i, lens[i]) for i in range(T)],
                       head_major=head_major)
    kv.token_stride, kv.head_stride = (D, cap * D) if head_major else (Hkv * D, D)       # (also where every cache is empty)
    kv.max_len = max(lens)
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()      # noqa: E731
    forest = dsbd.Forest(np.repeat(np.arange(P), trees).astype(np.int32), (np.arange(T + 1) * per).astype(np.int32),
                         np.where(np.arange(N) % per == 0, -1, np.arange(N) - 1).astype(np.int32), None, n_prompts=P,
                         max_tree_nodes=per, max_depth=depth, max_prompt_trees=trees, device="cuda")
    plan = dsbd.NextBeams.allocate(forest, W_cap)
    plan.n_next, plan.src_tree, plan.path_len, plan.path = i32(n_next), i32(src_tree), i32(path_len), i32(path)
    # the first destination of a tree continues in its buffer (of every second tree in one plane only)
    pool = [torch.full((P * W_cap,) + shape[1:], -1.0, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    dst, taken = ([], []), set()
    for j in range(P * W_cap):
        b = int(src_tree.reshape(-1)[j])
        first = b >= 0 and b not in taken
        taken.add(b)
        for plane in range(2):
            stays = first and (plane == 0 or b % 2 == 0)
            dst[plane].append(dev[plane][b] if stays else pool[plane][j])
    out = dsbd.KVDst(dst[0], dst[1], kv, head_major=head_major)
    n, fault = dsbd.dsbd_commit_kv(forest, kv, tree[0].cuda(), tree[1].cuda(), plan, W_cap, out)
    torch.cuda.synchronize()
    assert int(fault.item()) == 0
    assert np.array_equal(n.cpu().numpy(), rlen)
    for (p, s), want in rk.items():
        for plane, ref in ((0, want), (1, rv[(p, s)])):
            got = dst[plane][p * W_cap + s]
            got = got[:, :ref.shape[0]].transpose(0, 1) if head_major else got[:ref.shape[0]]
            assert np.array_equal(bits(got), ref), (p, s, plane)
    # nothing behind a destination's length, and no unused slot, is touched
    for j in range(P * W_cap):
        for plane in range(2):
            t = pool[plane][j]
            rest = t[:, int(rlen.reshape(-1)[j]):] if head_major else t[int(rlen.reshape(-1)[j]):]
            assert bool((rest == -1.0).all())


def test_commit_with_a_far_bound_on_the_lengths():
    """A caller's bound on the cache lengths may be far above them: as many chunks as one dimension of a launch holds."""
    import paper_2409_16560_amd as dsbd
    gen = torch.Generator().manual_seed(3)
    src = [torch.randn((20, 1, 8), generator=gen).to(torch.bfloat16).cuda() for _ in range(2)]
    tree = [torch.randn((1, 1, 8), generator=gen).to(torch.bfloat16).cuda() for _ in range(2)]
    i32 = lambda *a: torch.tensor(a, dtype=torch.int32, device="cuda")      # noqa: E731
    forest = dsbd.Forest(np.zeros(1, np.int32), np.array([0, 1], np.int32), np.array([-1], np.int32), None, n_prompts=1,
                         max_tree_nodes=1, max_depth=0, max_prompt_trees=1, device="cuda")
    kv = dsbd.PrefixKV([src[0][:19]], [src[1][:19]])
    kv.max_len = (1 << 27) + 1
    plan = dsbd.NextBeams.allocate(forest, 1)
    plan.n_next, plan.src_tree, plan.path_len, plan.path = i32(1), i32([0]), i32([1]), i32([[0]])
    dst = [torch.full((20, 1, 8), -1.0, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    n, fault = dsbd.dsbd_commit_kv(forest, kv, tree[0], tree[1], plan, 1, dsbd.KVDst([dst[0]], [dst[1]], kv))
    torch.cuda.synchronize()
    assert int(fault.item()) == 0 and int(n.item()) == 20
    for plane in range(2):
        assert torch.equal(dst[plane][:19], src[plane][:19]) and torch.equal(dst[plane][19], tree[plane][0])
