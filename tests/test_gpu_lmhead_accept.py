"""GPU parity: hb_tree_verify_attn_clearing + hb_lmhead_accept_cleared (LM head, acceptance and the append to
every layer's cache in two launches) give the oracle's results bit for bit, and so does hb_lmhead_accept."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import tree_accept_ref, kv_compact_ref
from parity import bits

pytestmark = pytest.mark.gpu


def _trees(kind):
    if kind == "mixed":  # a tree, no nodes, a lone root, the widest tree, a chain
        return [W.seeded_tree(1), np.array([], dtype=np.int32), W.chain_tree(1), W.seeded_tree(2, n_nodes=64), W.chain_tree(9)]
    return [W.chain_tree(4)] if kind == "one chain" else [W.seeded_tree(b) for b in range(16)]


@pytest.mark.parametrize("kind,dtype,layers,short", [
    ("mixed", "bf16", 3, 0), ("mixed", "f32", 1, 0), ("mixed", "bf16", 0, 0), ("mixed", "bf16", 1, 2),
    ("one chain", "f32", 1, 0), ("one chain", "bf16", 3, 1), ("16 trees", "bf16", 1, 0)])
def test_lm_head_acceptance_and_append(kind, dtype, layers, short):
    """short: max_path so many nodes below the deepest path; layers 3: through tables of pointers."""
    import paper_2509_18824_amd as hb
    import paper_2509_18824_amd.step as S
    Hq, Hkv, D, V = 8, 4, 128, 1000
    trees = _trees(kind)
    inps = [W.make_verify_inputs(50 + l, dtype, Hq, Hkv, D, [11 + 7 * b for b in range(len(trees))], trees, poison=False)
            for l in range(max(layers, 1))]
    inp = inps[0]
    T, max_path = inp.total_nodes, max(inp.max_path - short, 1)
    rng = np.random.default_rng(6)
    target = rng.integers(0, V, size=T)
    draft, _ = W.plant_draft_ids(6, [t for t in trees if len(t)], target, V)
    want = tree_accept_ref(inp.node_offset.numpy(), inp.parent.numpy(), draft, target, max_path)
    refs = [kv_compact_ref(bits(x.k_tree), bits(x.v_tree), bits(x.k_pool), bits(x.v_pool), inp.block_table.numpy(),
                           inp.prefix_len.numpy(), inp.node_offset.numpy(), want[0], want[1]) for x in inps]
    devs, desc = [S.to_device(x) for x in inps], S.desc_for(inp)
    dev, td = devs[0], devs[0].q.dtype
    # row t of the hidden states points at entry target[t] and nowhere else
    weight = torch.eye(V, Hq * D, dtype=td, device="cuda")
    hidden = weight[torch.from_numpy(target).cuda()].contiguous()
    i32 = lambda *shape: torch.full(shape, -7, dtype=torch.int32, device="cuda")
    B = len(trees)
    ids, alen, path, toks, bonus, slots, new_len = i32(T), i32(B), i32(B, max_path), i32(B, max_path), i32(B), i32(B, max_path), i32(B)
    keys = torch.full((8 * T,), 255, dtype=torch.uint8, device="cuda")  # larger than any key, were it not cleared
    table = lambda name: torch.tensor([getattr(d, name).data_ptr() for d in devs], dtype=torch.int64, device="cuda")
    names = ("k_tree", "v_tree", "k_pool", "v_pool")
    kv = [table(n) for n in names] if layers > 1 else [getattr(dev, n) for n in names]
    out, ref_out = torch.empty_like(dev.q), torch.empty_like(dev.q)
    ws = S.alloc_workspace(hb.hb_tree_verify_attn_workspace_bytes(desc))
    args = (desc, dev.q, dev.k_tree, dev.v_tree, dev.k_pool, dev.v_pool, dev.block_table, dev.prefix_len, dev.node_offset, dev.parent)
    hb.hb_tree_verify_attn(*args, ref_out, None, ws)
    hb.hb_tree_verify_attn_clearing(*args, out, None, ws, keys, T)
    assert not keys.any() and torch.equal(out.view(torch.uint8), ref_out.view(torch.uint8))
    hb.hb_lmhead_accept_cleared(desc, hidden, weight, torch.from_numpy(np.asarray(draft, dtype=np.int32)).cuda(), dev.node_offset,
                                dev.parent, max_path, ids, alen, path, toks, bonus, keys, layers, kv, dev.block_table,
                                dev.prefix_len, slots, new_len)
    torch.cuda.synchronize()
    assert np.array_equal(ids.cpu().numpy(), target)
    for got, ref in zip((alen, path, toks, bonus), want):
        assert np.array_equal(got.cpu().numpy(), ref)
    if layers:
        assert np.array_equal(slots.cpu().numpy(), refs[0][2]) and np.array_equal(new_len.cpu().numpy(), refs[0][3])
        for d, (ref_k, ref_v, _, _) in zip(devs, refs):
            assert np.array_equal(bits(d.k_pool), ref_k) and np.array_equal(bits(d.v_pool), ref_v)
    else:
        assert (slots == -7).all() and (new_len == -7).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_malformed_trees_and_rows_that_name_no_token(dtype):
    """The results of the three calls that it stands for, bit for bit, also for parents that do not precede their nodes or
    are below -1, drafted ids outside the vocabulary and rows without a logit that counts (all NaN, all -inf, one +inf)."""
    import paper_2509_18824_amd as hb
    import paper_2509_18824_amd.step as S
    K, V, n = 256, 500, 12
    trees = [W.seeded_tree(b, n_nodes=n, levels=4, root_fanout=4) for b in range(6)]
    inp = W.make_verify_inputs(8, dtype, 2, 1, 128, [5, 40, 17, 3, 64, 31], trees, poison=False)
    T, B, mp = inp.total_nodes, len(trees), inp.max_path
    rng = np.random.default_rng(2)
    parent = inp.parent.numpy().copy()
    parent[[3, n + 2, 2 * n + 5]] = [3, 7, 11]           # itself, a later node, the last
    parent[[3 * n + 4, 4 * n + 1]] = [-2, -2147483648]
    parent[5 * n] = 5                                    # a root with a parent
    g = torch.Generator().manual_seed(3)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    weight = torch.randn((V, K), generator=g).to(td)
    weight[:, 0] = 1.0
    hidden = torch.randn((T, K), generator=g).to(td)
    hidden[::7] = float("nan")
    hidden[2::9] = 0.0
    hidden[2::9, 0] = float("-inf")
    hidden[4::11, 3] = float("inf")
    dev, desc, weight, hidden = S.to_device(inp), S.desc_for(inp), weight.cuda(), hidden.cuda()
    par = torch.from_numpy(parent).cuda()
    i32 = lambda *shape: torch.full(shape, -7, dtype=torch.int32, device="cuda")
    new = lambda: (i32(T), i32(B), i32(B, mp), i32(B, mp), i32(B), i32(B, mp), i32(B))
    pools = [(dev.k_pool.clone(), dev.v_pool.clone()) for _ in range(3)]
    ids, alen, path, toks, bonus, slots, new_len = want = new()
    hb.hb_lmhead_argmax(hidden, weight, ids, None, S.alloc_workspace(8 * T))
    # drafted: the target's choice after the parent, where there is one, and here and there no token at all
    t = ids.cpu().numpy()
    off = inp.node_offset.numpy()
    draft = np.array([t[off[i // n] + max(parent[i], 0)] if 0 <= parent[i] < n else 1 for i in range(T)], dtype=np.int32)
    draft[rng.integers(0, T, 6)] = [-1, V, 2147483647, -2147483648, 0, 1]
    draft = torch.from_numpy(draft).cuda()
    hb.hb_tree_accept(B, n, dev.node_offset, par, draft, ids, mp, alen, path, toks, bonus)
    hb.hb_kv_compact(desc, dev.k_tree, dev.v_tree, *pools[0], dev.block_table, dev.prefix_len, dev.node_offset, alen, path, mp,
                     slots, new_len)
    for call, kv in ((hb.hb_lmhead_accept, pools[1]), (hb.hb_lmhead_accept_cleared, pools[2])):
        keys = torch.zeros(8 * T, dtype=torch.uint8, device="cuda")
        if call is hb.hb_lmhead_accept:
            keys.fill_(255)
        got = new()
        call(desc, hidden, weight, draft, dev.node_offset, par, mp, *got[:5], keys, 1, (dev.k_tree, dev.v_tree, *kv),
             dev.block_table, dev.prefix_len, *got[5:])
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))
        assert all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(kv, pools[0]))
    assert (alen > 1).any() and (t[::7] == t[0]).all()


@pytest.mark.parametrize("dtype,nodes", [("f32", 4), ("bf16", 8), ("bf16", 40)])
def test_a_second_call_on_the_same_keys(dtype, nodes):
    """hb_lmhead_accept needs nothing of its keys: the second call's rows name other tokens than the first's, with smaller
    logits, and so do both calls on keys that were never set.  Each way of the LM head by the number of rows."""
    import paper_2509_18824_amd as hb
    import paper_2509_18824_amd.step as S
    B, K, V = 2, 256, 1000
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    desc = S.make_desc(dtype, B, 2, 1, 128, 16, 4, 8, B * nodes, nodes, 1.0)
    off = torch.tensor([0, nodes, 2 * nodes], dtype=torch.int32, device="cuda")
    parent = torch.from_numpy(np.concatenate([W.chain_tree(nodes)] * B).astype(np.int32)).cuda()
    weight = torch.eye(V, K, dtype=td, device="cuda")
    i32 = lambda *shape: torch.full(shape, -7, dtype=torch.int32, device="cuda")
    keys = torch.full((8 * B * nodes,), 255, dtype=torch.uint8, device="cuda")
    rng = np.random.default_rng(nodes)
    for size in (4.0, 1.0):
        target = rng.integers(0, K, size=B * nodes)
        draft = np.roll(target, 1)  # every node names what the target chooses after its parent
        hidden = (size * weight[torch.from_numpy(target).cuda()]).contiguous()
        ids, alen, path, toks, bonus = i32(B * nodes), i32(B), i32(B, nodes), i32(B, nodes), i32(B)
        hb.hb_lmhead_accept(desc, hidden, weight, torch.from_numpy(draft.astype(np.int32)).cuda(), off, parent, nodes, ids, alen,
                            path, toks, bonus, keys)
        torch.cuda.synchronize()
        assert np.array_equal(ids.cpu().numpy(), target)
        assert (alen == nodes).all() and np.array_equal(toks.cpu().numpy().reshape(-1), target)


@pytest.mark.parametrize("B,max_path,layers", [
    (3, 1 << 23, 1),         # more than 2^24 path slots, most of which no tree of 64 nodes reaches
    (3, 1 << 23, 0),
    (70000, 64, 1),          # more workgroups than the grid has: each takes several
    (70000, 200, 0)])
def test_more_path_slots_than_a_grid_has_threads(B, max_path, layers):
    """Chains of two nodes that share pages: the root is always accepted, its child by every second sequence."""
    import paper_2509_18824_amd as hb
    import paper_2509_18824_amd.step as S
    K, V, page, T = 8, 16, 16, 2 * B
    rng = np.random.default_rng(B)
    target = rng.integers(0, K, size=T)
    draft = np.where(np.arange(T) % 4 == 1, np.roll(target, 1), (np.roll(target, 1) + 1) % V)
    t32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    # sequence b: positions 3 (b % 5) .. + 1 of page b / 5, nobody else's
    pages = B // 5 + 1
    desc = S.make_desc("f32", B, 1, 1, 8, page, 1, pages, T, 2, 1.0)
    off, parent = t32(2 * np.arange(B + 1)), t32(np.tile([-1, 0], B))
    block_table, prefix = t32(np.arange(B)[:, None] // 5), t32(3 * (np.arange(B) % 5))
    weight = torch.eye(V, K, device="cuda")
    hidden = weight[torch.from_numpy(target).cuda()].contiguous()
    i32 = lambda *shape: torch.full(shape, -7, dtype=torch.int32, device="cuda")
    ids, alen, path, toks, bonus, slots, new_len = (i32(T), i32(B), i32(B, max_path), i32(B, max_path), i32(B),
                                                    i32(B, max_path), i32(B))
    k_tree, v_tree = torch.randn(T, 1, 8, device="cuda"), torch.randn(T, 1, 8, device="cuda")
    k_pool, v_pool = torch.zeros(pages, 1, page, 8, device="cuda"), torch.zeros(pages, 1, page, 8, device="cuda")
    keys = torch.empty(8 * T, dtype=torch.uint8, device="cuda")
    hb.hb_lmhead_accept(desc, hidden, weight, t32(draft), off, parent, max_path, ids, alen, path, toks, bonus, keys, layers,
                        (k_tree, v_tree, k_pool, v_pool), block_table, prefix, slots, new_len)
    torch.cuda.synchronize()
    assert np.array_equal(ids.cpu().numpy(), target)
    want = 1 + (np.arange(B) % 2 == 0)
    assert np.array_equal(alen.cpu().numpy(), want)
    took = torch.arange(max_path, device="cuda") < alen[:, None]
    assert torch.equal(path, torch.where(took, torch.arange(max_path, dtype=torch.int32, device="cuda"), -1))
    assert torch.equal(toks[:, :2].cpu(), torch.from_numpy(np.where(want[:, None] == 2, target.reshape(B, 2),
                                                                    np.stack([target[::2], -np.ones(B)], 1))).int())
    assert (toks[:, 2:] == -1).all()
    assert np.array_equal(bonus.cpu().numpy(), np.where(want == 2, target[1::2], target[::2]))
    if not layers:
        assert (slots == -7).all() and (new_len == -7).all()
        return
    assert torch.equal(new_len, prefix + alen)
    at = block_table * page + prefix[:, None] + torch.arange(max_path, dtype=torch.int32, device="cuda")
    assert torch.equal(slots, torch.where(took, at, -1))
    two = alen == 2
    for tree, pool in ((k_tree, k_pool), (v_tree, v_pool)):
        ref = torch.zeros_like(pool).view(-1, 8)
        ref[at[:, 0].long()] = tree[::2, 0]
        ref[at[two, 1].long()] = tree[1::2, 0][two]
        assert torch.equal(pool.view(-1, 8), ref)
