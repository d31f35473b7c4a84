"""GPU parity: hb_tree_accept_sample is bit-exact against the oracle (every decision of the rule
is an integer expression, so there is exactly one correct result)."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import tree_accept_ref, tree_accept_sample_ref

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def step():
    import paper_2509_18824_amd.step as s
    return s


def _u32(rng, n):
    return rng.integers(0, 2 ** 32, size=n, dtype=np.uint64).astype(np.uint32)


def _both(step, trees, draft, P, Q, u_acc, u_bon, max_path):
    off = np.concatenate([[0], np.cumsum([len(t) for t in trees])]).astype(np.int32)
    par = (np.concatenate(trees) if len(off) > 1 and off[-1] > 0 else np.zeros(0)).astype(np.int32)
    P32, Q32 = P.astype(np.float32), Q.astype(np.float32)
    ref = tree_accept_sample_ref(off, par, draft, P32, Q32, u_acc, u_bon, max_path)
    t = lambda a: torch.from_numpy(np.asarray(a, dtype=np.int32)).cuda()
    bits = lambda a: torch.from_numpy(np.asarray(a, dtype=np.uint32).view(np.int32)).cuda()
    got = step.tree_accept_sample(t(off), t(par), t(draft), torch.from_numpy(P32).cuda(), torch.from_numpy(Q32).cuda(),
                                  bits(u_acc), bits(u_bon), max_path, max(max((len(x) for x in trees), default=1), 1))
    torch.cuda.synchronize()
    for g, r, name in zip(got, ref, ("accept_len", "accept_path", "out_tokens", "bonus_id")):
        assert np.array_equal(g.cpu().numpy(), r), (name, g.cpu().numpy(), r)
    return ref


def _draw_drafts(rng, trees, Q, V):
    """Children of a node carry distinct tokens drawn from the node's q without replacement."""
    off = np.concatenate([[0], np.cumsum([len(t) for t in trees])])
    draft = np.zeros(off[-1], dtype=np.int64)
    for b, t in enumerate(trees):
        for node in range(len(t)):
            kids = [c for c in range(len(t)) if t[c] == node]
            if kids:
                q = Q[off[b] + node].astype(np.float64)
                toks = rng.choice(V, size=len(kids), replace=False, p=q / q.sum())
                draft[off[b] + np.array(kids)] = toks
    return draft


@pytest.mark.parametrize("V", [7, 300, 4097])
def test_random_trees_and_distributions(step, V):
    rng = np.random.default_rng(V)
    for trial in range(6):
        B = int(rng.integers(1, 7))
        trees = []
        for _ in range(B):
            n = int(rng.integers(1, 40))
            par = [-1]
            for i in range(1, n):
                free = [x for x in range(i) if par.count(x) < min(V, 5)]
                par.append(int(rng.choice(free)))
            trees.append(np.array(par, dtype=np.int32))
        total = sum(len(t) for t in trees)
        # peaked target, flatter draft that resembles it: acceptances and rejections both happen
        logits = rng.standard_normal((total, V)) * 2.0
        P = np.exp(logits); P /= P.sum(1, keepdims=True)
        Qm = np.exp(0.7 * logits + 0.8 * rng.standard_normal((total, V))); Qm /= Qm.sum(1, keepdims=True)
        draft = _draw_drafts(rng, trees, Qm, V)
        ref = _both(step, trees, draft, P, Qm, _u32(rng, total), _u32(rng, B), 8)
        assert (ref[0] >= 1).all()


def test_acceptance_statistics_are_sane_on_chains(step):
    """8-node chains drafted from q = p: every node is accepted, whatever the uniforms; with an
    unrelated q most chains stop early.  (Bit-exactness against the oracle is checked inside.)"""
    rng = np.random.default_rng(5)
    V, B = 2000, 16
    trees = [W.chain_tree(8) for _ in range(B)]
    P = rng.dirichlet(np.full(V, 0.05), size=8 * B)
    draft = _draw_drafts(rng, trees, P, V)
    ref = _both(step, trees, draft, P, P.copy(), _u32(rng, 8 * B), _u32(rng, B), 8)
    assert (ref[0] == 8).all()
    Q = rng.dirichlet(np.full(V, 0.05), size=8 * B)
    draft = _draw_drafts(rng, trees, Q, V)
    ref = _both(step, trees, draft, P, Q, _u32(rng, 8 * B), _u32(rng, B), 8)
    assert ref[0].mean() < 3.0


def test_one_hot_distributions_equal_greedy_acceptance_and_edge_cases(step):
    rng = np.random.default_rng(9)
    V = 50
    trees = [W.seeded_tree(3), np.array([], dtype=np.int32), W.chain_tree(1), W.seeded_tree(4, n_nodes=64)]
    off = np.concatenate([[0], np.cumsum([len(t) for t in trees])])
    total = int(off[-1])
    target = rng.integers(0, V, size=total)
    draft, _ = W.plant_draft_ids(7, [trees[0], trees[2], trees[3]], np.concatenate([target[:60], target[60:]]), V)
    P = np.zeros((total, V)); P[np.arange(total), target] = 1.0
    Q = np.full((total, V), 1.0 / V)
    ref = _both(step, trees, draft, P, Q, _u32(rng, total), _u32(rng, 4), 7)
    want = tree_accept_ref(off, np.concatenate(trees), draft, target, 7)
    for g, w in zip(ref, want):
        assert np.array_equal(g, w)
    assert ref[0][1] == 0 and ref[3][1] == -1  # the sequence without nodes emits nothing
    # zero rows: nothing can be accepted and no last token exists (-1); max_path = 1: root only
    Z = np.zeros((total, V))
    ref = _both(step, trees, draft, Z, Q, _u32(rng, total), _u32(rng, 4), 7)
    assert list(ref[0]) == [1, 0, 1, 1] and list(ref[3]) == [-1, -1, -1, -1]
    _both(step, trees, draft, P, Q, _u32(rng, total), _u32(rng, 4), 1)


def test_full_vocabulary_chains(step):
    """The shape the paper measures: 8-node chains, batch 16, vocabulary 152064."""
    rng = np.random.default_rng(11)
    V, B = 152064, 16
    trees = [W.chain_tree(8) for _ in range(B)]
    logits = (rng.standard_normal((8 * B, V)) * 3.0).astype(np.float32)
    P = np.exp(logits - logits.max(1, keepdims=True)); P /= P.sum(1, keepdims=True)
    noise = rng.standard_normal((8 * B, V)).astype(np.float32)
    Q = np.exp(0.9 * logits + 0.6 * noise); Q /= Q.sum(1, keepdims=True)
    draft = _draw_drafts(rng, trees, Q, V)
    ref = _both(step, trees, draft, P, Q, _u32(rng, 8 * B), _u32(rng, B), 8)
    assert 1.0 < ref[0].mean() < 8.0


@pytest.mark.parametrize("V", [2559, 2561, 10240, 64 * 2560, 64 * 2560 + 1, 128 * 2560 + 77])
def test_vocabularies_around_the_shares_of_the_wavefronts(step, V):
    """One and two wavefronts, a whole workgroup, 64 and 65 partners of an exchange, and a vocabulary
    whose end does not fit the registers; several rejections at the root, some accepted children."""
    rng = np.random.default_rng(V)
    trees = [np.array([-1] + [0] * 6 + [1, 2, 3, 7], dtype=np.int32), W.chain_tree(3), W.chain_tree(1)]
    total = sum(len(t) for t in trees)
    logits = rng.standard_normal((total, V)) * 2.0
    P = np.exp(logits); P /= P.sum(1, keepdims=True)
    Q = np.exp(0.7 * logits + rng.standard_normal((total, V))); Q /= Q.sum(1, keepdims=True)
    for trial in range(3):
        _both(step, trees, _draw_drafts(rng, trees, Q, V), P, Q, _u32(rng, total), _u32(rng, 3), 4)


class _Case:
    """One batch on the GPU with the oracle's answer; calls it with a workspace and a stream of the caller's."""

    def __init__(self, seed, V, trees, max_path):
        rng = np.random.default_rng(seed)
        self.off = np.concatenate([[0], np.cumsum([len(t) for t in trees])]).astype(np.int32)
        par, total = np.concatenate(trees).astype(np.int32), int(self.off[-1])
        logits = rng.standard_normal((total, V)) * 2.0
        P = np.exp(logits); P /= P.sum(1, keepdims=True)
        Q = np.exp(0.7 * logits + rng.standard_normal((total, V))); Q /= Q.sum(1, keepdims=True)
        draft = _draw_drafts(rng, trees, Q, V)
        P, Q, ua, ub = P.astype(np.float32), Q.astype(np.float32), _u32(rng, total), _u32(rng, len(trees))
        self.ref = tree_accept_sample_ref(self.off, par, draft, P, Q, ua, ub, max_path)
        i32 = lambda a: torch.from_numpy(np.asarray(a).astype(np.uint32).view(np.int32)).cuda()
        self.inputs = [i32(self.off), i32(par), i32(draft), torch.from_numpy(P).cuda(), torch.from_numpy(Q).cuda(), i32(ua), i32(ub)]
        self.B, self.V, self.max_path, self.nodes = len(trees), V, max_path, max(len(t) for t in trees)

    def outputs(self):
        shapes = (self.B,), (self.B, self.max_path), (self.B, self.max_path), (self.B,)
        return [torch.full(s, -7, dtype=torch.int32, device="cuda") for s in shapes]

    def call(self, out, workspace, max_polls=None, stream=None):
        import paper_2509_18824_amd as hb
        args = (self.B, self.nodes, *self.inputs, self.max_path, *out, workspace)
        if max_polls is None:
            hb.hb_tree_accept_sample(*args, stream=stream)
        else:
            hb.hb_tree_accept_sample_polls(*args, max_polls, stream=stream)

    def check(self, out):
        for g, r in zip(out, self.ref):
            assert np.array_equal(g.cpu().numpy(), r), (g.cpu().numpy(), r)


_WIDE_TREE = np.array([-1] + [0] * 6 + [1, 2, 3, 7], dtype=np.int32)


@pytest.mark.parametrize("max_polls", [0, 1, 3, 40])
@pytest.mark.parametrize("V", [5121, 10241, 152064, 128 * 2560 + 77])
def test_waits_that_run_out_give_the_same_results(V, max_polls):
    """Partners that give up waiting (at once, or after some looks) leave the sequence to one workgroup."""
    case = _Case(V + 1, V, [_WIDE_TREE, W.chain_tree(3), W.chain_tree(1)], 4)
    out = case.outputs()
    case.call(out, torch.empty(case.B * V, dtype=torch.int32, device="cuda"), max_polls)
    torch.cuda.synchronize()
    case.check(out)


def test_workspace_of_an_earlier_launch_at_every_alignment():
    """One buffer, full of other things, for launches of a large vocabulary, smaller odd ones and other
    batches; it may start 4 bytes off an 8-byte boundary, and nothing beside it is touched."""
    cases = [_Case(1, 327757, [_WIDE_TREE], 4), _Case(2, 5121, [_WIDE_TREE, W.chain_tree(2), _WIDE_TREE], 4),
             _Case(3, 10243, [W.chain_tree(3)] * 2, 3)]
    guard = 64
    buf = torch.full((max(c.B * c.V for c in cases) + 2 * guard + 1,), -1, dtype=torch.int32, device="cuda")
    assert buf.data_ptr() % 8 == 0
    for rounds in range(2):
        for c in cases:
            for shift in (0, 1):
                first, last = guard + shift, guard + shift + c.B * c.V
                beside = buf.clone()
                out = c.outputs()
                c.call(out, buf[first:last])
                torch.cuda.synchronize()
                c.check(out)
                assert torch.equal(buf[:first], beside[:first]) and torch.equal(buf[last:], beside[last:])


def test_launches_on_two_streams():
    """Two batches on two streams at a time, several times over, each with its own workspace."""
    cases = [_Case(11, 152064, [_WIDE_TREE, W.chain_tree(3)] * 8, 4), _Case(12, 152064, [_WIDE_TREE] * 4, 4)]
    streams = [torch.cuda.Stream() for _ in cases]
    ws = [torch.empty(c.B * c.V, dtype=torch.int32, device="cuda") for c in cases]
    outs = [[c.outputs() for _ in range(6)] for c in cases]
    torch.cuda.synchronize()
    for i in range(6):
        for c, s, w, o in zip(cases, streams, ws, outs):
            c.call(o[i], w, stream=s)
    torch.cuda.synchronize()
    for c, o in zip(cases, outs):
        for out in o:
            c.check(out)


@pytest.mark.parametrize("V", [1, 255, 257, 5119, 5120, 5121, 7680, 7681])
def test_vocabularies_around_the_one_workgroup(step, V):
    """Up to 5120 tokens a sequence is one workgroup's, 256 values a pass; from 5121 on three wavefronts share
    it, from 7681 four."""
    rng = np.random.default_rng(V + 5)
    trees = [np.array([-1] + [0] * min(6, V) + [1] * min(3, V - 1), dtype=np.int32), W.chain_tree(3), np.array([], dtype=np.int32), W.chain_tree(1)]
    total = sum(len(t) for t in trees)
    logits = rng.standard_normal((total, V)) * 2.0
    P = np.exp(logits); P /= P.sum(1, keepdims=True)
    Q = np.exp(0.7 * logits + rng.standard_normal((total, V))); Q /= Q.sum(1, keepdims=True)
    for trial in range(4):
        _both(step, trees, _draw_drafts(rng, trees, Q, V), P, Q, _u32(rng, total), _u32(rng, 4), 4)


@pytest.mark.parametrize("V", [60, 2000, 6001, 30011])
def test_rows_that_sum_to_more_than_one(V, monkeypatch):
    """Rows scaled to sums of 0.6 up to nearly 4, in one wavefront's share too: every sum and product is
    held (the oracle's residual, made of Python integers here, has no limit)."""
    import oracle.stochastic_acceptance as A

    def residual(p, q, s_p, s_q):
        r = [max(a * s_q - b * s_p, 0) for a, b in zip(p.tolist(), q.tolist())]
        div = max(sum(r) >> A.FIX_BITS, 1)
        return np.array([x // div for x in r], dtype=np.int64) if sum(r) else p

    monkeypatch.setattr(A, "residual", residual)
    rng = np.random.default_rng(V)
    trees = [_WIDE_TREE, W.chain_tree(3)] * 4
    total = sum(len(t) for t in trees)
    logits = rng.standard_normal((total, V)) * 2.0
    P = np.exp(logits); P /= P.sum(1, keepdims=True)
    Q = np.exp(0.7 * logits + rng.standard_normal((total, V))); Q /= Q.sum(1, keepdims=True)
    draft = _draw_drafts(rng, trees, Q, V)
    scale = lambda: rng.choice([0.6, 1.0, 1.9, 2.0, 2.6, 3.9], size=(total, 1))
    P *= scale()
    Q *= scale()
    P[::3, 5] = 1.5  # one token with nearly all of it
    P[::3] *= 3.9 / P[::3].sum(1, keepdims=True)
    import paper_2509_18824_amd.step as step
    _both(step, trees, draft, P, Q, _u32(rng, total), _u32(rng, len(trees)), 4)


def test_replays_from_a_hip_graph():
    """Captured with its clearing kernel, replayed between other launches in the same workspace: the
    counter, the leave words and the slots are as new every time."""
    case, other = _Case(21, 30011, [_WIDE_TREE, W.chain_tree(3)] * 2, 4), _Case(22, 20002, [_WIDE_TREE] * 3, 4)
    ws = torch.full((max(case.B * case.V, other.B * other.V),), -1, dtype=torch.int32, device="cuda")
    out, out_other = case.outputs(), other.outputs()
    case.call(out, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        case.call(out, ws)
    for i in range(4):
        for o in out:
            o.fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        case.check(out)
        other.call(out_other, ws, 0 if i % 2 else None)  # leaves its own counts behind
        torch.cuda.synchronize()
        other.check(out_other)
