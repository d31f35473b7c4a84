"""The workloads whose speed this repository cares about, one pass of each through the public calls.

The framework verifies drafted token trees and chains on the target model and does what lies around
that: it builds the draft tree, runs the draft's intermediate layer and accepts greedily or by
sampling.  Six kinds of pass cover it:

  step    attention of one layer, LM head with argmax, acceptance, compaction (``VerifyStep``)
  layers  a stack of whole decoder layers, then the same (``VerifyLayerStack`` with ``mlp``)
  attn    tree-verify attention alone (``tree_verify_attn``)
  draft   construction of the draft tree from the draft model's logits (``DraftTreeBuilder``)
  meta    the draft's intermediate layer on a batch of tokens (``MetaQueryLayer``, ``fc_concat``)
  sample  sampling acceptance of a verified tree (``tree_accept_sample``)

Shapes are those of the repository's workloads (28 query and 4 key/value heads of 128, hidden size
3584, feed-forward width 18944, vocabulary 152064, 60-node trees and 8-node chains).  Inputs are
made on the GPU from the seed alone.  Scores of a head are as sharp as the head's place says (from
near-uniform to a handful of keys), and every node's hidden state points at one vocabulary entry as
a trained model's does, so that the greedy token has a margin.
"""
import math

import numpy as np
import torch

import paper_2509_18824_amd.step as S
import workloads as W

_PAGE = 16
_ROPE_THETA = 1e6
_EPS = 1e-6


def listed():
    model = {"Hq": 28, "Hkv": 4, "D": 128}
    bf = {"dtype": "bf16", **model, "vocab": 152064}
    return [
        # a unit-sized model in float32 with a chain of four: what a step costs when nothing is big
        {"name": "step_f32_chain4_b1", "kind": "step", "dtype": "f32", "B": 1, "tree": "chain", "nodes": 4, "L_min": 256,
         "L_max": 256, "Hq": 4, "Hkv": 1, "D": 64, "vocab": 1000},
        # one user, one drafted tree behind a context of half image, half text positions
        {"name": "step_tree60_b1", "kind": "step", "B": 1, "tree": "tree", "nodes": 60, "L_min": 2048, "L_max": 2048, **bf},
        # a serving batch with chain drafts, the drafting mode of the paper's measurements
        {"name": "step_chain8_b16", "kind": "step", "B": 16, "tree": "chain", "nodes": 8, "L_min": 1024, "L_max": 4096, **bf},
        # the serving batch with drafted trees: the benchmark's step
        {"name": "step_tree60_b16", "kind": "step", "B": 16, "tree": "tree", "nodes": 60, "L_min": 1024, "L_max": 4096, **bf},
        # whole decoder layers: one user's chain (the weights are streamed for eight tokens) ...
        {"name": "layers_chain8_b1", "kind": "layers", "B": 1, "tree": "chain", "nodes": 8, "L_min": 2048, "L_max": 2048,
         "layers": 8, "ffn": 18944, **bf},
        # ... the serving batch with chains ...
        {"name": "layers_chain8_b16", "kind": "layers", "B": 16, "tree": "chain", "nodes": 8, "L_min": 1024, "L_max": 4096,
         "layers": 8, "ffn": 18944, **bf},
        # ... and with trees: the most work a verification pass is asked for
        {"name": "layers_tree60_b16", "kind": "layers", "B": 16, "tree": "tree", "nodes": 60, "L_min": 1024, "L_max": 4096,
         "layers": 8, "ffn": 18944, **bf},
        # two long interleaved contexts: attention is what grows
        {"name": "attn_tree60_b2_32k", "kind": "attn", "dtype": "bf16", "B": 2, "tree": "tree", "nodes": 60, "L_min": 32768,
         "L_max": 32768, "lse": False, **model},
        # draft trees for the serving batch: five levels, ten candidates each
        {"name": "draft_tree60_b16", "kind": "draft", "B": 16, "K": 10, "T": 5, "nodes": 60, "vocab": 152064, "dtype": "f32"},
        # the intermediate layer on the tokens that a batch's last step accepted ...
        {"name": "meta_96", "kind": "meta", "S": 96, "L": 28, "D": 3584, "H": 28, "Q": 3},
        # ... and on a prompt
        {"name": "meta_2048", "kind": "meta", "S": 2048, "L": 28, "D": 3584, "H": 28, "Q": 3},
        # acceptance by sampling, for the serving batch's trees
        {"name": "sample_tree60_b16", "kind": "sample", "B": 16, "tree": "tree", "nodes": 60, "vocab": 152064},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _drawn_tree(rng, most):
    """A tree or a chain of at most ``most`` nodes per sequence."""
    if most >= 20 and rng.random() < 0.5:
        return {"tree": "tree", "nodes": rng.randint(20, min(64, most))}
    return {"tree": "chain", "nodes": rng.randint(2, max(2, min(16, most)))}


def _drawn_lengths(rng, B, most_total, most=32768):
    hi = _log_int(rng, 128, max(160, min(most, most_total // B)))
    return {"L_min": rng.choice([hi, max(1, hi // 4), max(1, hi // 2)]), "L_max": hi}


def draw(rng):
    kind = rng.choice(["step", "step", "layers", "layers", "attn", "draft", "meta", "sample"])
    Hq, Hkv = rng.choice([(28, 4), (28, 4), (32, 8), (16, 2)])
    heads = {"dtype": "bf16", "Hq": Hq, "Hkv": Hkv, "D": 128}
    vocab = rng.choice([152064, _log_int(rng, 32000, 152000)])
    if kind == "step" and rng.random() < 0.25:
        B = rng.randint(1, 4)
        return {"kind": "step", "dtype": "f32", "B": B, "tree": "chain", "nodes": rng.randint(1, 8),
                **_drawn_lengths(rng, B, 2048, 1024), "Hq": 4, "Hkv": rng.choice([1, 2]), "D": 64, "vocab": _log_int(rng, 500, 4000)}
    if kind in ("step", "layers"):
        B = _log_int(rng, 1, 16)
        case = {"kind": kind, "B": B, **_drawn_tree(rng, 64), **_drawn_lengths(rng, B, 40000), "vocab": vocab, **heads}
        if kind == "layers":
            case.update(layers=rng.randint(1, 8), ffn=64 * _log_int(rng, 64, 296))
        if B * case["nodes"] > 960:
            case["nodes"] = 960 // B
        return case
    if kind == "attn":
        B = _log_int(rng, 1, 32)
        return {"kind": "attn", "B": B, **_drawn_tree(rng, 64), **_drawn_lengths(rng, B, 80000), "lse": rng.random() < 0.5, **heads}
    if kind == "draft":
        K, T = rng.randint(2, 12), rng.randint(2, 6)
        most = min(64, 1 + K + (T - 1) * K * K)
        return {"kind": "draft", "B": _log_int(rng, 1, 16), "K": K, "T": T, "nodes": rng.randint(min(4, most), most),
                "vocab": vocab, "dtype": rng.choice(["f32", "f32", "bf16"])}
    if kind == "meta":
        D, H = rng.choice([(3584, 28), (3584, 28), (2048, 16), (4096, 32)])
        return {"kind": "meta", "S": _log_int(rng, 4, 1800), "L": rng.randint(12, 32) if D < 4096 else rng.randint(12, 24),
                "D": D, "H": H, "Q": rng.randint(1, 3)}
    return {"kind": "sample", "B": _log_int(rng, 1, 16), **_drawn_tree(rng, 60), "vocab": vocab}


def _lengths(case, rng):
    """Ragged prefix lengths, spread evenly over [L_min, L_max] with a jitter, in random order."""
    B, lo, hi = case["B"], case["L_min"], case["L_max"]
    at = (np.arange(B) + rng.random(B)) / B
    return rng.permutation(lo + np.floor(at * (hi - lo + 1)).astype(np.int64).clip(0, hi - lo))


def _trees(case, seed):
    n = case["nodes"]
    if case["tree"] == "chain":
        return [W.chain_tree(n)] * case["B"]
    return [W.seeded_tree(seed * 64 + b, n_nodes=n, levels=6, root_fanout=min(10, n - 6)) for b in range(case["B"])]


class _Batch:
    """Page tables, trees and the attention descriptor of a batch; ``kv`` makes a filled cache."""

    def __init__(self, case, seed):
        rng = np.random.default_rng(seed)
        self.gen = torch.Generator(device="cuda").manual_seed(seed)
        self.dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
        self.trees = _trees(case, seed)
        self.lens = _lengths(case, rng)
        self.max_path = max(int(W.tree_depths(t).max()) + 1 for t in self.trees)
        self.Hq, self.Hkv, self.D, self.T = case["Hq"], case["Hkv"], case["D"], case["B"] * case["nodes"]
        pages = [-(-(int(L) + self.max_path) // _PAGE) for L in self.lens]
        self.num_blocks = case["B"] * (-(-(case["L_max"] + self.max_path) // _PAGE)) + 4  # the pool has room for the longest
        ids = rng.permutation(self.num_blocks)
        table = np.full((case["B"], max(pages) + 1), ids[-1], dtype=np.int32)
        for b, n in enumerate(pages):
            at = sum(pages[:b])
            table[b, :n] = ids[at:at + n]
        i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
        self.block_table, self.prefix_len = i32(table), i32(self.lens)
        self.node_offset = i32(np.arange(case["B"] + 1) * case["nodes"])
        self.parent = i32(np.concatenate(self.trees))
        self.desc = S.make_desc(self.dtype, case["B"], self.Hq, self.Hkv, self.D, _PAGE, table.shape[1], self.num_blocks,
                                self.T, case["nodes"], self.D ** -0.5, hint=int(self.lens.max()))

    def normal(self, *shape, std=1.0, dtype=None):
        return torch.empty(shape, dtype=dtype or self.dtype, device="cuda").normal_(0.0, std, generator=self.gen)

    def kv(self, *lead):
        return self.normal(*lead, 2, self.num_blocks, self.Hkv, _PAGE, self.D)

    def device_inputs(self, kv):
        """Queries (head h of a group is sharper the higher h), K and V of the nodes, the cache."""
        q = self.normal(self.T, self.Hq, self.D) * torch.linspace(0.5, 3.0, self.Hq, device="cuda", dtype=self.dtype)[:, None]
        return S.DeviceInputs(q, self.normal(self.T, self.Hkv, self.D), self.normal(self.T, self.Hkv, self.D), kv[0], kv[1],
                              self.block_table, self.prefix_len, self.node_offset, self.parent)

    def tokens(self, vocab):
        """A distinct token per node: what the target will choose after it."""
        return torch.randperm(vocab, generator=self.gen, device="cuda")[:self.T]

    def draft_ids(self, seed, target, vocab):
        ids, _ = W.plant_draft_ids(seed, self.trees, target.cpu().numpy(), vocab)
        return torch.from_numpy(ids).cuda()


def _hidden_of(batch, dev):
    """The attention output of every node over its prefix alone (its few tree keys left out), float32:
    the direction that the LM head's row for the node's token is given."""
    n, G = len(batch.trees[0]), batch.Hq // batch.Hkv
    out = torch.empty((batch.T, batch.Hq, batch.D), device="cuda")
    for b, L in enumerate(batch.lens):
        L, rows = int(L), slice(b * n, (b + 1) * n)
        pages = batch.block_table[b, :-(-L // _PAGE)].long()
        k, v = (p[pages].float().permute(1, 0, 2, 3).reshape(batch.Hkv, -1, batch.D)[:, :L] for p in (dev.k_pool, dev.v_pool))
        for g in range(batch.Hkv):
            heads = slice(g * G, (g + 1) * G)
            s = dev.q[rows, heads].float().reshape(n * G, batch.D) @ k[g].t() * batch.D ** -0.5
            out[rows, heads] = (torch.softmax(s, dim=1) @ v[g]).view(n, G, batch.D)
    return out.view(batch.T, -1)


def _prepare_step(case, seed):
    batch = _Batch(case, seed)
    kv = batch.kv()
    dev = batch.device_inputs(kv)
    vocab, target = case["vocab"], batch.tokens(case["vocab"])
    weight = batch.normal(vocab, batch.Hq * batch.D, std=0.02)
    h = _hidden_of(batch, dev)
    weight[target] += (0.5 * h / h.norm(dim=1, keepdim=True)).to(batch.dtype)
    return {"kv": kv, "step": S.VerifyStep(batch.desc, dev, weight, batch.draft_ids(seed, target, vocab), batch.max_path)}


def _prepare_layers(case, seed):
    batch = _Batch(case, seed)
    n_layers, K, F, vocab = case["layers"], batch.Hq * batch.D, case["ffn"], case["vocab"]
    kv = batch.kv(n_layers)
    w = lambda n, k, std=0.02: batch.normal(n, k, std=std)
    small = 0.02 / math.sqrt(2 * n_layers)  # projections back into the residual stream
    gain = lambda: 1.0 + batch.normal(K, std=0.1)
    mlp = {"norm1": [gain() for _ in range(n_layers)], "norm2": [gain() for _ in range(n_layers)], "norm_f": gain(), "eps": _EPS,
           "w_gate_up": [w(2 * F, K) for _ in range(n_layers)], "w_down": [w(K, F, small) for _ in range(n_layers)]}
    w_qkv = [w((batch.Hq + 2 * batch.Hkv) * batch.D, K) for _ in range(n_layers)]
    w_o = [w(K, K, small) for _ in range(n_layers)]
    lm_weight, target = w(vocab, K), batch.tokens(vocab)
    row = lm_weight[target].float()
    hidden = batch.normal(batch.T, K, std=0.87, dtype=torch.float32) + 0.5 * math.sqrt(K) * row / row.norm(dim=1, keepdim=True)
    stack = S.VerifyLayerStack(batch.desc, batch.device_inputs(kv[0]), [(kv[l, 0], kv[l, 1]) for l in range(n_layers)], w_qkv, w_o,
                               lm_weight, batch.draft_ids(seed, target, vocab), batch.max_path, hidden.to(batch.dtype), _ROPE_THETA, mlp)
    return {"kv": kv, "step": stack}


def _prepare_attn(case, seed):
    batch = _Batch(case, seed)
    dev = batch.device_inputs(batch.kv())
    ws = S.alloc_workspace(S.hb.hb_tree_verify_attn_workspace_bytes(batch.desc))
    return {"desc": batch.desc, "dev": dev, "lse": case["lse"], "ws": ws}


def _next_token_logits(gen, rows, vocab):
    """float32 [rows, vocab] shaped like a language model's next-token scores: falling with the
    logarithm of a token's rank (a few tokens carry most of the mass)."""
    u = torch.rand((rows, vocab), generator=gen, device="cuda")
    return u.mul_(vocab).log1p_().mul_(-1.2)


def _noisy(base, gen, std=0.7):
    return torch.empty_like(base).normal_(0.0, std, generator=gen).add_(base)


def _prepare_draft(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    rows = [case["B"]] + [case["B"] * case["K"]] * (case["T"] - 1)
    logits = [_noisy(_next_token_logits(gen, r, case["vocab"]), gen).to(dtype) for r in rows]
    root = torch.randint(0, case["vocab"], (case["B"],), generator=gen, device="cuda", dtype=torch.int32)
    return {"B": case["B"], "K": case["K"], "T": case["T"], "nodes": case["nodes"], "logits": logits, "root": root}


def _prepare_meta(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    n, L, D, H, Q = case["S"], case["L"], case["D"], case["H"], case["Q"]
    bf = lambda *shape, std=1.0: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)
    w = lambda rows, cols: bf(rows, cols, std=cols ** -0.5)
    feats = bf(n, L, D) + bf(1, L, D, std=0.5)  # layers differ systematically
    layers = [L // 8, L // 2, L - 2, L - 1][:Q]
    layer = S.MetaQueryLayer(bf(Q, D, std=2.0), w(D, D), w(D, D), w(D, D), w(D, D), w(D, Q * D), H, layers)
    return {"layer": layer, "feats": feats, "embed": bf(n, D), "w_a": w(D, D), "w_b": w(D, D)}


def _prepare_sample(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    trees, V = _trees(case, seed), case["vocab"]
    n, T = case["nodes"], case["B"] * case["nodes"]
    base = _next_token_logits(gen, T, V)
    p = torch.softmax(_noisy(base, gen), dim=1)
    q = torch.softmax(_noisy(base, gen), dim=1)
    # the children of a node are drawn from the draft's distribution without replacement (the k
    # largest of log q plus Gumbel noise), in the order drawn
    children = [[np.flatnonzero(t == i) for i in range(n)] for t in trees]
    draft = torch.randint(0, V, (T,), generator=gen, device="cuda", dtype=torch.int32)
    for b in range(case["B"]):
        inner = [i for i in range(n) if len(children[b][i])]
        at = torch.tensor([b * n + i for i in inner], device="cuda")
        noise = torch.rand((len(inner), V), generator=gen, device="cuda").clamp_(1e-20).log_().neg_().log_().neg_()
        best = noise.add_(q[at].clamp_min_(1e-30).log_()).topk(max(len(children[b][i]) for i in inner), dim=1).indices
        slot = torch.tensor([b * n + int(c) for i in inner for c in children[b][i]], device="cuda")
        pick = torch.tensor([(r, j) for r, i in enumerate(inner) for j in range(len(children[b][i]))], device="cuda")
        draft[slot] = best[pick[:, 0], pick[:, 1]].int()
    bits = lambda k: torch.randint(-2 ** 31, 2 ** 31, (k,), generator=gen, device="cuda", dtype=torch.int64).int()
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    return {"node_offset": i32(np.arange(case["B"] + 1) * n), "parent": i32(np.concatenate(trees)), "draft": draft, "p": p, "q": q,
            "u_accept": bits(T), "u_bonus": bits(case["B"]), "nodes": n,
            "max_path": max(int(W.tree_depths(t).max()) + 1 for t in trees)}


_PREPARE = {"step": _prepare_step, "layers": _prepare_layers, "attn": _prepare_attn, "draft": _prepare_draft,
            "meta": _prepare_meta, "sample": _prepare_sample}


def prepare(case, seed):
    state = _PREPARE[case["kind"]](case, seed)
    state["kind"] = case["kind"]
    return state


def run(state):
    kind = state["kind"]
    if kind in ("step", "layers"):
        s = state["step"]
        s.run()
        hidden = s.out if kind == "step" else s.final_hidden
        return {"hidden": hidden, "target_ids": s.target_ids, "accept_len": s.accept_len, "accept_path": s.accept_path,
                "out_tokens": s.out_tokens, "bonus": s.bonus, "out_slots": s.out_slots, "new_len": s.new_len, "kv": state["kv"]}
    if kind == "attn":
        return S.tree_verify_attn(state["desc"], state["dev"], want_lse=state["lse"], workspace=state["ws"])
    if kind == "draft":
        builder = S.DraftTreeBuilder(state["B"], state["K"], state["T"])
        for logits in state["logits"]:
            builder.grow(*S.topk_logprob(logits, state["K"]))
        return builder.finalize(state["nodes"], state["root"])
    if kind == "meta":
        f_c, x = state["layer"].run(state["feats"])
        return f_c, x, S.fc_concat(x, state["embed"], state["w_a"], state["w_b"])
    return S.tree_accept_sample(state["node_offset"], state["parent"], state["draft"], state["p"], state["q"], state["u_accept"],
                                state["u_bonus"], state["max_path"], state["nodes"])


def work(case):
    """Bytes and operations of one pass: every input read once, every output written once."""
    kind = case["kind"]
    if kind == "draft":
        rows = case["B"] * (1 + (case["T"] - 1) * case["K"])
        return {"bytes": rows * case["vocab"] * (4 if case["dtype"] == "f32" else 2), "flops": 3.0 * rows * case["vocab"]}
    if kind == "meta":
        n, L, D, Q, rows = case["S"], case["L"], case["D"], case["Q"], case["H"] * case["Q"]
        weights = (2 + Q + 2) * D * D + 2 * rows * D
        # the queries are folded into the keys, the values are projected after the mixing
        flops = 2.0 * n * (2 * rows * L * D + 3 * Q * D * D + 2 * D * D)
        return {"bytes": 2.0 * (n * L * D + weights + n * D + n * (Q + 2) * D), "flops": flops}
    if kind == "sample":
        # the two rows of every node visited: the root and what is accepted below it, about two more
        visited = min(3.0, case["nodes"])
        return {"bytes": case["B"] * visited * 2 * case["vocab"] * 4, "flops": case["B"] * visited * 4.0 * case["vocab"]}
    size = 4 if case["dtype"] == "f32" else 2
    T, K = case["B"] * case["nodes"], case["Hq"] * case["D"]
    keys = case["B"] * (case["L_min"] + case["L_max"]) / 2
    attn_bytes = size * ((keys + T) * case["Hkv"] * case["D"] * 2 + 2 * T * K)
    attn_flops = 4.0 * case["D"] * case["Hq"] * case["nodes"] * keys
    if kind == "attn":
        return {"bytes": attn_bytes, "flops": attn_flops}
    head_bytes, head_flops = size * case["vocab"] * K, 2.0 * T * K * case["vocab"]
    if kind == "step":
        return {"bytes": attn_bytes + head_bytes, "flops": attn_flops + head_flops}
    weights = (case["Hq"] + 2 * case["Hkv"]) * case["D"] * K + K * K + 3 * case["ffn"] * K
    n = case["layers"]
    return {"bytes": n * (attn_bytes + size * weights) + head_bytes, "flops": n * (attn_flops + 2.0 * T * weights) + head_flops}


def tolerance(case):
    """About four times what the paths were measured to be off by against float64 references."""
    kind = case["kind"]
    if kind == "sample":
        return "exact"  # integers throughout
    if kind == "draft":  # ids by comparison, log-probabilities from float32 sums: 5e-8 seen
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.002}
    if case.get("dtype") == "f32":  # 4e-7 seen
        return {"rel": 2e-6, "max": 1e-5, "differ": 0.002}
    if kind == "layers":  # roundings to bf16 add up over eight layers: 1e-2 seen
        return {"rel": 0.03, "max": 0.2, "differ": 0.002}
    if kind == "meta":  # 3e-3 seen
        return {"rel": 0.01, "max": 0.06, "differ": 0.002}
    return {"rel": 0.008, "max": 0.07, "differ": 0.002}  # attention: 2e-3 seen
