"""GPU parity: hb_tree_verify_attn against the CPU oracle, element by element on sizes the
oracle finishes in seconds, and on every node at the full workload sizes."""
import numpy as np
import pytest
import torch

import workloads as W
from parity import check_attn, oracle_attn

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    import paper_2509_18824_amd as m
    return m


@pytest.fixture(scope="module")
def step():
    import paper_2509_18824_amd.step as s
    return s


def _run(step, inp, **kw):
    dev = step.to_device(inp)
    desc = step.desc_for(inp, **kw)
    out, lse = step.tree_verify_attn(desc, dev)
    torch.cuda.synchronize()
    return out, lse, desc


def _algos(hb, inp):
    """Every kernel the library offers for this shape (a descriptor it cannot take plans 0 splits)."""
    import paper_2509_18824_amd.step as s
    algos = [hb.HB_ATTN_SCALAR]
    if hb.hb_tree_verify_attn_num_splits(s.desc_for(inp, algo=hb.HB_ATTN_MFMA)) > 0:
        algos.append(hb.HB_ATTN_MFMA)
    return algos


def test_matrix_core_kernel_takes_the_bf16_workloads(hb, step):
    """The workloads with bf16 KV, head_dim 128 and page 16 must run on the MFMA kernel, both when
    asked for explicitly and by default (so the parity tests below really cover it)."""
    for cfg in (1, 2, 3, 4):
        inp = W.make_config(cfg, scale_down=32)
        assert hb.HB_ATTN_MFMA in _algos(hb, inp)
    assert hb.HB_ATTN_MFMA not in _algos(hb, W.make_config(0))


def test_config0_fp32_chain(hb, step):
    for peaked in (False, True):
        inp = W.make_config(0, peaked=peaked)
        ref = oracle_attn(inp)
        for splits in (1, 2, 0):
            out, lse, _ = _run(step, inp, num_splits=splits)
            check_attn(inp, out, lse, ref=ref, label=f"cfg0 peaked={peaked} splits={splits}")


@pytest.mark.parametrize("peaked", [False, True])
def test_config1_single_sequence_bf16(hb, step, peaked):
    inp = W.make_config(1, peaked=peaked)
    ref = oracle_attn(inp)
    for algo in _algos(hb, inp):
        for splits in (1, 2, 7, 0):
            out, lse, _ = _run(step, inp, num_splits=splits, algo=algo)
            check_attn(inp, out, lse, ref=ref, label=f"cfg1 algo={algo} splits={splits} peaked={peaked}")


@pytest.mark.parametrize("cfg,scale_down", [(2, 8), (3, 16), (4, 8)])
@pytest.mark.parametrize("peaked", [False, True])
def test_scaled_copies_of_the_batched_workloads(hb, step, cfg, scale_down, peaked):
    """Same structure as the big workloads (ragged lengths, permuted pages, 60-node trees), with
    prefixes short enough for the oracle to cover every node."""
    inp = W.make_config(cfg, peaked=peaked, scale_down=scale_down)
    ref = oracle_attn(inp)
    for algo in _algos(hb, inp):
        for splits in (1, 3, 0):
            out, lse, _ = _run(step, inp, num_splits=splits, algo=algo)
            check_attn(inp, out, lse, ref=ref, label=f"cfg{cfg}/{scale_down} algo={algo} splits={splits}")


def test_ragged_edges_and_odd_shapes(hb, step):
    """Empty prefix, prefix shorter than a page, lengths around page and tile boundaries,
    single-node trees, a 64-node tree, group sizes 1 and 8, head dims 64 and 128."""
    trees = [W.chain_tree(1), W.chain_tree(8), W.seeded_tree(1), W.seeded_tree(2, n_nodes=64),
             W.seeded_tree(3, n_nodes=17, levels=4, root_fanout=4), W.chain_tree(3), W.seeded_tree(4)]
    lens = [0, 5, 16, 63, 64, 65, 1000]
    # (8, 8), (8, 4) and (28, 4) / (8, 1) give 64, 128 and 448 / 512 query rows per kv head: the
    # three workgroup shapes of the matrix-core kernel
    for dtype, Hq, Hkv, D in [("bf16", 28, 4, 128), ("bf16", 8, 8, 128), ("bf16", 8, 4, 128), ("bf16", 8, 1, 128),
                              ("f32", 6, 2, 64), ("bf16", 4, 2, 64), ("f32", 4, 4, 128)]:
        inp = W.make_verify_inputs(77, dtype, Hq, Hkv, D, lens, trees, kv_std=1.0, q_std=1.0)
        ref = oracle_attn(inp)
        for algo in _algos(hb, inp):
            for splits in (1, 4, 0):
                out, lse, _ = _run(step, inp, num_splits=splits, algo=algo)
                check_attn(inp, out, lse, ref=ref, label=f"edges {dtype} Hq={Hq} Hkv={Hkv} D={D} algo={algo} s={splits}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D", [8, 72, 136, 256])
def test_scalar_kernel_blocks_and_wavefronts(hb, step, dtype, D):
    """Head dimensions of one, two and four elements per lane with and without a remainder, and
    prefixes around one block of 64 keys and one round of the four wavefronts (256 keys)."""
    trees = [W.chain_tree(2), W.seeded_tree(1), W.chain_tree(1), W.seeded_tree(2, n_nodes=64), W.chain_tree(20), W.chain_tree(3)]
    inp = W.make_verify_inputs(78, dtype, 4, 2, D, [0, 1, 192, 255, 257, 600], trees, kv_std=1.0, q_std=1.0)
    ref = oracle_attn(inp)
    for splits in (1, 2, 0):
        out, lse, _ = _run(step, inp, num_splits=splits, algo=hb.HB_ATTN_SCALAR)
        check_attn(inp, out, lse, ref=ref, label=f"scalar {dtype} D={D} splits={splits}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D", [64, 72])
def test_scalar_kernel_keys_with_scores_of_minus_infinity(hb, step, dtype, D):
    """Keys whose score is -inf have no weight beside any other, also where they fill the first block, a
    wavefront's only one, a whole chunk, or everything but a node's own path; where a row has no other
    keys, its result is NaN, as the definition's."""
    trees = [W.chain_tree(2), W.seeded_tree(1), W.chain_tree(3), W.chain_tree(4), W.chain_tree(2)]
    inp = W.make_verify_inputs(81, dtype, 4, 2, D, [600, 300, 64, 900, 100], trees, kv_std=1.0, q_std=1.0)
    inp.q[..., 0] = inp.q[..., 0].abs() + 0.25
    masked = [list(range(0, 128)) + list(range(256, 520)), range(64, 128), range(0, 64), list(range(0, 200)) + list(range(250, 900)), range(0, 100)]
    for b, positions in enumerate(masked):
        for p in positions:
            inp.k_pool[int(inp.block_table[b, p // inp.page]), :, p % inp.page, 0] = float("-inf")
    last = int(inp.node_offset[4])
    inp.k_tree[last:, :, 0] = float("-inf")
    with np.errstate(invalid="ignore"):
        ref, ref_lse = oracle_attn(inp)
    assert np.isfinite(ref[:last]).all() and np.isnan(ref[last:]).all()
    for splits in (1, 2, 3, 0):
        out, lse, _ = _run(step, inp, num_splits=splits, algo=hb.HB_ATTN_SCALAR)
        got, got_lse = W.widen(out), W.widen(lse)
        assert np.isnan(got[last:]).all(), splits
        tol = 1e-5 if dtype == "f32" else 2e-2
        assert np.abs(got[:last] - ref[:last]).max() <= tol and np.abs(got_lse[:last] - ref_lse[:last]).max() <= 1e-4, splits


@pytest.mark.parametrize("D,page", [(8, 16), (40, 4), (64, 16), (64, 48)])
@pytest.mark.parametrize("lens", [[0], [1, 63, 64, 65], [447, 448, 449, 0, 20], [900], [2, 0, 260]])
def test_float32_rows_of_few_workgroups(hb, step, D, page, lens):
    """The float32 kernel of few workgroups, in which a wavefront has K and V of 64 keys in flight and the tree one of its own:
    prefixes around a block of 64 keys and a round of its seven wavefronts (448 keys), trees of one to 64 nodes, poisoned
    slots and off-path nodes; and 70 sequences, 300 or 512 workgroups, which it leaves to the other kernel."""
    trees = [W.chain_tree(2), W.seeded_tree(2, n_nodes=13, levels=4, root_fanout=4), W.chain_tree(1), W.chain_tree(5), W.chain_tree(3)][:len(lens)]
    for Hq, Hkv in ((2, 1), (3, 3)):
        inp = W.make_verify_inputs(91 + D, "f32", Hq, Hkv, D, lens, trees, page=page, kv_std=1.0, q_std=1.0)
        ref = oracle_attn(inp)
        for splits in (1, 2, 0):
            out, lse, _ = _run(step, inp, num_splits=splits)
            check_attn(inp, out, lse, ref=ref, label=f"f32 D={D} page={page} {lens} splits={splits}")
    for trees in ([W.chain_tree(1)] * 70, [W.seeded_tree(3, n_nodes=64)] * 4, [W.seeded_tree(3, n_nodes=64), W.chain_tree(7)],
                  [W.seeded_tree(3, n_nodes=64)] * 2 + [W.chain_tree(22)]):
        inp = W.make_verify_inputs(92, "f32", 2, 1, D, (lens * 70)[:len(trees)], trees, page=page, kv_std=1.0, q_std=1.0)
        out, lse, _ = _run(step, inp)
        check_attn(inp, out, lse, ref=oracle_attn(inp), label=f"f32 D={D} {len(trees)} trees")


@pytest.mark.parametrize("nodes,heads,L,splits,hint,eager", [
    (64, 4, 100, 1, 0, True), (65, 4, 100, 1, 0, False),      # one round of 256 CUs
    (40, 4, 300, 2, 0, True), (54, 3, 300, 2, 0, False),      # 320 chunks of rows, 324
    (4, 4, 100, 1, 17, True), (4, 4, 100, 1, 16, False)])     # prefixes known to be longer than 16 positions
def test_float32_rows_by_the_kernel_of_few_workgroups(step, nodes, heads, L, splits, hint, eager):
    """Both sides of the lines of that kernel, by its name, and the results of both."""
    from torch.profiler import ProfilerActivity, profile
    L = min(L, hint or L)
    trees = [W.seeded_tree(4, n_nodes=min(nodes, 60)) if nodes >= 20 else W.chain_tree(nodes)] + ([W.chain_tree(nodes - 60)] if nodes > 60 else [])
    inp = W.make_verify_inputs(95, "f32", heads, 1, 64, [L] * len(trees), trees, kv_std=1.0, q_std=1.0)
    desc, dev = step.desc_for(inp, num_splits=splits, hint=hint), step.to_device(inp)
    step.tree_verify_attn(desc, dev)
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as trace:
        out, lse = step.tree_verify_attn(desc, dev)
        torch.cuda.synchronize()
    names = [e.name for e in trace.events() if "attn_scalar" in e.name]
    assert len(names) == 1 and ("attn_scalar_eager_kernel" in names[0]) == eager
    check_attn(inp, out, lse, ref=oracle_attn(inp), label=f"f32 {nodes} x {heads}")


def test_float32_rows_of_few_workgroups_with_scores_of_minus_infinity(hb, step):
    """As above for whole blocks, wavefronts and rows of keys without weight."""
    trees = [W.chain_tree(2), W.chain_tree(3), W.chain_tree(4), W.chain_tree(2)]
    inp = W.make_verify_inputs(93, "f32", 4, 2, 64, [600, 64, 900, 100], trees, kv_std=1.0, q_std=1.0)
    inp.q[..., 0] = inp.q[..., 0].abs() + 0.25
    masked = [list(range(0, 128)) + list(range(256, 520)), range(0, 64), list(range(0, 200)) + list(range(250, 900)), range(0, 100)]
    for b, positions in enumerate(masked):
        for p in positions:
            inp.k_pool[int(inp.block_table[b, p // inp.page]), :, p % inp.page, 0] = float("-inf")
    last = int(inp.node_offset[3])
    inp.k_tree[last:, :, 0] = float("-inf")
    with np.errstate(invalid="ignore"):
        ref, ref_lse = oracle_attn(inp)
    assert np.isfinite(ref[:last]).all() and np.isnan(ref[last:]).all()
    for splits in (1, 2, 3, 0):
        out, lse, _ = _run(step, inp, num_splits=splits)
        got, got_lse = W.widen(out), W.widen(lse)
        assert np.isnan(got[last:]).all(), splits
        assert np.abs(got[:last] - ref[:last]).max() <= 1e-5 and np.abs(got_lse[:last] - ref_lse[:last]).max() <= 1e-4, splits


@pytest.mark.parametrize("dtype,splits", [("f32", 16), ("bf16", 16), ("bf16", 5), ("bf16", 12)])
def test_a_row_does_not_depend_on_the_merge_that_it_takes(step, dtype, splits):
    """Few partial results are merged by one kernel, many (more than 8 MB of them) by another: the same arithmetic in the same
    order, so a sequence's rows are the same bits alone and in a batch."""
    lens = [1000, 2000, 300, 1500, 17, 2000, 900, 1200, 0, 1900, 640, 64, 5, 1100, 700, 1999]
    inp = W.make_verify_inputs(94, dtype, 28, 4, 128, lens, [W.chain_tree(8)] * len(lens))
    dev = step.to_device(inp)
    many, many_lse = step.tree_verify_attn(step.desc_for(inp, num_splits=splits), dev)
    rows = inp.total_nodes * 28 * splits * 128 * 4
    assert rows > 8 << 20 and rows // len(lens) <= 8 << 20
    for b in range(len(lens)):
        n0, n1 = int(inp.node_offset[b]), int(inp.node_offset[b + 1])
        one = step.DeviceInputs(dev.q[n0:n1], dev.k_tree[n0:n1], dev.v_tree[n0:n1], dev.k_pool, dev.v_pool, dev.block_table[b:b + 1],
                                dev.prefix_len[b:b + 1], dev.node_offset[b:b + 2] - n0, dev.parent[n0:n1])
        desc = step.make_desc(dtype, 1, 28, 4, 128, inp.page, inp.max_blocks, inp.num_blocks, n1 - n0, 8, inp.softmax_scale, splits)
        out, lse = step.tree_verify_attn(desc, one)
        assert torch.equal(out, many[n0:n1]) and torch.equal(lse, many_lse[n0:n1]), (b, lens[b])


@pytest.mark.parametrize("nodes", [8, 60])
@pytest.mark.parametrize("lens", [[1], [191], [193], [2048], [640, 64, 1500], [300] * 8, [100, 900, 0, 500, 70, 1400, 33, 256, 812]])
def test_short_pieces_of_a_few_sequences(hb, step, nodes, lens):
    """Sequences that do not occupy the workers with long pieces are cut from 3 (chains) or 4 tiles (trees)
    on: one sequence around one and two pieces, many pieces of one, unequal lengths (pieces as long
    as the longest sequence's); without a length hint the page table's span decides."""
    trees = [W.chain_tree(8) if nodes == 8 else W.seeded_tree(10 + i) for i in range(len(lens))]
    inp = W.make_verify_inputs(79, "bf16", 28, 4, 128, lens, trees, kv_std=1.0, q_std=1.0)
    ref = oracle_attn(inp)
    for hint in (0, max(lens)):
        out, lse, _ = _run(step, inp, num_splits=0, algo=hb.HB_ATTN_MFMA, hint=hint)
        check_attn(inp, out, lse, ref=ref, label=f"pieces {nodes} {lens} hint={hint}")


@pytest.mark.parametrize("n_nodes", [20, 33, 64])
@pytest.mark.parametrize("lens", [[0, 1, 31, 32, 33, 63], [64, 65, 95, 96, 97, 127, 128, 129], [255, 256, 257, 320]])
def test_tile_counts_and_tails_of_the_eight_wavefront_shape(hb, step, n_nodes, lens):
    """More than 128 rows: one to six tiles a workgroup and half-empty last blocks, whole and in pieces;
    trees that end in the first and in the second block of their tile, and one that fills it."""
    trees = [W.seeded_tree(40 + i, n_nodes=n_nodes, levels=4, root_fanout=5) for i in range(len(lens))]
    inp = W.make_verify_inputs(81, "bf16", 28, 4, 128, lens, trees, kv_std=1.0, q_std=1.0)
    ref = oracle_attn(inp)
    for splits in (1, 3, 0):
        out, lse, _ = _run(step, inp, num_splits=splits, algo=hb.HB_ATTN_MFMA)
        check_attn(inp, out, lse, ref=ref, label=f"tails {n_nodes} {lens} s={splits}")


def test_schedules_of_the_matrix_core_kernel(hb, step):
    """With num_splits = 0 the kernel cuts the KV itself, on the device, from the prefix lengths:
    work-proportionally when that finishes first (one long sequence among short ones: pieces of
    several sequences per workgroup, rows written directly next to rows that go through the
    merge), with equal pieces per sequence otherwise (equal lengths), and with host-planned
    chunks for more than 64 sequences."""
    cases = {
        "one long, many short": ([3000, 0, 70, 1, 130, 64, 17, 300], 8),
        "equal lengths": ([1536] * 4, 4),
        "more than 64 sequences": ([33 + 7 * i for i in range(66)], 66),
    }
    for name, (lens, B) in cases.items():
        trees = [W.seeded_tree(10 + i, n_nodes=15 + (i * 11) % 46) for i in range(B)]
        inp = W.make_verify_inputs(91, "bf16", 28, 4, 128, lens, trees, kv_std=1.0, q_std=1.0)
        ref = oracle_attn(inp)
        out, lse, desc = _run(step, inp, num_splits=0, algo=hb.HB_ATTN_MFMA, hint=max(lens))
        check_attn(inp, out, lse, ref=ref, label=f"schedule: {name}")
        out2, lse2, _ = _run(step, inp, num_splits=0, algo=hb.HB_ATTN_MFMA)  # no length hint
        check_attn(inp, out2, lse2, ref=ref, label=f"schedule, no hint: {name}")


def test_poisoned_tree_nodes_off_the_path_do_not_leak(hb, step):
    """Inputs already carry NaN in every slot past the prefix and in unmapped pages.  Here the
    tree K/V of one branch is additionally set to Inf/NaN: nodes outside that branch must be
    bitwise unchanged."""
    inp = W.make_config(1)
    par = inp.trees()[0]
    bad = 1  # first child of the root; poison it and all its descendants
    sub = [i for i in range(len(par)) if bad in _path(par, i)]
    clean = [i for i in range(len(par)) if i not in sub]
    for algo in _algos(hb, inp):
        base, lse0, _ = _run(step, inp, algo=algo)
        dirty = W.make_config(1)
        dirty.k_tree[sub] = float("inf")
        dirty.v_tree[sub] = float("nan")
        got, lse1, _ = _run(step, dirty, algo=algo)
        assert torch.equal(base[clean].view(torch.int16), got[clean].view(torch.int16))
        assert torch.equal(lse0[clean], lse1[clean])


def _path(par, i):
    out = []
    while i >= 0:
        out.append(i); i = int(par[i])
    return out


def test_results_are_deterministic(hb, step):
    inp = W.make_config(2, scale_down=8)
    for algo in _algos(hb, inp):
        a, la, _ = _run(step, inp, algo=algo)
        b, lb, _ = _run(step, inp, algo=algo)
        assert torch.equal(a.view(torch.int16), b.view(torch.int16)) and torch.equal(la, lb)


@pytest.mark.parametrize("cfg,tree", [(2, "tree"), (3, "tree"), (4, "tree"), (4, "chain8")])
def test_full_size_workloads_every_node(hb, step, cfg, tree):
    """Full sizes, default launch configuration (the one the benchmark times), with and without
    the length hint the benchmark passes; the oracle recomputes every node of every sequence.
    The 8-node-chain run of the full-step workload takes the four-wavefront kernel with the
    device-side KV cut over 16 ragged prefixes."""
    inp = W.make_config(cfg, tree=tree)
    ref = oracle_attn(inp)
    hint = int(inp.prefix_len.max())
    for kw in (dict(), dict(hint=hint)):
        out, lse, desc = _run(step, inp, **kw)
        check_attn(inp, out, lse, ref=ref, label=f"cfg{cfg} {tree} full {kw}")
        assert torch.isfinite(out.float()).all()
        # per-row check as well: a wrong row must not hide in the batch-wide norms
        got, want = W.widen(out), ref[0]
        rel_rows = np.linalg.norm(got - want, axis=2) / np.linalg.norm(want, axis=2)
        assert rel_rows.max() <= 3e-2, f"cfg{cfg} {tree}: worst row rel err {rel_rows.max():.3e}"
    if cfg == 3 and hb.HB_ATTN_MFMA in _algos(hb, inp):
        # only 8 (sequence, kv head) pairs: the KV-sharing kernel must split the long context
        assert hb.hb_tree_verify_attn_num_splits(desc) > 1


def _planted_scores(inp, log2_scores):
    """Overwrite sequence 0 so that the prefix key at position p scores log2_scores[p] (in log2
    units, i.e. score * log2(e)) against a query that is c_r * e_0, c_r = 1 for row 0 and
    slightly different for other rows; all other key components are 0, V stays random."""
    L = len(log2_scores)
    assert int(inp.prefix_len[0]) == L
    ln2 = float(np.log(2.0))
    q = torch.zeros_like(inp.q, dtype=torch.float32)
    T, Hq, _ = inp.q.shape
    # row-dependent gain: rows cross the rescale threshold at different blocks
    gain = 1.0 + 0.03125 * (torch.arange(T * Hq).reshape(T, Hq) % 5).float()
    q[:, :, 0] = gain / inp.softmax_scale
    inp.q.copy_(q.to(inp.q.dtype))
    kt = torch.zeros_like(inp.k_tree, dtype=torch.float32)
    kt[:, :, 0] = float(log2_scores[-1]) * ln2  # tree keys score like the last prefix key
    inp.k_tree.copy_(kt.to(inp.k_tree.dtype))
    for p in range(L):
        blk = int(inp.block_table[0, p // inp.page])
        row = torch.zeros(inp.D)
        row[0] = float(log2_scores[p]) * ln2
        inp.k_pool[blk, :, p % inp.page] = row.to(inp.k_pool.dtype)
    return inp


@pytest.mark.parametrize("shape", ["tree60_gqa7", "chain8_gqa7", "tree20_gqa1"])
def test_reference_exponent_of_the_online_softmax_under_climbing_scores(hb, step, shape):
    """The matrix-core kernel keeps a per-row reference exponent that moves only when a score
    outgrows it by a fixed slack (2^8).  Scores that climb by just under / just over that slack
    from one 32-key block to the next, by fractions of it, that ramp from 60 below to 60 above,
    that jump up once at the very end, and that fall all the way: each must still give the
    oracle's output and log-sum-exp."""
    Hq, Hkv, tree = {"tree60_gqa7": (28, 4, W.seeded_tree(5)), "chain8_gqa7": (28, 4, W.chain_tree(8)),
                     "tree20_gqa1": (2, 2, W.seeded_tree(6, n_nodes=20))}[shape]
    nblk = 40
    L = 32 * nblk
    blk = np.arange(L) // 32
    jitter = np.random.default_rng(0).uniform(-0.5, 0.0, size=L)
    patterns = {
        "step 7.9": 7.9 * blk, "step 8.1": 8.1 * blk, "step 3.9": 3.9 * blk, "step 16.3": 16.3 * blk,
        "ramp -60..60": np.linspace(-60.0, 60.0, L) / np.log(2.0),
        "late jump": np.where(np.arange(L) == L - 3, 90.0, 0.0) + jitter,
        "falling": -7.9 * blk + jitter,
        "sawtooth": 7.9 * (blk % 3) + 8.1 * (blk // 3) + jitter,
    }
    for name, sc in patterns.items():
        inp = W.make_verify_inputs(321, "bf16", Hq, Hkv, 128, [L], [tree], kv_std=1.0, q_std=1.0)
        inp = _planted_scores(inp, sc)
        ref = oracle_attn(inp)
        for splits in (1, 0, 3):
            out, lse, _ = _run(step, inp, num_splits=splits, algo=hb.HB_ATTN_MFMA)
            check_attn(inp, out, lse, ref=ref, label=f"{shape} {name} splits={splits}")


def test_device_side_cut_on_random_batches(hb, step):
    """Seeded random batches (1..20 sequences, prefix lengths 0..2500 with a bias to short ones,
    trees of 15..60 nodes) through the matrix-core kernel with the library's own KV cut."""
    rng = np.random.default_rng(2024)
    for case in range(6):
        B = int(rng.integers(1, 21))
        lens = [int(x) for x in np.minimum(rng.geometric(1.0 / 400.0, size=B) - 1, 2500)]
        if case == 0:
            lens[0] = 2500
        trees = [W.seeded_tree(1000 * case + i, n_nodes=int(rng.integers(15, 61))) for i in range(B)]
        inp = W.make_verify_inputs(500 + case, "bf16", 8, 2, 128, lens, trees, kv_std=1.0, q_std=1.0)
        ref = oracle_attn(inp)
        out, lse, _ = _run(step, inp, num_splits=0, algo=hb.HB_ATTN_MFMA, hint=max(max(lens), 1))
        check_attn(inp, out, lse, ref=ref, label=f"random batch {case}: B={B} lens={lens}")
