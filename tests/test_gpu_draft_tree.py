"""GPU parity of the draft tree's construction: hb_topk_logprob (token ids exact, log-probabilities
within 2e-5 of the float64 definition: float32 exp/log and a float32 sum over the vocabulary),
hb_tree_grow and hb_tree_finalize (bit-exact: integer outputs, and scores that are one float32
addition each)."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import DraftTreeRef, topk_logprob_ref

pytestmark = pytest.mark.gpu

LOGP_TOL = 2e-5


@pytest.fixture(scope="module")
def S():
    import paper_2509_18824_amd.step as s
    return s


def _topk_case(S, x, k, bf16=False):
    t = torch.from_numpy(x).cuda()
    if bf16:
        t = t.to(torch.bfloat16)
        x = t.float().cpu().numpy()
    ids, logp = S.topk_logprob(t.contiguous(), k)
    torch.cuda.synchronize()
    rid, rlogp = topk_logprob_ref(x, k)
    assert np.array_equal(ids.cpu().numpy(), rid)
    got = logp.cpu().numpy()
    assert np.abs(got - rlogp).max() <= LOGP_TOL, np.abs(got - rlogp).max()
    assert (got <= 0).all()


@pytest.mark.parametrize("M,V,k", [(5, 1000, 4), (3, 2049, 32), (7, 33, 8), (3, 1001, 5), (1, 16384, 10),
                                   (2, 16385, 10), (40, 32000, 10), (1, 7, 7)])
def test_topk_small_shapes(S, M, V, k):
    _topk_case(S, W.make_draft_logits(11 + M, M, V), k)


@pytest.mark.parametrize("M,V,k", [(4, 5000, 16), (2, 40000, 10)])
def test_topk_equal_logits_go_to_the_lower_token_id(S, M, V, k):
    _topk_case(S, W.make_draft_logits(21, M, V, ties=True), k)
    x = np.zeros((2, 3000), dtype=np.float32)  # everything equal, signed zeros mixed in
    x[0, ::2] = -0.0
    _topk_case(S, x, 9)
    x = np.full((1, 2500), -np.inf, dtype=np.float32)  # -inf entries are ordinary, just last
    x[0, [2000, 17]] = [1.0, 1.0]
    ids, logp = S.topk_logprob(torch.from_numpy(x).cuda(), 4)
    assert ids.cpu().numpy().tolist() == [[17, 2000, 0, 1]]
    assert np.allclose(logp.cpu().numpy()[0, :2], -np.log(2.0), atol=1e-6) and np.isneginf(logp.cpu().numpy()[0, 2:]).all()


@pytest.mark.parametrize("M,V,k,bf16,ties", [(3, 16388, 10, False, False),   # last chunk: a single 16-byte vector
                                              (70, 32768, 12, True, True),     # bf16, more than a thousand chunks
                                              (600, 4096, 10, False, False),   # one chunk per row, two rounds of rows
                                              (33, 40008, 32, True, False)])   # bf16, last chunk of one vector, k = 32
def test_topk_rows_of_whole_vectors(S, M, V, k, bf16, ties):
    """Rows that consist of whole 16-byte vectors (vector loads all the way, no ragged end), with
    a last chunk of a single vector, many more chunks than resident workgroups, bf16 and ties."""
    _topk_case(S, W.make_draft_logits(41 + M, M, V, ties=ties), k, bf16=bf16)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("M,V,k", [(6, 16385, 10), (9, 16391, 32), (5, 33003, 7), (8, 9, 9), (4, 1027, 12), (17, 2, 1)])
def test_topk_rows_that_start_anywhere(S, M, V, k, bf16):
    """Rows of odd length start at every offset inside a 16-byte piece: values before the first and
    behind the last whole piece, chunks of one value, rows without a whole piece."""
    _topk_case(S, W.make_draft_logits(51 + M, M, V), k, bf16=bf16)


def test_topk_masked_and_not_finite(S):
    """Masked ranges (-inf) that fill whole chunks and all but a few values of one, a plateau of
    more equal values than the candidate list holds, and NaN entries, which count as -inf."""
    x = W.make_draft_logits(61, 5, 40001)
    x[0, 16384:32768] = -np.inf
    x[1, 100:] = -np.inf
    x[2, 5000:9000] = 50.0
    _topk_case(S, x, 10)
    _topk_case(S, x, 10, bf16=True)
    y = x.copy()
    y[3, ::3] = np.nan
    y[4, 16384:32768] = np.nan
    x[3, ::3] = -np.inf
    x[4, 16384:32768] = -np.inf
    ids, logp = S.topk_logprob(torch.from_numpy(y).cuda(), 10)
    rid, rlogp = topk_logprob_ref(x, 10)
    assert np.array_equal(ids.cpu().numpy(), rid) and np.abs(logp.cpu().numpy() - rlogp).max() <= LOGP_TOL


@pytest.mark.parametrize("bf16", [False, True])
def test_topk_signalling_nan_counts_as_minus_infinity(S, bf16):
    """Signalling NaNs beside the only values of a masked row, in every place of a 16-byte piece, in the
    values outside the pieces, and among ordinary values."""
    dtype, snan = (np.int16, 0x7F81) if bf16 else (np.int32, 0x7F800001)
    V = 20003
    x = np.full((18, V), -np.inf, dtype=np.float32)
    at = []
    for m in range(17):
        x[m, 800 + m] = 5.0
        at += [(m, 800 + (m & ~7) + i) for i in range(8) if (m & ~7) + i != m]
    x[9:17, :] = -np.inf  # these rows hold their value where a row of odd length starts or ends
    for m in range(9, 17):
        x[m, m - 9 if m < 13 else V - 1 - (m - 13)] = 5.0
        at += [(m, i) for i in range(8) if x[m, i] != 5.0] + [(m, V - 1 - i) for i in range(8) if x[m, V - 1 - i] != 5.0]
    x[17] = W.make_draft_logits(71, 1, V)[0]
    at += [(17, int(i)) for i in np.argsort(-x[17])[:40:2]]
    bits = (torch.from_numpy(x).to(torch.bfloat16).view(torch.int16) if bf16 else torch.from_numpy(x).view(torch.int32)).numpy().copy()
    ref = torch.from_numpy(bits.copy()).view(torch.bfloat16 if bf16 else torch.float32).float().numpy()
    for m, i in at:
        bits[m, i] = dtype(snan)
        ref[m, i] = -np.inf
    t = torch.from_numpy(bits).cuda().view(torch.bfloat16 if bf16 else torch.float32)
    ids, logp = S.topk_logprob(t, 3)
    rid, rlogp = topk_logprob_ref(ref, 3)
    assert np.array_equal(ids.cpu().numpy(), rid)
    got, fin = logp.cpu().numpy(), np.isfinite(rlogp)
    assert np.abs(got[fin] - rlogp[fin]).max() <= LOGP_TOL and np.isneginf(got[~fin]).all()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("V", [7, 33, 100, 16384 + 40, 40001])
def test_topk_masks_of_the_types_lowest_value(S, V, bf16):
    """Rows and chunks whose every value is the type's lowest finite one, with and without -inf, and one
    chunk of ordinary values beside them: the difference to the maximum is finite, its scaled parts are not."""
    low = float(torch.finfo(torch.bfloat16 if bf16 else torch.float32).min)
    k = min(V, 10)
    x = np.full((5, V), low, dtype=np.float32)
    x[1, 1::2] = -np.inf
    x[2, :5] = [3.0, 2.0, 1.0, 0.0, -1.0]
    x[3, -5:] = [3.0, 2.0, 1.0, 0.0, -1.0]
    x[4] = -low
    t = torch.from_numpy(x).cuda().to(torch.bfloat16 if bf16 else torch.float32)
    x = t.float().cpu().numpy()
    ids, logp = S.topk_logprob(t, k)
    rid, rlogp = topk_logprob_ref(x, k)
    assert np.array_equal(ids.cpu().numpy(), rid)
    got, want = logp.cpu().numpy(), rlogp.astype(np.float32)
    # the log-probability is a float32 sum of the maximum and the logarithm of the exponentials' sum:
    # at the type's ends that logarithm is lost in the maximum's rounding, in the result as in its bound
    tol = np.where(np.abs(x.max(1, keepdims=True)) > 1e30, np.float32(np.log(V)), LOGP_TOL)
    near = np.isfinite(want) & (np.abs(want) < 1e30)
    assert (np.abs(got - want)[near] <= np.broadcast_to(tol, got.shape)[near]).all(), (got, want)
    assert np.array_equal(got[~near] < -1e30, want[~near] < -1e30) and not np.isnan(got).any()


@pytest.mark.parametrize("V", [9, 60, 250])
def test_topk_few_values_of_large_magnitude(S, V):
    """Too few values for a threshold, with a common offset of some thousands: the exponentials are those
    of the differences to the maximum (the offset's product with log2 e alone is off by 1e-4)."""
    x = (W.make_draft_logits(91, 4, V) + np.float32(-3000.0)).astype(np.float32)
    ids, logp = S.topk_logprob(torch.from_numpy(x).cuda(), min(V, 9))
    rid, rlogp = topk_logprob_ref(x, min(V, 9))
    assert np.array_equal(ids.cpu().numpy(), rid)
    # lse = maximum + log(sum) and logit - lse round once each at 3000 (half a unit of 2^-12 each)
    assert np.abs(logp.cpu().numpy() - rlogp).max() <= 2.0 ** -12 + LOGP_TOL


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("V", [3000, 16384, 40001])
def test_topk_values_that_leave_the_first_ones_behind(S, V, bf16):
    """The exponentials' reference starts with a thread's first values: masks there (-inf and the type's lowest),
    ramps that rise or fall by hundreds from piece to piece, a common offset; whole and partial chunks."""
    x = W.make_draft_logits(95, 6, V)
    x[0, :V // 3] = -np.inf
    x[1, :V // 3] = float(torch.finfo(torch.bfloat16 if bf16 else torch.float32).min)
    x[2] = np.linspace(-5000, 5000, V)
    x[3] = np.linspace(5000, -5000, V)
    x[4] -= np.float32(30000.0)
    x[5, V // 2:] += np.float32(100.0)
    t = torch.from_numpy(x).cuda().to(torch.bfloat16 if bf16 else torch.float32)
    x = t.float().cpu().numpy()
    ids, logp = S.topk_logprob(t, 10)
    rid, rlogp = topk_logprob_ref(x, 10)
    assert np.array_equal(ids.cpu().numpy(), rid)
    # lse rounds at the maximum's size: half a unit of 2^-11 below 8192, of 2^-9 at 30000
    tol = LOGP_TOL + np.array([0, 0, 2.0 ** -12, 2.0 ** -12, 2.0 ** -10, 0])[:, None]
    assert (np.abs(logp.cpu().numpy() - rlogp) <= tol).all(), np.abs(logp.cpu().numpy() - rlogp).max(1)


def _topk_us(S, x, k=10):
    """Shortest of five means of twenty calls."""
    ids, logp = S.topk_logprob(x, k)
    best = float("inf")
    for _ in range(5):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        for _ in range(20):
            S.topk_logprob(x, k)
        end.record()
        torch.cuda.synchronize()
        best = min(best, start.elapsed_time(end) / 20 * 1e3)
    return best, ids, logp


@pytest.mark.parametrize("offset", [1000.0, 10000.0, -30000.0])
def test_topk_takes_no_longer_for_a_common_offset(S, offset):
    """Distinct float32 logits that share an offset keep to the path of the plain ones: a threshold of 16 bits,
    which everything reaches, took 2 to 8 times as long.  Twice leaves room for the clock."""
    g = torch.Generator(device="cuda").manual_seed(7)
    x = torch.randn((160, 152064), generator=g, device="cuda")
    plain, _, _ = _topk_us(S, x)
    x += offset
    shifted, ids, logp = _topk_us(S, x)
    assert torch.equal(x.gather(1, ids.long()), torch.topk(x, 10, dim=1).values)
    # lse and logit - lse round once each at the offset's size
    lse = torch.logsumexp(x.double(), 1, keepdim=True)
    assert (logp.double() - (x.double().gather(1, ids.long()) - lse)).abs().max() <= abs(offset) * 2.0 ** -23 + LOGP_TOL
    assert shifted <= 2.0 * plain, (plain, shifted)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("mask", [-65504.0, -1e9, -1e10, -1e20, -1e30, -2e38])
def test_topk_takes_no_longer_for_scattered_masks(S, mask, bf16):
    """Nine tenths of the tokens at a large negative value, so that many threads begin with nothing else: the
    exponentials' reference must not become an infinity there (2.3 times as long).  1.6 leaves room for the clock."""
    g = torch.Generator(device="cuda").manual_seed(8)
    x = torch.randn((160, 152064), generator=g, device="cuda").to(torch.bfloat16 if bf16 else torch.float32)
    drop = torch.rand(x.shape, generator=g, device="cuda") < 0.9
    plain, _, _ = _topk_us(S, x.masked_fill(drop, float("-inf")))
    x = x.masked_fill(drop, mask)
    masked, ids, logp = _topk_us(S, x)
    assert torch.equal(x.gather(1, ids.long()), torch.topk(x, 10, dim=1).values)
    lse = torch.logsumexp(x.double(), 1, keepdim=True)
    assert (logp.double() - (x.double().gather(1, ids.long()) - lse)).abs().max() <= LOGP_TOL
    assert masked <= 1.6 * plain, (plain, masked)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("V", [700, 16384, 40001])
def test_topk_of_values_around_the_least_reference(S, V, bf16):
    """Chunks whose every value lies above, at and below -2^30 / log2 e, where the exponentials' reference stops,
    spread by less and by more than float32 resolves there, and ordinary values behind such ones."""
    rng = np.random.default_rng(96)
    edge = -(2.0 ** 30) / np.log2(np.e)
    x = np.empty((6, V), dtype=np.float32)
    x[0] = edge + 1e3 * rng.standard_normal(V)
    x[1] = edge - 2e4 * rng.random(V)
    x[2] = edge + 2e4 * rng.random(V)
    x[3] = -1e10 + 1e5 * rng.standard_normal(V)
    x[4] = -3e20 * (1 + rng.random(V))
    x[5] = np.where(np.arange(V) < V // 2, -1e10, rng.standard_normal(V))
    t = torch.from_numpy(x).cuda().to(torch.bfloat16 if bf16 else torch.float32)
    x = t.float().cpu().numpy()
    ids, logp = S.topk_logprob(t, 10)
    rid, rlogp = topk_logprob_ref(x, 10)
    assert np.array_equal(ids.cpu().numpy(), rid)
    # lse and logit - lse round once each at the maximum's size (half a unit of 2^-23 of it at most)
    tol = LOGP_TOL + np.abs(x.max(1, keepdims=True)) * 2.0 ** -23
    assert (np.abs(logp.cpu().numpy() - rlogp) <= tol).all(), np.abs(logp.cpu().numpy() - rlogp).max(1)


def test_topk_full_vocabulary_every_row_of_a_level(S):
    """The shape of one level of the batch-16 workload: 160 rows (16 sequences x 10 frontier
    nodes) over the vocabulary of 152064, float32; and the root level's 16 rows in bf16."""
    _topk_case(S, W.make_draft_logits(31, 160, 152064), 10)
    _topk_case(S, W.make_draft_logits(32, 16, 152064), 10, bf16=True)


def _grow_both(S, B, K, T, N, V, seed, ties=False, uniform=False):
    builder = S.DraftTreeBuilder(B, K, T)
    refs = [DraftTreeRef(K, T) for _ in range(B)]
    for level in range(T):
        F = 1 if level == 0 else K
        if uniform:
            ids = torch.arange(K, dtype=torch.int32).repeat(B * F, 1).cuda() + 100 * level
            logp = torch.full((B * F, K), -2.0, dtype=torch.float32).cuda()
        else:
            logits = torch.from_numpy(W.make_draft_logits(seed * 100 + level, B * F, V, ties=ties)).cuda()
            ids, logp = S.topk_logprob(logits, K)
        frontier, slot = builder.grow(ids, logp)
        torch.cuda.synchronize()
        ids_h = ids.cpu().numpy().reshape(B, F, K)
        logp_h = logp.cpu().numpy().reshape(B, F, K)
        for b in range(B):
            rf, rs = refs[b].grow(ids_h[b], logp_h[b])
            assert frontier[b].cpu().numpy().tolist() == rf, (level, b)
            assert slot[b].cpu().numpy().tolist() == rs, (level, b)
    root = torch.arange(B, dtype=torch.int32).cuda() + 7
    out = builder.finalize(N, root)
    torch.cuda.synchronize()
    n = N
    h = {k: v.cpu().numpy() for k, v in out.items()}
    assert h["node_offset"].tolist() == [b * n for b in range(B + 1)]
    import paper_2509_18824_amd as hb
    for b in range(B):
        parent, ids, depth, anc, cand, score = refs[b].finalize(N, 7 + b)
        sl = slice(b * n, (b + 1) * n)
        assert len(parent) == n
        assert np.array_equal(h["parent"][sl], parent), b
        assert np.array_equal(h["draft_ids"][sl], ids), b
        assert np.array_equal(h["depth"][sl], depth), b
        assert np.array_equal(h["anc_mask"][sl].view(np.uint64), anc), b
        assert np.array_equal(h["node_cand"][sl], cand), b
        assert np.array_equal(h["node_score"][sl].view(np.uint32), score.view(np.uint32)), b
        hb.hb_tree_validate_host(h["parent"][sl].tolist())
    return h


def test_tree_of_the_batch16_workload_shape(S):
    """16 sequences, 10 children per node, 5 levels, 60 nodes: the tree shape the verification
    workloads use."""
    h = _grow_both(S, 16, 10, 5, 60, 32000, seed=1)
    assert h["depth"].max() <= 5 and h["depth"].max() >= 2


@pytest.mark.parametrize("B,K,T,N", [(1, 1, 5, 6), (3, 2, 2, 4), (2, 4, 3, 1), (2, 3, 3, 22), (5, 8, 4, 64),
                                     (2, 32, 2, 40), (1, 7, 1, 8)])
def test_tree_shapes_and_edges(S, B, K, T, N):
    """Chains (K = 1), root-only trees (N = 1), everything kept (N - 1 = all candidates), the
    widest node (K = 32), the largest tree (64 nodes), a single level."""
    h = _grow_both(S, B, K, T, N, 5000, seed=B + K + T)
    if K == 1:
        assert h["parent"].tolist() == [-1, 0, 1, 2, 3, 4]


def test_tree_with_equal_scores(S):
    _grow_both(S, 2, 3, 3, 9, 0, seed=0, uniform=True)
    _grow_both(S, 4, 6, 4, 48, 3000, seed=9, ties=True)


@pytest.mark.parametrize("B,K,T,N", [(2, 22, 2, 64), (2, 16, 3, 64), (3, 8, 9, 33), (1, 31, 5, 64), (1, 8, 64, 2), (2, 2, 64, 64)])
def test_trees_from_many_candidates(S, B, K, T, N):
    """506 candidates (one wavefront), 528 and 520 (four), 3875 and 4040 (most of what they hold), chains of 64
    levels; distinct scores, ties, and all equal."""
    _grow_both(S, B, K, T, N, 3000, seed=K + T)
    _grow_both(S, B, K, T, N, 3000, seed=K + T, ties=True)
    _grow_both(S, B, K, T, N, 0, seed=0, uniform=True)


@pytest.mark.parametrize("B,K,T,N", [(2, 1, 64, 40), (2, 2, 17, 64), (1, 2, 32, 33), (2, 2, 33, 64), (1, 2, 64, 9), (2, 3, 30, 64)])
def test_trees_of_every_run_length(S, B, K, T, N):
    """64 candidates (one a lane), 66 and 126 (two), 130 and 254 (four), 264 (eight)."""
    _grow_both(S, B, K, T, N, 3000, seed=K + T)
    _grow_both(S, B, K, T, N, 3000, seed=K + T, ties=True)
    _grow_both(S, B, K, T, N, 0, seed=0, uniform=True)


def test_finalising_few_candidates_takes_less_than_many(S):
    """6 and 55 candidates against 410, in graphs: 3.5 and 3.6 us against 7.1 (6.6 and 6.7 when every lane kept eight)."""
    def us(B, K, T, N):
        builder = S.DraftTreeBuilder(B, K, T)
        for level in range(T):
            logits = torch.from_numpy(W.make_draft_logits(level, B * (K if level else 1), 2000)).cuda()
            builder.grow(*S.topk_logprob(logits, K))
        root = torch.zeros(B, dtype=torch.int32, device="cuda")
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            out = builder.finalize(N, root)
        torch.cuda.synchronize()
        args = [out[k] for k in ("node_offset", "parent", "draft_ids", "depth", "anc_mask", "node_cand", "node_score")]
        import paper_2509_18824_amd as hb
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            for _ in range(50):
                hb.hb_tree_finalize(B, K, T, N, builder.cand_score, builder.cand_token, builder.cand_parent, root, *args)
        best = float("inf")
        for _ in range(8):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            graph.replay()
            end.record()
            torch.cuda.synchronize()
            best = min(best, start.elapsed_time(end) / 50 * 1e3)
        return best

    many = us(16, 10, 5, 60)
    assert us(16, 2, 2, 4) <= 0.75 * many and us(16, 5, 3, 40) <= 0.75 * many


def test_tree_build_replays_from_a_hip_graph(S):
    """Top-k, growth of every level and finalisation only enqueue kernels (no allocation, no
    memset): captured once, replayed on changing logits with eager builds in between, every replay
    equals the eager build bit for bit."""
    import paper_2509_18824_amd as hb
    B, K, T, N, V = 4, 5, 3, 24, 6000
    levels = [torch.empty((B * (1 if l == 0 else K), V), dtype=torch.float32, device="cuda") for l in range(T)]
    ids = [torch.empty((x.shape[0], K), dtype=torch.int32, device="cuda") for x in levels]
    lps = [torch.empty((x.shape[0], K), dtype=torch.float32, device="cuda") for x in levels]
    ws = S.alloc_workspace(hb.hb_topk_logprob_workspace_bytes(B * K, V, K))
    builder = S.DraftTreeBuilder(B, K, T)
    root = torch.arange(B, dtype=torch.int32, device="cuda")
    n = B * N
    i32 = lambda m: torch.empty(m, dtype=torch.int32, device="cuda")
    outs = [i32(B + 1), i32(n), i32(n), i32(n), torch.empty(n, dtype=torch.int64, device="cuda"), i32(n),
            torch.empty(n, dtype=torch.float32, device="cuda")]

    def build():
        for l in range(T):
            hb.hb_topk_logprob(levels[l], K, ids[l], lps[l], ws)
            hb.hb_tree_grow(B, K, T, l, ids[l], lps[l], builder.cand_score, builder.cand_token, builder.cand_parent,
                            builder.frontier, builder.frontier_slot)
        hb.hb_tree_finalize(B, K, T, N, builder.cand_score, builder.cand_token, builder.cand_parent, root, *outs)

    def fill(seed):
        for l, x in enumerate(levels):
            x.copy_(torch.from_numpy(W.make_draft_logits(seed * 10 + l, x.shape[0], V)))

    fill(0)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        build()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        build()
    seen = set()
    for seed in (1, 2, 3):
        fill(seed)
        build()
        torch.cuda.synchronize()
        eager = [t.clone() for t in outs]
        for t in outs:
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(eager, outs):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
        hb.hb_tree_validate_host(outs[1][:N].cpu().tolist())
        seen.add(tuple(outs[2].cpu().tolist()))
    assert len(seen) == 3  # the logits, and with them the trees, did change between replays
