"""GPU parity: hb_lmhead_argmax against the float64 oracle.

Margin rule: where the oracle's top-1 logit leads the runner-up by more than EPS, the GPU id
must be the oracle's; elsewhere (a near tie that fp32 accumulation order may flip) it must be
one of the two.  EPS = 1e-4 * |h| * |w|_typ bounds the fp32 accumulation error of a K-term dot
product (K * 2^-24 * sum|h_k w_k| is a few 1e-6 of that product for K = 3584)."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import lmhead_logits_ref

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def step():
    import paper_2509_18824_amd.step as s
    return s


def _check(hidden, weight, ids, mx, rows=None, block=192):
    rows = np.arange(hidden.shape[0]) if rows is None else np.asarray(rows)
    w = W.widen(weight)
    w_rms = np.sqrt((w * w).sum(1).mean())
    got_all = ids.cpu().numpy()
    mx_all = mx.cpu().numpy() if mx is not None else None
    n_clear = 0
    for i0 in range(0, len(rows), block):  # blocks of rows bound the float64 logits in memory
        rb = rows[i0:i0 + block]
        h = W.widen(hidden)[rb]
        logits = lmhead_logits_ref(h, w)
        r = np.arange(len(rb))
        top1 = np.argmax(logits, axis=1)  # first maximum = lowest id
        best = logits[r, top1]
        if logits.shape[1] > 1:
            rest = logits.copy()
            rest[r, top1] = -np.inf
            top2 = np.argmax(rest, axis=1)
        else:
            top2 = top1
        margin = best - logits[r, top2]
        eps = 1e-4 * np.linalg.norm(h, axis=1) * w_rms
        got = got_all[rb]
        clear = margin > eps
        assert (got[clear] == top1[clear]).all(), "argmax differs where the margin is clear"
        assert np.logical_or(got == top1, got == top2)[~clear].all()
        if mx_all is not None:
            assert np.abs(mx_all[rb] - logits[r, got]).max() <= 1e-2
        n_clear += int(clear.sum())
    return n_clear


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
# K % 64 == 0 takes the matrix-core kernel: the shapes below cover its four hidden-tile heights
# (64 .. 256 rows), one and several hidden tiles, odd and even numbers of K steps, and
# vocabularies below, at and above one 256-row tile
@pytest.mark.parametrize("M,K,V", [(1, 8, 1), (5, 64, 1000), (60, 136, 777), (128, 512, 4099), (300, 264, 513),
                                   (250, 192, 1500), (300, 256, 777), (1000, 128, 3000), (380, 64, 600),
                                   (64, 320, 256), (193, 448, 255)])
def test_small_shapes(step, dtype, M, K, V):
    hidden, weight = W.make_lmhead_inputs(M * 7 + V, M, K, V, dtype=dtype, w_std=0.05)
    ids, mx = step.lmhead_argmax(hidden.cuda(), weight.cuda())
    torch.cuda.synchronize()
    _check(hidden, weight, ids, mx)


@pytest.mark.parametrize("M,K,V", [(1, 64, 16385), (64, 128, 16384), (64, 64, 20480), (60, 192, 81920), (8, 64, 81921),
                                   (61, 64, 152064), (128, 64, 152065), (100, 128, 164000), (65, 64, 36864), (70, 192, 17000),
                                   (33, 4096, 16400), (128, 2048, 24600), (192, 64, 20480), (129, 64, 20481), (256, 128, 24600),
                                   (255, 64, 40960), (256, 64, 40961), (1, 1024, 5), (64, 1024, 129), (65, 1024, 300),
                                   (64, 1088, 12288), (128, 1024, 12288), (60, 1024, 12289), (128, 2048, 16384),
                                   (100, 2112, 16384), (1, 640, 16385), (64, 704, 20480), (128, 1536, 17000), (65, 1600, 36864), (100, 512, 66000),
                                   (128, 128, 131073), (8, 128, 81921), (60, 192, 65537), (192, 2112, 20500), (129, 2112, 24577), (256, 2112, 24600), (255, 2112, 40960), (250, 2112, 40961)])
def test_runs_of_vocabulary_rows(step, M, K, V):
    """Up to 128 rows, and some calls of up to 256, a workgroup has a run of vocabulary rows for itself: runs that are missing,
    ragged, one tile, one row more, several tiles; both sides of the lines.  Two rows, the first and the last of the vocabulary
    among them, are equal and far ahead for some hidden rows."""
    hidden, weight = W.make_lmhead_inputs(M + V, M, K, V, dtype="bf16", w_std=0.05)
    rng = np.random.default_rng(M + V)
    rows = range(0, M, 7)
    places = 1 + np.sort(rng.choice(V - 2, (len(rows), 2), replace=False), axis=1)
    places[0] = 0, V - 1
    for m, at in zip(rows, places):  # the same row in two places: the lower one wins
        weight[at] = hidden[m].float().mul(0.5).to(weight.dtype)
    ids, mx = step.lmhead_argmax(hidden.cuda(), weight.cuda())
    torch.cuda.synchronize()
    _check(hidden, weight, ids, mx)
    assert (ids.cpu().numpy()[list(rows)] == places[:, 0]).all()


@pytest.mark.parametrize("K,V", [(64, 300), (1024, 300), (1024, 12288), (1088, 12300), (192, 17000), (2048, 24600), (4096, 17000), (2048, 70000), (3584, 36000), (2048, 100000)])
def test_equal_rows_and_any_number_of_hidden_rows(step, K, V):
    """A row's sum over K has one order, wherever it lies in the vocabulary and however many hidden rows there are: of equal rows in
    one tile, two tiles of a run, or the runs of two workgroups the lowest wins, and a hidden row has the same id and the same
    bits of its largest logit in every call that it is part of."""
    gen = torch.Generator(device="cuda").manual_seed(K + V)
    weight = torch.empty((V, K), dtype=torch.bfloat16, device="cuda").normal_(0, 0.05, generator=gen)
    hidden = torch.empty((960, K), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=gen)
    rng = np.random.default_rng(K + V)
    apart = [1, 4, 16, 70, 200, 305, V // 256, V // 8, V // 2]
    lower, used = {}, set()
    for i, m in enumerate(list(range(24)) + list(range(24, 960, 40))):
        d = apart[i % len(apart)]
        at = [int(v) for v in rng.permutation(max(1, V - d)) if v + d < V and not used & {int(v), int(v) + d}][:1]
        for v in at:
            used |= {v, v + d}
            weight[[v, v + d]] = hidden[m] * 0.5
            lower[m] = v
    assert len(lower) > 40
    all_ids, all_mx = step.lmhead_argmax(hidden, weight)
    for M in (1, 8, 24, 64, 65, 100, 128, 129, 192, 200, 256, 257, 320, 480, 700, 960):
        ids, mx = step.lmhead_argmax(hidden[:M].contiguous(), weight)
        assert torch.equal(ids, all_ids[:M]) and torch.equal(mx, all_mx[:M]), M
        got = ids.cpu().numpy()
        assert all(got[m] == v for m, v in lower.items() if m < M), M


@pytest.mark.parametrize("M,K,V", [(257, 64, 41000), (320, 128, 16500), (385, 64, 50001), (448, 64, 9000), (577, 128, 6000), (700, 64, 32001),
                                   (769, 64, 20000), (900, 128, 2100), (2100, 64, 1000), (200, 2048, 45000), (130, 4096, 42000),
                                   (193, 64, 32768), (193, 64, 32769), (250, 128, 90001)])
def test_tile_heights_by_rounds(step, M, K, V):
    """Rows a little beyond a tile's height, where many low tiles would hold fewer padded rows; several heights and numbers of
    hidden tiles; one hidden tile; up to 256 rows on both sides of the 128 vocabulary tiles that two hidden tiles meet in one
    round."""
    hidden, weight = W.make_lmhead_inputs(M + V, M, K, V, dtype="bf16", w_std=0.05)
    ids, mx = step.lmhead_argmax(hidden.cuda(), weight.cuda())
    torch.cuda.synchronize()
    _check(hidden, weight, ids, mx, rows=np.unique(np.concatenate([np.arange(0, M, max(1, M // 150)), [M - 1]])))


def _kernel(call):
    """The LM head kernel that a call runs, as it is in the source with its template arguments."""
    import re
    from torch.profiler import ProfilerActivity, profile
    call()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as trace:
        call()
        torch.cuda.synchronize()
    names = [m[0] for m in (re.search(r"lmhead_(few|mfma)_kernel<[^>]*>", e.name) for e in trace.events()) if m]
    assert len(names) == 1, names
    return names[0]


@pytest.mark.parametrize("M,K,V,kernel", [(1, 1024, 1, "few_kernel<1, 1, true>"), (64, 4096, 4096, "few_kernel<1, 1, true>"),
                                          (65, 4096, 4096, "few_kernel<1, 1, false>"), (64, 1024, 12288, "few_kernel<1, 1, true>"),
                                          (128, 1024, 12288, "few_kernel<1, 2, false>"), (64, 2048, 16384, "few_kernel<1, 1, true>"),
                                          (128, 2048, 16384, "few_kernel<1, 2, false>"), (64, 2112, 12289, "few_kernel<2, 1, true>"),
                                          (128, 4096, 16384, "few_kernel<2, 1, true>"), (128, 960, 12288, "mfma_kernel<1, false>"),
                                          (129, 1024, 4096, "mfma_kernel<1, false>"),
                                          (64, 640, 16385, "few_kernel<1, 2, true>"), (64, 576, 65536, "mfma_kernel<1, true>"),
                                          (64, 128, 65537, "few_kernel<1, 5, true>"), (64, 64, 131072, "mfma_kernel<1, true>"), (64, 64, 131073, "few_kernel<1, 5, true>"), (65, 1536, 16385, "few_kernel<2, 2, true>"),
                                          (65, 1472, 65536, "mfma_kernel<2, true>"), (65, 512, 65537, "few_kernel<2, 5, true>"),
                                          (65, 448, 131072, "mfma_kernel<2, true>"), (128, 128, 131073, "few_kernel<2, 5, true>"),
                                          (128, 64, 131073, "mfma_kernel<2, true>"), (192, 2112, 24576, "few_kernel<2, 3, false>"),
                                          (192, 2048, 24576, "mfma_kernel<2, false>"), (192, 2112, 40961, "mfma_kernel<3, true>")])
def test_kernels_of_few_hidden_rows(step, M, K, V, kernel):
    """One or two hidden tiles of 64 rows, one or two of 128, or 256-row tiles: both sides of every line.  The equal rows above
    are compared across them."""
    hidden, weight = (torch.zeros((n, K), dtype=torch.bfloat16, device="cuda") for n in (M, V))
    assert _kernel(lambda: step.lmhead_argmax(hidden, weight, want_max=False)) == "lmhead_" + kernel


@pytest.mark.parametrize("K,kernel", [(3355392, "few_kernel<1, 1, true>"), (3355456, "mfma_kernel<1, true>")])
def test_rows_of_megabytes(step, K, kernel):
    """A tile of 320 rows ends below 2 GB, as the few rows' 32-bit offsets want it, up to K = 3355392; longer rows are the other
    kernel's.  Every hidden row is one of the vocabulary's, the last but one twice: its largest logit is K exactly."""
    gen = torch.Generator(device="cuda").manual_seed(K)
    weight = torch.randint(0, 2, (10, K), device="cuda", generator=gen, dtype=torch.int8).mul_(2).sub_(1).bfloat16()
    weight[9] = weight[8]
    hidden = weight[[7, 9, 0]].contiguous()
    assert _kernel(lambda: step.lmhead_argmax(hidden, weight, want_max=False)) == "lmhead_" + kernel
    ids, mx = step.lmhead_argmax(hidden, weight)
    assert ids.tolist() == [7, 8, 0] and mx.tolist() == [K] * 3


@pytest.mark.parametrize("M,K,V,kernel", [(8, 512, 16384, "lmhead_mfma_kernel<1, true>"), (64, 512, 16384, "lmhead_mfma_kernel<1, true>"),
                                          (65, 512, 16384, "lmhead_mfma_kernel<1, false>"), (192, 512, 60000, "lmhead_mfma_kernel<3, true>"),
                                          (960, 64, 152064, "lmhead_mfma_kernel<3, false>")])
def test_weights_of_one_hidden_tile_are_streamed(step, M, K, V, kernel):
    """With one hidden tile nobody shares a weight tile, and its loads carry the non-temporal hint (second template argument)."""
    hidden, weight = (torch.zeros((n, K), dtype=torch.bfloat16, device="cuda") for n in (M, V))
    assert _kernel(lambda: step.lmhead_argmax(hidden, weight, want_max=False)) == kernel


@pytest.mark.parametrize("M,K,V", [(65, 64, 32768), (128, 128, 32769), (128, 192, 32700), (129, 64, 20480), (192, 128, 20481),
                                   (193, 64, 16384), (256, 128, 16385), (256, 192, 300)])
def test_tile_height_of_few_vocabulary_tiles(step, M, K, V):
    """128, 80 and 64 vocabulary tiles of 256 are the most that two, three and four hidden tiles of 64 rows meet
    in one round of CUs; one tile more takes the taller hidden tile."""
    hidden, weight = W.make_lmhead_inputs(M + V, M, K, V, dtype="bf16", w_std=0.05)
    ids, mx = step.lmhead_argmax(hidden.cuda(), weight.cuda())
    torch.cuda.synchronize()
    _check(hidden, weight, ids, mx)


@pytest.mark.parametrize("K,V", [(4096, 4096), (2048, 8192), (4096, 16384)])
def test_128_rows_take_hardly_longer_than_64_on_few_vocabulary_tiles(step, K, V):
    """Where a launch occupies a few CUs only, a tile of 128 rows took 1.15 to 1.34 times as long as one of 64."""
    weights = [torch.randn((V, K), device="cuda", dtype=torch.bfloat16) for _ in range(8)]

    def us(M):
        hidden = torch.randn((M, K), device="cuda", dtype=torch.bfloat16)
        ids = torch.empty(M, dtype=torch.int32, device="cuda")
        ws = step.alloc_workspace(step.hb.hb_lmhead_argmax_workspace_bytes(M))
        step.hb.hb_lmhead_argmax(hidden, weights[0], ids, None, ws)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for i in range(16):
                step.hb.hb_lmhead_argmax(hidden, weights[i % 8], ids, None, ws)
        best = float("inf")
        for _ in range(6):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            graph.replay()
            end.record()
            torch.cuda.synchronize()
            best = min(best, start.elapsed_time(end) / 16 * 1e3)
        return best

    low, high = us(64), us(128)
    assert high <= 1.12 * low, (low, high)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
# 1 .. 32 rows of whole 16-byte pieces take the few-rows kernel (eight rows and sixteen vocabulary
# entries per workgroup, 256 or 512 elements of K per step); 33 rows or a broken piece the tiles
@pytest.mark.parametrize("M,K,V", [(1, 8, 15), (8, 264, 16), (9, 504, 17), (31, 1032, 65), (32, 520, 1000),
                                   (33, 520, 64), (7, 250, 100)])
def test_few_rows(step, dtype, M, K, V):
    hidden, weight = W.make_lmhead_inputs(M * 5 + V, M, K, V, dtype=dtype, w_std=0.05)
    ids, mx = step.lmhead_argmax(hidden.cuda(), weight.cuda())
    torch.cuda.synchronize()
    _check(hidden, weight, ids, mx)


def test_work_units_of_the_left_over_cus(step):
    """960 rows are five 192-row hidden tiles: six lockstep groups occupy 30 of an XCD's 32 CUs.
    With 152 vocabulary tiles (19 per XCD) the other two CUs take the XCD's first tile as five
    (vocabulary tile, hidden tile) units, which saves the groups their fourth round.  Every row
    is checked against the oracle over the whole vocabulary, and winners are planted in the tiles
    that travel that way (vocabulary ids below 8 * 256) and in the ragged last tile."""
    M, K, V = 960, 192, 152 * 256 - 100
    hidden, weight = W.make_lmhead_inputs(4242, M, K, V, dtype="bf16", w_std=0.05)
    rng = np.random.default_rng(7)
    planted = {}
    for m in rng.choice(M, size=120, replace=False):
        v = int(rng.integers(0, 2048)) if m % 3 else int(rng.integers(V - 156, V))
        weight[v] = (hidden[m].float() * 0.5).to(weight.dtype)
        planted[int(m)] = v
    ids, mx = step.lmhead_argmax(hidden.cuda(), weight.cuda())
    torch.cuda.synchronize()
    _check(hidden, weight, ids, mx)
    got = ids.cpu().numpy()
    hit = sum(int(got[m]) == v for m, v in planted.items())
    assert hit >= 100  # a later planted row can only lose to another planted row of the same kind


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_planted_winner_ties_and_nan(step, dtype):
    M, K, V = 70, 256, 3000
    hidden, weight = W.make_lmhead_inputs(5, M, K, V, dtype=dtype, w_std=0.02)
    rng = np.random.default_rng(0)
    plant = rng.choice(V, size=M, replace=False)
    for m in range(0, M, 2):
        weight[plant[m]] = hidden[m] * 0.5  # logit = |h|^2 / 2, far above the N(0, 0.02) rows
    # exact ties: three identical rows, the lowest id must win
    tie = sorted(rng.choice(V, size=3, replace=False).tolist())
    while set(tie) & set(plant.tolist()):
        tie = sorted(rng.choice(V, size=3, replace=False).tolist())
    for v in tie:
        weight[v] = hidden[1] * 0.75
    ids, mx = step.lmhead_argmax(hidden.cuda(), weight.cuda())
    ids = ids.cpu().numpy()
    assert (ids[0::2] == plant[0::2]).all()
    assert ids[1] == tie[0]
    # a NaN logit never wins
    weight[7] = float("nan")
    ids2, _ = step.lmhead_argmax(hidden.cuda(), weight.cuda())
    ids2 = ids2.cpu().numpy()
    assert (ids2 != 7).all() and (ids2[0::2] == plant[0::2]).all()


def test_deterministic(step):
    hidden, weight = W.make_lmhead_inputs(9, 200, 512, 20000, w_std=0.02)
    h, w = hidden.cuda(), weight.cuda()
    a, am = step.lmhead_argmax(h, w)
    b, bm = step.lmhead_argmax(h, w)
    assert torch.equal(a, b) and torch.equal(am, bm)


@pytest.fixture(scope="module")
def full_weight():
    return W.make_lmhead_inputs(4000, 960, 3584, 152064, dtype="bf16")


@pytest.mark.parametrize("M", [960, 128])
def test_full_vocabulary_every_row(step, full_weight, M):
    """hidden 3584 x vocab 152064 (the full-step workload; M = 960 tree nodes, or 128 for the
    8-node-chain run); the oracle recomputes every row over the whole vocabulary."""
    hidden, weight = full_weight
    hidden = hidden[:M].contiguous()
    ids, mx = step.lmhead_argmax(hidden.cuda(), weight.cuda())
    torch.cuda.synchronize()
    n_clear = _check(hidden, weight, ids, mx)
    assert n_clear >= 0.9 * M
    assert (ids >= 0).all() and (ids < 152064).all()
