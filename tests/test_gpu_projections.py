"""GPU parity: positions, rotary table, fused QKV projection + rotary embedding, output projection
against the float64 oracle.

Tolerances (bf16 outputs of fp32-accumulated products of bf16 inputs): the result is rounded once
to bf16 (relative 2^-9 = 2e-3); fp32 accumulation over K <= 3584 terms adds well under 1e-5
relative to the sum of magnitudes.  Tested as: max abs error <= 1e-2 * (1 + |ref|) elementwise and
relative L2 error <= 4e-3."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import tree_positions_ref, rope_ref, qkv_rope_project_ref, linear_ref, rmsnorm_ref, swiglu_ref

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    import paper_2509_18824_amd as m
    return m


def _close(got, ref, label):
    got = W.widen(got)
    err = np.abs(got - ref)
    assert np.isfinite(got).all(), label
    assert (err <= 1e-2 * (1.0 + np.abs(ref))).all(), f"{label}: max abs err {err.max():.3e}"
    rel = np.linalg.norm(got - ref) / max(np.linalg.norm(ref), 1e-30)
    assert rel <= 4e-3, f"{label}: rel L2 {rel:.3e}"


def test_positions_and_rope_table(hb):
    rng = np.random.default_rng(0)
    trees = [W.seeded_tree(1), np.array([], dtype=np.int32), W.chain_tree(8), W.seeded_tree(2, n_nodes=64), W.chain_tree(1)]
    off = np.concatenate([[0], np.cumsum([len(t) for t in trees])]).astype(np.int32)
    par = np.concatenate(trees).astype(np.int32)
    L = np.array([32768, 5, 0, 4095, 17], dtype=np.int32)
    t = lambda a: torch.from_numpy(a).cuda()
    pos = torch.full((int(off[-1]),), -1, dtype=torch.int32, device="cuda")
    hb.hb_tree_positions(len(trees), 64, t(off), t(par), t(L), pos)
    ref = tree_positions_ref(off, par, L)
    assert np.array_equal(pos.cpu().numpy(), ref)
    for theta in (1e4, 1e6):
        cos = torch.empty((pos.numel(), 64), dtype=torch.float32, device="cuda")
        sin = torch.empty_like(cos)
        hb.hb_rope_table(128, theta, pos, cos, sin)
        ang = ref[:, None].astype(np.float64) * theta ** (-np.arange(64) / 64.0)
        assert np.abs(cos.cpu().numpy() - np.cos(ang)).max() <= 2e-7
        assert np.abs(sin.cpu().numpy() - np.sin(ang)).max() <= 2e-7


@pytest.mark.parametrize("T,K,Hq,Hkv,bias", [(960, 3584, 28, 4, True), (128, 3584, 28, 4, False), (77, 128, 2, 1, True),
                                             (300, 320, 3, 3, False), (300, 320, 3, 3, True), (1, 64, 1, 1, True), (513, 192, 8, 2, True),
                                             (100, 256, 2, 1, True), (1, 512, 1, 1, True), (16, 768, 3, 3, False),
                                             (128, 1024, 4, 2, True)])
def test_qkv_projection_with_rotary_embedding(hb, T, K, Hq, Hkv, bias):
    _qkv_case(hb, T, K, Hq, Hkv, bias, False)


@pytest.mark.parametrize("T,K,Hq,Hkv,bias", [(128, 3584, 28, 4, True), (100, 256, 2, 1, True), (1, 512, 1, 1, False),
                                             (64, 768, 3, 3, True), (65, 1024, 4, 2, False), (300, 320, 3, 3, True),
                                             (288, 3584, 28, 4, True), (200, 1024, 3, 1, False), (512, 2048, 2, 2, True),
                                             (513, 2048, 2, 1, True)])
def test_qkv_projection_split_over_k(hb, T, K, Hq, Hkv, bias):
    """The workspace variant: at most 512 tokens take the split-K path when K has enough steps
    (one or several hidden tiles per weight tile and K part), up to 1024 tokens when the cost
    model expects a gain, anything else the ordinary one."""
    _qkv_case(hb, T, K, Hq, Hkv, bias, True)


def _qkv_case(hb, T, K, Hq, Hkv, bias, with_workspace):
    g = torch.Generator().manual_seed(T * 7 + K)
    hidden = torch.randn((T, K), generator=g).to(torch.bfloat16)
    w = (torch.randn(((Hq + 2 * Hkv) * 128, K), generator=g) * (1.0 / np.sqrt(K))).to(torch.bfloat16)
    b = (torch.randn((Hq + 2 * Hkv) * 128, generator=g) * 0.5).to(torch.bfloat16) if bias else None
    pos = torch.randint(0, 40000, (T,), generator=g, dtype=torch.int32)
    theta = 1e6
    cos = torch.empty((T, 64), dtype=torch.float32, device="cuda")
    sin = torch.empty_like(cos)
    hb.hb_rope_table(128, theta, pos.cuda(), cos, sin)
    q = torch.full((T, Hq, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    k = torch.full((T, Hkv, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    v = torch.full((T, Hkv, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    if with_workspace:
        nbytes = hb.hb_proj_workspace_bytes(T, K, (Hq + 2 * Hkv) * 128)
        assert nbytes == 0 if (K < 512 or T > 1024) else (nbytes > 0 or T > 512)
        ws = torch.full((max(nbytes, 16),), 0xFF, dtype=torch.uint8, device="cuda")  # NaN patterns: nothing may be read unwritten
        hb.hb_qkv_rope_project_ws(hidden.cuda(), w.cuda(), None if b is None else b.cuda(), cos, sin, q, k, v, ws)
    else:
        hb.hb_qkv_rope_project(hidden.cuda(), w.cuda(), None if b is None else b.cuda(), cos, sin, q, k, v)
    torch.cuda.synchronize()
    rq, rk, rv = qkv_rope_project_ref(W.widen(hidden), W.widen(w), None if b is None else W.widen(b), pos.numpy(),
                                      Hq, Hkv, 128, theta)
    _close(q, rq, "q"); _close(k, rk, "k"); _close(v, rv, "v")


@pytest.mark.parametrize("T,K,N,res", [(960, 3584, 3584, True), (128, 3584, 3584, False), (50, 64, 4, True),
                                       (333, 448, 1000, False), (700, 256, 260, True),
                                       (128, 3584, 3584, True), (37, 256, 20, True), (5, 512, 1000, False),
                                       (96, 10752, 3584, False), (1, 256, 4, True)])
def test_output_projection(hb, T, K, N, res):
    _out_case(hb, T, K, N, res, False)


@pytest.mark.parametrize("T,K,N,res", [(1025, 64, 260, True), (1100, 128, 2308, False), (1537, 192, 2560, True),
                                       (193, 256, 4612, True), (2049, 64, 4608, False), (129, 448, 1284, True)])
def test_output_projection_with_units_dealt_across_weight_tiles(hb, T, K, N, res):
    """Weight tiles that are no multiple of the XCDs, one to seven K steps, ragged last tiles of both kinds."""
    _out_case(hb, T, K, N, res, False)


@pytest.mark.parametrize("T,K,N,res", [(128, 3584, 3584, True), (96, 10752, 3584, False), (37, 256, 20, True),
                                       (5, 512, 1000, False), (1, 1024, 4, True), (64, 2048, 260, True),
                                       (129, 512, 512, True), (288, 3584, 3584, True), (300, 1024, 520, False),
                                       (512, 2048, 260, True), (450, 768, 2052, True), (960, 18944, 3584, True),
                                       (768, 9472, 520, False), (1024, 4096, 260, True), (1025, 4096, 260, True)])
def test_output_projection_split_over_k(hb, T, K, N, res):
    _out_case(hb, T, K, N, res, True)


# Up to 16 tokens stream: 8 and 16 are token tiles of the streaming kernel; 8 K steps give every
# wavefront one, 9 the first one two; 64 steps are the most whose tokens stay in registers; 16-row
# tiles with and without a remainder (N = 4: no partner rows; 20, 12); more tiles than workgroups.
# 17 to 33 tokens by whichever way is expected to be faster there
@pytest.mark.parametrize("T,K,N,res", [(1, 512, 4, True), (8, 576, 20, False), (9, 4096, 36, True), (16, 4160, 12, True),
                                       (17, 512, 100, False), (32, 4160, 264, True), (33, 4160, 264, True),
                                       (8, 4160, 4620, True), (20, 576, 16404, False), (3, 1024, 9000, True)])
def test_output_projection_of_few_tokens(hb, T, K, N, res):
    _out_case(hb, T, K, N, res, False)
    _out_case(hb, T, K, N, res, True)


@pytest.mark.parametrize("T,K,Hq,Hkv,bias", [(1, 512, 1, 1, True), (8, 3584, 28, 4, True), (16, 4160, 3, 1, False),
                                             (17, 576, 6, 2, True), (32, 4160, 28, 4, False), (24, 1024, 16, 2, True)])
def test_qkv_projection_of_few_tokens(hb, T, K, Hq, Hkv, bias):
    _qkv_case(hb, T, K, Hq, Hkv, bias, False)


@pytest.mark.parametrize("T,K,F", [(1, 512, 4), (7, 576, 12), (8, 3584, 18944), (16, 4160, 100), (31, 1024, 9004), (32, 4160, 264)])
def test_gated_silu_projection_of_few_tokens(hb, T, K, F):
    test_gated_silu_projection(hb, T, K, F, False)


# Long rows over few weight rows, and many short ones, around the 17 and 32 tokens between which the stream, tiles of few
# rows and the split over K each have their shapes
@pytest.mark.parametrize("T,K,N,res", [(25, 12288, 260, True), (24, 18944, 1024, False), (32, 18944, 2048, True), (17, 18944, 20, False),
                                       (32, 512, 16404, True), (33, 2048, 1000, False), (33, 1024, 4, True), (40, 8192, 2052, True)])
def test_output_projection_around_the_end_of_the_stream(hb, T, K, N, res):
    assert hb.hb_proj_workspace_bytes(T, K, N) > 0 or N > 16384
    _out_case(hb, T, K, N, res, True)
    _out_case(hb, T, K, N, res, False)


@pytest.mark.parametrize("T,K,Hq,Hkv,bias", [(33, 512, 1, 1, True), (24, 12288, 6, 1, False), (20, 3584, 28, 4, True)])
def test_qkv_projection_around_the_end_of_the_stream(hb, T, K, Hq, Hkv, bias):
    _qkv_case(hb, T, K, Hq, Hkv, bias, True)


# tiles of few rows, weights below and above the size from which their loads are non-temporal
@pytest.mark.parametrize("T,K,F,ws", [(33, 4160, 16128, False), (40, 4160, 16136, False), (128, 4160, 16136, True), (24, 2048, 4100, True)])
def test_gated_silu_projection_of_one_tile_of_tokens(hb, T, K, F, ws):
    test_gated_silu_projection(hb, T, K, F, ws)


# All tokens in one tile: 64 and 128 tokens are its sizes; one K step and odd numbers of them (two go to a stage
# where they can), ragged last tiles, K whole and in parts
@pytest.mark.parametrize("T,K,N", [(17, 64, 4), (33, 192, 100), (64, 576, 4100), (65, 1088, 4612), (127, 832, 9004), (128, 1536, 260),
                                   (128, 9728, 516), (100, 128, 20484), (40, 256, 30724), (96, 320, 40960), (20, 576, 41000)])
def test_output_projection_of_all_tokens_at_once(hb, T, K, N):
    for ws in (False, True):
        _out_case(hb, T, K, N, T % 2 == 1, ws)


@pytest.mark.parametrize("T,K,Hq,Hkv,bias", [(17, 64, 1, 1, True), (64, 320, 5, 1, False), (65, 1536, 12, 4, True), (128, 192, 40, 8, True),
                                             (100, 3584, 28, 4, False)])
def test_qkv_projection_of_all_tokens_at_once(hb, T, K, Hq, Hkv, bias):
    for ws in (False, True):
        _qkv_case(hb, T, K, Hq, Hkv, bias, ws)


@pytest.mark.parametrize("T,K,F", [(17, 64, 4), (64, 192, 4100), (65, 576, 8204), (128, 1088, 12300), (33, 2112, 16388), (128, 64, 20480)])
def test_gated_silu_projection_of_all_tokens_at_once(hb, T, K, F):
    for ws in (False, True):
        test_gated_silu_projection(hb, T, K, F, ws)


# Rows or parts of K a multiple of 4 KB apart, 15 million weights and more: the workgroups begin at K steps of their own.  One
# and several K steps of a stage, whole and in parts, one token over; the sizes below the line stand in the tests above.
@pytest.mark.parametrize("T,K,N,ws", [(24, 2048, 7328, False), (100, 4096, 4100, False), (33, 6144, 2564, False), (128, 8192, 4096, True),
                                      (64, 16384, 1028, True), (17, 12288, 6272, True)])
def test_output_projection_of_rows_that_meet_on_few_channels(hb, T, K, N, ws):
    _out_case(hb, T, K, N, T % 2 == 1, ws)


@pytest.mark.parametrize("T,K,F", [(17, 2048, 4100), (40, 6144, 2052), (128, 4096, 4100), (64, 8192, 1028)])
def test_gated_projection_of_rows_that_meet_on_few_channels(hb, T, K, F):
    test_gated_silu_projection(hb, T, K, F, False)


def _kernels(call):
    """Names of the projection kernels that a call runs, each as it is in the source with its template arguments."""
    import re
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as trace:
        call()
        torch.cuda.synchronize()
    names = [re.search(r"proj_(\w+)_kernel(<[^>]*>)", e.name) for e in trace.events()]
    short = lambda t: re.sub(r"\(hb::[^)]*\)+", "", t)  # the enumerations' names
    return [m[1] + short(m[2].replace("(anonymous namespace)::", "")) for m in names if m]


# Every way a product can go, asserted by the kernel's name.  few<kind, 16-row groups of a tile, tokens, K steps of a stage>
# (kind 0 plain, 1 rotary, 2 gated, 3 partial sums), stream<kind, groups of eight tokens, tokens in registers>,
# mfma<64-token tiles, rotary, gated, non-temporal>
@pytest.mark.parametrize("T,K,N,ws,kernel", [
    (24, 14336, 260, False, "stream<0, 4, false>"), (20, 1472, 41000, False, "stream<0, 4, true>"),
    (32, 4160, 41000, True, "stream<0, 4, false>"),
    (40, 512, 260, False, "few<0, 1, 64, 2>"), (96, 576, 260, False, "few<0, 1, 128, 1>"), (64, 576, 4100, False, "few<0, 2, 64, 1>"),
    (40, 64, 8196, False, "few<0, 4, 64, 1>"), (100, 128, 8196, False, "few<0, 4, 128, 2>"), (40, 64, 16388, False, "few<0, 6, 64, 1>"),
    (100, 64, 16388, False, "few<0, 6, 128, 1>"), (40, 64, 24580, False, "few<0, 8, 64, 1>"), (100, 64, 24580, False, "few<0, 8, 128, 1>"),
    (40, 64, 32772, False, "few<0, 10, 64, 1>"), (100, 64, 32772, False, "few<0, 10, 128, 1>"),
    (32, 8192, 516, True, "few<3, 2, 64, 2>"), (40, 7168, 3072, True, "few<3, 6, 64, 1>"), (128, 7168, 8192, True, "few<3, 8, 128, 1>"),
    (40, 7168, 4612, True, "few<3, 10, 64, 1>"), (100, 7168, 10240, True, "few<3, 10, 128, 1>"),
    (40, 8192, 8192, True, "splitk<1>"), (100, 8192, 8192, True, "splitk<2>")])
def test_every_way_of_the_output_projection(hb, T, K, N, ws, kernel):
    names = _kernels(lambda: _out_case(hb, T, K, N, T % 2 == 0, ws))
    assert names == ([kernel, "reduce<false, false>"] if kernel.startswith(("few<3", "splitk")) else [kernel])


@pytest.mark.parametrize("T,K,Hq,Hkv,bias,ws,kernel", [
    (24, 5120, 12, 4, True, False, "stream<1, 4, false>"), (32, 4096, 28, 2, False, False, "stream<1, 4, true>"),
    (64, 64, 65, 1, True, False, "few<1, 4, 64, 1>"), (128, 128, 64, 8, True, False, "few<1, 4, 128, 2>"),
    (40, 64, 130, 3, True, False, "few<1, 6, 64, 1>"), (128, 64, 130, 3, False, False, "few<1, 6, 128, 1>"),
    (64, 64, 200, 5, False, False, "few<1, 8, 64, 1>"), (128, 64, 200, 5, True, False, "few<1, 8, 128, 1>"),
    (40, 64, 270, 11, True, False, "few<1, 10, 64, 1>"), (128, 128, 270, 11, False, False, "few<1, 10, 128, 1>"),
    (100, 7168, 40, 8, True, True, "few<3, 8, 128, 1>"), (40, 8192, 64, 8, True, True, "few<3, 10, 64, 1>"),
    (100, 8192, 64, 8, False, True, "few<3, 10, 128, 1>")])
def test_every_way_of_the_qkv_projection(hb, T, K, Hq, Hkv, bias, ws, kernel):
    names = _kernels(lambda: _qkv_case(hb, T, K, Hq, Hkv, bias, ws))
    assert names == ([kernel, "reduce<true, false>"] if kernel.startswith("few<3") else [kernel])


@pytest.mark.parametrize("T,K,F,ws,kernel", [
    (17, 2048, 16384, False, "stream<2, 4, true>"), (32, 2048, 16384, True, "stream<2, 4, true>"), (24, 8192, 4100, False, "stream<2, 4, false>"),
    (32, 4160, 2052, False, "few<2, 2, 64, 1>"), (40, 64, 4100, False, "few<2, 4, 64, 1>"), (100, 128, 4100, False, "few<2, 4, 128, 2>"),
    (40, 64, 8196, False, "few<2, 6, 64, 1>"), (100, 64, 8196, False, "few<2, 6, 128, 1>"), (40, 2112, 12292, False, "few<2, 8, 64, 1>"),
    (100, 2112, 12292, False, "few<2, 8, 128, 1>"), (40, 2112, 16388, False, "few<2, 10, 64, 1>"), (100, 2112, 16388, False, "few<2, 10, 128, 1>"),
    (64, 2048, 16384, True, "few<2, 10, 64, 1>"), (100, 2048, 16384, False, "mfma<1, false, true, false>"), (288, 2048, 1000, True, "splitk<1>"),
    (160, 3584, 18944, False, "mfma<3, false, true, true>"), (240, 3584, 18944, False, "mfma<4, false, true, true>"),
    (500, 2048, 16384, False, "mfma<4, false, true, false>")])
def test_every_way_of_the_gated_projection(hb, T, K, F, ws, kernel):
    names = _kernels(lambda: test_gated_silu_projection(hb, T, K, F, ws))
    assert names == ([kernel, "reduce<false, true>"] if kernel.startswith("splitk") else [kernel])


# 17 to 32 tokens on rows, or parts of them, a multiple of 4 KB apart, by what few rows take since the workgroups begin at K
# steps of their own: whole rows, eight parts and the tallest tiles are theirs, short parts in lower tiles the stream's
@pytest.mark.parametrize("T,K,N,kernel", [(32, 4096, 20480, "few<0, 6, 64, 1>"), (32, 16384, 4096, "few<3, 8, 64, 1>"),
                                          (17, 8192, 10240, "few<3, 10, 64, 1>"), (32, 8192, 4096, "stream<0, 4, false>")])
def test_ways_of_rows_that_meet_on_few_channels(hb, T, K, N, kernel):
    names = _kernels(lambda: _out_case(hb, T, K, N, T % 2 == 0, True))
    assert names == ([kernel, "reduce<false, false>"] if kernel.startswith("few<3") else [kernel])


# Tiles whose K steps two groups of wavefronts share: pair<kind (0 plain, 1 rotary, 2 gated, 3 partial sums), 32-row
# tiles of weights, of tokens>.  Odd and even K steps in all and per part, ragged last tiles of both kinds, one token over.
@pytest.mark.parametrize("kind,T,K,N,ws,kernel", [
    ("plain", 2000, 1088, 3580, False, "pair<0, 7, 4>"), ("plain", 2047, 1024, 3500, False, "pair<0, 7, 4>"),
    ("plain", 513, 10752, 3588, False, "pair<0, 4, 4>"), ("plain", 400, 3584, 3584, False, "pair<0, 4, 4>"),
    ("plain", 961, 3584, 3460, True, "pair<0, 4, 4>"), ("plain", 1121, 2112, 3588, True, "pair<0, 4, 5>"),
    ("plain", 400, 3584, 3584, True, "pair<3, 4, 4>"), ("plain", 513, 10752, 3588, True, "pair<3, 7, 4>"),
    ("plain", 288, 3584, 3584, True, "pair<3, 4, 5>"),
    ("rope", 960, 192, 35, False, "pair<1, 4, 5>"), ("rope", 961, 256, 36, True, "pair<1, 4, 5>"),
    ("rope", 300, 2048, 20, False, "pair<1, 4, 4>"), ("rope", 288, 3584, 36, True, "pair<3, 4, 4>"),
    ("gated", 520, 320, 4092, False, "pair<2, 4, 5>"), ("gated", 400, 2048, 4092, True, "pair<2, 4, 4>")])
def test_projections_whose_k_steps_two_groups_share(hb, kind, T, K, N, ws, kernel):
    if kind == "plain":
        names = _kernels(lambda: _out_case(hb, T, K, N, T % 2 == 0, ws))
    elif kind == "rope":
        names = _kernels(lambda: _qkv_case(hb, T, K, N - 2 * (N // 9), N // 9, T % 2 == 0, ws))
    else:
        names = _kernels(lambda: test_gated_silu_projection(hb, T, K, N, ws))
    assert names[0] == kernel and len(names) == (2 if kernel.startswith("pair<3") else 1)


# Both sides of the lines between these tiles and the ones of 256 rows, which are ahead of them where they stand here
@pytest.mark.parametrize("kind,T,K,N,ws,kernel", [
    ("plain", 256, 2048, 5656, True, "pair<3, 4, 4>"), ("plain", 336, 1408, 1784, True, "splitk"), ("plain", 1014, 1152, 292, True, "pair<0, 4, 4>"),
    ("plain", 700, 2048, 3588, True, "pair<0, 4, 4>"),
    ("plain", 3840, 1408, 928, False, "mfma"), ("plain", 4491, 2560, 644, True, "mfma"), ("plain", 1100, 2112, 900, False, "pair<0, 4, 4>"),
    ("plain", 3068, 1152, 1696, False, "mfma"), ("plain", 1446, 1280, 3328, False, "mfma"), ("plain", 2250, 1920, 2824, False, "pair<0, 7, 4>"),
    ("rope", 384, 1728, 28, True, "splitk"), ("rope", 150, 1664, 40, True, "pair<1, 4, 4>"),
    ("gated", 242, 2688, 3008, True, "splitk"), ("gated", 520, 1152, 320, True, "pair<2, 4, 4>")])
def test_the_lines_between_the_tiles_of_more_than_128_tokens(hb, kind, T, K, N, ws, kernel):
    if kind == "plain":
        names = _kernels(lambda: _out_case(hb, T, K, N, T % 2 == 0, ws))
    elif kind == "rope":
        names = _kernels(lambda: _qkv_case(hb, T, K, N - 2 * (N // 9), N // 9, T % 2 == 0, ws))
    else:
        names = _kernels(lambda: test_gated_silu_projection(hb, T, K, N, ws))
    assert names[0].startswith(kernel) and len(names) == (2 if kernel in ("splitk", "pair<3, 4, 4>") else 1)


@pytest.mark.parametrize("T,K,N,res,fused", [
    (128, 18944, 3584, True, True), (1, 3584, 3584, True, False), (100, 3584, 3584, False, True), (300, 3584, 3592, True, True),
    (960, 18944, 3584, True, True), (960, 3584, 3584, True, False), (40, 8192, 8192, True, True), (40, 8192, 8200, False, False),
    (40, 7168, 8, True, True)])
def test_projection_and_normalisation_are_the_two_calls_one_after_the_other(hb, T, K, N, res, fused):
    """Rows of a few threads to the widest that one launch takes, and ways without parts of K.  One launch adds the squares
    in another order: 1e-6 of the scale at most, which may turn a rounding to bf16, by one step of 2^-7 of the value at
    most and seldom (about 1e-6 / 2^-9 of the values)."""
    g = torch.Generator().manual_seed(T + K + N)
    bf = lambda *shape, std=1.0: (torch.randn(shape, generator=g) * std).to(torch.bfloat16).cuda()
    x, w, r, gain = bf(T, K), bf(N, K, std=K ** -0.5), bf(T, N) if res else None, 1.0 + bf(N, std=0.1)
    ws = torch.full((max(hb.hb_proj_workspace_bytes(T, K, N), 16),), 0xFF, dtype=torch.uint8, device="cuda")
    out, norm, out2, norm2 = (torch.full((T, N), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(4))
    hb.hb_out_project_ws(x, w, r, out, ws)
    hb.hb_rmsnorm(out, gain, 1e-6, norm)
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as trace:
        hb.hb_out_project_norm_ws(x, w, r, out2, gain, 1e-6, norm2, ws)
        torch.cuda.synchronize()
    assert torch.isfinite(norm).all() and torch.equal(out, out2)
    off = (norm.float() - norm2.float()).abs()
    assert (off <= 2 ** -7 * norm.float().abs()).all() and (off > 0).float().mean() <= 5e-3
    assert any("proj_reduce_norm_kernel" in e.name for e in trace.events()) == fused


@pytest.mark.parametrize("T,K,N,fused", [(536, 12544, 512, False), (300, 7488, 1016, False), (300, 7488, 1024, True), (128, 7488, 512, True),
                                         (300, 4992, 4096, True), (300, 4992, 4104, False), (200, 4992, 4104, True), (300, 4992, 5120, True)])
def test_projection_and_normalisation_in_one_launch_where_that_is_ahead(hb, T, K, N, fused):
    test_projection_and_normalisation_are_the_two_calls_one_after_the_other(hb, T, K, N, T % 2 == 0, fused)


@pytest.mark.parametrize("K,N,gated", [(14336, 4096, False), (18944, 3584, False), (4096, 28672, True)])
def test_seventeen_tokens_take_hardly_longer_than_sixteen(hb, K, N, gated):
    """Shapes where the stream stays ahead beyond 16 tokens: 25 and 26 us, 31 and 32, 43 and 44 by it; 33, 39 and 54 by tiles
    of few rows.  Four weight matrices in turn, in a graph."""
    weights = [torch.randn((N, K), device="cuda", dtype=torch.bfloat16) for _ in range(4)]

    def us(T):
        x = torch.randn((T, K), device="cuda", dtype=torch.bfloat16)
        out = torch.empty((T, N // 2 if gated else N), device="cuda", dtype=torch.bfloat16)
        run = (lambda w: hb.hb_swiglu_project(x, w, out, None)) if gated else (lambda w: hb.hb_out_project(x, w, None, out))
        run(weights[0])
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for i in range(12):
                run(weights[i % 4])
        best = float("inf")
        for _ in range(6):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            graph.replay()
            end.record()
            torch.cuda.synchronize()
            best = min(best, start.elapsed_time(end) / 12 * 1e3)
        return best

    sixteen, seventeen = us(16), us(17)
    assert seventeen <= 1.2 * sixteen, (sixteen, seventeen)


def _out_case(hb, T, K, N, res, with_workspace):
    g = torch.Generator().manual_seed(T + K + N)
    x = torch.randn((T, K), generator=g).to(torch.bfloat16)
    w = (torch.randn((N, K), generator=g) * (1.0 / np.sqrt(K))).to(torch.bfloat16)
    r = torch.randn((T, N), generator=g).to(torch.bfloat16) if res else None
    out = torch.full((T, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    if with_workspace:
        nbytes = hb.hb_proj_workspace_bytes(T, K, N)
        ws = torch.full((max(nbytes, 16),), 0xFF, dtype=torch.uint8, device="cuda")
        hb.hb_out_project_ws(x.cuda(), w.cuda(), None if r is None else r.cuda(), out, ws)
    else:
        hb.hb_out_project(x.cuda(), w.cuda(), None if r is None else r.cuda(), out)
    torch.cuda.synchronize()
    _close(out, linear_ref(W.widen(x), W.widen(w), None if r is None else W.widen(r)), "out")


@pytest.mark.parametrize("T,K,eps", [(960, 3584, 1e-6), (128, 3584, 1e-6), (1, 8, 0.0), (7, 8200, 1e-5), (33, 72, 1e-2),
                                     (5, 16384, 1e-6)])
def test_rmsnorm(hb, T, K, eps):
    """Rows that fit the registers a thread keeps (K <= 8192), longer ones, the shortest."""
    g = torch.Generator().manual_seed(T + K)
    x = (torch.randn((T, K), generator=g) * 3.0 + 0.5).to(torch.bfloat16)
    w = (1.0 + 0.3 * torch.randn(K, generator=g)).to(torch.bfloat16)
    out = torch.full((T, K), float("nan"), dtype=torch.bfloat16, device="cuda")
    hb.hb_rmsnorm(x.cuda(), w.cuda(), eps, out)
    torch.cuda.synchronize()
    _close(out, rmsnorm_ref(W.widen(x), W.widen(w), eps), "rmsnorm")
    xin = x.cuda()
    hb.hb_rmsnorm(xin, w.cuda(), eps, xin)   # in place
    torch.cuda.synchronize()
    assert torch.equal(xin, out)


@pytest.mark.parametrize("T,K,F,ws", [(960, 3584, 18944, False), (128, 3584, 18944, True), (128, 3584, 18944, False),
                                      (77, 128, 132, True), (300, 320, 100, False), (1, 64, 4, True),
                                      (513, 192, 520, True), (40, 1024, 260, True), (288, 2048, 1000, True)])
def test_gated_silu_projection(hb, T, K, F, ws):
    """Gate and up projection in one pass with silu(gate) * up in the epilogue: the feed-forward
    width of the target model's shape for trees (960 tokens) and chains (128 tokens, split over K),
    ragged feature counts (the last tile holds fewer than 128 features), a single token."""
    g = torch.Generator().manual_seed(T * 3 + K + F)
    x = torch.randn((T, K), generator=g).to(torch.bfloat16)
    w = (torch.randn((2 * F, K), generator=g) * (1.5 / np.sqrt(K))).to(torch.bfloat16)
    out = torch.full((T, F), float("nan"), dtype=torch.bfloat16, device="cuda")
    wsp = None
    if ws:
        nbytes = hb.hb_proj_workspace_bytes(T, K, 2 * F)
        wsp = torch.full((max(nbytes, 16),), 0xFF, dtype=torch.uint8, device="cuda")
    hb.hb_swiglu_project(x.cuda(), w.cuda(), out, wsp)
    torch.cuda.synchronize()
    _close(out, swiglu_ref(W.widen(x), W.widen(w)), "swiglu")


@pytest.mark.parametrize("scale_down,K,tree", [(16, 512, "tree"), (1, 3584, "tree"), (1, 3584, "chain8")])
def test_projected_qkv_feed_the_attention(hb, scale_down, K, tree):
    """hidden -> QKV + rotary -> tree-verify attention -> output projection, against the oracle
    chained the same way on the bf16 tensors the GPU hands from step to step; also one whole layer
    of the batch-16 workload at full size (960 tree tokens, and 128 tokens of 8-node chains, which
    take the split-K projections; hidden size 3584, prefixes of 1024-4096 tokens)."""
    import paper_2509_18824_amd.step as S
    from oracle import tree_attn_ref
    inp = W.make_config(4, scale_down=scale_down, tree=tree)
    T, Hq, Hkv, D = inp.total_nodes, inp.Hq, inp.Hkv, inp.D
    g = torch.Generator().manual_seed(5)
    hidden = torch.randn((T, K), generator=g).to(torch.bfloat16)
    wqkv = (torch.randn(((Hq + 2 * Hkv) * D, K), generator=g) / np.sqrt(K)).to(torch.bfloat16)
    wo = (torch.randn((K, Hq * D), generator=g) / np.sqrt(Hq * D)).to(torch.bfloat16)
    dev = S.to_device(inp)
    pos = torch.empty(T, dtype=torch.int32, device="cuda")
    hb.hb_tree_positions(inp.B, 64, dev.node_offset, dev.parent, dev.prefix_len, pos)
    cos = torch.empty((T, 64), dtype=torch.float32, device="cuda"); sin = torch.empty_like(cos)
    hb.hb_rope_table(D, 1e6, pos, cos, sin)
    ws = S.alloc_workspace(max(hb.hb_proj_workspace_bytes(T, K, (Hq + 2 * Hkv) * D), hb.hb_proj_workspace_bytes(T, Hq * D, K)))
    hb.hb_qkv_rope_project_ws(hidden.cuda(), wqkv.cuda(), None, cos, sin, dev.q, dev.k_tree, dev.v_tree, ws)
    desc = S.desc_for(inp)
    out, _ = S.tree_verify_attn(desc, dev, want_lse=False)
    y = torch.empty((T, K), dtype=torch.bfloat16, device="cuda")
    hb.hb_out_project_ws(out.view(T, -1), wo.cuda(), hidden.cuda(), y, ws)
    torch.cuda.synchronize()
    ref_pos = tree_positions_ref(inp.node_offset.numpy(), inp.parent.numpy(), inp.prefix_len.numpy())
    rq, rk, rv = qkv_rope_project_ref(W.widen(hidden), W.widen(wqkv), None, ref_pos, Hq, Hkv, D, 1e6)
    _close(dev.q, rq, "q"); _close(dev.k_tree, rk, "k"); _close(dev.v_tree, rv, "v")
    ref_attn, _ = tree_attn_ref(W.widen(dev.q), W.widen(dev.k_tree), W.widen(dev.v_tree), W.widen(inp.k_pool),
                                W.widen(inp.v_pool), inp.block_table.numpy(), inp.prefix_len.numpy(),
                                inp.node_offset.numpy(), inp.parent.numpy(), inp.softmax_scale)
    got_attn = W.widen(out)
    assert np.linalg.norm(got_attn - ref_attn) / np.linalg.norm(ref_attn) <= 1e-2
    _close(y, linear_ref(got_attn.reshape(T, -1), W.widen(wo), W.widen(hidden)), "layer output")
