"""GPU parity of the draft model's intermediate layer (meta-query cross-attention, Section 3.1.1,
Eq. 1, with the skip connection and fc1 of Section 3.1.2) against the float64 oracle.

Tolerance: the path is bf16 with fp32 accumulation; the projected values, the attention output
before the output projection and the layer's output are each rounded to bf16 (relative 2^-9), so
outputs of unit scale carry errors of a few 1e-3 in the worst element; asserted: relative L2
error <= 1e-2 and max-abs error <= 2e-2 * (1 + max |reference|), the bar of the attention tests."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import fc_concat_ref, linear_ref, meta_query_attn_ref

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import paper_2509_18824_amd.step as s
    return s


def _close(got, ref, what):
    got = got.float().cpu().numpy().astype(np.float64)
    err = np.abs(got - ref)
    rel = np.linalg.norm(got - ref) / max(np.linalg.norm(ref), 1e-30)
    assert rel <= 1e-2 and err.max() <= 2e-2 * (1 + np.abs(ref).max()), (what, rel, err.max())
    return rel


def _run(S, seed, n_tok, L, D, H, Q, layers, peaked=False, zero_wo=False):
    x = W.make_meta_inputs(seed, n_tok, L, D, H, Q, peaked=peaked)
    if zero_wo:
        x["w_o"] = torch.zeros_like(x["w_o"])
    g = {k: v.cuda() for k, v in x.items()}
    layer = S.MetaQueryLayer(g["f_q"], g["w_q"], g["w_k"], g["w_v"], g["w_o"], g["w_fc1"], H, residual_layers=layers)
    f_c, out = layer.run(g["feats"])
    torch.cuda.synchronize()
    w = {k: v.float().numpy().astype(np.float64) for k, v in x.items()}
    ref_c = meta_query_attn_ref(w["f_q"], w["feats"], w["w_q"], w["w_k"], w["w_v"], w["w_o"], H, residual_layers=layers)
    _close(f_c, ref_c, "f_c")
    _close(out, linear_ref(ref_c, w["w_fc1"]), "fc1")
    return f_c, ref_c, x


@pytest.mark.parametrize("n_tok,L,D,H,Q,layers", [
    (5, 6, 256, 2, 3, [0, 2, 5]),        # small: one row tile, layers in one column tile
    (3, 28, 512, 4, 3, [1, 13, 27]),     # 28 layers (two column tiles, the second ragged)
    (7, 32, 768, 3, 4, None),            # 32 layers, four queries, no skip connection
    (2, 17, 1024, 32, 3, [0, 8, 16]),    # 96 (head, query) rows: every row tile
    (1, 1, 256, 2, 1, [0]),              # one layer, one head, one query
    (9, 5, 4352, 34, 2, [0, 4]),         # 17 slices of D over 9 workgroup columns (two slices each, the last one), a ragged
                                         # second token group, more than 4096 features (two column blocks in the mixing)
    (150, 4, 256, 2, 2, None),           # many tokens, a single slice
])
def test_small_shapes(S, n_tok, L, D, H, Q, layers):
    _run(S, 3 + n_tok, n_tok, L, D, H, Q, layers)
    _run(S, 13 + n_tok, n_tok, L, D, H, Q, layers, peaked=True)


def test_target_model_shape(S):
    """28 layers of hidden size 3584, 28 heads of 128, three queries: the 96 tokens that a
    batch of 16 sequences commits per step at most."""
    _run(S, 40, 96, 28, 3584, 28, 3, [2, 14, 27])
    _run(S, 41, 24, 28, 3584, 28, 3, [2, 14, 27], peaked=True)


@pytest.mark.parametrize("n_tok,L,D,H,Q,layers", [
    (1, 1, 256, 2, 1, [0]),               # 4 tokens and 2 heads per workgroup: one token, one layer
    (7, 28, 768, 6, 3, [1, 13, 27]),      # ... a ragged second group
    (130, 31, 1280, 10, 4, None),         # ... all four queries; odd layers
    (1025, 5, 512, 4, 2, [0, 4]),         # 4 tokens and 4 heads
    (421, 17, 1280, 10, 3, [0, 8, 16]),   # 4 heads, the last group with 2
    (3601, 3, 256, 2, 1, [2]),            # 16 tokens, 4 heads per workgroup, one token in the last group
    (1203, 4, 768, 6, 2, [0, 3]),
    (1203, 32, 768, 6, 3, [0, 8, 31]),
    (3203, 4, 768, 6, 4, None),
    (2203, 2, 1280, 10, 1, [1]),          # ... three groups of heads
    (2203, 12, 1280, 10, 2, [1, 11]),
    (2203, 9, 1280, 10, 3, None),
])
def test_values_projected_after_the_mixing(S, n_tok, L, D, H, Q, layers):
    """hb_meta_query_attn_project at sizes of each of its forms, at the edges of its token groups, head
    groups and layer tiles: the attention output before the output projection, on sampled tokens
    (the first, the last and 30 others).  Rounded once to bf16 (2^-9 relative to the element): 4e-3
    relative in the norm leaves room for the float32 softmax."""
    import paper_2509_18824_amd as hb
    x = W.make_meta_inputs(5 + n_tok, n_tok, L, D, H, Q, peaked=True)
    g = {k: v.cuda() for k, v in x.items()}
    layer = S.MetaQueryLayer(g["f_q"], g["w_q"], g["w_k"], g["w_v"], g["w_o"], g["w_fc1"], H, residual_layers=layers)
    new = lambda: torch.full((n_tok, Q, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    pre, res = new(), new() if layers is not None else None
    ws = S.alloc_workspace(hb.binding.hb_meta_query_attn_project_workspace_bytes(n_tok, D, H, Q))
    hb.binding.hb_meta_query_attn_project(H, Q, g["feats"], g["w_v"], layer.a_fold, layers, pre, res, ws)
    torch.cuda.synchronize()
    if layers is not None:
        assert torch.equal(res, g["feats"][:, layers, :])
    assert torch.isfinite(pre).all()
    pick = np.unique(np.concatenate([[0, n_tok - 1], np.random.default_rng(5).integers(0, n_tok, 30)]))
    w = {k: v.float().numpy().astype(np.float64) for k, v in x.items() if k != "feats"}
    feats = x["feats"][torch.from_numpy(pick)].float().numpy().astype(np.float64)
    ref = meta_query_attn_ref(w["f_q"], feats, w["w_q"], w["w_k"], w["w_v"], np.eye(D), H)
    got = pre[torch.from_numpy(pick).cuda()].float().cpu().numpy().astype(np.float64).reshape(len(pick), -1)
    assert np.linalg.norm(got - ref) <= 4e-3 * np.linalg.norm(ref)


@pytest.mark.parametrize("n_tok,L,D,H,Q,layers", [
    (2060, 28, 1024, 8, 3, [0, 5, 27]),   # 16 tokens: 24 hq rows, all of LDS; 28 layers are the most of 7 loads a slice
    (2040, 24, 1792, 14, 3, [1, 2, 23]),  # 21 rows; 6 loads
    (2203, 25, 1280, 10, 3, None),        # 4 heads, 7 loads
    (2061, 29, 1024, 8, 3, None),         # three slices of 32 features, 24 rows
    (2040, 32, 1792, 14, 3, [31, 0, 7]),  # ... 21 rows, all layers
    (2047, 32, 1024, 8, 2, [31, 0]),      # 4 heads, two wavefronts each, 8 loads
    (700, 30, 1024, 8, 4, None),          # 4 tokens, four queries
    (690, 7, 256, 2, 1, [6]),             # 4 tokens, one row a head
])
def test_sixteen_tokens_per_workgroup(S, n_tok, L, D, H, Q, layers):
    test_values_projected_after_the_mixing(S, n_tok, L, D, H, Q, layers)


@pytest.mark.parametrize("n_tok,L,D,H,Q,layers,form", [
    (501, 7, 256, 2, 1, None, "project<2>"),
    (1030, 9, 512, 4, 3, [4, 0, 8], "project<4>"),
    (2061, 24, 256, 2, 1, [23], "wide<1, 4, 6>"),
    (2101, 25, 256, 2, 1, None, "wide<1, 4, 7>"),
    (2131, 32, 256, 2, 1, [31], "wide<1, 4, 8>"),
    (1875, 5, 768, 6, 2, [0, 4], "wide<2, 4, 6>"),
    (2102, 28, 256, 2, 2, None, "wide<2, 4, 7>"),
    (2132, 29, 256, 2, 2, [0, 28], "wide<2, 4, 8>"),
    (2050, 24, 256, 2, 3, [12, 0, 23], "wide<3, 4, 6>"),
    (2203, 28, 256, 2, 3, None, "wide<3, 4, 7>"),
    (2251, 31, 256, 2, 3, [15, 0, 30], "wide<3, 4, 8>"),
    (2319, 12, 256, 2, 4, None, "wide<4, 4, 6>"),
    (2370, 28, 256, 2, 4, None, "wide<4, 4, 7>"),
    (2541, 32, 256, 2, 4, None, "wide<4, 4, 8>"),
    (2066, 5, 768, 6, 1, [4], "wide<1, 8, 6>"),
    (2064, 28, 768, 6, 1, None, "wide<1, 8, 7>"),
    (2077, 29, 768, 6, 1, [28], "wide<1, 8, 8>"),
    (2064, 24, 768, 6, 2, [0, 23], "wide<2, 8, 6>"),
    (2071, 25, 1024, 8, 2, None, "wide<2, 8, 7>"),
    (2063, 32, 1024, 8, 2, [0, 31], "wide<2, 8, 8>"),  # 16 rows and all of LDS
    (2065, 6, 768, 6, 3, [3, 0, 5], "wide<3, 8, 6>"),
    (1500, 25, 1280, 10, 3, None, "wide<3, 8, 7>"),  # 15 rows in two tiles of 16
    (2064, 28, 1024, 8, 3, [14, 0, 27], "wide<3, 8, 7>"),  # 24 rows and all of LDS
    (2061, 32, 1024, 8, 3, [16, 0, 31], "wide<3, 8, 8>"),  # ... and three slices of 32 features
    # where the lines between the forms matter: 6 to 30 % ahead of the next one
    (480, 21, 2048, 16, 3, None, "project<4>"), (350, 26, 2560, 20, 4, None, "project<4>"),
    (1247, 15, 3584, 28, 1, [14], "wide<1, 8, 6>"), (1147, 14, 4096, 32, 3, None, "wide<3, 4, 6>"),
])
def test_every_form_of_the_projection_after_the_mixing(S, n_tok, L, D, H, Q, layers, form):
    """... each asserted by its kernel's name: project<16-column tiles of a wavefront> for 4 tokens a workgroup, wide<queries,
    16-column tiles, feature loads of a wavefront> for 16."""
    import re
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as trace:
        test_values_projected_after_the_mixing(S, n_tok, L, D, H, Q, layers)
    names = [m[1] + m[2] for m in (re.search(r"meta_(project|project_wide)_kernel(<[^>]*>)", e.name) for e in trace.events()) if m]
    assert names == [form.replace("wide", "project_wide")]


@pytest.mark.parametrize("n_tok,L,D,H,Q,layers,form,shared", [
    (10, 28, 2048, 16, 3, [27, 0, 5], "wide<3, 4, 7>", True), (17, 32, 1280, 10, 1, None, "wide<1, 4, 8>", True),
    (40, 5, 2304, 18, 2, [4, 0], "wide<2, 4, 6>", True), (300, 30, 3584, 28, 3, None, "wide<3, 8, 8>", True),  # slices of 32 features
    (320, 24, 3072, 24, 3, [0, 23, 7], "wide<3, 4, 6>", True), (640, 25, 2048, 16, 1, [3], "wide<1, 8, 7>", True),
    (512, 2, 3328, 26, 2, None, "wide<2, 8, 6>", True), (513, 2, 3328, 26, 2, [1, 0], "wide<2, 4, 6>", False),  # 26 heads in a round by fours
    (512, 2, 5120, 40, 1, [1], "wide<1, 8, 6>", True), (513, 2, 5120, 40, 1, None, "wide<1, 8, 6>", False),
    (9, 28, 2048, 16, 3, [27, 0, 5], "project<2>", False), (321, 24, 1024, 8, 3, None, "project<4>", False), (17, 9, 768, 6, 2, [8, 1], "project<2>", False), (49, 9, 2048, 16, 3, None, "project<2>", False)])
def test_workgroups_that_share_d(S, n_tok, L, D, H, Q, layers, form, shared):
    """Probabilities made in front and float32 sums of the shares added up behind: shares of unequal and of the
    shortest length, ragged tokens, both forms; and both sides of the lines."""
    import re
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as trace:
        test_values_projected_after_the_mixing(S, n_tok, L, D, H, Q, layers)
    names = [m[1] + (m[2] or "") for m in (re.search(r"meta_(project|project_wide|softmax|sum)_kernel(<[^>]*>)?", e.name) for e in trace.events()) if m]
    form = form.replace("wide", "project_wide")
    assert names == (["softmax", form, "sum"] if shared else [form])


def test_a_workspace_without_room_for_shares(S):
    """One that holds the partial scores and W_v's copy only (sized for more tokens, say) is taken, by the form that shares
    nothing, and nothing behind it is touched; a byte less is refused."""
    import paper_2509_18824_amd as hb
    n_tok, L, D, H, Q = 40, 12, 2048, 16, 2
    least = -(-hb.hb_meta_query_attn_workspace_bytes(n_tok, D, H, Q) // 256) * 256 + D * D * 2
    most = hb.hb_meta_query_attn_project_workspace_bytes(n_tok, D, H, Q)
    assert most > least
    x = {k: v.cuda() for k, v in W.make_meta_inputs(3, n_tok, L, D, H, Q).items()}
    layer = S.MetaQueryLayer(x["f_q"], x["w_q"], x["w_k"], x["w_v"], x["w_o"], x["w_fc1"], H)
    ws = torch.full((most,), 77, dtype=torch.uint8, device="cuda")
    out = [torch.empty(n_tok, Q, D, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    hb.hb_meta_query_attn_project(H, Q, x["feats"], x["w_v"], layer.a_fold, None, out[0], None, ws[:least])
    assert (ws[least:] == 77).all()
    hb.hb_meta_query_attn_project(H, Q, x["feats"], x["w_v"], layer.a_fold, None, out[1], None, ws)
    assert (out[0].float() - out[1].float()).norm() <= 4e-3 * out[1].float().norm()
    with pytest.raises(RuntimeError):
        hb.hb_meta_query_attn_project(H, Q, x["feats"], x["w_v"], layer.a_fold, None, out[0], None, ws[:least - 1])



@pytest.mark.parametrize("n_tok,L,D,H,Q", [(7, 28, 768, 6, 3), (1203, 5, 768, 6, 2), (1025, 5, 512, 4, 2)])
@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
def test_a_token_with_features_that_are_not_finite(S, n_tok, L, D, H, Q, bad):
    """Its own rows are NaN whether values are projected before or after the mixing (an infinite score
    leaves no finite probability times a finite value); every other token's are as without it."""
    import paper_2509_18824_amd as hb
    x = W.make_meta_inputs(9, n_tok, L, D, H, Q)
    g = {k: v.cuda() for k, v in x.items()}
    layer = S.MetaQueryLayer(g["f_q"], g["w_q"], g["w_k"], g["w_v"], g["w_o"], g["w_fc1"], H)

    def both(feats):
        v_proj = torch.empty(n_tok * L, D, dtype=torch.bfloat16, device="cuda")
        hb.hb_out_project(feats.view(n_tok * L, D), g["w_v"], None, v_proj)
        first, after = (torch.empty(n_tok, Q, D, dtype=torch.bfloat16, device="cuda") for _ in range(2))
        ws = S.alloc_workspace(hb.hb_meta_query_attn_workspace_bytes(n_tok, D, H, Q))
        hb.hb_meta_query_attn(H, Q, feats, v_proj.view(n_tok, L, D), layer.a_fold, None, first, None, ws)
        ws = S.alloc_workspace(hb.hb_meta_query_attn_project_workspace_bytes(n_tok, D, H, Q))
        hb.hb_meta_query_attn_project(H, Q, feats, g["w_v"], layer.a_fold, None, after, None, ws)
        torch.cuda.synchronize()
        return first, after

    clean = both(g["feats"])
    feats, at = g["feats"].clone(), n_tok - 2
    feats[at, L - 1, 129] = bad
    for got, want in zip(both(feats), clean):
        assert torch.isnan(got[at]).all()
        assert torch.equal(got[:at], want[:at]) and torch.equal(got[at + 1:], want[at + 1:])


def test_prefill_scale_on_sampled_tokens(S):
    """1024 tokens of the target model's shape (one workgroup column per two slices of D in the
    score kernel, 128 token groups); every token is independent of the others, so the oracle
    checks 24 sampled ones."""
    n_tok, L, D, H, Q, layers = 1024, 28, 3584, 28, 3, [2, 14, 27]
    x = W.make_meta_inputs(77, n_tok, L, D, H, Q)
    g = {k: v.cuda() for k, v in x.items()}
    layer = S.MetaQueryLayer(g["f_q"], g["w_q"], g["w_k"], g["w_v"], g["w_o"], g["w_fc1"], H, residual_layers=layers)
    f_c, out = layer.run(g["feats"])
    torch.cuda.synchronize()
    pick = np.sort(np.random.default_rng(5).choice(n_tok, 24, replace=False))
    pick[0], pick[-1] = 0, n_tok - 1
    w = {k: v.float().numpy().astype(np.float64) for k, v in x.items() if k != "feats"}
    feats = x["feats"][torch.from_numpy(pick)].float().numpy().astype(np.float64)
    ref_c = meta_query_attn_ref(w["f_q"], feats, w["w_q"], w["w_k"], w["w_v"], w["w_o"], H, residual_layers=layers)
    _close(f_c[torch.from_numpy(pick).cuda()], ref_c, "f_c")
    _close(out[torch.from_numpy(pick).cuda()], linear_ref(ref_c, w["w_fc1"]), "fc1")


def test_zero_initialised_output_projection_passes_the_feature_levels_through(S):
    """Section 3.1.2: with W_o at zero the layer's output is the three residual features, bit for bit."""
    f_c, ref_c, x = _run(S, 50, 9, 28, 512, 4, 3, [0, 13, 27], zero_wo=True)
    want = torch.cat([x["feats"][:, l, :] for l in (0, 13, 27)], dim=1)
    assert torch.equal(f_c.cpu(), want)


def test_fc_over_a_concatenation(S):
    rng = np.random.default_rng(7)
    bf = lambda a: torch.from_numpy(a.astype(np.float32)).to(torch.bfloat16)
    a, b = bf(rng.normal(size=(33, 512))), bf(rng.normal(size=(33, 512)))
    w = bf(rng.normal(0, 1024 ** -0.5, size=(512, 1024)))
    out = S.fc_concat(a.cuda(), b.cuda(), w[:, :512].contiguous().cuda(), w[:, 512:].contiguous().cuda())
    torch.cuda.synchronize()
    f = lambda t: t.float().numpy().astype(np.float64)
    _close(out, fc_concat_ref(f(a), f(b), f(w)), "fc2")


@pytest.mark.parametrize("n_tok,K,N,kernels", [
    (96, 3584, 3584, ("few", "reduce")), (40, 4096, 516, ("few", "reduce")),       # parts of K from one half each
    (300, 3584, 3584, ("pair", "reduce")), (2048, 3584, 3584, ("pair",)),          # ... and tiles that change over
    (2030, 1088, 3580, ("pair",)),                                                # at an odd step
    (5, 512, 1000, ("stream", "stream")), (6144, 576, 3584, ("mfma", "mfma"))])    # one product after the other
def test_fc_over_two_halves_in_one_product(S, n_tok, K, N, kernels):
    import re
    from torch.profiler import ProfilerActivity, profile
    g = torch.Generator().manual_seed(n_tok)
    bf = lambda *shape, std=1.0: (torch.randn(shape, generator=g) * std).to(torch.bfloat16)
    a, b, w_a, w_b = bf(n_tok, K), bf(n_tok, K), bf(N, K, std=K ** -0.5), bf(N, K, std=K ** -0.5)
    dev = [t.cuda() for t in (a, b, w_a, w_b)]
    with profile(activities=[ProfilerActivity.CUDA]) as trace:
        out = S.fc_concat(*dev)
        torch.cuda.synchronize()
    names = [m[1] for m in (re.search(r"proj_([a-z]+)_kernel", e.name) for e in trace.events()) if m]
    assert tuple(names) == kernels
    pick = np.unique(np.concatenate([[0, n_tok - 1], np.random.default_rng(1).integers(0, n_tok, 60)]))
    _close(out[pick], fc_concat_ref(W.widen(a[pick]), W.widen(b[pick]), np.concatenate([W.widen(w_a), W.widen(w_b)], axis=1)), "fc2")
