"""The library calls that the step classes make, recorded in place of the library (no GPU): their names, their order and
what the caller is told of them."""
import pytest
import torch

import workloads as W
import paper_2509_18824_amd.step as S


@pytest.fixture
def calls(monkeypatch):
    """Every library call that enqueues work is noted by its name instead, with its arguments."""
    made = []
    for name in dir(S.hb):
        if name.startswith("hb_") and not name.endswith(("_bytes", "_splits", "_rows", "_error", "_version")):
            monkeypatch.setattr(S.hb, name, lambda *args, _name=name, **kwargs: made.append((_name[3:], args)))
    return made


def _inputs():
    inp = W.make_verify_inputs(3, "bf16", 4, 2, 128, [20, 9], [W.chain_tree(3), W.seeded_tree(1, n_nodes=12, levels=3)], poison=False)
    return inp, S.to_device(inp, "cpu"), S.desc_for(inp)


@pytest.mark.parametrize("compact,layers", [(True, 1), (1, 1), (2, 1), ("yes", 1), (False, 0), (0, 0), (None, 0)])
def test_any_true_value_asks_for_the_append(calls, compact, layers):
    inp, dev, desc = _inputs()
    step = S.VerifyStep(desc, dev, torch.empty(50, 512, dtype=torch.bfloat16), torch.zeros(inp.total_nodes, dtype=torch.int32), inp.max_path)
    step.run(compact=compact)
    assert [c for c, _ in calls] == ["tree_verify_attn_clearing", "lmhead_accept_cleared"]
    assert calls[1][1][13] == layers


def _stack(n_layers, whole, norm_f=True):
    inp, dev, desc = _inputs()
    K, F, T = inp.Hq * inp.D, 64, inp.total_nodes
    t = lambda *shape: torch.empty(shape, dtype=torch.bfloat16)
    mlp = dict(norm1=[t(K)] * n_layers, norm2=[t(K)] * n_layers, w_gate_up=[t(2 * F, K)] * n_layers,
               w_down=[t(K, F)] * max(n_layers, 1), eps=1e-6) if whole else None
    if whole and norm_f:
        mlp["norm_f"] = t(K)
    return S.VerifyLayerStack(desc, dev, [(dev.k_pool, dev.v_pool)] * n_layers, [t((inp.Hq + 2 * inp.Hkv) * inp.D, K)] * max(n_layers, 1),
                              [t(K, K)] * max(n_layers, 1), t(50, K), torch.zeros(T, dtype=torch.int32), inp.max_path, t(T, K), mlp=mlp)


@pytest.mark.parametrize("n_layers,whole,norm_f,compact", [(2, True, True, True), (2, True, False, True), (1, True, True, False),
                                                           (3, False, False, True), (0, True, True, True), (0, False, False, True)])
def test_every_call_of_a_stack_is_told_by_its_name(calls, n_layers, whole, norm_f, compact):
    """on_call hears of each kind of work before the one call that does it, joined or not in a plain run."""
    told = []
    _stack(n_layers, whole, norm_f).run(compact=compact, on_call=lambda name: (told.append(name), calls.append((name, None))))
    layer = (["rmsnorm"] if whole else []) + ["qkv_rope_project", "tree_verify_attn", "out_project"]
    layer += ["rmsnorm", "swiglu_project", "down_project"] if whole else []
    assert told == (["positions"] + n_layers * layer + (["rmsnorm"] if whole and norm_f else []) + ["lmhead_argmax", "tree_accept"]
                    + (["kv_compact"] if compact else []) + ["end"])
    # what follows a name is the call it names; positions are two
    names = [c for c, args in calls]
    library = {"positions": ["tree_positions", "rope_table"], "qkv_rope_project": ["qkv_rope_project_ws"],
               "tree_verify_attn": ["tree_verify_attn_clearing"], "out_project": ["out_project_ws"],
               "down_project": ["out_project_ws"], "kv_compact": ["kv_compact_layers"], "end": []}
    assert names == [n for t in told for n in [t] + library.get(t, [t])]


@pytest.mark.parametrize("n_layers", [0, 2])
def test_a_plain_run_of_a_stack(calls, n_layers):
    """Without layers there is no attention that clears the LM head's keys: the call that needs nothing of them."""
    _stack(n_layers, True).run()
    layer = ["qkv_rope_project_ws", "tree_verify_attn_clearing", "out_project_norm_ws", "swiglu_project", "out_project_norm_ws"]
    assert [c for c, _ in calls] == (["tree_positions", "rope_table", "rmsnorm"] + n_layers * layer
                                     + ["lmhead_accept_cleared" if n_layers else "lmhead_accept"])
    assert [args[14] for c, args in calls if c == "tree_verify_attn_clearing"] == [0, 15][:n_layers]
