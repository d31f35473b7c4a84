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
