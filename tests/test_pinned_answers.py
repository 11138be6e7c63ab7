"""How much pinned memory the exported arrays of a program may take together (CPU: the accounting alone)."""
import gc

import numpy as np
import pytest
import torch

from paper_2209_07663_amd import binding


@pytest.fixture
def accounting(monkeypatch):
    """The accounting on its own, with ordinary memory in the place of pinned memory, and a small allowance."""
    acc = binding._PinnedAnswers()
    monkeypatch.setattr(binding, "_pinned", acc)
    monkeypatch.setattr(binding, "PINNED_HELD", 1 << 16)
    made, real = [], torch.empty

    def empty(*args, pin_memory=False, **kw):
        made.append(pin_memory)
        return real(*args, **kw)
    monkeypatch.setattr(binding.torch, "empty", empty)
    monkeypatch.setattr(binding.torch.cuda, "current_stream", lambda device: type("S", (), {"synchronize": lambda s: None})())
    acc.made = made
    return acc


def _answer(n=4000):
    return binding._to_numpy({"keys": torch.arange(n), "acc": torch.zeros(0)})


def test_held_answers_are_pinned_up_to_the_allowance_and_no_further(accounting):
    held = [_answer() for _ in range(5)]                       # 32000 bytes each: 32 KB of the pool
    assert sum(accounting.made) == 4 and accounting.held == 1 << 16    # two answers of two arrays
    assert all((a["keys"] == np.arange(4000)).all() for a in held)
    held.pop(0)
    gc.collect()
    assert accounting.held == 1 << 15
    held.append(_answer())
    assert accounting.held == 1 << 16


def test_a_view_or_a_tensor_of_an_answer_still_holds_it(accounting):
    view = _answer()["keys"][10:20]
    gc.collect()
    assert accounting.held == 1 << 15
    tensor = torch.from_numpy(view)
    del view
    gc.collect()
    assert accounting.held == 1 << 15 and int(tensor[0]) == 10
    del tensor
    gc.collect()
    assert accounting.held == 0


def test_an_answer_too_large_or_refused_by_the_host_takes_the_pageable_way(accounting, monkeypatch):
    monkeypatch.setattr(binding, "PINNED_MOST", 1000)
    assert _answer()["keys"][-1] == 3999 and not accounting.made and accounting.held == 0
    monkeypatch.setattr(binding, "PINNED_MOST", 1 << 20)

    def refused(*args, **kw):
        raise RuntimeError("no pinned memory")
    monkeypatch.setattr(binding.torch, "empty", refused)
    assert _answer()["keys"][-1] == 3999 and accounting.held == 0


def test_a_failed_copy_gives_everything_back(accounting, monkeypatch):
    def failed(device):
        raise RuntimeError("copy failed")
    monkeypatch.setattr(binding.torch.cuda, "current_stream", failed)
    with pytest.raises(RuntimeError):
        _answer()
    assert accounting.held == 0
