"""The binding's calls over a list of blocks (Nova.entropy_blocks, Nova.select_blocks) with too short lists or none, on the
CPU: the library reads one entry per block of every host array, so such a call must not reach it."""
import pytest
import torch

from paper_2602_01345_amd import binding


@pytest.fixture
def nova(monkeypatch):
    """A Nova whose library notes the calls it gets and launches nothing."""
    class Library:
        def __init__(self):
            self.calls = []

        def __getattr__(self, name):
            return lambda *args: self.calls.append(name) or 0
    monkeypatch.setattr(binding, "_ptr", lambda t: 16)
    monkeypatch.setattr(binding, "_stream", lambda: 0)
    n = object.__new__(binding.Nova)
    n.lib, n.ctx = Library(), None
    return n


def _ts(n, *shape):
    return [torch.zeros(shape) for _ in range(n)]


@pytest.mark.parametrize("logits,entropy,mean", [(3, 2, None), (3, 3, 2), (3, 0, 3), (1, 0, None)])
@pytest.mark.parametrize("mixed", [False, True])
def test_entropy_blocks_of_too_short_lists(nova, logits, entropy, mean, mixed):
    ls = _ts(logits, 2, 4, 8)
    if mixed and ls:
        ls[-1] = torch.zeros(2, 4, 16)                 # another shape: one call per block
    with pytest.raises(ValueError):
        nova.entropy_blocks(ls, _ts(entropy, 2, 4), None if mean is None else _ts(mean, 2))
    assert nova.lib.calls == []


@pytest.mark.parametrize("entropy,k,idx,mask", [(3, 2, 3, 3), (3, 3, 2, 3), (3, 3, 3, 2), (1, 0, 1, 1)])
def test_select_blocks_of_too_short_lists(nova, entropy, k, idx, mask):
    with pytest.raises(ValueError):
        nova.select_blocks(_ts(entropy, 2, 4), [1] * k, _ts(idx, 2, 1), _ts(mask, 2, 4))
    assert nova.lib.calls == []


def test_no_blocks_is_no_call(nova):
    nova.entropy_blocks([], [])
    nova.entropy_blocks([], [], [])
    nova.select_blocks([], [], [], [])
    assert nova.lib.calls == []


@pytest.mark.parametrize("more", [0, 1])
def test_enough_entries_are_one_call(nova, more):
    nova.entropy_blocks(_ts(3, 2, 4, 8), _ts(3 + more, 2, 4), _ts(3 + more, 2))
    nova.select_blocks(_ts(3, 2, 4), [1, 2, 0] + [0] * more, _ts(3 + more, 2, 2), _ts(3 + more, 2, 4))
    assert nova.lib.calls == ["nova_entropy_blocks", "nova_select_blocks"]
