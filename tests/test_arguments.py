"""Packing of a call's lists for the C-ABI: kinds and per-field entries from
any iterable, missing ones zero or null, too many refused."""
import pytest

torch = pytest.importorskip("torch")

import paper_2609_10165_amd as gcr


@pytest.mark.parametrize("form", [list, tuple, iter, lambda x: (k for k in x), lambda x: map(int, x),
                                  torch.tensor])
def test_kinds_from_any_iterable(form):
    assert list(gcr._kinds(form([1, 0, 2]), 3)) == [1, 0, 2]
    assert list(gcr._kinds(form([1, 2]), 4)) == [1, 2, 0, 0]
    assert list(gcr._kinds(form([2] * 9), 9)) == [2] * 9
    with pytest.raises(IndexError):
        gcr._kinds(form([1, 0, 2]), 2)


@pytest.mark.parametrize("form", [list, tuple, iter, lambda x: (k for k in x)])
def test_entries_from_any_iterable(form):
    assert list(gcr._opt_array(form([None, None]), 2, torch.uint8)) == [None] * 2
    assert list(gcr._opt_array(form([None]), 10, torch.uint8)) == [None] * 10
    with pytest.raises(IndexError):
        gcr._opt_array(form([None] * 3), 2, torch.uint8)
    with pytest.raises(ValueError):
        gcr._opt_array(form([torch.zeros(3)]), 2, torch.uint8)
