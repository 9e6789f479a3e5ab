"""The Python binding where its native half does not load."""
import sys

import pytest
import torch

import paper_2402_05396_amd as T
from paper_2402_05396_amd import build


@pytest.mark.parametrize("why", ["absent", "other torch"])
def test_calls_go_the_general_way(monkeypatch, why):
    monkeypatch.setattr(T, "_native", None)
    if why == "absent":
        monkeypatch.setitem(sys.modules, T.__name__ + "._binding", None)     # importing it raises ImportError
        monkeypatch.delattr(T, "_binding", raising=False)
    else:
        monkeypatch.setattr(build, "binding_tag", lambda: "torch 1.0, Python 3.10")
        assert build.stale()
    with pytest.warns(RuntimeWarning, match="ctypes"), pytest.raises(TypeError, match="device tensor"):
        T.gather_features(torch.zeros((3, 4)), torch.zeros(2, dtype=torch.int32))     # refused by the general half
    with pytest.raises(TypeError, match="nbr"):                                       # and no second warning
        T.candidate_encodings(torch.zeros((3, 4)), torch.zeros(3))


def test_the_built_one_fits():
    assert build.binding_fits()
