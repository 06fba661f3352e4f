"""Lengths of the layer, target and guide-star parameters that the binding hands to the library.

The library reads 4 doubles per layer, 3 per target and 5 per guide star, so the arrays hold that many
whatever the caller's tuples hold: short ones are filled with 0 at the end of the array, long ones refused.
"""
import types

import pytest
import torch

from paper_1408_0698_amd import shwfs

STREAM = types.SimpleNamespace(cuda_stream=0)
LAYER = (torch.zeros((40, 40)), 0.05, 0.0, 20.0, 20.0)


@pytest.fixture
def calls(monkeypatch):
    """(entry point, arguments) of the calls, which go no further."""
    seen = []

    def record(name):
        return lambda *args: (seen.append((name, args)), 0)[1]

    names = ("shw_project_layers", "shw_uplink_tilt")
    monkeypatch.setattr(shwfs, "_lib", types.SimpleNamespace(**{n: record(n) for n in names}))
    return seen


def _project(targets, layers=(LAYER,)):
    shwfs.project_layers(list(layers), 8, 0.05, targets, torch.zeros((max(1, len(targets)), 8, 8)), stream=STREAM)


def _uplink(lgs, layers=(LAYER,)):
    shwfs.uplink_tilt(list(layers), lgs, 0.4, 8, torch.zeros((max(1, len(lgs)), 2), dtype=torch.float64), stream=STREAM)


@pytest.mark.parametrize("targets,want", [
    ([], [0, 0, 0]), ([(1e-6, 2e-6, 9e4)], [1e-6, 2e-6, 9e4]), ([(1e-6, 2e-6)], [1e-6, 2e-6, 0]),
    ([(1, 2, 3), (4, 5)], [1, 2, 3, 4, 5, 0]), ([(1, 2), (3, 4)], [1, 2, 3, 4, 0, 0]), ([()], [0, 0, 0])])
def test_target_parameters(calls, targets, want):
    _project(targets)
    assert calls[0][0] == "shw_project_layers" and calls[0][1][8] == len(targets) and list(calls[0][1][9]) == want


@pytest.mark.parametrize("lgs,want", [
    ([], [0] * 5), ([(1, 2, 3, 4, 9e4)], [1, 2, 3, 4, 9e4]), ([(1, 2, 3, 4)], [1, 2, 3, 4, 0]),
    ([(1, 2, 3, 4, 5), (6,)], [1, 2, 3, 4, 5, 6, 0, 0, 0, 0])])
def test_guide_star_parameters(calls, lgs, want):
    _uplink(lgs)
    assert calls[0][0] == "shw_uplink_tilt" and calls[0][1][6] == len(lgs) and list(calls[0][1][7]) == want


@pytest.mark.parametrize("call", [_project, _uplink])
@pytest.mark.parametrize("layers,want", [
    ((LAYER, LAYER), [0.05, 0, 20, 20] * 2), ((LAYER[:4],), [0.05, 0, 20, 0]), ((LAYER, LAYER[:2]), [0.05, 0, 20, 20, 0.05, 0, 0, 0]),
    ((LAYER + (7.0,),), [0.05, 0, 20, 20])])
def test_layer_parameters(calls, call, layers, want):
    call([], layers)
    assert calls[0][1][0] == len(layers) and list(calls[0][1][5]) == want


def test_too_many_parameters_are_refused(calls):
    with pytest.raises(IndexError):
        _project([(0, 0, 9e4, 1), (0, 0, 9e4)])
    with pytest.raises(IndexError):
        _uplink([(1, 2, 3, 4, 5, 6)])
    assert not calls


def test_numbers_of_every_kind(calls):
    """Whatever float() takes: integers, numpy and torch scalars, texts."""
    import numpy as np
    _project([(1, np.float32(2.5), torch.tensor(3.0))])
    _project([(np.int64(1), "2.5", True)])
    assert [list(c[1][9]) for c in calls] == [[1, 2.5, 3], [1, 2.5, 1]]
    with pytest.raises(TypeError):
        _project([(1, 2, None)])
    with pytest.raises(ValueError):
        _project([(1, 2, "high")])
