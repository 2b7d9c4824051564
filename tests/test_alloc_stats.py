"""`alloc_stats` is a dictionary like any other, to copy, save and set back, and up to date whenever it is looked at (no GPU: blocks that are
nowhere are given back)."""
import copy
import json
import pickle

import pytest

import paper_2204_02662_amd as epp

KEYS = ["allocs", "frees", "bytes", "live"]


@pytest.fixture
def stats():
    held = dict(epp.alloc_stats)
    epp.alloc_stats.update(dict.fromkeys(KEYS, 0))
    yield epp.alloc_stats
    epp.alloc_stats.update(held)


def _free(blocks):
    for _ in range(blocks):
        epp._TORCH_FREE_FN(None, None)  # (as the library calls it)


@pytest.mark.parametrize("read", [lambda s: {k: s[k] for k in s}, dict, lambda s: s.copy(), lambda s: json.loads(json.dumps(s)),
                                  lambda s: {**s}, lambda s: dict(s.items()), lambda s: dict(zip(s, s.values())), lambda s: s | {},
                                  lambda s: {} | s, lambda s: eval(repr(s)), copy.copy, copy.deepcopy, lambda s: {k: s.get(k) for k in KEYS},
                                  lambda s: pickle.loads(pickle.dumps(s)), lambda s: {} if s == dict.fromkeys(KEYS, 0) else dict(s)])
def test_looked_at(read, stats):
    assert isinstance(stats, dict) and list(stats) == KEYS
    _free(3)
    got = read(stats)
    assert type(got) is dict and got == {"allocs": 0, "frees": 3, "bytes": 0, "live": -3}
    _free(1)
    assert got["frees"] == 3 and stats["frees"] == 4


def test_set_back(stats):
    _free(2)
    stats["frees"] = 0  # (a key on its own: the others go on)
    _free(1)
    assert stats == {"allocs": 0, "frees": 1, "bytes": 0, "live": -3}
    _free(1)
    stats.update(frees=0, live=0)
    assert dict(stats) == dict.fromkeys(KEYS, 0)
    _free(1)
    stats["frees"] -= 1
    assert stats["frees"] == 0 and stats.pop("live") == -1
    _free(1)
    assert stats == {"allocs": 0, "frees": 1, "bytes": 0, "live": -1}
