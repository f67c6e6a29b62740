"""Per-query parameter sets marshalled by column: the values that reading them one by
one with p["k"] and p.get(name, default) gives, for every kind of mapping."""

import collections
import math
import types

import numpy as np
import pytest

import paper_2107_05537_amd as pm

DEFAULTS = (("c", 1.5), ("confidence", 1 - 1 / math.e), ("beta", -1.0), ("r_min", 0.0))


class Row:
    """A mapping without `in` or a length."""

    def __init__(self, **kw):
        self._kw = kw

    def __getitem__(self, name):
        return self._kw[name]

    def get(self, name, default=None):
        return self._kw.get(name, default)


SETS = [{"k": 3}, {"k": 10, "c": 2}, {"k": np.int64(7), "beta": np.float32(0.25)},
        {"k": 1, "r_min": 1e-3, "confidence": 0.9}, {"k": True, "c": "1.25"}]


@pytest.mark.parametrize("kind", [dict, types.MappingProxyType,
                                  lambda p: collections.defaultdict(float, p),
                                  lambda p: collections.ChainMap({}, p),
                                  lambda p: Row(**p)],
                         ids=["dict", "proxy", "defaultdict", "chain", "row"])
@pytest.mark.parametrize("count", [0, 1, 3, 5])
def test_columns(kind, count):
    params = [kind(p) for p in SETS[:count]]
    rows, largest = pm._query_args(params)
    assert largest == max([int(p["k"]) for p in params] or [1])
    for i, p in enumerate(params):
        assert rows[i].k == int(p["k"]) and rows[i].reserved == 0
        for name, default in DEFAULTS:
            assert getattr(rows[i], name) == float(SETS[i].get(name, default)), (i, name)
    # nothing is added to the caller's sets
    for i, p in enumerate(params):
        if not isinstance(p, Row):
            assert dict(p) == SETS[i]


def test_refused_sets():
    for bad in ({}, {"k": None}, {"k": 2, "c": None}):
        for other in ({"k": 1}, Row(k=1)):
            with pytest.raises((KeyError, TypeError)):
                pm._query_args([other, bad])
    wide = [{"k": 2 ** 40 + 5}, {"k": -1}]
    rows, largest = pm._query_args(wide)
    assert (rows[0].k, rows[1].k, largest) == (5, -1, 2 ** 40 + 5)
