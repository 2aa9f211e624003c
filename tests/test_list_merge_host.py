"""The searches around the list merge's sizes are decided: on their recipe the
float64 oracle finds at most two of the 24 queries whose path hangs on a
rounding, at every size and queue (CPU only)."""
import pytest

import oracle as O
import workloads as W
from test_gpu_list_merge import SIZES, SMALL


@pytest.fixture(scope="module")
def case():
    w = SMALL
    x, q = W.make_base(w), W.make_queries(w)
    return (w, x, q, *W.build_graph(x, w.R, w.cand), *W.directions_for(w))


@pytest.mark.parametrize("ef", SIZES)
def test_paths_are_decided(case, ef):
    w, x, q, g, entry, A, B = case
    for pool in (ef, -2, 0):
        if pool == 0 and ef > 128:
            continue
        r = O.search(x, g, entry, q, min(10, ef), ef, w.L, w.m, A, B, w.metric, 0.1, pool=pool, precision=64)
        assert (r["fragile"] == 0).sum() >= 22, (ef, pool)
