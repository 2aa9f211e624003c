"""Searches whose lists are merged a chunk of 64 entries at a time, at sizes
around the chunks and around the 256 entries merged together, with the list as
the queue, a queue of two lists and the unbounded one, against the oracle
(both parity rules, on the integer-valued recipe, where nearly every query's
path is decided exactly)."""
import numpy as np
import pytest

import workloads as W
from parity import check_both

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2402_11354_amd")

pytestmark = pytest.mark.gpu

SMALL = W.SIFT_LIKE.with_sizes(n=6000, nq=24)


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(torch.device("cuda:0"))


@pytest.fixture(scope="module")
def case():
    w = SMALL
    x, q = W.make_base(w), W.make_queries(w)
    g, entry = W.build_graph(x, w.R, w.cand)
    A, B = W.directions_for(w)
    idx = P.peos_build_tables(T(x), T(g), entry, w.L, w.m, T(A), T(B), w.metric)
    return w, x, q, g, entry, A, B, idx


SIZES = [1, 63, 64, 65, 128, 129, 192, 193, 256, 257, 520]


# (the unbounded queue holds 16 lists, up to the kernel's 2048 entries)
@pytest.mark.parametrize("ef,pool", [(e, p) for e in SIZES for p in ("list", -2, 0) if p != 0 or e <= 128])
def test_list_sizes_around_the_chunks(case, ef, pool):
    w, x, q, g, entry, A, B, idx = case
    p = ef if pool == "list" else pool
    k = min(10, ef)
    print("[gpu] list", ef, "pool", p, flush=True)
    ids, d, st = P.search(idx, T(q), k, ef, eps=0.1, pool=p)
    torch.cuda.synchronize()
    check_both((ids.cpu().numpy(), d.cpu().numpy(), st.cpu().numpy()), x, g, entry, q, k, ef, w.L, w.m, A, B,
               w.metric, 0.1, pool=p, min_checked=0.5, label=f"ef={ef} pool={p}")
