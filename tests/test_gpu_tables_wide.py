"""Projection tables of more than 16 directions, whose tiles are dealt to
several workgroups per 16 queries: few and many queries, blocks with and
without a partly filled group of 16, one to eight direction tiles, against the
float64 oracle with the tolerance of the other table tests (single-precision
sums of at most 960 products of order one)."""
import numpy as np
import pytest

import oracle as O

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2402_11354_amd")

pytestmark = pytest.mark.gpu


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(torch.device("cuda:0"))


@pytest.mark.parametrize("nq", [1, 16, 33, 700])
@pytest.mark.parametrize("d,L,m", [(960, 16, 128), (20, 5, 48), (4, 1, 32), (256, 8, 32), (96, 12, 112),
                                   (128, 32, 64), (320, 5, 80)])
def test_wide_tables(d, L, m, nq):
    rng = np.random.default_rng([d, L, m, nq])
    x = rng.normal(size=(40, d)).astype(np.float32)
    g = ((np.arange(40)[:, None] + np.arange(1, 5)[None, :]) % 40).astype(np.int32)
    A = rng.normal(size=(L, m, d // L)).astype(np.float32)
    B = rng.normal(size=(m, d)).astype(np.float32)
    q = (rng.normal(size=(nq, d)) * 3).astype(np.float32)
    idx = P.peos_build_tables(T(x), T(g), 0, L, m, T(A), T(B), P.PEOS_METRIC_L2)
    tables = torch.full((nq, L + 1, m), np.nan, dtype=torch.float32, device="cuda:0")
    norms = torch.full((nq,), np.nan, dtype=torch.float32, device="cuda:0")
    print("[gpu] tables", d, L, m, nq, flush=True)
    P.peos_query_tables(idx, T(q), tables, norms)
    torch.cuda.synchronize()
    pick = np.unique(np.linspace(0, nq - 1, 40).astype(int))
    ref = np.stack([O.query_table(q[i], L, m, A, B) for i in pick])
    np.testing.assert_allclose(tables.cpu().numpy()[pick], ref, rtol=0, atol=2e-5)
    assert not bool(torch.isnan(tables).any())
    np.testing.assert_allclose(norms.cpu().numpy(), np.linalg.norm(q.astype(np.float64), axis=1), rtol=2e-6)
