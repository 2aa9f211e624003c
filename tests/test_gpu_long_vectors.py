"""Vectors past 3,200 coordinates: the build holds 256 of them (or a group of
blocks) on the chip at a time, so the dimension has no limit there.  Records,
tables and searches against the oracle; the vectors are small integers, so that
every distance (at most 4096 x 15^2, below 2^24) is exact in single precision.
Scalars: single-precision sums of up to 4096 positive terms in 16 chains and a
tree, relative error at most (d/16 + 6) 2^-24; tables: chains of up to d products
of order |q_i'| |a_i|, at most d 2^-24 of the sum of their sizes."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from parity import check_both

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2402_11354_amd")

pytestmark = pytest.mark.gpu


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(torch.device("cuda:0"))


@pytest.mark.parametrize("d,L,perm", [(3328, 16, False), (4096, 8, False), (4096, 2, True), (3328, 32, True)])
def test_long_vectors(d, L, perm):
    n, nq, R, m, k, ef = 400, 12, 16, 16, 5, 32
    rng = np.random.default_rng([d, L])
    x = rng.integers(0, 16, (n, d)).astype(np.float32)
    q = rng.integers(0, 16, (nq, d)).astype(np.float32)
    g, entry = W.build_graph(x, R, 32)
    A = rng.normal(size=(L, m, d // L)).astype(np.float32)
    B = rng.normal(size=(m, d)).astype(np.float32)
    p = rng.permutation(d).astype(np.int32) if perm else None
    print("[gpu] long vectors", d, L, perm, flush=True)
    idx = P.peos_build_tables(T(x), T(g), entry, L, m, T(A), T(B), P.PEOS_METRIC_L2, perm=None if p is None else T(p))
    lay = idx.layout()
    rec = idx._keep[-1].cpu().numpy().reshape(n, lay.node_stride)
    codes = rec[:, lay.codes_offset:lay.codes_offset + lay.code_bytes * R].reshape(n, R, -1)
    sc = rec[:, lay.scalars_offset:lay.scalars_offset + 16 * R].copy().view(np.float32).reshape(n, R, 4)
    xp, qp = (x, q) if p is None else (x[:, p], q[:, p])
    rc, rs, _ = O.build_tables(xp, g, L, m, A, B)
    valid = g >= 0
    assert np.array_equal(codes[..., :L + 1][valid], rc[valid])
    rel = (d / 16 + 6) * 2.0 ** -24
    np.testing.assert_allclose(sc[..., 1][valid], rs[..., 0][valid], rtol=rel)
    np.testing.assert_allclose(sc[..., 2][valid], rs[..., 1][valid], rtol=0, atol=4 * rel)
    tables = torch.empty((nq, L + 1, m), dtype=torch.float32, device="cuda:0")
    norms = torch.empty((nq,), dtype=torch.float32, device="cuda:0")
    P.peos_query_tables(idx, T(q), tables, norms)
    ref = np.stack([O.query_table(v, L, m, A, B) for v in qp])
    qn = np.linalg.norm(q.astype(np.float64), axis=1, keepdims=True)
    # sum of |q'_k| |a_k| of each entry, at most |q'| |a| with |q'| <= 1
    size = max(np.linalg.norm(A, axis=2).max(), np.linalg.norm(B, axis=1).max())
    np.testing.assert_allclose(tables.cpu().numpy(), ref, rtol=0, atol=d * 2.0 ** -24 * size)
    np.testing.assert_allclose(norms.cpu().numpy(), qn[:, 0], rtol=d / 4 * 2.0 ** -24)
    for mode in (P.PEOS_MODE_PEOS, P.PEOS_MODE_EXHAUSTIVE):
        ids, dd, st = P.search(idx, T(q), k, ef, eps=0.1, mode=mode, pool=ef)
        torch.cuda.synchronize()
        check_both((ids.cpu().numpy(), dd.cpu().numpy(), st.cpu().numpy()), x, g, entry, q, k, ef, L, m, A, B,
                   W.L2, 0.1, mode=mode, pool=ef, perm=p, min_checked=0.5, label=f"d={d} mode={mode}")
