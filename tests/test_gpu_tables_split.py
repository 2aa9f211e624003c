"""Projection tables of more than 16 directions where their tiles do not come in
fours (one block, odd numbers of direction tiles, blocks longer than one load
stage), against the float64 oracle with the tolerance of the other table tests
(single-precision sums of at most 960 products of order one), and the same bits
whichever queries go with them."""
import numpy as np
import pytest

import oracle as O

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2402_11354_amd")

pytestmark = pytest.mark.gpu


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(torch.device("cuda:0"))


def check(d, L, m, nq, flags=0, perm=False):
    rng = np.random.default_rng([d, L, m, nq])
    x = rng.normal(size=(40, d)).astype(np.float32)
    g = ((np.arange(40)[:, None] + np.arange(1, 5)[None, :]) % 40).astype(np.int32)
    A = rng.normal(size=(L, m, d // L)).astype(np.float32)
    B = rng.normal(size=(m, d)).astype(np.float32)
    q = (rng.normal(size=(nq, d)) * 3).astype(np.float32)
    p = rng.permutation(d).astype(np.int32) if perm else np.arange(d, dtype=np.int32)
    idx = P.peos_build_tables(T(x), T(g), 0, L, m, T(A), T(B), P.PEOS_METRIC_L2, flags=flags,
                              perm=T(p) if perm else None)

    def tables(rows):
        out = torch.full((len(rows), L + 1, m), np.nan, device="cuda:0",
                         dtype=torch.float16 if flags & P.PEOS_FLAG_FP16 else torch.float32)
        norms = torch.full((len(rows),), np.nan, dtype=torch.float32, device="cuda:0")
        P.peos_query_tables(idx, T(rows), out, norms)
        torch.cuda.synchronize()
        return out.cpu().numpy(), norms.cpu().numpy()

    print("[gpu] tables", d, L, m, nq, flush=True)
    out, norms = tables(q)
    assert not np.isnan(out).any()
    pick = np.unique(np.linspace(0, nq - 1, 40).astype(int))
    ref = np.stack([O.query_table(q[i][p], L, m, A, B) for i in pick])
    if flags & P.PEOS_FLAG_FP16:  # half an ulp of the half, on top
        np.testing.assert_allclose(out[pick], ref, rtol=2.0 ** -11, atol=2e-5)
    else:
        np.testing.assert_allclose(out[pick], ref, rtol=0, atol=2e-5)
    np.testing.assert_allclose(norms, np.linalg.norm(q.astype(np.float64), axis=1), rtol=2e-6)
    few, few_norms = tables(q[:5])
    assert np.array_equal(few, out[:5]) and np.array_equal(few_norms, norms[:5])


@pytest.mark.parametrize("nq", [5, 50])
@pytest.mark.parametrize("d,L,m", [(960, 1, 32), (256, 1, 48), (96, 3, 112), (900, 3, 80), (64, 2, 16 * 7),
                                   (12, 1, 128)])
def test_tables_of_leftover_tiles(d, L, m, nq):
    check(d, L, m, nq)


# (more than 8,192 queries fill the chip without the tiles being dealt out;
# 45,000 of 9 x 128 floats outgrow the last-level cache)
@pytest.mark.parametrize("d,L,m,nq,flags", [(128, 8, 32, 8193, 0), (20, 5, 48, 8205, 0), (4, 1, 32, 9000, 0),
                                            (128, 8, 32, 8200, P.PEOS_FLAG_FP16), (256, 4, 48, 8301, 0),
                                            (128, 8, 64, 8192, 0), (64, 8, 128, 60_001, 0), (400, 5, 32, 24_600, 0),
                                            (400, 5, 32, 16_000, 0), (640, 16, 32, 12_300, 0), (256, 4, 64, 8_300, 0)])
def test_tables_of_many_queries(d, L, m, nq, flags):
    check(d, L, m, nq, flags)


# rows too long to be staged, and a permutation of the coordinates: the general
# form, with and without steps past whole groups of eight
@pytest.mark.parametrize("perm", [False, True])
@pytest.mark.parametrize("d,L,m,nq", [(1024, 16, 16, 35), (1040, 4, 48, 3), (1036, 1, 16, 16), (2048, 32, 32, 17)])
def test_tables_of_unstaged_rows(d, L, m, nq, perm):
    check(d, L, m, nq, perm=perm)


@pytest.mark.parametrize("d,L,m,nq", [(128, 8, 16, 35), (20, 5, 48, 7), (900, 3, 32, 18), (4, 1, 16, 1)])
def test_tables_of_permuted_rows(d, L, m, nq):
    check(d, L, m, nq, perm=True)
