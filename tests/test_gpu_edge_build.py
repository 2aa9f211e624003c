"""Edge records at the edges of the build's tiles against the oracle: node
degrees that fill, straddle and overfill the 16-edge tiles, blocks of 4 to 172
coordinates, vectors shorter and longer than the part held on the chip at a
time, 16 to 128 directions, absent and zero-length edges.  Codes are integer
decisions and bit-exact; the scalars keep the tolerances of the other record
tests (single-precision sums against float64)."""
import numpy as np
import pytest

import oracle as O

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2402_11354_amd")

pytestmark = pytest.mark.gpu


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(torch.device("cuda:0"))


def inputs(n, d, R, L, m):
    rng = np.random.default_rng([n, d, R, L, m])
    x = rng.normal(0, 3, (n, d)).astype(np.float32)
    x[1] = x[0]  # a zero-length edge 0 -> 1
    x[2, : d // 2] = x[0, : d // 2]  # and zero blocks
    g = np.full((n, R), -1, np.int32)
    for v in range(n):
        others = rng.permutation(np.delete(np.arange(n), v))[:R]
        keep = rng.random(len(others)) < 0.9
        g[v, : len(others)][keep] = others[keep]
    g[0, 0] = 1
    if R > 1:
        g[0, 1] = 2
        g[0, 2:] = np.where(np.isin(g[0, 2:], (1, 2)), -1, g[0, 2:])
    A = rng.normal(size=(L, m, d // L)).astype(np.float32)
    B = rng.normal(size=(m, d)).astype(np.float32)
    return x, g, A, B


SHAPES = [(97, 4, 1, 1, 16), (150, 20, 17, 5, 48), (130, 96, 33, 12, 32), (90, 260, 48, 5, 16),
          (70, 516, 64, 3, 128), (41, 960, 20, 16, 16), (66, 128, 32, 32, 16), (3, 64, 16, 4, 16),
          (70, 128, 32, 8, 16), (70, 128, 33, 4, 32), (40, 320, 31, 5, 16), (60, 128, 32, 8, 128),
          (45, 480, 24, 6, 32)]


@pytest.mark.parametrize("perm", [False, True])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_records_at_tile_edges(shape, perm):
    n, d, R, L, m = shape
    x, g, A, B = inputs(*shape)
    p = np.random.default_rng(d).permutation(d).astype(np.int32) if perm else None
    print("[gpu] build", shape, "perm" if perm else "", flush=True)
    idx = P.peos_build_tables(T(x), T(g), 0, L, m, T(A), T(B), P.PEOS_METRIC_L2,
                              perm=None if p is None else T(p))
    lay = idx.layout()
    rec = idx._keep[-1].cpu().numpy().reshape(n, lay.node_stride)
    codes = rec[:, lay.codes_offset:lay.codes_offset + lay.code_bytes * R].reshape(n, R, -1)
    sc = rec[:, lay.scalars_offset:lay.scalars_offset + 16 * R].copy().view(np.float32).reshape(n, R, 4)
    rc, rs, _ = O.build_tables(x if p is None else x[:, p], g, L, m, A, B)
    valid = g >= 0
    assert np.array_equal(codes[..., :L + 1][valid], rc[valid])
    assert np.all(codes[..., L + 1:] == 0) and np.all(codes[~valid] == 0) and np.all(sc[~valid] == 0)
    ge, ne, wreg, swres = (sc[..., i][valid].astype(np.float64) for i in range(4))
    r_ne, r_wreg, r_wres, r_ge = (rs[..., i][valid] for i in range(4))
    np.testing.assert_allclose(ne, r_ne, rtol=2e-6)
    np.testing.assert_allclose(wreg, r_wreg, rtol=0, atol=2e-6)
    np.testing.assert_allclose(swres, np.sqrt(L) * r_wres, rtol=0, atol=2e-5 if L <= 16 else 4e-5)
    np.testing.assert_allclose(ge, r_ge, rtol=0, atol=2e-6 * (x.astype(np.float64) ** 2).sum(1).max())


@pytest.mark.parametrize("perm", [False, True])
@pytest.mark.parametrize("shape", [(97, 4, 1, 1, 16), (130, 96, 33, 3, 32), (90, 260, 48, 1, 16),
                                   (70, 516, 64, 3, 128), (150, 16, 17, 4, 48),
                                   (70, 128, 32, 2, 16), (60, 64, 32, 4, 32)], ids=str)
def test_compact_records_at_tile_edges(shape, perm):
    n, d, R, L, m = shape
    x, g, A, B = inputs(*shape)
    p = np.random.default_rng(d).permutation(d).astype(np.int32) if perm else None
    print("[gpu] compact build", shape, "perm" if perm else "", flush=True)
    idx = P.peos_build_tables(T(x), T(g), 0, L, m, T(A), T(B), P.PEOS_METRIC_L2,
                              flags=P.PEOS_FLAG_COMPACT, perm=None if p is None else T(p))
    lay = idx.layout()
    rec = idx._keep[-1].cpu().numpy().reshape(n, lay.node_stride)
    hdr, cg, ci = O.compact_tables(x, g, L, P.PEOS_METRIC_L2, perm=p)
    got = rec[:, lay.scalars_offset:lay.scalars_offset + 2 * R].reshape(n, R, 2)
    valid = g >= 0
    assert np.array_equal(rec[:, :16].copy().view(np.float32), np.asarray(hdr, np.float32))
    assert np.array_equal(got[..., 0][valid], np.asarray(cg)[valid])
    assert np.array_equal(got[..., 1][valid], np.asarray(ci)[valid])
    codes = rec[:, lay.codes_offset:lay.codes_offset + 4 * R].reshape(n, R, 4)
    rc, _, _ = O.build_tables(x if p is None else x[:, p], g, L, m, A, B)
    assert np.array_equal(codes[..., :L][valid], rc[..., 1:][valid])
    assert np.all(codes[..., L:] == 0) and np.all(codes[~valid] == 0)
