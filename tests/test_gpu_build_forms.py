"""Edge records of sparse rows (tiles without an edge, nodes without one, graphs
of a few nodes), and of the other metrics and the half scalars at the edges of
the build's tiles: codes bit for bit the oracle's, an absent edge all zeros, and
the scalars of one form exactly those of the full-precision l2 form (the same
single-precision sums) where the form keeps them."""
import numpy as np
import pytest

import oracle as O

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2402_11354_amd")

pytestmark = pytest.mark.gpu


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(torch.device("cuda:0"))


class Records:
    def __init__(self, x, g, L, m, A, B, metric, flags, C, perm):
        n, R = g.shape
        idx = P.peos_build_tables(T(x), T(g), 0, L, m, T(A), T(B), metric, flags=flags,
                                  simhash_dirs=T(C) if flags & P.PEOS_FLAG_SIMHASH else None,
                                  perm=None if perm is None else T(perm))
        lay = idx.layout()
        rec = idx._keep[-1].cpu().numpy()[:n * lay.node_stride].reshape(n, lay.node_stride)
        self.codes = rec[:, lay.codes_offset:lay.codes_offset + lay.code_bytes * R].reshape(n, R, -1)
        sb = lay.scalar_bytes
        self.scal = rec[:, lay.scalars_offset:lay.scalars_offset + sb * R].reshape(n, R, sb).copy()
        self.sig = rec[:, lay.simhash_offset:lay.simhash_offset + 8 * R].copy().view(np.uint64)


def inputs(n, d, R, L, m, rows):
    rng = np.random.default_rng([n, d, R, L, m])
    x = rng.normal(0, 3, (n, d)).astype(np.float32)
    g = np.full((n, R), -1, np.int32)
    for v in range(n):
        others = rng.permutation(np.delete(np.arange(n), v))[:R]
        if rows == "last":  # only the row's last slots
            others = others[:2]
            g[v, R - len(others):] = others
        elif rows == "few":  # every other node has none, the rest short rows
            others = others[: v % 2 * 3]
            g[v, : len(others)] = others
        else:
            keep = rng.random(len(others)) < 0.9
            g[v, : len(others)][keep] = others[keep]
    A = rng.normal(size=(L, m, d // L)).astype(np.float32)
    B = rng.normal(size=(m, d)).astype(np.float32)
    C = rng.normal(size=(64, d)).astype(np.float32)
    return x, g, A, B, C


@pytest.mark.parametrize("rows", ["last", "few", "most"])
@pytest.mark.parametrize("shape", [(2, 128, 32, 8, 16), (2, 960, 64, 16, 128), (70, 20, 17, 5, 48), (900, 32, 40, 8, 16),
                                   (2100, 16, 3, 4, 32)], ids=str)
def test_sparse_rows(shape, rows):
    n, d, R, L, m = shape
    x, g, A, B, C = inputs(*shape, rows)
    print("[gpu] sparse build", shape, rows, flush=True)
    rc, _, _ = O.build_tables(x, g, L, m, A, B)
    valid = g >= 0
    for flags in (0, P.PEOS_FLAG_SIMHASH, P.PEOS_FLAG_FP16):
        r = Records(x, g, L, m, A, B, P.PEOS_METRIC_L2, flags, C, None)
        assert np.array_equal(r.codes[..., :L + 1][valid], rc[valid])
        assert not r.codes[..., L + 1:].any() and not r.codes[~valid].any() and not r.scal[~valid].any()
        if flags & P.PEOS_FLAG_SIMHASH:
            assert not r.sig[~valid].any()
            for v, j in np.argwhere(valid)[:200]:
                assert r.sig[v, j] == O.simhash_bits(x[g[v, j]] - x[v], C)[0], (v, j)


@pytest.mark.parametrize("rows", ["last", "few"])
@pytest.mark.parametrize("perm", [False, True])
def test_sparse_compact_rows(rows, perm):
    n, d, R, L, m = shape = (61, 96, 33, 3, 32)
    x, g, A, B, C = inputs(*shape, rows)
    p = np.random.default_rng(1).permutation(d).astype(np.int32) if perm else None
    r = Records(x, g, L, m, A, B, P.PEOS_METRIC_L2, P.PEOS_FLAG_COMPACT, C, p)
    _, cg, ci = O.compact_tables(x, g, L, P.PEOS_METRIC_L2, perm=p)
    rc, _, _ = O.build_tables(x if p is None else x[:, p], g, L, m, A, B)
    valid = g >= 0
    assert np.array_equal(r.codes[..., :L][valid], rc[..., 1:][valid]) and not r.codes[~valid].any()
    assert np.array_equal(r.scal[..., 0][valid], np.asarray(cg)[valid])
    assert np.array_equal(r.scal[..., 1][valid], np.asarray(ci)[valid])
    assert not r.scal[~valid].any()


@pytest.mark.parametrize("perm", [False, True])
@pytest.mark.parametrize("shape", [(90, 260, 33, 5, 16), (40, 516, 20, 3, 48), (60, 384, 17, 8, 128), (70, 128, 64, 8, 32)],
                         ids=str)
def test_metrics_and_half_scalars(shape, perm):
    n, d, R, L, m = shape
    x, g, A, B, C = inputs(*shape, "most")
    x[1] = x[0]  # a zero-length edge
    g[0, 0] = 1
    g[0, 1:] = np.where(g[0, 1:] == 1, -1, g[0, 1:])
    p = np.random.default_rng(d).permutation(d).astype(np.int32) if perm else None
    print("[gpu] forms", shape, "perm" if perm else "", flush=True)
    make = lambda metric, flags: Records(x, g, L, m, A, B, metric, flags, C, p)
    full = make(P.PEOS_METRIC_L2, 0)
    rc, _, _ = O.build_tables(x if p is None else x[:, p], g, L, m, A, B)
    valid = g >= 0
    assert np.array_equal(full.codes[..., :L + 1][valid], rc[valid])
    s = full.scal.view(np.float32).reshape(n, R, 4)
    ge, en, wreg, swres = (s[..., i] for i in range(4))
    for metric in (P.PEOS_METRIC_L2, P.PEOS_METRIC_ANGULAR, P.PEOS_METRIC_IP):
        g_e = ge if metric == P.PEOS_METRIC_L2 else np.zeros_like(ge)
        other = make(metric, 0)
        assert np.array_equal(other.codes, full.codes)
        assert np.array_equal(other.scal.view(np.float32).reshape(n, R, 4), np.stack([g_e, en, wreg, swres], -1))
        half = make(metric, P.PEOS_FLAG_FP16)
        assert np.array_equal(half.codes, full.codes)
        with np.errstate(divide="ignore", invalid="ignore"):
            gp = np.where(en > 0, g_e / en, np.float32(0)).astype(np.float32)
            ie = np.where(en > 0, np.float32(1) / en, np.float32(np.inf)).astype(np.float32)
            want = np.stack([gp, ie, wreg, swres], -1).astype(np.float16)
        want[~valid] = 0
        assert np.array_equal(half.scal.view(np.float16).reshape(n, R, 4), want)
