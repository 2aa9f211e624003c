"""SimHash signatures at the edges of the build's tiles (partly filled groups of
16 coordinates, vectors past the 256 held on the chip at a time, tiles that
straddle nodes), with the sign vectors starting at every float of a 16-byte
line: the bits are integer decisions and exact."""
import numpy as np
import pytest

import oracle as O

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2402_11354_amd")

pytestmark = pytest.mark.gpu


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(torch.device("cuda:0"))


@pytest.mark.parametrize("shape,first", [((150, 20, 17, 5, 48), 1), ((90, 260, 33, 5, 16), 2),
                                         ((60, 384, 33, 8, 128), 3), ((3, 64, 16, 4, 16), 0),
                                         ((40, 516, 20, 3, 16), 1)], ids=str)
def test_signatures_at_tile_edges(shape, first):
    n, d, R, L, m = shape
    rng = np.random.default_rng(shape)
    x = rng.normal(0, 3, (n, d)).astype(np.float32)
    g = np.full((n, R), -1, np.int32)
    for v in range(n):
        others = rng.permutation(np.delete(np.arange(n), v))[:R]
        keep = rng.random(len(others)) < 0.9
        g[v, : len(others)][keep] = others[keep]
    A = rng.normal(size=(L, m, d // L)).astype(np.float32)
    B = rng.normal(size=(m, d)).astype(np.float32)
    C = rng.normal(size=(64, d)).astype(np.float32)
    held = torch.full((64 * d + 4,), np.nan, dtype=torch.float32, device="cuda:0")
    Ct = held[first:first + 64 * d].view(64, d)
    Ct.copy_(T(C))
    assert Ct.data_ptr() % 16 == 4 * first
    print("[gpu] simhash build", shape, "first", first, flush=True)
    idx = P.peos_build_tables(T(x), T(g), 0, L, m, T(A), T(B), P.PEOS_METRIC_L2, flags=P.PEOS_FLAG_SIMHASH,
                              simhash_dirs=Ct)
    lay = idx.layout()
    rec = idx._keep[-1].cpu().numpy().reshape(n, lay.node_stride)
    sig = rec[:, lay.simhash_offset:lay.simhash_offset + 8 * R].copy().view(np.uint64)
    codes = rec[:, lay.codes_offset:lay.codes_offset + lay.code_bytes * R].reshape(n, R, -1)
    rc, _, _ = O.build_tables(x, g, L, m, A, B)
    valid = g >= 0
    assert np.array_equal(codes[..., :L + 1][valid], rc[valid])
    assert np.all(sig[~valid] == 0)
    for v, j in np.argwhere(valid):
        assert sig[v, j] == O.simhash_bits(x[g[v, j]] - x[v], C)[0], (v, j)
