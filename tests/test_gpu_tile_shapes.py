"""Product tiles of the grouped GEMM on launches of many shapes: one level of
leaves whose widths and sets sit at and beside the edges of the tiles (32, 64,
128) and of the k chunks, R_L and R_U of equal and of different sizes, complex
blocks, and a batch.  The 32-wide tiles stage their operands through registers,
the wider ones load them straight into LDS where their type allows; every
entry sums the same products in the same order, so the results are equal bit
for bit.  Marked gpu."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-11, "mixed_fp32": 1e-5, "mixed_bf16x3": 1e-5}
ROOT = 130
WIDTHS = [1, 15, 16, 17, 31, 33, 63, 64, 65, 127, 128, 129]
ROWS = [129, 1, 17, 63, 64, 65, 127, 128, 33, 16, 31, 15]
COLS = [64, 16, 1, 129, 65, 31, 33, 15, 127, 128, 17, 63]


def leaves(widths, rows, cols, seed, dtype=float):
    """Leaves of the given widths, each coupled to its first rows / columns of a
    dense root of ROOT columns, and the dense matrix."""
    n = sum(widths) + ROOT
    rng = np.random.default_rng(seed)
    m = np.zeros((n, n), bool)
    o, r0 = 0, n - ROOT
    for w, r, c in zip(widths, rows, cols):
        m[o:o + w, o:o + w] = True
        m[r0:r0 + r, o:o + w] = True
        m[o:o + w, r0:r0 + c] = True
        o += w
    m[r0:, r0:] = True
    a = np.where(m, rng.uniform(-1, 1, (n, n)), 0).astype(dtype)
    if dtype == complex:
        a += 1j * np.where(m, rng.uniform(-1, 1, (n, n)), 0)
    np.fill_diagonal(a, 0)
    a[np.arange(n), np.arange(n)] = np.abs(a).sum(1) + 1
    s = sp.csc_matrix(a)
    s.sort_indices()
    return s, a


def table(levels, tile):
    return [4, levels, 1, tile, tile, tile, 1, 0] + [tile, tile, 1, 0] * levels


def selected(s, a):
    """What get_selected returns: A^{-1}(j, i) for the stored entries (i, j)."""
    inv = np.linalg.inv(a)
    j = np.repeat(np.arange(a.shape[0]), np.diff(s.indptr))
    return inv[j, s.indices]


def check(handles, runner, mats, prec):
    got = {}
    for tile in (32, 64, 128):
        print("[case] tile shapes", prec, tile, flush=True)
        runner.set_tuning(table(runner.info["nlevels"], tile), prec)
        runner.run(prec)
        assert runner.level_stats(1)["tile35"] == tile
        got[tile] = [h.export(sort=False)[2] for h in handles]
        for h, (s, a), x in zip(handles, mats, got[tile]):
            assert np.array_equal(x, got[32][handles.index(h)])
            ref = selected(s, a)
            assert np.abs(h.get_selected() - ref).max() / np.abs(ref).max() <= TOL[prec]


@pytest.fixture(scope="module")
def si():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1708_04539_amd import selinv
    return selinv


@pytest.mark.parametrize("kind", ["symmetrized", "exact", "complex"])
@pytest.mark.parametrize("prec", ["fp64", "mixed_fp32", "mixed_bf16x3"])
def test_one_level_of_many_shapes(si, kind, prec):
    rows, cols = (ROWS, COLS) if kind == "exact" else (ROWS, ROWS)
    s, a = leaves(WIDTHS, rows, cols, 3, complex if kind == "complex" else float)
    h = si.SelInv(a.shape[0], s.indptr.astype(np.int64), s.indices, None, 1024, 0, 0,
                  symbolic="exact" if kind == "exact" else "symmetrized", complex_values=kind == "complex")
    st = h.structure()
    two = 2 if kind == "complex" else 1  # columns of the real form
    assert np.diff(st["xsup"]).tolist() == [two * w for w in WIDTHS + [ROOT]]
    assert np.diff(st["rl_ptr"]).tolist() == [two * r for r in rows + [0]]
    assert np.diff(st["ru_ptr"]).tolist() == [two * c for c in cols + [0]]
    h.factor(s.data)
    check([h], h, [(s, a)], prec)


@pytest.mark.parametrize("prec", ["fp64", "mixed_fp32", "mixed_bf16x3"])
def test_batch_of_many_shapes(si, prec):
    mats = [leaves(WIDTHS[k::3], ROWS[k::3], ROWS[k::3], k) for k in range(3)]
    handles = [si.SelInv(a.shape[0], s.indptr.astype(np.int64), s.indices, None, 1024, 0, 0).factor(s.data)
               for s, a in mats]
    for k, h in enumerate(handles):
        assert np.diff(h.structure()["xsup"]).tolist() == WIDTHS[k::3] + [ROOT]
    b = si.Batch(handles)
    check(handles, b, mats, prec)
    b.close()
