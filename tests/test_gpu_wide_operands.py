"""Products whose G_K is 2 GiB or more: the tiles that load their operands
straight into LDS address such an operand with one descriptor per load.  The
32-wide tiles stage it through registers with 64-bit addresses; both sum the
same products in the same order.  Marked gpu."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu


def test_g_of_two_gib():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1708_04539_amd import selinv as si
    # arrow matrix: node 0 coupled to all others, which elimination makes dense
    n, cap = 17500, 1024
    rng = np.random.default_rng(4)
    row, col = rng.uniform(-1, 0, n), rng.uniform(-1, 0, n)
    d = np.concatenate([[np.abs(row[1:]).sum() + 1.0], np.abs(col[1:]) + rng.uniform(0.5, 1.5, n - 1)])
    i = np.arange(1, n)
    a = sp.csc_matrix((np.concatenate([d, row[1:], col[1:]]),
                       (np.concatenate([np.arange(n), 0 * i, i]), np.concatenate([np.arange(n), i, 0 * i]))),
                      shape=(n, n))
    a.sort_indices()
    print("[case] arrow", n, flush=True)
    s = si.SelInv(n, a.indptr.astype(np.int64), a.indices.astype(np.int32), None, cap, 0, 0)
    c = np.diff(s.structure()["rl_ptr"])
    assert 8 * int(c.max()) ** 2 >= 1 << 31
    s.factor_device(torch.from_numpy(a.data).cuda())
    print("[case] factored", flush=True)
    L = s.info["nlevels"]
    got = {}
    for tile in (32, 64):
        s.set_tuning([4, L, 1, 0, 0, 0, 1, 0] + [0, 0, 0, 0] * (L - 1) + [tile, 0, 0, 0], "fp64")
        s.run("fp64")
        assert s.level_stats(L - 1)["tile35"] == tile
        got[tile] = s.get_selected()
        print("[case] tile", tile, flush=True)
    assert np.array_equal(got[32], got[64])
    # the inverse of an arrow matrix: z = 1 / (d_0 - sum row col / d)
    z = 1.0 / (d[0] - (row[1:] * col[1:] / d[1:]).sum())
    u, v = -z * row[1:] / d[1:], -z * col[1:] / d[1:]  # inverse's first row and column
    diag = np.concatenate([[z], 1.0 / d[1:] + col[1:] * row[1:] * z / d[1:] ** 2])
    # out[p] = A^{-1}(j, i) for the entry (i, j)
    ref = sp.csc_matrix((np.concatenate([diag, v, u]),
                         (np.concatenate([np.arange(n), 0 * i, i]), np.concatenate([np.arange(n), i, 0 * i]))),
                        shape=(n, n))
    ref.sort_indices()
    assert np.abs(got[64] - ref.data).max() / np.abs(ref.data).max() <= 1e-11
    s.close()
