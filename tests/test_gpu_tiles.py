"""Product tiles of the grouped GEMM at the sizes where they can go wrong:
operands one short of, at and one past the edges of the tiles (64, 128) and of
the k chunks (16, 32), down to single rows and columns.  Marked gpu.

The 32-wide tiles stage their operands through registers; the wider FP64 and
FP32 ones load them straight into LDS.  Every entry sums the same products in
the same order in both, so the results are compared bit for bit, and with the
oracle at the parity bar."""
import numpy as np
import pytest

from oracle import Oracle
from workloads import random_sparse

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-11, "mixed_fp32": 1e-5, "mixed_bf16x3": 1e-5}


def table(levels, tile):
    """Tuning table with one tile edge on every launch class, per-phase launches."""
    return [4, levels, 1, tile, tile, tile, 0, 0] + [tile, tile, 1, 0] * levels


# Only sum(sizes) enters the matrix below, a random pattern that fills in: its
# supernodes are as wide as the cap, the last one the remainder.  Chosen widths
# and sets, several in one launch, are in test_gpu_tile_shapes.py.
def split_matrix(sizes, seed):
    """Dense diagonal blocks of the given sizes, each coupled to all later
    ones: supernode k has sizes[k] columns and c = sum(sizes[k+1:])."""
    n = sum(sizes)
    return random_sparse(n, 0.7, seed)


# supernode widths from the first (deepest) to the root; c_L = c_U is the sum
# of the widths that follow
SIZES = [
    (1, 1, 1),
    (15, 16, 17, 1),
    (31, 33, 32, 63),
    (65, 63, 64, 1),
    (64, 129, 127, 2),
    (200, 3, 130, 61),
    (48, 80, 112, 16, 96),
]


@pytest.mark.parametrize("sizes", SIZES, ids=["_".join(map(str, s)) for s in SIZES])
@pytest.mark.parametrize("prec", ["fp64", "mixed_fp32", "mixed_bf16x3"])
def test_tile_widths_agree(sizes, prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1708_04539_amd import selinv as si
    cap = max(sizes)
    got = {}
    for tile in (32, 64, 128):
        # one matrix per supernode width as the cap, so that every width and
        # every remainder of it occurs
        for c in sorted(set(sizes)):
            print("[case]", sizes, prec, "tile", tile, "cap", c, flush=True)
            cp, ri, v, _ = split_matrix(sizes, 11)
            s = si.SelInv(sum(sizes), cp, ri, None, c, 0, 100)
            s.factor(v)
            s.set_tuning(table(s.info["nlevels"], tile), prec)
            s.run(prec)
            r, col, x = s.export(sort=False)
            if tile == 32:
                o = Oracle(sum(sizes), cp, ri, None, c, 0, 0, 100).factor(v).selinv()
                got[c] = x
                r2, c2, ref = o.export()
                k = np.lexsort((r, col))
                assert np.array_equal(r[k], r2) and np.array_equal(col[k], c2)
                assert np.abs(x[k] - ref).max() / np.abs(ref).max() <= TOL[prec]
            else:
                assert np.array_equal(x, got[c])
            s.close()
    assert cap in got


# diagonal tiles of the device LU: one 64-wide block in 16-column panels, its
# last panel ragged, and a second block
@pytest.mark.parametrize("n", [1, 15, 16, 17, 32, 33, 48, 63, 64, 65, 81, 129])
def test_device_lu_tile_edges(n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1708_04539_amd import selinv as si
    print("[case] device LU, one dense block of", n, flush=True)
    cp, ri, v, _ = random_sparse(n, 1.0, n)
    s = si.SelInv(n, cp, ri, None, n, n, 0)
    assert s.info["max_s"] == n
    s.factor_device(torch.from_numpy(v).cuda())
    s.run("fp64")
    r, c, x = s.export()
    o = Oracle(n, cp, ri, None, n, n, 0, 0).factor(v).selinv()
    r2, c2, ref = o.export()
    assert np.array_equal(r, r2) and np.array_equal(c, c2)
    assert np.abs(x - ref).max() / np.abs(ref).max() <= TOL["fp64"]


@pytest.mark.parametrize("k", [0, 15, 16, 40, 63, 64, 79])
def test_device_lu_names_the_first_zero_pivot(k):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1708_04539_amd import selinv as si
    print("[case] device LU, zero pivot at", k, flush=True)
    n = 80
    a = np.full((n, n), 0.25) + np.diag(np.full(n, float(n)))
    a[k, :] = 0.0  # an exactly zero row of the block: its pivot is zero whatever precedes it
    cp = np.arange(0, n * n + 1, n, dtype=np.int64)
    ri = np.tile(np.arange(n, dtype=np.int32), n)
    s = si.SelInv(n, cp, ri, None, n, n, 0)
    with pytest.raises(si.SelinvError) as e:
        s.factor_device(torch.from_numpy(a.T.ravel().copy()).cuda())
    assert e.value.status == "ZERO_PIVOT" and f"permuted column {k} " in str(e.value)


# the level sweep's own choices (no tuning): level launches at every size, the
# prologue of the lower levels forked or not; neither changes a result
@pytest.mark.parametrize("dims,cap", [((5, 4), 8), ((45, 165), 139), ((77, 81), 128), ((160, 150), 96)],
                         ids=["5x4", "45x165", "77x81", "160x150"])
@pytest.mark.parametrize("prec", ["fp64", "mixed_fp32"])
def test_policy_sweep_equals_plain_levels(dims, cap, prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1708_04539_amd import selinv as si
    from workloads import config_grid
    print("[case] sweep policy", dims, prec, flush=True)
    w = config_grid("p", dims, "box", "sym_perturbed", 0.1, 0, cap, 64, delta=0.15)
    s = si.SelInv(w.n, w.colptr, w.rowind, w.perm, w.max_super, w.relax, w.pad_pct).factor(w.values)
    st = torch.cuda.Stream()
    s.run(prec, stream=st)
    assert s.sweep_is_persistent(prec) == 0
    _, _, x = s.export(sort=False)
    for _ in range(3):
        s.run(prec, stream=st, graph=True)
        _, _, g = s.export(sort=False)
        assert np.array_equal(x, g)
    L = s.info["nlevels"]
    for fork in (0, 1):  # side stream from the first wide level on, none
        s.set_tuning([4, L, 1, 0, 0, 0, fork, 0] + [0, 0, 0, 0] * L, prec)
        s.run(prec, stream=st)
        _, _, y = s.export(sort=False)
        assert np.array_equal(x, y)


# G_K read in place by the level sweep's own choice (no tuning) against a stored
# G: the sides of the choice (s and c around one tile, 32- and 64-wide tiles,
# plans with and without codes for every G_K)
@pytest.mark.parametrize("dims,cap,budget", [((9, 7), 16, -1), ((64, 64), 64, -1), ((128, 96), 130, -1),
                                             ((200, 200), 32, -1), ((64, 64), 64, 0), ((64, 64), 64, 5000)],
                         ids=["9x7", "64x64", "128x96", "200x200", "64x64-maps", "64x64-some"])
@pytest.mark.parametrize("prec", ["fp64", "mixed_fp32", "mixed_bf16x3"])
def test_policy_in_place_levels(dims, cap, budget, prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1708_04539_amd import selinv as si
    from workloads import config_grid
    print("[case] in-place levels", dims, cap, budget, prec, flush=True)
    w = config_grid("p", dims, "box", "sym_perturbed", 0.1, 3, cap, 32, delta=0.15)
    s = si.SelInv(w.n, w.colptr, w.rowind, w.perm, w.max_super, w.relax, w.pad_pct)
    s.set_gather_code_budget(budget)
    s.factor(w.values)
    s.run(prec)
    _, _, x = s.export(sort=False)
    L = s.info["nlevels"]
    in_place = [d for d in range(L) if s.level_stats(d)["gather_fused"] == 2]
    # (9x7: every level is made of small supernodes and keeps G_K in LDS)
    assert bool(in_place) == (budget < 0 and dims != (9, 7))
    s.set_gather_form("stored")
    s.run(prec)
    assert not any(s.level_stats(d)["gather_fused"] == 2 for d in range(L))
    _, _, y = s.export(sort=False)
    assert np.array_equal(x, y)


# 64x64 gather tiles whose rows share one supernode and whose columns share
# one (all three blocks they can come from, full and ragged) beside those that
# straddle supernodes: read through the maps, the source codes, and against
# the oracle
@pytest.mark.parametrize("n,density,cap", [(400, 0.01, 64), (400, 0.01, 65), (400, 0.01, 130), (330, 0.7, 64),
                                           (330, 0.7, 63), (330, 0.7, 129), (449, 0.004, 200)])
@pytest.mark.parametrize("prec", ["fp64", "mixed_fp32", "mixed_bf16x3"])
def test_gather_tiles_of_one_supernode(n, density, cap, prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1708_04539_amd import selinv as si
    print("[case] gather tiles", n, density, cap, prec, flush=True)
    cp, ri, v, _ = random_sparse(n, density, 5)
    o = Oracle(n, cp, ri, None, cap, 0, 0, 100).factor(v).selinv()
    r2, c2, ref = o.export()
    got = []
    for budget in (0, -1):
        s = si.SelInv(n, cp, ri, None, cap, 0, 100)
        s.set_gather_code_budget(budget)
        s.factor(v)
        for form in ("stored", "auto"):
            s.set_gather_form(form)
            s.run(prec)
            r, c, x = s.export(sort=False)
            got.append(x)
        s.close()
    k = np.lexsort((r, c))
    assert np.array_equal(r[k], r2) and np.array_equal(c[k], c2)
    assert np.abs(got[0][k] - ref).max() / np.abs(ref).max() <= TOL[prec]
    for x in got[1:]:
        assert np.array_equal(x, got[0])


# small supernodes handled whole by one workgroup: operand edges at and beside
# the blocks of 16 (k and rows) and 32 (split-BF16 k chunks), against the
# per-phase launches bit for bit and the oracle
@pytest.mark.parametrize("n,density,cap", [(2, 1.0, 1), (17, 1.0, 16), (33, 1.0, 17), (49, 1.0, 15), (65, 1.0, 1),
                                           (80, 1.0, 33), (97, 1.0, 48), (127, 1.0, 63), (128, 1.0, 64),
                                           (120, 0.02, 64), (128, 0.02, 5)])
@pytest.mark.parametrize("prec", ["fp64", "mixed_fp32", "mixed_bf16x3"])
def test_small_supernodes_equal_the_per_phase_launches(n, density, cap, prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1708_04539_amd import selinv as si
    print("[case] small supernodes", n, density, cap, prec, flush=True)
    cp, ri, v, _ = random_sparse(n, density, 7)
    s = si.SelInv(n, cp, ri, None, cap, 0, 100)
    s.factor(v)
    s.run(prec)
    assert sum(s.level_stats(d)["small_count"] for d in range(s.info["nlevels"])) > 0
    r, c, x = s.export(sort=False)
    s.set_tuning(table(s.info["nlevels"], 32), prec)
    s.run(prec)
    assert sum(s.level_stats(d)["small_count"] for d in range(s.info["nlevels"])) == 0
    assert np.array_equal(s.export(sort=False)[2], x)
    s.close()
    r2, c2, ref = Oracle(n, cp, ri, None, cap, 0, 0, 100).factor(v).selinv().export()
    k = np.lexsort((r, c))
    assert np.array_equal(r[k], r2) and np.array_equal(c[k], c2)
    assert np.abs(x[k] - ref).max() / np.abs(ref).max() <= TOL[prec]
