"""The launch choices a handle makes by itself (no tuning table) and the
tuner's return to them.  Marked gpu."""
import numpy as np
import pytest

from workloads import config_grid

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def si():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1708_04539_amd import selinv
    return selinv


def grid(si, dims, cap, leaf=64):
    w = config_grid("p", dims, "box", "sym_perturbed", 0.1, 3, cap, leaf, delta=0.15)
    return w, si.SelInv(w.n, w.colptr, w.rowind, w.perm, w.max_super, w.relax, w.pad_pct)


def in_place_levels(s):
    return [d for d in range(s.info["nlevels"]) if s.level_stats(d)["gather_fused"] == 2]


# a tuning that ends with the size policy installs a table that runs it: the
# levels the policy reads in place, and its side stream (only on the larger
# grid).  The tuner's timings decide whether a call ends there, so it is called
# until one does.
@pytest.mark.parametrize("dims,cap,forks", [((64, 64), 64, False), ((256, 256), 128, True)], ids=["64x64", "256x256"])
def test_kept_policy_runs_the_policy(si, dims, cap, forks):
    import torch
    w, s = grid(si, dims, cap)
    s.factor(w.values)
    s.run("fp64")
    want = in_place_levels(s)
    assert want
    x = s.get_selected()
    L = s.info["nlevels"]
    st = torch.cuda.Stream()
    for k in range(60):
        print("[case] tune", dims, k, flush=True)
        ms_policy, ms_tuned = s.tune("fp64", reps=1, stream=st)
        t = s.get_tuning("fp64")
        if not any(t[3:6]) and not any(t[8 + 4 * d] or t[9 + 4 * d] for d in range(L)):
            break
    else:
        pytest.skip("every tuning was faster than the policy")
    assert ms_tuned == ms_policy
    assert [d for d in range(L) if t[11 + 4 * d]] == want
    assert t[6] == (0 if forks else 1)
    s.run("fp64")
    assert in_place_levels(s) == want and np.array_equal(s.get_selected(), x)


# the levels read in place by default take their codes from the gather's own
# array: no allocation of one code per entry of every G_K, whose failure (a
# bounded hook) would fail a run that a stored G can do without it
def test_in_place_levels_need_no_code_array(si):
    import torch
    print("[case] in-place levels under a bounded hook", flush=True)
    refuse = []

    def alloc(nbytes):
        if any(r <= nbytes < r + 64 for r in refuse):
            return None
        return torch.cuda.caching_allocator_alloc(nbytes, torch.cuda.current_device())

    si.set_allocator("custom", alloc=alloc, free=torch.cuda.caching_allocator_delete)
    try:
        w, s = grid(si, (96, 80), 64, 32)
        s.factor(w.values)
        st = s.structure()
        refuse.append(4 * int((np.diff(st["rl_ptr"]) * np.diff(st["ru_ptr"])).sum()))
        s.run("fp64")
        assert in_place_levels(s)
        x = s.get_selected()
        for form in ("stored", "in_products"):
            s.set_gather_form(form)
            s.run("fp64")
            assert np.array_equal(s.get_selected(), x)
        s.close()
    finally:
        si.set_allocator("torch")


def chains(parts):
    """Independent band matrices, `count` of n columns coupled at distances 1
    and c: natural order gives each a chain of supernodes with about c rows."""
    import scipy.sparse as sp
    blocks = []
    for count, n, c in parts:
        r = np.random.default_rng(n + c)
        offs = [-c, -1, 0, 1, c]
        m = sp.diags([r.uniform(-1, 0, n - abs(k)) if k else np.full(n, 5.0) for k in offs], offs)
        blocks += [m] * count
    a = sp.block_diag(blocks, format="csc")
    a.sort_indices()
    return a.shape[0], a.indptr.astype(np.int64), a.indices.astype(np.int32), a.data


def level_shapes(s):
    """Per level: supernodes, widest, largest c, mean and size-weighted mean of c_L c_U."""
    st = s.structure()
    w, cl, cu = np.diff(st["xsup"]), np.diff(st["rl_ptr"]), np.diff(st["ru_ptr"])
    out = []
    for d in range(s.info["nlevels"]):
        k = (st["level"] == d) & (cl + cu > 0)
        g = (cl[k] * cu[k]).astype(float)
        out.append((k.sum(), w[k].max(initial=0), max(cl[k].max(initial=0), cu[k].max(initial=0)),
                    g.mean() if k.any() else 0.0, (g * g).sum() / g.sum() if k.any() else 0.0))
    return out


# long products read G_K in place only where that is faster: the mixed forms not
# beyond c = 160, nor where the gather's tiles are whole blocks (s = 64); FP64
# not beyond 320 on levels of a few supernodes
@pytest.mark.parametrize("parts,cap,prec,want", [
    ([(1, 500, 200)], 32, "mixed_fp32", False), ([(1, 500, 200)], 32, "mixed_bf16x3", False),
    ([(1, 500, 200)], 32, "fp64", True), ([(1, 292, 100)], 32, "mixed_fp32", True),
    ([(4, 500, 120)], 64, "mixed_fp32", False), ([(4, 500, 120)], 48, "mixed_fp32", True),
    ([(1, 900, 400)], 64, "fp64", False), ([(8, 900, 400)], 64, "fp64", True)])
def test_in_place_by_product_length(si, parts, cap, prec, want):
    print("[case] in place", parts, cap, prec, flush=True)
    n, cp, ri, v = chains(parts)
    s = si.SelInv(n, cp, ri, None, cap, cap, 100).factor(v)
    s.run(prec)
    c = parts[0][2]
    shapes = level_shapes(s)
    full = [d for d, x in enumerate(shapes) if x[2] >= c and x[1] == cap]
    got = in_place_levels(s)
    assert full and all((d in got) == want for d in full), (got, shapes)
    x = s.get_selected()
    for form in ("stored", "in_products"):
        s.set_gather_form(form)
        s.run(prec)
        assert np.array_equal(s.get_selected(), x)


# a level of many thin supernodes and a few with a large G_K: the few take most
# of the time, so the mixed forms weigh each G_K by its size
@pytest.mark.parametrize("prec", ["mixed_fp32", "mixed_bf16x3", "fp64"])
def test_in_place_weighs_g_by_size(si, prec):
    import torch
    print("[case] in place, few large G_K among many", prec, flush=True)
    n, cp, ri, v = chains([(900, 64 * 3 + 70, 70), (24, 64 * 3 + 250, 250)])
    s = si.SelInv(n, cp, ri, None, 64, 64, 100).factor_device(torch.from_numpy(v).cuda())
    s.run(prec)
    shapes = level_shapes(s)
    d = [d for d, x in enumerate(shapes) if x[0] > 900 and x[3] < 6500 < 9000 < x[4]]
    assert d
    got = in_place_levels(s)
    assert all((k in got) == (prec == "fp64") for k in d), (got, shapes)
    x = s.get_selected()
    s.set_gather_form("stored")
    s.run(prec)
    assert np.array_equal(s.get_selected(), x)
