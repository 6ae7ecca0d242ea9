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
