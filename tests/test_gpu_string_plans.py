"""What surrounds the sigma of up to 10 orbitals: the shapes without string
operators, and how plans lay out, schedule and bound its operands (needs an
MI355X)."""
import ctypes
import sys

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
EPS = np.finfo(np.float64).eps


def _log(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("n,na,nb", [(0, 0, 0), (1, 0, 0), (1, 1, 0), (1, 1, 1)])
def test_noalloc_sigma_of_no_and_one_orbital(n, na, nb):
    """mbefci_sigma_noalloc of 0 and 1 orbitals (one determinant each): H_00 c
    = (e_core + na h + nb h + na nb (00|00)) c.  The pointers are not null
    (the library reads nothing through them for 0 orbitals)."""
    from paper_1910_03527_amd import Context
    _log("noalloc", n, na, nb)
    h, g, c, out = _dev([0.75]), _dev([0.5]), _dev([2.0]), _dev([float("nan")])
    ctx = Context(0)
    try:
        rc = ctx._L.mbefci_sigma_noalloc(
            ctx._h, n, na, nb, *(ctypes.c_void_p(t.data_ptr()) for t in (h, g)), 0.25,
            *(ctypes.c_void_p(t.data_ptr()) for t in (c, out)), ctx._stream())
        assert rc == 0
        torch.cuda.synchronize()
        # exact in double precision
        assert float(out[0]) == 2.0 * (0.25 + 0.75 * (na + nb) + 0.5 * na * nb)
    finally:
        ctx.close()


def test_small_plan_leaves_the_units_of_larger_ones_open(tmp_path):
    """One CASCI has one length of work unit: the tuner keeps its tile width and
    times a batch of the same size anew; the energies are the same bit for bit
    (identical problems, and the order of every sum is fixed)."""
    from paper_1910_03527_amd import Context
    cache = tmp_path / "tune.txt"
    h, g = W.synthetic(8, 31)
    hd, gd = _dev(h), _dev(g)

    def entry():
        return [int(x) for x in cache.read_text().splitlines()[-1].split()]

    c = Context(0, tune_cache=str(cache))
    try:
        _log("tune one CAS(8,8)")
        e1 = c.casci([hd], [gd], 4, 4)[0]
        n, _, steps = entry()
        assert (n, steps) == (8, -1)  # 70 strings: one step per unit
        ms = c.last_stats["ms_tune"]
        c.casci([hd], [gd], 4, 4)
        assert c.last_stats["ms_tune"] - ms < 1.0  # kept
        _log("tune 400 CAS(8,8)s")
        e = c.casci([hd] * 400, [gd] * 400, 4, 4)
        n, _, steps = entry()
        assert n == 8 and (steps >= 4 or steps <= -5)
        assert all(x == e1 for x in e)
    finally:
        c.close()
    # read back and kept by the same plan
    _log("reread")
    c = Context(0, tune_cache=str(cache))
    try:
        assert all(x == e1 for x in c.casci([hd] * 400, [gd] * 400, 4, 4))
        assert entry() == [n, entry()[1], steps]
    finally:
        c.close()


# CASCIs, sigma_pass_mb and a cap (bytes) that held them when sigma contracted
# every pair (W and G of the workspace instead of string Hamiltonians)
@pytest.mark.parametrize("n,na,nb,count,pass_mb,cap", [
    (10, 5, 0, 64, 0, 17197056), (10, 5, 1, 64, 1, 29999104), (9, 4, 0, 100, 0, 18319360),
    (9, 4, 4, 24, 1, 53829632), (4, 1, 2, 500, 1, 61396992), (10, 1, 0, 100, 0, 15620096)])
def test_workspace_cap_holds_what_it_held(n, na, nb, count, pass_mb, cap):
    """Plans whose string Hamiltonians are more than a cap leaves room for form
    them pass by pass: the energies of an uncapped solve bit for bit, batched
    and one launch sequence per CASCI."""
    from paper_1910_03527_amd import BATCHED, Context, PER_LAUNCH
    _log("cap", n, na, nb, count)
    hg = [W.synthetic(n, 50 + i) for i in range(3)]
    hs = [_dev(hg[i % 3][0]) for i in range(count)]
    gs = [_dev(hg[i % 3][1]) for i in range(count)]
    res = []
    for kw in ({}, dict(max_workspace=cap, sigma_pass_mb=pass_mb)):
        c = Context(0, mode=BATCHED, **kw)
        try:
            res.append(c.casci(hs, gs, na, nb))
            if kw and count <= 64:
                c.set_opts(mode=PER_LAUNCH)
                assert c.casci(hs, gs, na, nb) == res[0]
        finally:
            c.close()
    assert res[0] == res[1]


def test_expansion_with_operands_formed_in_passes():
    """An expansion of 6 to 10 orbitals in sigma passes of 1 MiB under a cap
    (2.1 GB of it for vectors and RDM partials): energies, increments and
    gradients of the uncapped one bit for bit.  A cap with room changes nothing."""
    from paper_1910_03527_amd import Context
    p = W.problem("hubbard16")
    h, g = _dev(p.h1), _dev(p.eri)
    res = []
    for kw in ({}, dict(max_workspace=2300 << 20, sigma_pass_mb=1),
               dict(max_workspace=16 << 30, sigma_pass_mb=1)):
        _log("expansion", kw)
        c = Context(0, tile=64, **kw)
        try:
            r = c.mbe_forward(h, g, p.occ, p.ref, p.exp, p.max_order, want_increments=True)
            dh, dg = c.mbe_backward([1.0] * (p.max_order + 1))
            names = {k["name"] for k in c.time_kernels(reps=1)}
            res.append((r["e_total"], r["increments"], dh.cpu().numpy(), dg.cpu().numpy()))
        finally:
            c.close()
        assert ("sigma_operands" in names) == (kw.get("max_workspace") == 2300 << 20), names
    for r in res[1:]:
        assert r[0] == res[0][0] and r[1] == res[0][1]
        assert np.array_equal(r[2], res[0][2]) and np.array_equal(r[3], res[0][3])


def test_cap_counts_the_plan_in_hand_only():
    """Under a cap a plan's G and W give way to the next plan's: a batch of
    252 x 1 strings (its operands are most of the workspace), then one CASCI of
    12 orbitals (its G is), under the largest of what either takes alone."""
    from paper_1910_03527_amd import Context
    h, g = (_dev(x) for x in W.synthetic(10, 51))
    h12, g12 = (_dev(x) for x in W.synthetic(12, 52))
    ref = Context(0, conv_tol=1e-3)
    want = [ref.casci([h] * 400, [g] * 400, 5, 0), ref.casci([h12], [g12], 5, 2)]
    ref.close()
    # the batch takes 100 MB in passes, G of 12 orbitals (78 rows of 792 x 66
    # strings) 33 MB
    c = Context(0, conv_tol=1e-3, max_workspace=120 << 20)
    try:
        for _ in range(2):
            _log("batch, then 12 orbitals")
            assert c.casci([h] * 400, [g] * 400, 5, 0) == want[0]
            assert c.casci([h12], [g12], 5, 2) == want[1]
    finally:
        c.close()


def test_probed_mfma_peak_is_that_of_the_faster_form():
    """Independent chains of the 16x16x4 form end at 50 TFLOP/s, of the 4x4x4
    form (which sigma of up to 10 orbitals issues) at 65 to 78.6."""
    from paper_1910_03527_amd import Context
    _log("probe")
    c = Context(0)
    try:
        assert 55.0 < c.probe_peaks()["fp64_mfma_tflops"] < 80.0
    finally:
        c.close()
