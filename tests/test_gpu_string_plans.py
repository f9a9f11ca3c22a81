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
