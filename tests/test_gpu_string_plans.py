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
