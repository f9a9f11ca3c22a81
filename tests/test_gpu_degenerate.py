"""Degenerate and vanishing P-space blocks (needs an MI355X)."""
import sys

import numpy as np
import pytest

import workloads as W
from oracle import fci

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _log(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


def _atomic(n, u=4.0, t=0.0):
    """Hubbard chain in the site basis: diagonal degenerate, hopping t."""
    h = np.zeros((n, n))
    for i in range(n - 1):
        h[i, i + 1] = h[i + 1, i] = -t
    g = np.zeros((n,) * 4)
    for i in range(n):
        g[i, i, i, i] = u
    return h, g


@pytest.mark.parametrize("n,na,nb,t", [(4, 2, 2, 1e-9), (4, 2, 2, 1.0), (6, 3, 3, 1e-3),
                                       (8, 4, 4, 1e-9), (8, 4, 4, 1e-3), (8, 4, 4, 1.0)])
def test_equal_casci_of_a_batch_are_bitwise_equal(n, na, nb, t):
    """A hundred copies of one CASCI with a nearly degenerate P-space: the bracket
    of its lowest eigenvalue is one choice of the block, so all agree bit for
    bit, and none is below the oracle's ground state."""
    from paper_1910_03527_amd import Context
    _log("copies", n, t)
    h, g = _atomic(n, t=t)
    hd, gd = _dev(h), _dev(g)
    c = Context(0, conv_tol=1e-9)
    try:
        e = c.casci([hd] * 100, [gd] * 100, na, nb)
    finally:
        c.close()
    assert len(set(e)) == 1
    occ, every = list(range(na)), list(range(n))
    # exact whole-space P-spaces of n = 4, else an upper bound; conv_tol 1e-9
    # bounds the distance to an eigenvalue
    exact = fci.casci(h, g, 0.0, occ, every)
    assert e[0] >= exact - 1e-8
    if n == 4:
        assert e[0] <= exact + 1e-8
    if t <= 1e-3:  # the lowest multiplet: within 4 t^2 / U of zero per bond
        assert abs(e[0]) <= 4 * n * t * t + 1e-8


@pytest.mark.parametrize("n,na,nb,u", [(2, 1, 1, 0.0), (4, 2, 2, 0.0), (8, 4, 4, 0.0), (9, 4, 4, 0.0),
                                       (7, 3, 3, 4.0), (9, 4, 4, 4.0), (9, 2, 5, 4.0)])
def test_vanishing_pspace_block(n, na, nb, u):
    """No hopping: the P-space holds only determinants without a doubly occupied
    site, a block of zeros (for u = 0 the whole Hamiltonian vanishes).  The
    lowest energy is 0, exactly: every term of sigma on such a vector is."""
    from paper_1910_03527_amd import Context
    _log("vanishing block", n, na, nb, u)
    h, g = _atomic(n, u)
    c = Context(0)
    try:
        e = c.casci([_dev(h)], [_dev(g)], na, nb)[0]
        c.set_opts(precond=1)
        e1 = c.casci([_dev(h)], [_dev(g)], na, nb)[0]
    finally:
        c.close()
    assert abs(e) <= 1e-12 and abs(e1) <= 1e-12, (e, e1)
