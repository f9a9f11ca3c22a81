"""Kernels whose tiles, register blocks and size classes end raggedly (needs an
MI355X):

* sigma from string operators (up to 10 orbitals) at the shapes where its
  16-string blocks, wave tiles, LDS passes and empty strings meet their edges,
  through mbefci_sigma and mbefci_sigma_noalloc.  Bound, element by element:
  an entry of sigma is a sum of at most npair^2 products (pq|rs) D_pq,rs c plus
  the one-electron and diagonal terms, so K = npair^2 + 2 npair roundings of
  eps/2 each against |H| |c| on either side.
* P-space reductions at the ends of their size classes: the same energies as
  from unit-vector guesses to the sum of both solvers' quadratic errors
  (conv_tol^2 over a gap of at least 1e-3), far below the 1e-9 asserted, and no
  more sigma products (a wrong factor shows as lost iterations).
* RDMs at 7, 8, 12 and 13 orbitals, where the workgroup changes its size,
  against the oracle's for the same CI vector; sums of at most ndet products of
  determinant weights: ndet eps, times 8 for the products of links.
"""
import sys

import numpy as np
import pytest

import workloads as W
from oracle import fci, rdm

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
EPS = np.finfo(np.float64).eps


def _log(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


@pytest.fixture(scope="module")
def ctx():
    from paper_1910_03527_amd import Context
    c = Context(0)
    yield c
    c.close()


# (orbitals, alpha, beta electrons): one and two strings, the fewest and the
# most links, empty and full strings, 1..17 strings beside 16-string blocks,
# many alpha with few beta strings and the reverse, every LDS pass count
SIGMA = [(2, 1, 1), (2, 2, 1), (3, 0, 2), (3, 2, 1), (4, 2, 2), (4, 4, 1), (5, 1, 3), (5, 2, 0),
         (6, 3, 2), (6, 6, 3), (7, 1, 3), (7, 4, 0), (7, 4, 6), (8, 4, 1), (8, 0, 4), (8, 3, 3),
         (9, 1, 4), (9, 4, 1), (9, 8, 2), (9, 3, 3), (10, 1, 1), (10, 9, 1), (10, 1, 5),
         (10, 5, 1), (10, 0, 5), (10, 2, 3)]


@pytest.mark.parametrize("n,na,nb", SIGMA)
def test_sigma_of_ragged_shapes(ctx, n, na, nb):
    _log("string sigma", n, na, nb)
    h, g = W.synthetic(n, 4000 + 100 * n + 10 * na + nb)
    H = fci.hamiltonian(h, g, 0.5, fci.string_masks(range(n), na), fci.string_masks(range(n), nb))
    c = np.random.default_rng(n + na).standard_normal(H.shape[0])
    npair = n * (n + 1) // 2
    bound = (npair * npair + 2 * npair) * EPS * (abs(H) @ abs(c))
    got = ctx.sigma(_dev(h), _dev(g), na, nb, _dev(c), 0.5).cpu().numpy()
    out = torch.full((c.size,), float("nan"), dtype=torch.float64, device="cuda")
    noalloc = ctx.sigma_noalloc(_dev(h), _dev(g), na, nb, _dev(c), out, 0.5).cpu().numpy()
    assert np.all(abs(got - H @ c) <= bound)
    assert np.all(abs(noalloc - H @ c) <= bound)


@pytest.mark.parametrize("n,na,nb,pspace", [(8, 4, 4, 24), (8, 4, 4, 48), (8, 4, 4, 49),
                                            (8, 4, 4, 76), (9, 4, 4, 80), (9, 4, 4, 81),
                                            (9, 4, 4, 112), (7, 3, 4, 112)])
def test_pspace_size_classes(n, na, nb, pspace):
    from paper_1910_03527_amd import Context
    _log("pspace class", n, na, nb, pspace)
    h, g = W.synthetic(n, 900 + n)
    res = []
    for p in (0, pspace):
        c = Context(0, pspace=p)
        e = c.casci([_dev(h)], [_dev(g)], na, nb)[0]
        res.append((e, c.last_stats["sigma_calls"]))
        c.close()
    assert abs(res[0][0] - res[1][0]) < 1e-9
    assert res[1][1] <= res[0][1], res


@pytest.mark.parametrize("n,na,nb", [(7, 3, 2), (8, 2, 3), (12, 1, 2), (13, 1, 2)])
def test_rdm_workgroup_sizes(ctx, n, na, nb):
    _log("rdm", n, na, nb)
    h, g = W.synthetic(n, 60 + n)
    r = ctx.casci_one(_dev(h), _dev(g), na, nb, want_ci=True, want_rdm=True)
    am, bm = fci.string_masks(range(n), na), fci.string_masks(range(n), nb)
    c = r["ci"].cpu().numpy().reshape(len(am), len(bm))
    d1, d2 = rdm.rdm12(am, bm, c, n)
    tol = 8 * c.size * EPS
    assert np.max(abs(r["rdm1"].cpu().numpy() - d1)) <= tol
    assert np.max(abs(rdm.sym8(r["rdm2"].cpu().numpy()) - rdm.sym8(d2))) <= tol
