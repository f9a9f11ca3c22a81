"""Sigma of up to 10 orbitals in plans large enough for its large tiles and long
work units (needs an MI355X).

One CASCI takes 16 x 16 same-spin tiles and one step of alpha strings per unit.
Plans of at least 2,048 tiles of 32 x 64 strings take those, and units hold
several steps as soon as that leaves 1,024 of them: the links, integral rows and
C rows of the next strings are then carried from step to step.  Here both run
with unequal spins (a string Hamiltonian of its own for each, padded by
itself), for the shortest and the longest lists of links, ragged last tiles and
ragged last units.  The order of every sum is the same in every form, so
energies and CI vectors equal those of single CASCIs bit for bit; single CASCIs
are compared with the oracle's H element by element.

Bound of that comparison: an entry of sigma is a chain of at most K = Na + Nb +
2 (1 + na (n - na)) + 2 (1 + nb (n - nb)) additions and products, each rounded by
at most eps / 2 of a partial sum that is at most |H| |c|.  Independent roundings
add like sqrt(K); six standard deviations (eps / sqrt(12) each at most).
"""
import sys
from math import comb

import numpy as np
import pytest

import workloads as W
from oracle import fci

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
EPS = np.finfo(np.float64).eps


def _log(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


def _count(n, na, nb):
    """CASCIs for 2,048 large tiles and units of at least three steps."""
    tiles = -(-comb(n, na) // 32) * -(-comb(n, nb) // 64)
    return max(-(-2048 // tiles), -(-3 * 4 * 1024 // comb(n, na)))


SHAPES = [(5, 1, 3), (6, 2, 3), (7, 2, 4), (8, 2, 5), (8, 4, 1), (9, 2, 5), (9, 5, 2), (10, 1, 4),
          (10, 5, 2), (10, 2, 5), (10, 4, 5)]


# every width compiled for the size (128 columns not for 8 and 9 orbitals, one
# wave per string up to 9)
CASES = [(*s, t) for s in SHAPES for t in (32, 64, 128, -32, -64)
         if not (t == 128 and s[0] in (8, 9)) and not (t < 0 and s[0] > 9)]


@pytest.mark.parametrize("n,na,nb,tile", CASES)
def test_batches_of_unequal_spins(tmp_path, n, na, nb, tile):
    from paper_1910_03527_amd import Context
    count = _count(n, na, nb)
    _log("batch", n, na, nb, tile, count)
    cache = tmp_path / "tune.txt"
    cache.write_text(f"{n} {tile} 16\n")
    hg = [tuple(_dev(x) for x in W.synthetic(n, 7100 + 10 * n + i)) for i in range(3)]
    one = Context(0)
    c = Context(0, tune_cache=str(cache))
    try:
        ref = [one.casci([h], [g], na, nb, want_ci=True) for h, g in hg]
        es, cis = c.casci([hg[i % 3][0] for i in range(count)], [hg[i % 3][1] for i in range(count)],
                          na, nb, want_ci=True)
        assert c.last_stats["ms_tune"] < 50.0  # the forced schedule
        assert all(es[i] == ref[i % 3][0][0] for i in range(count))
        assert all(torch.equal(cis[i], ref[i % 3][1][0]) for i in range(count))
    finally:
        one.close()
        c.close()


@pytest.mark.parametrize("n,na,nb", [(5, 1, 3), (7, 2, 4), (8, 4, 4), (9, 5, 2), (9, 4, 4), (10, 2, 5),
                                     (10, 5, 2), (10, 3, 3)])
def test_sigma_to_rounding(n, na, nb):
    from paper_1910_03527_amd import Context
    _log("sigma", n, na, nb)
    h, g = W.synthetic(n, 7100 + 10 * n)
    H = fci.hamiltonian(h, g, 0.5, fci.string_masks(range(n), na), fci.string_masks(range(n), nb))
    c = np.random.default_rng(n).standard_normal(H.shape[0])
    want = H.astype(np.longdouble) @ c.astype(np.longdouble)
    K = comb(n, na) + comb(n, nb) + 2 * (1 + na * (n - na)) + 2 * (1 + nb * (n - nb))
    bound = 6.0 * np.sqrt(K / 12.0) * EPS * (abs(H) @ abs(c))
    ctx = Context(0)
    try:
        got = ctx.sigma(_dev(h), _dev(g), na, nb, _dev(c), 0.5).cpu().numpy()
    finally:
        ctx.close()
    assert np.all(abs(got - want) <= bound), float(np.max(abs(got - want) / bound))
