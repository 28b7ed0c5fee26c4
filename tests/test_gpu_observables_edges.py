"""Observables at the edges of their kernels' tiles, against the CPU oracle.

Tolerance: both sides sum FP64 values with compensation; a chain's Rg^2 comes
from sums about its first bead, which lose at most the factor N + 1 <= 129 of
the FP64 rounding (129 * 2^-53 * a few operations < 1e-13), so 1e-12 relative.
"""
import numpy as np
import pytest

from paper_2606_09356_amd import workloads as W
from tests.test_gpu_parity import make_pair

pytestmark = pytest.mark.gpu
KEYS = ("Re2", "Re2_err", "Rg2", "Rg2_err", "Ebond_per_chain", "Enb_per_chain")


def check(g, orcs):
    for k, o in enumerate(orcs):
        a, b, c = g.observables(k), o.observables(), g.observables(k)
        for key in KEYS:
            assert abs(a[key] - b[key]) <= 1e-12 * max(1.0, abs(b[key])), (k, key, a[key], b[key])
        assert a == c          # a second call repeats the first bit for bit


# one chain, lanes just below and above a wave, two chains per wave with a
# ragged last tile, odd and even ends; cell counts that leave 1..3 cells over
@pytest.mark.parametrize("r,cw", [("f32", 16), ("cell", 32), ("cell", 16)])
@pytest.mark.parametrize("N,chains,grid", [(2, 1, (4, 4, 4)), (2, 129, (5, 5, 5)), (3, 33, (5, 5, 7)), (31, 5, (4, 5, 9)),
                                           (64, 3, (6, 5, 5)), (65, 7, (7, 7, 7)), (128, 2, (5, 7, 5)),
                                           (33, 700, (23, 21, 25))])
def test_observables_at_tile_edges(N, chains, grid, r, cw):
    s = W.diblock_system(chains, N, 0.5, 20.0, 50.0, tuple(0.23 * g for g in grid), grid)
    t = W.diblock_system(chains + 1, N, 0.5, 10.0, 30.0, tuple(0.25 * g for g in grid), grid, ham_form=1)
    g, orcs = make_pair([s, t], r, cw, reorder_every=1)
    check(g, orcs)
    g.close()


def test_observables_of_more_tiles_than_the_grid_holds():
    """More wave tiles than waves of the resident grid (1280 blocks of four)."""
    s = W.diblock_system(6000, 100, 0.5, 20.0, 50.0, (17.0, 17.0, 17.0), (68, 68, 67))
    g, orcs = make_pair([s], "f32", 16)
    check(g, orcs)
    g.close()


@pytest.mark.parametrize("r", ["f32", "cell"])
def test_observables_far_from_the_origin(r):
    """A chain's sums are taken about its first bead, so images cost no precision."""
    s = W.diblock_system(50, 40, 0.5, 20.0, 50.0, (2.0, 2.0, 2.0), (8, 8, 8))
    xyz = W.gaussian_walks(s, seed=9) + 4.0e4
    g, orcs = make_pair([s], r, 16)
    g.set_positions(0, xyz)
    orcs[0].set_positions(xyz)
    a, b = g.observables(0), orcs[0].observables()
    # the oracle sums positions of 4e4 (2^-53 * 4e4 * 2 per coordinate difference)
    for key in KEYS:
        assert abs(a[key] - b[key]) <= 1e-9 * max(1.0, abs(b[key])), (key, a[key], b[key])
    g.close()
    assert np.isfinite(list(a.values())).all()
