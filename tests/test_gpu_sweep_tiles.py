"""Sweep parity at the edges of its tiles and lists, against the CPU oracle.

Bars as in the parity tests: counts bit-exact, stored state equal for every
bead (a decision mismatch needs an FP32 energy rounding next to u, at most
one in 1e6; these systems have fewer than 2e4 beads).
"""
import numpy as np
import pytest

from paper_2606_09356_amd import workloads as W
from paper_2606_09356_amd.soma import Soma
from tests.test_gpu_parity import SEED, make_pair, same_state

pytestmark = pytest.mark.gpu


def ragged(N, chains, edge=0.23, chiN=30.0):
    """A system on a grid of unequal, non-dyadic cells at about two beads per cell."""
    m = max(4, int(round((N * chains / 2.0) ** (1.0 / 3.0))))
    grid = (m, m + 1, max(4, m - 1))
    return W.diblock_system(chains, N, 0.4, chiN, 45.0, tuple(edge * g for g in grid), grid)


def check_sweeps(g, orcs, sweeps=2):
    for s in range(sweeps):
        g.sweep(1)
        for k, o in enumerate(orcs):
            o.sweep(SEED, s)
            o.density()
            o.fields()
            assert (g.density(k) == o.counts).all(), (k, s)
            assert same_state(g, k, o).all(), (k, s)


# chain counts around the tile capacities: one chain, one tile less or more
# than full, lanes ending on a wave or stream-tile boundary (62 lanes)
@pytest.mark.parametrize("til,wpb", [(0, 1), (0, 4), (1, 3), (1, 16), (2, 1), (2, 5)])
@pytest.mark.parametrize("N,chains", [(2, 1), (2, 62), (2, 63), (3, 125), (31, 4), (32, 5), (63, 3), (64, 31), (65, 2),
                                      (127, 9), (128, 1), (128, 63)])
def test_tile_tables_at_their_edges(N, chains, til, wpb):
    systems = [ragged(N, chains), ragged(max(2, N // 2), chains + 1)]
    g, orcs = make_pair(systems, "cell" if chains % 2 else "f32", 16, density_mode=3 if til else 0, packed_tiles=til,
                        waves_per_block=wpb)
    check_sweeps(g, orcs)
    g.close()


# beads many images away take the general wrap in every cell lookup, with
# positive and negative indexes, in dyadic and other grids
@pytest.mark.parametrize("r,cw,dm,til", [("f32", 16, 2, 0), ("f32", 32, 0, 2), ("cell", 16, 1, 0), ("cell", 32, 3, 1)])
@pytest.mark.parametrize("edge", [0.25, 0.23])
def test_images_take_the_general_wrap(r, cw, dm, til, edge):
    s = ragged(24, 300, edge)
    rng = np.random.default_rng(5)
    xyz = W.gaussian_walks(s, seed=3).reshape(3, s.n_chains, s.N)
    xyz += (rng.integers(-40, 41, size=(3, s.n_chains, 1)) * np.array(s.box)[:, None, None])
    xyz = np.ascontiguousarray(xyz.reshape(3, -1))
    g, orcs = make_pair([s], r, cw, density_mode=dm, packed_tiles=til)
    g.set_positions(0, xyz)
    orcs[0].set_positions(xyz)
    assert (g.density(0) == orcs[0].density()).all()
    check_sweeps(g, orcs)
    g.close()


# length of a wave's list of changed beads: none (tiny moves), up to every
# bead on three faces (moves of almost a cell edge in a fine grid)
@pytest.mark.parametrize("dm", [0, 2, 3])
@pytest.mark.parametrize("delta", [1e-4, 0.02, 0.05])
def test_change_lists_of_every_length(delta, dm):
    s = W.diblock_system(200, 32, 0.5, 5.0, 10.0, (1.275, 1.275, 1.275), (25, 25, 25), move_halfwidth=delta)
    s.Re = 4.0          # soft bonds, so that almost every move is accepted
    g, orcs = make_pair([s], "f32", 16, density_mode=dm)
    check_sweeps(g, orcs)
    if delta == 0.05:
        assert orcs[0].counts.sum() == s.n_beads and g.observables(0)["accept_ratio"] > 0.5
    g.close()


def test_counters_near_their_limits():
    """The sweep counter and system id are Philox words: large values, two calls against one."""
    s = ragged(16, 40)
    outs = []
    for split in ((3,), (1, 2)):
        with Soma([s], seed=2**63 + 5, pos_repr="f32", sys_id_base=2**31 - 3, density_mode=1) as g:
            g.set_sweep(2**33 + 1)
            for n in split:
                g.sweep(n)
            outs.append((g.state(0), g.density(0)))
    assert (outs[0][0] == outs[1][0]).all() and (outs[0][1] == outs[1][1]).all()
