"""Initial walks and placements on wave tiles against the CPU oracle, at the tiles' edges.

Bars: the walks are FP64 sums in the oracle's order, but logarithm, sine and
cosine come from two math libraries (each within an ulp or so), so a stored
FP32 value may differ by one rounding where the FP64 sums straddle it: at most
one FP32 ulp of the coordinate, in at most 1 % of the values.
"""
import numpy as np
import pytest

import oracle
from paper_2606_09356_amd import workloads as W
from paper_2606_09356_amd.soma import Soma

pytestmark = pytest.mark.gpu
SEED = 77


def system(N, chains, walls=None):
    s = W.diblock_system(chains, N, 0.5, 20.0, 50.0, (5.0, 4.0, 6.0), (20, 16, 24))
    s.walls = walls
    return s


@pytest.mark.parametrize("walls", [None, (3, 20)])
@pytest.mark.parametrize("N,chains", [(2, 1), (2, 65), (3, 43), (33, 7), (64, 5), (127, 3), (128, 2)])
def test_walks_at_tile_edges(N, chains, walls):
    s = system(N, chains, walls)
    with Soma([s], seed=SEED, pos_repr="f32", sys_id_base=5) as g:
        o = oracle.OracleSystem(s, sys_id=5, mode=oracle.MODE_F32)
        o.set_positions(o.init_walks(SEED))
        a, b = g.state(0), o.xf
        off = np.abs(a - b)
        assert (off <= np.spacing(np.abs(b))).all()
        assert (off > 0).mean() <= 0.01
        if walls:
            z = a[2] / 0.25
            assert (z >= walls[0]).all() and (z < walls[1]).all()


@pytest.mark.parametrize("N,chains", [(2, 65), (31, 9), (64, 3), (128, 5)])
def test_placement_repeats_across_chain_orders(N, chains):
    """A placement depends on logical ids only: the same in any physical chain order, and walls hold."""
    s = system(N, chains, walls=(2, 22))
    phi = np.zeros((2, 20, 16, 24), np.float32)
    phi[:, :, :, 8:16] = 1.0
    phi = phi.reshape(2, -1)
    out = []
    for sweeps in (0, 3):
        with Soma([s], seed=SEED, pos_repr="cell", coupling=True, reorder_every=1) as g:
            g.sweep(sweeps)
            g.place_from_fields(0, phi)
            f, c = g.state(0)
            out.append((f, c))
            assert g.density(0).sum() == s.n_beads
            assert (c[2] >= 2).all() and (c[2] < 22).all()
    assert (out[0][0] == out[1][0]).all() and (out[0][1] == out[1][1]).all()
