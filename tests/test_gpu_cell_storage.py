"""The stored order of the cells (bricks, padding, linear order): exact against the oracle.

Grids whose y and z are and are not multiples of the brick, of one or a few
cells (stored linearly), in batches that mix both.
"""
import numpy as np
import pytest

from paper_2606_09356_amd import workloads as W
from paper_2606_09356_amd.soma import Soma
from tests.test_gpu_parity import SEED, make_pair, same_state

pytestmark = pytest.mark.gpu
GRIDS = [(8, 8, 8), (5, 9, 10), (7, 11, 13), (1, 12, 16), (16, 1, 12), (12, 16, 1), (2, 3, 4), (3, 5, 6), (1, 1, 1), (9, 8, 31)]


def system(grid, N=12, edge=0.23, form=0):
    chains = max(3, int(2 * np.prod(grid)) // N)
    return W.diblock_system(chains, N, 0.5, 20.0, 50.0, tuple(edge * g for g in grid), grid, ham_form=form)


@pytest.mark.parametrize("r,cw,dm,til", [("f32", 16, 0, 0), ("cell", 32, 1, 2), ("f32", 32, 2, 1), ("cell", 16, 2, 2),
                                         ("cell", 16, 3, 0), ("f32", 32, 3, 2)])
def test_counts_fields_and_sweeps_in_every_order(r, cw, dm, til):
    systems = [system(g, form=k % 2) for k, g in enumerate(GRIDS)]
    g, orcs = make_pair(systems, r, cw, density_mode=dm, packed_tiles=til, reorder_every=2)
    for s in range(3):
        for k, o in enumerate(orcs):
            assert (g.density(k) == o.counts).all(), (k, s)
            w = o.omega
            assert np.abs(g.fields(k) - w).max() <= 4e-6 * max(1.0, np.abs(w).max()), (k, s)
            a, b = g.observables(k), o.observables()
            assert abs(a["Enb_per_chain"] - b["Enb_per_chain"]) <= 1e-12 * max(1.0, abs(b["Enb_per_chain"])), (k, s)
        g.sweep(1)
        for k, o in enumerate(orcs):
            o.sweep(SEED, s)
            o.density()
            o.fields()
            assert same_state(g, k, o).all(), (k, s)
    g.close()


@pytest.mark.parametrize("grid", [(5, 9, 10), (8, 8, 8), (3, 5, 6)])
def test_frozen_fields_and_targets_in_every_order(grid):
    """Frozen fields come back as they were set and move beads as the oracle's; targets likewise."""
    s = system(grid)
    rng = np.random.default_rng(2)
    w = rng.normal(0.0, 1.0, size=(2, s.n_cells)).astype(np.float32)
    g, orcs = make_pair([s], "f32", 16, coupling=True)
    o = orcs[0]
    g.set_fields(0, w)
    assert (g.fields(0) == w).all()
    o.set_fields(w)
    g.sweep(1)
    o.sweep(SEED, 0)
    assert same_state(g, 0, o).all()
    g.release_fields(0)
    phi = np.zeros((2, s.n_cells), np.float32)
    cell = s.n_cells // 2 + 1
    phi[:, cell] = 1.0                       # all targets in one cell
    g.place_from_fields(0, phi)
    rho = g.density(0).astype(np.float64)
    g.set_umbrella(0, 3.0)
    phi_of = rho * (s.n_cells / s.n_beads)
    base = g.fields(0)
    g.set_umbrella(0, 0.0)
    plain = g.fields(0)
    want = 3.0 * (phi_of - phi) / s.N
    assert np.abs((base - plain) - want).max() <= 1e-4 * max(1.0, np.abs(plain).max())
    g.close()


def test_density_to_unaligned_device_memory():
    import torch
    s = system((6, 9, 12))
    with Soma([s], seed=4) as g:
        want = g.density(0)
        buf = torch.zeros(2 * s.n_cells + 3, dtype=torch.int32, device="cuda")
        for off in (0, 1, 3):
            out = buf[off:off + 2 * s.n_cells]
            g.density_device(0, out)
            assert (out.cpu().numpy().reshape(2, -1) == want).all()
