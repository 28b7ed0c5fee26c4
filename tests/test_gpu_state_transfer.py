"""State transfer between the host and the stored (permuted, padded) layout: exact."""
import numpy as np
import pytest

from paper_2606_09356_amd import workloads as W
from paper_2606_09356_amd.soma import Soma, SomaError, SOMA_EINVAL

pytestmark = pytest.mark.gpu


def systems(N, chains):
    out = []
    for n, c in ((N, chains), (max(2, N - 1), chains + 3)):
        m = max(4, int(round((n * c / 2.0) ** (1.0 / 3.0))))
        out.append(W.diblock_system(c, n, 0.5, 20.0, 50.0, (0.23 * m, 0.25 * m, 0.24 * m), (m, m, m)))
    return out


@pytest.mark.parametrize("r", ["f32", "cell"])
@pytest.mark.parametrize("N,chains", [(2, 1), (3, 200), (32, 65), (65, 9), (127, 3), (128, 40)])
def test_state_round_trip_through_a_reordered_context(N, chains, r):
    sy = systems(N, chains)
    with Soma(sy, seed=11, pos_repr=r, reorder_every=1) as g, Soma(sy, seed=12, pos_repr=r, reorder_every=2) as h:
        g.sweep(3)
        h.sweep(5)           # another physical chain order
        for k, s in enumerate(sy):
            st = g.state(k)
            h.set_state(k, *(st if r == "cell" else (st,)))
            back = h.state(k)
            for a, b in zip(st if r == "cell" else (st,), back if r == "cell" else (back,)):
                assert (a == b).all()
            xyz = g.positions(k)
            assert (xyz == h.positions(k)).all()
            e = np.array([np.float32(b / n) for b, n in zip(s.box, s.grid)], np.float64)[:, None]
            want = st[1].astype(np.float64) * e + st[0].astype(np.float64) if r == "cell" else st.astype(np.float64)
            assert (xyz == want).all()
            assert (g.density(k) == h.density(k)).all()
        g.sweep(2)           # the scratch was used: sweeps and reorders go on from the state
        h.set_sweep(3)
        ref = Soma(sy, seed=11, pos_repr=r, reorder_every=1)
        ref.sweep(5)
        for k in range(2):
            a, b = g.state(k), ref.state(k)
            assert all((x == y).all() for x, y in zip(a, b)) if r == "cell" else (a == b).all()
        ref.close()


def test_bad_states_change_nothing():
    s = W.diblock_system(30, 17, 0.5, 20.0, 50.0, (2.0, 2.0, 3.0), (8, 8, 12))
    s.walls = (2, 10)
    for r in ("f32", "cell"):
        with Soma([s], seed=3, pos_repr=r) as g:
            st = g.state(0)
            f, c = (st if r == "cell" else (st, None))
            rho = g.density(0)
            bad = []
            for v in (np.nan, np.inf, -np.inf):
                x = f.copy()
                x[1, 77] = v
                bad.append((x, c))
            if r == "cell":
                for v in (0.25 * 2.0, -0.2501):
                    x = f.copy()
                    x[0, 509] = v
                    bad.append((x, c))
                for v in (1 << 22, -(1 << 22)):
                    y = c.copy()
                    y[1, 0] = v
                    bad.append((f, y))
                for v in (1, 10):
                    y = c.copy()
                    y[2, 5] = v
                    bad.append((f, y))
            else:
                for v in (0.499, 2.5):
                    x = f.copy()
                    x[2, 5] = v
                    bad.append((x, None))
            for x, y in bad:
                with pytest.raises(SomaError) as e:
                    g.set_state(0, x, y)
                assert e.value.code == SOMA_EINVAL
                now = g.state(0)
                assert (now[0] == f).all() and (now[1] == c).all() if r == "cell" else (now == f).all()
                assert (g.density(0) == rho).all()
            g.set_state(0, f, c)
