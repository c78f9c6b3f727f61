"""Forward gates on tall tiles: batches above the row count from which a d = 64
launch takes 96-row tiles (whole and partial last tiles, runs of a segment cut
by a tile's end) against the same structures alone, which take 64-row tiles."""
import numpy as np
import pytest

from gpu_helpers import assert_close
from paper_2412_20796_amd import synth
from test_gpu_model import _dev, bd  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu

TALL_ROWS = 131072  # edges + 2 x angles of a launch


@pytest.mark.parametrize("seed,S", [(1, 30), (2, 31), (3, 47)])
def test_tall_tiles_match_single_structures(bd, seed, S):
    b = synth.random_crystals(seed=700 + seed, n_struct=S, n_lo=40, n_hi=48)
    hp = bd.hparams(d=64, n_layers=2)
    params = _dev(synth.make_params(64, 2, seed=(seed, 1)))
    db, ws, g = bd.DeviceBatch.from_host(b), bd.Workspace(), bd.DeviceGraph(b.n_atoms, 64, 16, 64)

    def run(batch, save):
        bd.build_graph(hp, batch, g, ws)
        E, F, X = bd.forward(hp, batch, g, params, ws, save_for_backward=save)
        return E.cpu().numpy().copy(), F.cpu().numpy().copy(), X.cpu().numpy().copy()

    E, F, X = run(db, False)
    rows = g.n_edges + 2 * g.n_angles
    print("rows", rows, "edges % 96", g.n_edges % 96, "angles % 96", g.n_angles % 96)
    assert rows >= TALL_ROWS
    for got, want, name in zip(run(db, True), (E, F, X), ("energy", "forces", "stress")):
        assert np.array_equal(got, want), name
    one_E, one_F, one_X = [], [], []
    for k in range(S):
        a0, a1 = b.atom_ptr[k], b.atom_ptr[k + 1]
        one = synth.Batch(np.array([0, a1 - a0], np.int32), b.pos[a0:a1], b.lattice[k:k + 1], b.Z[a0:a1])
        e, f, x = run(bd.DeviceBatch.from_host(one), False)
        assert g.n_edges + 2 * g.n_angles < TALL_ROWS
        one_E.append(e)
        one_F.append(f)
        one_X.append(x)
    assert_close(E, np.concatenate(one_E), "energy")
    assert_close(F, np.concatenate(one_F), "forces")
    assert_close(X, np.concatenate(one_X), "stress")
