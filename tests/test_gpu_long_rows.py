"""Few atoms with many bonds and angles each (a bond cutoff as long as the atom
cutoff), for which several blocks form one atom's geometry: step parity with
one pass a block and several, whole and partial passes, and more bonds an atom
than have their vectors in LDS."""
import numpy as np
import pytest

from gpu_helpers import assert_close
from oracle import graph as og
from oracle import model as om
from paper_2412_20796_amd import synth
from test_gpu_model import _dev, bd  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,n,r_atom,r_bond", [(1, 1, 6.0, 4.0), (2, 3, 6.0, 5.5), (40, 9, 6.0, 4.5), (1, 1, 9.2, 9.2)])
def test_step_parity(bd, S, n, r_atom, r_bond):
    b = synth.random_crystals(seed=950 + n, n_struct=S, n_lo=n, n_hi=n, rho=(0.1, 0.1))
    ohp = om.HParams(d=64, n_layers=2, r_atom=r_atom, r_bond=r_bond)
    params = synth.make_params(64, 2, seed=(7, 1, n))
    targets = synth.make_targets(b, seed=(7, 2, n))
    ref_graph = og.build_graph(b.atom_ptr, b.pos, b.lattice, r_atom=r_atom, r_bond=r_bond)
    k = np.diff(ref_graph["bond_ptr"])
    print("atoms", b.n_atoms, "largest bonds an atom", k.max(), "angles", len(ref_graph["angle_b2"]))
    rl, rg, (rE, rF, rS), _ = om.step(ohp, b, params.astype(np.float64), targets, graph=ref_graph)
    hp = bd.hparams(d=64, n_layers=2, r_atom=r_atom, r_bond=r_bond)
    db, ws, g = bd.DeviceBatch.from_host(b), bd.Workspace(), bd.DeviceGraph(b.n_atoms, 64, 16, 64)
    loss, grad = bd.step(hp, db, g, _dev(params), [_dev(x) for x in targets], ws)
    assert_close(loss.cpu().numpy(), [rl], "loss")
    gg = grad.cpu().numpy()
    for name, (off, shape) in om.layout(ohp)[0].items():
        m = int(np.prod(shape))
        assert_close(gg[off:off + m], rg[off:off + m], "grad " + name)
    E, F, S_ = bd.forward(hp, db, g, _dev(params), ws, save_for_backward=False)
    assert_close(E.cpu().numpy(), rE, "energy")
    assert_close(F.cpu().numpy(), rF, "forces")
    assert_close(S_.cpu().numpy(), rS, "stress")
