"""Step parity with basis sizes other than 31: the depths at which the
matrix products change (whole and partial 16-deep steps, one step and more
than the widest launch keeps, rows whose stride is no multiple of 16 bytes),
on few rows (weights streamed) and on enough for the launches that keep the
weights in LDS; and the same for the conservative readout's gradients."""
import numpy as np
import pytest

from gpu_helpers import assert_close
from oracle import autodiff as oa
from oracle import graph as og
from oracle import model as om
from paper_2412_20796_amd import synth
from test_gpu_model import _dev, bd  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


def _params(hp, seed):
    rng = np.random.default_rng([seed, 41])
    lay, total = om.layout(hp)
    p = np.empty(total, np.float32)
    for name, (off, shape) in lay.items():
        n = int(np.prod(shape))
        if name in ("f_a", "f_b"):
            x = np.pi * np.arange(1, n + 1)
        elif name == "W_Z":
            x = rng.standard_normal(n)
        elif name.endswith(("g_c", "g_g")):
            x = np.ones(n)
        else:
            bound = 1.0 / np.sqrt(shape[0] if len(shape) > 1 else hp.d)
            x = rng.uniform(-bound, bound, n)
        p[off:off + n] = x
    return p


@pytest.mark.parametrize("R,K,d,S", [(1, 1, 64, 2), (16, 17, 64, 3), (33, 63, 64, 2), (64, 15, 128, 2), (33, 63, 64, 24),
                                     (2, 31, 64, 24), (16, 15, 64, 24), (31, 3, 128, 12),
                                     (48, 33, 128, 12)])
def test_step_parity(bd, R, K, d, S):
    b = synth.random_crystals(seed=500 + R, n_struct=S, n_lo=5, n_hi=8 if S < 4 else 30)
    ohp = om.HParams(d=d, n_layers=2, n_rbf=R, n_fourier=K)
    params = _params(ohp, R)
    targets = synth.make_targets(b, seed=(7, 2, R))
    ref_graph = og.build_graph(b.atom_ptr, b.pos, b.lattice)
    rl, rg, (rE, rF, rS), _ = om.step(ohp, b, params.astype(np.float64), targets, graph=ref_graph)
    hp = bd.hparams(d=d, n_layers=2, n_rbf=R, n_fourier=K)
    db, ws, g = bd.DeviceBatch.from_host(b), bd.Workspace(), bd.DeviceGraph(b.n_atoms, 64, 16, 64)
    loss, grad = bd.step(hp, db, g, _dev(params), [_dev(x) for x in targets], ws)
    print("E", g.n_edges, "A", g.n_angles)
    assert_close(loss.cpu().numpy(), [rl], "loss")
    gg = grad.cpu().numpy()
    for name, (off, shape) in om.layout(ohp)[0].items():
        n = int(np.prod(shape))
        assert_close(gg[off:off + n], rg[off:off + n], "grad " + name)
    E, F, S_ = bd.forward(hp, db, g, _dev(params), ws, save_for_backward=False)
    assert_close(E.cpu().numpy(), rE, "energy")
    assert_close(F.cpu().numpy(), rF, "forces")
    assert_close(S_.cpu().numpy(), rS, "stress")


@pytest.mark.parametrize("R,K", [(16, 17), (33, 35)])
def test_conservative_gradient(bd, R, K):
    b = synth.random_crystals(seed=540 + R, n_struct=2, n_lo=4, n_hi=7)
    ohp = om.HParams(n_layers=2, n_rbf=R, n_fourier=K, conservative=True)
    params = _params(ohp, R)
    targets = synth.make_targets(b, seed=(7, 2, R))
    ref_graph = og.build_graph(b.atom_ptr, b.pos, b.lattice)
    rl, rg = oa.loss_and_grad(ohp, b, ref_graph, params.astype(np.float64), targets)
    hp = bd.hparams(n_layers=2, n_rbf=R, n_fourier=K, conservative=True)
    db, ws, g = bd.DeviceBatch.from_host(b), bd.Workspace(), bd.DeviceGraph(b.n_atoms, 64, 16, 64)
    loss, grad = bd.step(hp, db, g, _dev(params), [_dev(x) for x in targets], ws)
    assert_close(loss.cpu().numpy(), [rl], "loss")
    gg, m = grad.cpu().numpy(), np.abs(rg).max()
    for name, (off, shape) in om.layout(ohp)[0].items():
        n = int(np.prod(shape))
        # the tolerance of the conservative training tests (first derivatives
        # multiplied by tangents that pass through the same chain again)
        scale = max(np.abs(rg[off:off + n]).max(), 1e-2 * m)
        err = np.abs(gg[off:off + n] - rg[off:off + n])
        assert (err <= 3e-5 * scale + 1e-4 * np.abs(rg[off:off + n])).all(), (name, err.max(), scale)
