"""Products of fp32 operands split into bf16 parts: the range, operands and
weights above the largest bf16 number (3.39e38) and infinite ones, on few rows
and on enough for the launches that keep the weights in LDS; and the rounding
of a single product (one-atom crystals, whose weight gradient of the energy
head's output layer and whose energy are products of two numbers) against that
of an fp32 multiplication."""
import numpy as np
import pytest

from oracle import model as om
from paper_2412_20796_amd import synth
from test_gpu_model import _dev, _setup, bd  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu

BIG = np.float32(3.4e38)


def _one_atom(d):
    b = synth.Batch(np.array([0, 1], np.int32), np.zeros((1, 3), np.float32),
                    (np.eye(3, dtype=np.float32) * np.float32(2.9))[None], np.array([14], np.int32))
    return b, synth.make_params(d, 1, seed=(61, 1, d)), om.layout(om.HParams(d=d, n_layers=1))[0]


def _grad_w3(bd, setup, b, p, off, d):
    hp, db, g, ws = setup
    bd.forward(hp, db, g, p, ws)
    z = lambda *s: _dev(np.zeros(s, np.float32))

    def run(dE):
        grad = bd.backward(hp, db, g, p, _dev(np.array([dE], np.float32)), z(1, 3), z(1, 3, 3), ws)
        return grad.cpu().numpy()[off:off + d].copy()

    return run


@pytest.mark.parametrize("d", [64, 128])
def test_operand_near_the_top_of_the_range(bd, d):
    b, params, lay = _one_atom(d)
    run = _grad_w3(bd, _setup(bd, b, d, 1), b, _dev(params), lay["E_W3"][0], d)
    a = run(1.0)  # h + m + l of the activations times one: exact
    assert (a != 0).all()
    big = run(BIG)
    assert np.all(np.abs(big / (a.astype(np.float64) * float(BIG)) - 1) <= 2.0 ** -22)
    assert np.array_equal(run(np.inf), np.where(a > 0, np.inf, -np.inf).astype(np.float32))
    assert np.array_equal(run(-np.inf), np.where(a > 0, -np.inf, np.inf).astype(np.float32))
    assert np.isnan(run(np.nan)).all()


def test_result_near_the_top_of_the_range(bd):
    """Products just below the largest fp32 number, whose operands' leading
    parts multiply to more, in every column of a weight gradient."""
    d, k = 64, 21
    b, params, lay = _one_atom(d)
    view = {n: params[o:o + int(np.prod(s))].reshape(s) for n, (o, s) in lay.items()}
    # activation k of the first layer is about 40 and the second layer does not
    # see it: the factors stay well inside the range
    view["E_b1"][k] = 40
    view["E_W2"][k] = 0
    hp, db, g, ws = _setup(bd, b, d, 1)
    z = lambda *s: _dev(np.zeros(s, np.float32))
    off = lay["E_W2"][0]
    w3 = view["E_W3"].copy()

    def run(p, dE):
        bd.forward(hp, db, g, p, ws)
        grad = bd.backward(hp, db, g, p, _dev(np.array([dE], np.float32)), z(1, 3), z(1, 3, 3), ws)
        return grad.cpu().numpy()[off:off + d * d].reshape(d, d)[k].astype(np.float64)

    for n in range(d):
        view["E_W3"][:] = 1e-3 * w3
        view["E_W3"][n] = 1000
        p = _dev(params)
        one = run(p, 1.0)
        dE = np.float32(float(np.finfo(np.float32).max) * (1 - 2.0 ** -12) / abs(one[n]))
        got, want = run(p, dE), one * float(dE)
        assert np.all(np.abs(got / want - 1) <= 2.0 ** -21), (n, got[n], want[n])


@pytest.mark.parametrize("S", [2, 18])
def test_weights_near_the_top_of_the_range(bd, S):
    """d = 128 heads with one weight of the force head's output layer at
    3.4e38, and one of the energy head's infinite."""
    d, k = 128, 37
    b = synth.random_crystals(seed=620, n_struct=S, n_lo=3 if S == 2 else 50, n_hi=6 if S == 2 else 50, rho=(0.09, 0.1))
    params = synth.make_params(d, 1, seed=(62, 1))
    lay = om.layout(om.HParams(d=d, n_layers=1))[0]
    view = {n: params[o:o + int(np.prod(s))].reshape(s) for n, (o, s) in lay.items()}
    for h in "EF":
        # activation k small and negative for every row: silu(-7 +- 0.1)
        view[h + "_W2"][:, k] *= 0.01
        view[h + "_b2"][k] = -7
        view[h + "_W3"][:] = 0
        view[h + "_b3"][:] = 0
    hp, db, g, ws = _setup(bd, b, d, 1)
    tiles = -(-g.n_edges // 32) - 2 * (-b.n_atoms // 32)
    print("E", g.n_edges, "tiles", tiles)
    assert (tiles >= 2048) == (S > 2)

    def run(wE, wF):
        view["E_W3"][k, 0], view["F_W3"][k, 0] = wE, wF
        E, F, _ = bd.forward(hp, db, g, _dev(params), ws, save_for_backward=False)
        return E.cpu().numpy(), F.cpu().numpy().astype(np.float64)

    E1, F1 = run(1.0, 1.0)
    assert (E1 < 0).all()
    E2, F2 = run(-np.inf, BIG)
    assert (E2 == np.inf).all()
    # forces are linear in the output layer: two roundings of a scalar an edge apart
    ref = F1 * float(BIG)
    assert np.isfinite(F2).all()
    assert np.abs(F2 - ref).max() <= 1e-5 * np.abs(ref).max()
    E3, _ = run(float(BIG), 1.0)
    assert np.all(np.abs(E3 / (E1.astype(np.float64) * float(BIG)) - 1) <= 1e-5)


def _rms(got, a, y):
    """rms relative errors of `got` and of the fp32 product a y."""
    want = a.astype(np.float64) * y
    rel = lambda x: float(np.sqrt(np.mean(np.square(x.astype(np.float64) / want - 1))))
    return rel(got), rel(a.astype(np.float32) * np.asarray(y, np.float32))


@pytest.mark.parametrize("d", [64, 128])
def test_weight_gradient_of_one_row(bd, d):
    b, params, lay = _one_atom(d)
    run = _grad_w3(bd, _setup(bd, b, d, 1), b, _dev(params), lay["E_W3"][0], d)
    a = run(1.0)  # h + m + l of the activations times one: exact
    assert (a != 0).all()
    ys = np.random.default_rng(d).uniform(1, 2, 1536 // d).astype(np.float32)
    got = np.stack([run(y) for y in ys])
    e, e32 = _rms(got, np.broadcast_to(a, got.shape), ys[:, None].astype(np.float64))
    print("rms", e, "fp32 product", e32)
    # the terms left out (2^-27.5 rms) and one rounding to fp32 (2^-25.6 rms): 1.04 of the rounding alone; 1,536 values
    # give the rms to 2 %
    assert e <= 1.1 * e32


def test_energy_of_one_weight(bd):
    d = 128
    b, params, lay = _one_atom(d)
    off = lay["E_W3"][0]
    params[lay["E_b3"][0]] = 0
    setup = _setup(bd, b, d, 1)

    def run(k, w):
        p = params.copy()
        p[off:off + d] = 0
        p[off + k] = w
        hp, db, g, ws = setup
        return bd.forward(hp, db, g, _dev(p), ws, save_for_backward=False)[0].cpu().numpy()[0]

    a = np.array([run(k, 1.0) for k in range(d)])
    y = np.random.default_rng(3).uniform(1, 2, (8, d)).astype(np.float32)
    got = np.array([[run(k, y[r, k]) for k in range(d)] for r in range(8)])
    e, e32 = _rms(got, np.broadcast_to(a, got.shape), y.astype(np.float64))
    print("rms", e, "fp32 product", e32)
    assert e <= 1.1 * e32  # as above
