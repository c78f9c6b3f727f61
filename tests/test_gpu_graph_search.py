"""The search kernels' variants against the oracle, bit-exact, at the sizes
where they change over: one or four wavefronts an atom (1,024 atoms), keys
placed by rank in a wavefront's 256 slots or in a block's, and the sort network
past 1,024 keys; cells thinner and wider than the cutoff in one batch."""
import numpy as np
import pytest

from gpu_helpers import assert_graph_equal
from oracle import graph as og
from paper_2412_20796_amd import synth
from test_gpu_graph import bd, gpu_graph  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


def _cat(parts):
    ptr = np.concatenate([[0], np.cumsum(np.concatenate([np.diff(p.atom_ptr) for p in parts]))]).astype(np.int32)
    return synth.Batch(ptr, np.concatenate([p.pos for p in parts]), np.concatenate([p.lattice for p in parts]),
                       np.concatenate([p.Z for p in parts]))


@pytest.mark.parametrize("n", [1023, 1024, 1025])
def test_wavefronts_per_atom(bd, n):
    b = _cat([synth.random_crystals(seed=310, n_struct=1, n_lo=700, n_hi=700),
              synth.random_crystals(seed=311, n_struct=1, n_lo=n - 700 - 3, n_hi=n - 700 - 3),
              synth.random_crystals(seed=312, n_struct=1, n_lo=3, n_hi=3)])
    assert b.n_atoms == n
    got, _ = gpu_graph(bd, b)
    assert_graph_equal(got, og.build_graph(b.atom_ptr, b.pos, b.lattice))


@pytest.mark.parametrize("r_atom,n", [(9.0, 1040), (9.5, 60), (15.0, 20), (15.0, 1030)])
def test_keys_per_atom(bd, r_atom, n):
    """About 260, 310 and 1,200 edges an atom."""
    m = min(n, 20) if r_atom > 10 else n
    parts = [synth.random_crystals(seed=320, n_struct=1, n_lo=m, n_hi=m, rho=(0.085, 0.085))]
    if n > m:  # one-atom cells make up the count: the reference tests every pair of images
        parts.append(synth.random_crystals(seed=340, n_struct=n - m, n_lo=1, n_hi=1, rho=(0.01, 0.012)))
    b = _cat(parts)
    assert b.n_atoms == n
    got, _ = gpu_graph(bd, b, r_atom=r_atom)
    ref = og.build_graph(b.atom_ptr, b.pos, b.lattice, r_atom=r_atom)
    print("largest row", int(np.diff(ref["edge_ptr"]).max()))
    assert_graph_equal(got, ref)


def test_many_crystals_and_more_than_one_pass(bd):
    """More crystals than are searched in LDS, and more than 1,024 (several
    rounds of the structure setup)."""
    b = synth.random_crystals(seed=350, n_struct=2100, n_lo=1, n_hi=2, rho=(0.02, 0.04))
    got, _ = gpu_graph(bd, b)
    assert_graph_equal(got, og.build_graph(b.atom_ptr, b.pos, b.lattice))
