"""Runs of atoms of the fused Allegro and MACE kernels against the FP64 oracles:
how the edges of consecutive atoms are packed into a workgroup's 128 rows, on
systems whose degrees differ from atom to atom.  Tolerances: tests/parity.py."""
import numpy as np
import pytest

from oracle import allegro as AO
from oracle import mace as MO
from paper_2506_04055_amd import synth
from parity import TOL, check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mlp():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2506_04055_amd import mlp as M
    M.lib()
    return M


def mixed(n_gas, degree, n_dense, seed):
    """A gas of the given mean degree with a cluster in its middle whose inner atoms have about 150 neighbours, so that runs
    of many atoms, of none with edges, and pieces of one atom follow each other."""
    rng = np.random.default_rng(seed)
    L = (n_gas * 4 / 3 * np.pi * 125 / degree) ** (1 / 3)
    pos = rng.uniform(0, L, (n_gas, 3))
    for _ in range(3):     # no close contacts
        d = pos[:, None].astype(np.float32) - pos[None].astype(np.float32)
        d -= np.float32(L) * np.round(d / np.float32(L))
        close = (np.triu((d ** 2).sum(2) < 1.5, 1)).any(0)
        pos[close] = rng.uniform(0, L, (close.sum(), 3))
    pos = pos[~close]
    if n_dense:
        c = synth.fcc_crystal(5, a=2.4, seed=seed, sigma=0.15).pos[:n_dense].astype(np.float64) + L / 2 - 6.0
        pos = np.concatenate([pos[(np.abs(pos - L / 2) > 7.5).any(1)], c])
    pos = (pos % L).astype(np.float32)
    pos[pos >= np.float32(L)] = 0
    return synth.System(pos, rng.integers(0, 2, len(pos)).astype(np.int32), np.array([L] * 3), len(pos))


def copies_of(s, k):
    """k^3 periodic copies; coordinates and box on a grid of 2^-14 A, so that every copy is exact in float32."""
    assert k * max(s.box) < 512
    q = 2.0 ** 14
    sh = np.stack(np.meshgrid(*[np.arange(k)] * 3, indexing="ij"), -1).reshape(-1, 1, 3) * s.box
    pos = (s.pos.astype(np.float64)[None] + sh).reshape(-1, 3)
    assert np.array_equal(pos * q, np.round(pos * q))
    return synth.System(pos.astype(np.float32), np.tile(s.species, k ** 3), s.box * k, s.n_atoms * k ** 3)


def on_grid(s):
    q = 2.0 ** 14
    box = np.ceil(np.asarray(s.box, np.float64) * q) / q
    pos = np.round(s.pos.astype(np.float64) * q) / q
    pos[pos >= box] = 0
    return synth.System(pos.astype(np.float32), s.species, box, s.n_atoms)


def run(mlp, label, oracle, hw, s, precision, copies=1):
    import torch
    h, w = hw
    if copies > 1:
        s = on_grid(s)
    print(f"[case] {label} {precision} n={s.n_atoms} x {copies}^3", flush=True)
    E_ref, F_ref, U_ref = oracle.energy_forces(h, w, s.pos, s.species, s.box, per_atom=True)
    if copies > 1:
        s = copies_of(s, copies)
        E_ref, F_ref, U_ref = E_ref * copies ** 3, np.tile(F_ref, (copies ** 3, 1)), np.tile(U_ref, copies ** 3)
    d = mlp.System(mlp.Model(h, w, precision), s.pos, s.species, s.box, skin=0.5)
    out = d.compute(atom_energy=True)
    torch.cuda.synchronize()
    U = out["atom_energy"].cpu().numpy().astype(np.float64)
    # (a dense cluster's net forces are differences of five times the edges: as in the tests of the dense crystals)
    check(label, precision, float(out["energy"].item()), E_ref, out["forces"].t().cpu().numpy().astype(np.float64), F_ref,
          f_scale=2.5)
    assert np.abs(U - U_ref).max() <= 20 * TOL[precision][0] * max(np.abs(U_ref).mean(), np.abs(U_ref).max() / 20)
    return d


# mean degrees from runs that the slots limit (60 atoms of half an edge each) to runs that the rows limit
@pytest.mark.parametrize("n,degree,dense", [(4000, 0.5, 0), (4000, 2.0, 500), (3000, 8.0, 500)])
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_allegro_runs(mlp, n, degree, dense, precision):
    run(mlp, f"allegro mixed {degree}", AO, synth.make_allegro_weights(2, seed=12, bias_scale=0.1),
        mixed(n, degree, dense, 21), precision)


# few neighbours: a kernel each for the radial MLP and the convolution (the first two), otherwise the edge kernels
@pytest.mark.parametrize("n,degree,dense", [(2500, 1.0, 0), (6000, 2.0, 300), (2500, 9.0, 300)])
@pytest.mark.parametrize("precision", ["fp32", "bf16", "bf16_node"])
def test_mace_routes(mlp, n, degree, dense, precision):
    import torch
    d = run(mlp, f"mace mixed {degree}", MO, synth.make_mace_weights(2, seed=12, bias_scale=0.1),
            mixed(n, degree, dense, 22), precision)
    E = float(d.energy.item())
    d.compute(forces=False)
    torch.cuda.synchronize()
    assert float(d.energy.item()) == E


def _water():
    return synth.water_box(4, 3.105, seed=7)


def _fcc():
    return synth.fcc_crystal(3, seed=6, sigma=0.1)


def _mixed():
    return mixed(300, 4.0, 250, 23)


# several runs per workgroup by the plan (copies of one cell, so that the cell's oracle serves)
@pytest.mark.parametrize("make,copies", [(_water, 5), (_fcc, 7), (_mixed, 6)])
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_allegro_large(mlp, make, copies, precision):
    run(mlp, f"allegro {make.__name__}", AO, synth.make_allegro_weights(2, seed=12, bias_scale=0.1), make(), precision, copies)


# more atoms per workgroup than waves in the forward, several runs per workgroup in the adjoint
@pytest.mark.parametrize("make,copies", [(_water, 5), (_fcc, 7), (_mixed, 5)])
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_mace_large(mlp, make, copies, precision):
    run(mlp, f"mace {make.__name__}", MO, synth.make_mace_weights(2, seed=12, bias_scale=0.1), make(), precision, copies)
