"""Two atoms in one place: the edge between them has no direction, so what
depends on it is NaN.  Nothing else may be, however the atoms are packed into
waves and workgroups."""
import numpy as np
import pytest

from paper_2506_04055_amd import synth

pytestmark = pytest.mark.gpu

L, RC = 58.0, 5.0


@pytest.fixture(scope="module")
def mlp():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2506_04055_amd import mlp as M
    M.lib()
    return M


def system(gap, n):
    """A gas (1,500 atoms: four neighbours each) with a pair of atoms `gap` apart alone in the first and in the last cell."""
    rng = np.random.default_rng(3)
    pos = rng.uniform(0, L, (n, 3))
    d = pos[:, None] - pos[None]
    d -= L * np.round(d / L)
    close = (np.triu((d ** 2).sum(2) < 0.8, 1)).any(0)     # (no other close contacts)
    pos = pos[~close]
    for corner in (0.5, L - 0.5):
        pos = pos[(np.abs(pos - corner) > 6.5).any(1)]
    first, last = np.full((2, 3), 0.5), np.full((2, 3), L - 0.5)
    first[1, 0] += gap
    last[1, 0] -= gap
    pos = np.concatenate([first, pos, last]).astype(np.float32)
    n = len(pos)
    return synth.System(pos, np.random.default_rng(4).integers(0, 2, n).astype(np.int32), np.array([L] * 3), n)


def far(s, depth):
    """The atoms farther than depth from the corner where the pairs are."""
    w = np.abs(np.asarray(s.pos, np.float64))
    return np.sqrt((np.minimum(w, L - w) ** 2).sum(1)) > depth + 1.5


MODELS = {
    # weights, atoms, and how many cutoffs an energy and a force reach
    "allegro": (lambda: synth.make_allegro_weights(2, seed=1, bias_scale=0.1), 1500, 0, 1),
    "mace": (lambda: synth.make_mace_weights(2, seed=1, bias_scale=0.1), 1500, 2, 4),
    "mace_two_waves": (lambda: synth.make_mace_weights(2, seed=1, bias_scale=0.1), 900, 2, 4),
    "painn32": (lambda: synth.make_weights(32, 8, 2, 2, seed=1, bias_scale=0.1), 1500, 2, 4),
    "painn64": (lambda: synth.make_weights(64, 20, 2, 2, seed=1, bias_scale=0.1), 1500, 2, 4),
}


@pytest.mark.parametrize("name", list(MODELS))
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_coincident_atoms_stay_apart(mlp, name, precision):
    import torch
    make, n, reach_u, reach_f = MODELS[name]
    h, w = make()
    out = []
    for gap in (0.9, 0.0):
        s = system(gap, n)
        d = mlp.System(mlp.Model(h, w, precision), s.pos, s.species, s.box, skin=0.5)
        print(f"[case] {name} {precision} gap {gap}", flush=True)
        r = d.compute(atom_energy=True)
        torch.cuda.synchronize()
        out.append((r["atom_energy"].cpu().numpy(), r["forces"].t().cpu().numpy()))
    (U0, F0), (U, F) = out
    ok_u, ok_f = far(s, reach_u * RC), far(s, reach_f * RC)
    if reach_u == 0:          # strictly local: the pairs' own energies alone
        ok_u = np.ones(s.n_atoms, bool)
        ok_u[[0, 1, -2, -1]] = False
    assert ok_u.sum() > n // 2 and ok_f.sum() > n // 5
    assert np.isnan(U[[0, 1, -2, -1]]).all() and np.isfinite(U0).all()
    print(f"[measured] {name} {precision}: {(~np.isfinite(U[ok_u])).sum()} of {ok_u.sum()} energies and "
          f"{(~np.isfinite(F[ok_f])).any(1).sum()} of {ok_f.sum()} forces that are not finite", flush=True)
    assert np.isfinite(U[ok_u]).all() and np.isfinite(F[ok_f]).all()
    # (a neighbour's energy sees the pair's other place, and a force the neighbour's energy)
    same_u, same_f = ok_u & far(s, max(reach_u, 1) * RC), ok_f & far(s, max(reach_f, 2) * RC)
    assert np.array_equal(U[same_u], U0[same_u]) and np.array_equal(F[same_f], F0[same_f])
