"""GPU tests of the local search with one individual per block at its edges:
poses that are not finite."""
import numpy as np
import pytest

from paper_2410_10447_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FIELDS = ("genotype", "acc_g2", "acc_dx2", "best_genotype", "best_energy", "energy", "iters_done")


@pytest.fixture(scope="module")
def setup():
    from paper_2410_10447_amd import dock
    grd = synth.grids(40, 10, 5)
    return dock, dock.Grids.from_synth(grd), grd, synth.force_field()


@pytest.mark.parametrize("atoms,torsions", [(24, 6), (28, 7), (48, 10), (60, 14), (64, 16), (65, 12), (112, 28)])
@pytest.mark.parametrize("steps", [1, 4])
def test_poses_that_are_not_finite(setup, atoms, torsions, steps):
    """A NaN or infinite gene, in every gene of the genotype in turn: the gradient
    and the state are those of a wave per individual, NaN where they are NaN. The
    one-wave loop adds the 0 d of an unused lane to two free accumulator slots, the
    shared one does not; where d is NaN this reaches no gradient that is finite
    otherwise, since any two torsions apart move atoms four bonds from each other,
    a kept pair, which carries the NaN too."""
    dock, G, grd, ff = setup
    lig = synth.ligand(atoms, torsions, 104)
    L = dock.Ligand(lig, ff)
    n, genes = 1100, L.n_genes
    gen = synth.genotypes(lig, grd, n, 3)
    for r in range(0, n, 2):
        gen[r, (r // 2) % genes] = (np.nan, np.inf, -np.inf)[(r // 2 // genes) % 3]
    gen = torch.from_numpy(gen).cuda()

    def search(rows):
        st, grad = dock.LSState.start(rows), torch.zeros_like(rows)
        dock.local_search([dock.LsJob(G, L, st, grad=grad)], steps, final_eval=False)
        return {**{f: getattr(st, f).cpu().numpy() for f in FIELDS}, "grad": grad.cpu().numpy()}

    whole = search(gen)
    assert np.isnan(whole["grad"][0::2]).any() and np.isfinite(whole["grad"][1::2]).all()
    for lo, hi in ((0, 250), (100, 600)):
        part = search(gen[lo:hi])
        for f, v in part.items():
            assert np.array_equal(v, whole[f][lo:hi], equal_nan=v.dtype != np.int32), (lo, hi, f)
