"""GPU tests of the scoring kernels' branches: energies without a gradient,
atoms outside the box beside atoms inside it, non-finite genotypes."""
import numpy as np
import pytest

from paper_2410_10447_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# ligand sizes whose pair batches number 0, 1, 2, 3, ... modulo 4 (the pair
# loops are unrolled by four), on one and two atoms per lane
SIZES = [(1, 0), (9, 1), (12, 2), (20, 4), (24, 6), (32, 8), (33, 5), (48, 10), (60, 14), (64, 16), (65, 12), (128, 32)]


@pytest.fixture(scope="module")
def setup():
    from paper_2410_10447_amd import dock
    grd = synth.grids(40, 10, 5)
    return dock, grd, dock.Grids.from_synth(grd), dock.Grids.from_synth(grd, corners=False), synth.force_field()


def _poses(lig, grd, n):
    gen = synth.genotypes(lig, grd, n, 3)
    gen[n // 2:, :3] *= 2.5               # whole and half ligands outside the box
    return torch.from_numpy(gen).cuda()


@pytest.mark.parametrize("atoms,torsions", SIZES)
def test_energy_alone_equals_energy_with_gradient(setup, atoms, torsions):
    """Bit for bit, in every reduction, on either map layout, one and two
    genotypes per wave."""
    dock, grd, G, Gp, ff = setup
    lig = synth.ligand(atoms, torsions, 104)
    L = dock.Ligand(lig, ff)
    gen = _poses(lig, grd, 101)
    two = (False, True) if atoms <= 32 else (False,)
    for grids in (G, Gp):
        for t in two:
            for v in range(1 if t else 5):
                E, g = dock.score_batch(grids, L, gen, variant=v, two_per_wave=t)
                E0, g0 = dock.score_batch(grids, L, gen, variant=v, two_per_wave=t, with_grad=False)
                torch.cuda.synchronize()
                assert g0 is None and torch.equal(E, E0), (v, t)
    print(f"{atoms} atoms: {L.n_batches} pair batches")


@pytest.mark.parametrize("two", [False, True])
@pytest.mark.parametrize("gene", [0, 3, 8])
def test_non_finite_genotypes_stay_in_their_row(setup, two, gene):
    """A NaN or infinite gene makes its own row's energy non-finite and leaves
    the others as they are."""
    dock, grd, G, _, ff = setup
    lig = synth.ligand(24, 6, 104)
    L = dock.Ligand(lig, ff)
    gen = _poses(lig, grd, 40)
    bad = gen.clone()
    bad[5, gene], bad[6, gene], bad[39, gene] = float("nan"), float("inf"), float("nan")
    rows = [r for r in range(40) if r not in (5, 6, 39)]
    for grad in (False, True):
        E, g = dock.score_batch(G, L, gen, two_per_wave=two, with_grad=grad)
        Eb, gb = dock.score_batch(G, L, bad, two_per_wave=two, with_grad=grad)
        torch.cuda.synchronize()
        assert torch.equal(E[rows], Eb[rows])
        assert not torch.isfinite(Eb[[5, 6, 39]]).any()
        if grad:
            assert torch.equal(g[rows], gb[rows])
