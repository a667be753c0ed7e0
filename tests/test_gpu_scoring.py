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


@pytest.mark.parametrize("atoms,torsions", [(1, 0), (20, 0), (24, 6), (48, 10), (60, 20), (64, 28)])
@pytest.mark.parametrize("n", [9000, 40001])
def test_energies_from_grouped_poses(setup, atoms, torsions, n):
    """More genotypes than waves: a wave makes the poses of 64 / (torsions + 1) of
    its genotypes at once (two to sixty-four; the last group is cut off). Energies
    are those of the gradient evaluation, which makes one at a time, bit for bit."""
    dock, grd, *maps, ff = setup
    lig = synth.ligand(atoms, torsions, 104)
    L = dock.Ligand(lig, ff)
    gen = torch.from_numpy(synth.genotypes(lig, grd, 1000, 3)).cuda().repeat(-(-n // 1000), 1)[:n].contiguous()
    gen[:, :3] += torch.linspace(-1.0, 1.0, n, device="cuda")[:, None]
    for G in maps:
        E, _ = dock.score_batch(G, L, gen, with_grad=False)
        want, _ = dock.score_batch(G, L, gen, with_grad=True)
        assert torch.equal(E, want)


@pytest.mark.parametrize("atoms,torsions", [(12, 2), (48, 10), (112, 28)])
@pytest.mark.parametrize("iterations", [1, 2, 9])
def test_random_search_reads_either_map_layout(setup, atoms, torsions, iterations):
    """The random search of the corner-expanded maps and of the plain ones (a kernel
    each): the same cells, so the same states bit for bit."""
    dock, grd, *maps, ff = setup
    lig = synth.ligand(atoms, torsions, 104)
    L = dock.Ligand(lig, ff)
    gen = torch.from_numpy(synth.genotypes(lig, grd, 70, 3)).cuda()
    normals = torch.randn((iterations, 70, L.n_genes), device="cuda", generator=torch.Generator("cuda").manual_seed(4))
    scale = torch.full((L.n_genes,), 0.3, device="cuda")
    states = []
    for G in maps:
        st = dock.SWState.start(gen, dock.score_batch(G, L, gen, with_grad=False)[0])
        dock.solis_wets(G, L, st, normals, scale)
        states.append(st)
    for f in ("genotype", "energy", "bias", "rho", "counts"):
        assert torch.equal(getattr(states[0], f), getattr(states[1], f)), f
