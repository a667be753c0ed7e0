"""GPU tests of the local search with one individual per block at its edges: which
calls take it, ligands without a pair beside others, several calls in flight, and
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


def _job(dock, G, ff, grd, atoms, torsions, n, **kw):
    lig = synth.ligand(atoms, torsions, 104)
    gen = torch.from_numpy(synth.genotypes(lig, grd, n, 3)).cuda()
    return dock.LsJob(G, dock.Ligand(lig, ff), dock.LSState.start(gen), **kw)


# (atoms, torsions): blocks per CU of eight waves, of four (0: not shared so)
LAYOUTS = {(1, 0): (0, 0), (12, 2): (1, 0), (24, 6): (1, 0), (28, 7): (1, 2), (48, 10): (1, 2), (64, 16): (1, 2),
           (65, 12): (1, 0), (112, 28): (1, 0)}


@pytest.mark.parametrize("atoms,torsions", sorted(LAYOUTS))
def test_which_calls_share(setup, atoms, torsions):
    """On either side of the numbers of individuals that the GPU holds in blocks of
    eight waves and of four, a quarter of them on other streams than the default
    one; and never when a wave each is asked for, on plain maps or beside another
    family."""
    dock, G, grd, ff = setup
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    eight, four = (per_cu * cu for per_cu in LAYOUTS[atoms, torsions])
    stream = torch.cuda.Stream()
    for n in sorted({1, cu // 4, cu // 4 + 1, cu // 2, cu // 2 + 1, cu, cu + 1, 2 * cu, 2 * cu + 1}):
        job = _job(dock, G, ff, grd, atoms, torsions, n)
        for calls, kw in ((1, {}), (4, dict(stream=stream))):
            want = 8 if n * calls <= eight else 4 if n * calls <= four else 0
            assert dock.ls_shared_waves([job], 5, **kw) == want, (n, calls)
    job = _job(dock, G, ff, grd, atoms, torsions, 10)
    assert dock.ls_shared_waves([job], 5, threads_per_ind=64) == 0
    assert dock.ls_shared_waves([job], 5, threads_per_ind=128) == 0
    assert dock.ls_shared_waves([job], 0, final_eval=False) == 0
    for kw in (dict(threads_per_ind=64), dict(plain_maps=True)):
        assert dock.ls_shared_waves([_job(dock, G, ff, grd, atoms, torsions, 10, **kw)], 5) == 0
    assert dock.ls_shared_waves([job, _job(dock, G, ff, grd, 20, 3, 10, threads_per_ind=128)], 5) == 0


@pytest.mark.parametrize("sizes", [((1, 0), (48, 10), (5, 0)), ((5, 0), (64, 16)), ((2, 0), (12, 2)), ((64, 16), (1, 0), (24, 6))])
def test_ligands_without_a_pair_beside_others(setup, sizes):
    """The most pair batches of a call decide its layout: ligands that have none run
    in the shared blocks of the others."""
    dock, G, grd, ff = setup
    make = lambda **kw: [_job(dock, G, ff, grd, a, t, 70 + k, **kw) for k, (a, t) in enumerate(sizes)]
    shared = make()
    assert dock.ls_shared_waves(shared, 6) == 8
    dock.local_search(shared, 6)
    for s, w in zip(shared, make(threads_per_ind=64)):
        assert dock.ls_shared_waves([w], 6) == 0
        dock.local_search([w], 6)
        for f in FIELDS:
            assert torch.equal(getattr(s.state, f), getattr(w.state, f)), f


@pytest.mark.parametrize("atoms,torsions,n", [(48, 10, 64), (48, 10, 128), (48, 10, 150), (48, 10, 500), (112, 28, 200)])
def test_several_calls_in_flight(setup, atoms, torsions, n):
    """Five calls at a time, one on the default stream and four on streams of their
    own, whose individuals are shared in smaller calls only: every one's state is
    that of the call alone."""
    dock, G, grd, ff = setup
    alone = _job(dock, G, ff, grd, atoms, torsions, n)
    dock.local_search([alone], 40)
    jobs = [_job(dock, G, ff, grd, atoms, torsions, n) for _ in range(5)]
    streams = [torch.cuda.Stream() for _ in range(4)]
    torch.cuda.synchronize()
    assert dock.ls_shared_waves(jobs[4:], 40) > 0
    workspaces = [dock.local_search([j], 40, workspace=torch.empty(dock.workspace_bytes(1), dtype=torch.uint8, device="cuda"),
                                    stream=s) for j, s in zip(jobs, streams + [None])]
    torch.cuda.synchronize()
    assert len(workspaces) == 5
    for j in jobs:
        for f in FIELDS:
            assert torch.equal(getattr(j.state, f), getattr(alone.state, f)), f
