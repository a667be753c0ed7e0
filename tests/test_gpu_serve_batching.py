"""Continuous batching without a clock: jobs that are all there at the start share
every launch, however warm the process is and however fast a job."""
import numpy as np
import pytest

from paper_2410_10447_amd import serve, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_jobs_that_are_there_share_every_launch():
    grids = [synth.grids(40, 10, 5), synth.grids(48, 10, 6)]
    ex = serve.GpuExecutor(grids, synth.force_field())
    specs = []
    for k, (atoms, torsions) in enumerate([(12, 2), (24, 6), (48, 10), (60, 14), (70, 12)]):
        lig = synth.ligand(atoms, torsions, 104)
        specs.append(serve.JobSpec(job_id=k, ligand=lig, grid_id=k % 2, arrival=0.0, iterations=40 + 10 * k,
                                   genotypes=synth.genotypes(lig, grids[k % 2], 40, k)))
    carried = []
    launch = ex.launch
    ex.launch = lambda plan, iters: (carried.append(len(plan)), launch(plan, iters))[1]

    def run(jobs, chunk_iters):
        st = serve.Server(ex, max_individuals=10_000, device_budget=1 << 30, chunk_iters=chunk_iters).run(jobs)
        assert len(st.completed) == len(jobs) and not st.failed
        return {r.spec.job_id: r.result for r in st.completed}

    for _ in range(2):
        carried.clear()
        mixed = run(specs, 16)
        # 40, 50, ... 80 steps in chunks of 16: three, four, four, five and five of them
        assert carried == [5, 5, 5, 4, 2]
    for s in specs:
        alone = run([s], 25)[s.job_id]
        for f in ("best_energy", "best_genotype"):
            assert np.array_equal(alone[f], mixed[s.job_id][f])
