"""GPU tests of the population steps between searches: the genetic step's two
ways of finding a run's best member (a wave up to 256 members, the block above),
and the start state written by one kernel, against the tensor operations it
stands for."""
import numpy as np
import pytest

from oracle import ga_ref as GA
from paper_2410_10447_amd import dock

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("runs,pop,genes", [(1, 1, 7), (4, 64, 39), (5, 255, 9), (3, 256, 17), (3, 257, 17), (2, 1000, 39)])
@pytest.mark.parametrize("elitism", [0, 1])
def test_genetic_step_around_the_wave_scan(runs, pop, genes, elitism):
    """Bit for bit; many equal energies, so that the first of the best decides,
    and runs of NaN and infinities only."""
    rng = np.random.default_rng(runs * 1000 + pop)
    E = rng.integers(-1, 4, (runs, pop)).astype(np.float32)
    E[0, rng.random(pop) < 0.3] = np.nan
    if runs > 2:
        E[1], E[2] = np.nan, np.inf
    arrays = (rng.normal(size=(runs, pop, genes)).astype(np.float32), E,
              rng.integers(0, pop, (runs, pop, 4), dtype=np.int32), rng.random((runs, pop, 3), dtype=np.float32),
              rng.integers(0, genes + 1, (runs, pop, 2), dtype=np.int32),
              rng.random((runs, pop, genes), dtype=np.float32),
              rng.normal(size=(runs, pop, genes)).astype(np.float32))
    children, best = dock.ga_step(*(torch.from_numpy(a).cuda() for a in arrays), 0.6, 0.8, 0.1, elitism)
    want, want_best = GA.ga_step(*arrays, 0.6, 0.8, 0.1, elitism)
    assert np.array_equal(best.cpu().numpy(), want_best)
    assert np.array_equal(children.cpu().numpy().view(np.uint32), want.view(np.uint32))


def _sources():
    base = torch.randn((600, 40), device="cuda")
    base[3, 2], base[5, 1], base[7, 0] = float("nan"), float("inf"), -0.0
    odd = torch.randn(1 + 17 * 33, device="cuda")
    return {"whole": base, "one gene": base[:1, :1], "columns": base[:, 3:20], "transposed": base.t(),
            "misaligned": odd[1:].view(33, 17), "none": base[:0], "repeated": base[:1].expand(9, 40),
            "double": base.double(), "gradient": base.clone().requires_grad_(), "host": base.cpu()}


@pytest.mark.parametrize("name", list(_sources()) if torch.cuda.is_available() else ["no GPU"])
def test_start_state(name):
    src = _sources()[name]
    st = dock.LSState.start(src)
    n = src.shape[0]
    want = {"genotype": src, "best_genotype": src, "acc_g2": torch.zeros_like(src), "acc_dx2": torch.zeros_like(src),
            "best_energy": torch.full((n,), float("inf")), "energy": torch.full((n,), float("nan")),
            "iters_done": torch.zeros(n, dtype=torch.int32)}
    for f, w in want.items():
        got = getattr(st, f)
        assert got.shape == w.shape and got.dtype == w.dtype and got.device == src.device, f
        assert got.is_contiguous() and (n == 0 or got.data_ptr() != src.data_ptr()), f
        got, w = got.detach().cpu().contiguous().numpy(), w.detach().cpu().contiguous().numpy()
        assert got.tobytes() == w.tobytes(), f
    assert st.genotype.requires_grad == src.requires_grad
