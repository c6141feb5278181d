"""The wave-per-child breeding kernels against the host driver, column for
column: k_max at the lane count and on both sides of it, populations around
the four individuals of a rank block, the 16 and 64 children of a packing
block and the 8,192 individuals past which a wave ranks eight, and a capture
on a stream without scratch (one workgroup breeds there)."""
import numpy as np
import pytest

from paper_1807_09932_amd import ebic
from tests.gpu_common import announce, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture()
def ctx():
    from paper_1807_09932_amd.ebic import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n_cols,pop,k_min,k_max,elite", [
    (64, 5, 1, 64, 1),       # k_max = n_cols = lanes: nothing left to insert or substitute
    (200, 130, 30, 64, 7),   # k_max at the lane count
    (200, 130, 30, 65, 7),   # one past it: the one-workgroup kernel
    (90, 2, 1, 20, 0),
    (90, 1025, 2, 30, 1024), # every child but one an elite
    (150, 4097, 2, 30, 200),
    (150, 8192, 2, 12, 400),
    (150, 8195, 2, 12, 8194),
])
def test_waves_equal_host(ctx, n_cols, pop, k_min, k_max, elite):
    import torch
    rng = np.random.default_rng(pop + k_max)
    ea = ebic.EA(n_cols, pop, k_min, k_max, elite=elite, p_crossover=0.6, p_mutation=0.9, seed=3 * pop)
    try:
        host = ea.population()
        p = ctx.population(offsets=host[0], cols=host[1])
        for g in (1, 2, 3):
            announce("breed waves", n_cols, pop, k_min, k_max, elite, g)
            # few distinct counts: equal fitnesses rank by index
            m = rng.integers(-1, 6, size=pop).astype(np.int32)
            best_h, _ = ea.step(m)
            p, best = ctx.breed(ea.params, g, p, torch.from_numpy(m).to(ctx.device))
            torch.cuda.synchronize()
            host = ea.population()
            offs = to_np(p.offsets)
            assert int(best.cpu()[0]) == best_h
            assert np.array_equal(host[0], offs), f"generation {g}: offsets differ"
            assert np.array_equal(host[1], to_np(p.cols)[: int(offs[-1])]), f"generation {g}: columns differ"
    finally:
        ea.close()


@pytest.mark.parametrize("warm", [False, True])
def test_breeding_under_capture(ctx, warm):
    """Captured with and without the stream's scratch in place; replays with
    other counts in the same buffer equal the host's generations."""
    import torch
    n, n_cols = 800, 120
    rng = np.random.default_rng(9)
    ea = ebic.EA(n_cols, n, 2, 30, seed=17)
    try:
        offs, cols, _ = ea.population()
        p = ctx.population(offsets=offs, cols=cols)
        m = torch.zeros(n, dtype=torch.int32, device=ctx.device)
        out = (torch.zeros(n + 1, dtype=torch.int32, device=ctx.device),
               torch.zeros(n * 30, dtype=torch.int32, device=ctx.device),
               torch.zeros(1, dtype=torch.int32, device=ctx.device))
        s = torch.cuda.Stream()
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            if warm:
                ctx.breed(ea.params, 1, p, m, stream=s, out=out)
                s.synchronize()
            announce("breed capture", warm)
            graph.capture_begin()
            ctx.breed(ea.params, 1, p, m, stream=s, out=out)
            graph.capture_end()
        for rnd in range(3):
            counts = rng.integers(-1, 50, size=n).astype(np.int32)
            m.copy_(torch.from_numpy(counts))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            e = ebic.EA(n_cols, n, 2, 30, seed=17)
            best, _ = e.step(counts)
            ho, hc, _ = e.population()
            e.close()
            got = to_np(out[0])
            assert int(out[2].cpu()[0]) == best
            assert np.array_equal(ho, got) and np.array_equal(hc, to_np(out[1])[: int(got[-1])]), rnd
    finally:
        ea.close()
