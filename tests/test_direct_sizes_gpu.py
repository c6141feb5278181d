"""Direct reads at the sizes where their arithmetic changes: a matrix of 2 to
4 GiB, whose 32-bit offsets and size have the highest bit set, and populations
whose groups would pass a grid's 2^32 threads (there also the pair bitmaps)."""
import numpy as np
import pytest

from paper_1807_09932_amd import ebic, gen
from tests.gpu_common import announce, assert_same, gpu_eval, oracle_eval

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1807_09932_amd.ebic import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("rows,cols", [(700_003, 1_000), (2_000_001, 536)])
def test_columns_between_two_and_four_gigabytes(ctx, rows, cols):
    """Compared with the oracle on the columns that are used: the first and
    last ones, and those on both sides of 2 GiB."""
    import torch
    ld = (rows + 63) // 64 * 64
    assert 1 << 31 < ld * cols * 4 < 1 << 32
    half = (1 << 31) // (ld * 4)  # the column that 2 GiB falls in
    g = torch.Generator(device="cuda").manual_seed(7)
    Xd = torch.empty(rows, cols, dtype=torch.float32, device="cuda").uniform_(-1, 1, generator=g)
    used = np.array([0, 1, half - 1, half, half + 1, cols - 3, cols - 2, cols - 1], np.int32)
    rng = np.random.default_rng(8)
    picks = [rng.permutation(used.size)[: int(rng.integers(1, used.size + 1))] for _ in range(40)]
    picks += [np.array([7]), np.array([0, 7]), np.arange(used.size)]
    X = Xd[:, torch.from_numpy(used.astype(np.int64)).cuda()].cpu().numpy()
    mat = ctx.upload(Xd)
    del Xd
    try:
        for negative in (True, False):
            announce("direct, 2 to 4 GiB", rows, cols, negative)
            offs, cc = gen.csr([used[p] for p in picks])
            so, sc = gen.csr([p.astype(np.int32) for p in picks])
            got = gpu_eval(ctx, mat, offs, cc, negative=negative, masks=True)
            want = oracle_eval(np.ascontiguousarray(X), so, sc, negative=negative, masks=True)
            assert_same(got, want, f"{rows}x{cols} negative={negative}")
    finally:
        ctx.release(mat)


@pytest.mark.parametrize("cols,n,shape", [
    (520, 34_000_000, None),                      # the default shape's 16 individuals per group
    (520, 600_000, (16, 1, ebic.STAGE_DIRECT)),
    (40, 600_000, (16, 1, ebic.STAGE_PAIRS)),
    (40, 600_000, (16, 1000, ebic.STAGE_PAIRS)),
])
def test_populations_past_the_grid(ctx, cols, n, shape):
    """Pairs of columns on rows without ties: every row rises or falls, and
    the number that falls is a table's entry (plain torch)."""
    import torch
    rows = 64
    g = torch.Generator(device="cuda").manual_seed(9)
    X = torch.rand(rows, cols, generator=g, device="cuda").argsort(1).argsort(1).float()
    a = torch.randint(0, cols, (n,), generator=g, device="cuda", dtype=torch.int32)
    b = (a + torch.randint(1, cols, (n,), generator=g, device="cuda", dtype=torch.int32)) % cols
    falls = (X[:, None, :] < X[:, :, None]).sum(0, dtype=torch.int32)
    pop = ebic.Population(torch.arange(0, 2 * n + 1, 2, dtype=torch.int32, device="cuda"),
                          torch.stack([a, b], 1).view(-1))
    mat = ctx.upload(X)
    try:
        if shape:
            ctx.set_launch_shape(1, shape[0], shape[1], shape[2], 0)
        announce("past the grid", cols, n, shape)
        m, neg, _, _ = ctx.eval(mat, pop, negative=True)
        assert bool((m == rows).all())
        assert bool((neg == falls.view(-1)[a.long() * cols + b.long()]).all())
    finally:
        ctx.set_launch_shape()
        ctx.release(mat)
