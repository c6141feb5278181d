"""Individuals finished together past the window, on panels that list tied
pairs: eight of uneven lengths, so that some are done while others still
compare, with the ties on late pairs of rows that follow the individuals in
either direction (a listed pair that went unseen would lose them).
Bit-exact against the oracle, in the two-kernel, one-kernel and batched
evaluation."""
import numpy as np
import pytest

from paper_1807_09932_amd import ebic, gen
from tests.gpu_common import announce, assert_same, gpu_eval, oracle_eval, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1807_09932_amd.ebic import Context
    c = Context(0)
    yield c
    c.close()


def _case(rows, cols, n):
    """Rows that rise or fall along `order`, each 2,048 of them with up to 32
    tied pairs of late neighbours; individuals of 2 .. cols columns."""
    rng = np.random.default_rng(rows + n)
    X = np.sort(rng.random((rows, cols)), axis=1)
    X[1::2] = -X[1::2]
    X = X.astype(np.float32)
    order = rng.permutation(cols)
    for chunk in range(0, rows, 2048):
        for t in range(int(rng.integers(1, 33))):
            r, j = int(rng.integers(chunk, min(rows, chunk + 2048))), int(rng.integers(8, cols - 1))
            X[r, j + 1] = X[r, j]
    Y = np.empty_like(X)
    Y[:, order] = X
    inds = []
    for i in range(n):
        k = (2, 9, 10, 12, 13, 17, 21, cols)[i % 8] if i < 16 else int(rng.integers(2, cols + 1))
        at = cols - k if i % 3 else int(rng.integers(0, cols - k + 1))
        c = order[at:at + k].astype(np.int32)
        inds.append(c[::-1].copy() if i % 2 else c)
    return Y, gen.csr(inds)


@pytest.mark.parametrize("rows,cols,n", [(1_000, 30, 8), (5_000, 40, 61), (34_000, 33, 130)])
def test_late_ties(ctx, rows, cols, n):
    import torch
    X, (offs, cc) = _case(rows, cols, n)
    want = oracle_eval(X, offs, cc)
    mat = ctx.upload(X)
    try:
        for shape in (None, (2, 16), (4, 256)):
            if shape:
                ctx.set_launch_shape(1, shape[0], shape[1], ebic.STAGE_PAIRS, 0)
            announce("late ties", rows, cols, n, shape)
            assert_same(gpu_eval(ctx, mat, offs, cc), want, f"{rows}x{cols} n={n} shape={shape}")
        ctx.set_launch_shape()
        pop = ctx.population(offsets=offs, cols=cc)
        outs = [ctx.outputs(mat, n, True) for _ in range(3)]
        announce("late ties, batched", rows, cols, n)
        ctx.eval_batch([ctx.request(mat, pop, o) for o in outs])
        torch.cuda.synchronize()
        for o in outs:
            assert_same(tuple(to_np(t) for t in o), want, f"{rows}x{cols} n={n} batched")
    finally:
        ctx.set_launch_shape()
        ctx.release(mat)
