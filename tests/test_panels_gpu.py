"""The pair-bitmap kernels at their own edges, bit-exact against the oracle:
rows around the 1,024-row panels, widths around the build's tiles (16 columns
a, runs of columns b, four staged together), chunks with exactly as many tied
pairs as their list holds and with one more, individuals that all wait for
their columns past the window (more and fewer than a step's eight), and a
batch long enough that its items are taken from the lists' counters."""
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


def _tie_free(rng, rows, cols):
    """Distinct values in every row (permuted ranks, shifted per row)."""
    X = np.argsort(rng.random((rows, cols)), axis=1).astype(np.float32)
    return X + rng.random((rows, 1)).astype(np.float32)


def _population(rng, cols, order, n):
    """Half along `order` (rows survive to the last column), half random."""
    inds = []
    for i in range(n):
        k = int(rng.integers(1, min(cols, 30) + 1))
        if i % 2:
            inds.append(order[np.sort(rng.choice(cols, k, replace=False))])
        else:
            inds.append(rng.permutation(cols)[:k].astype(np.int32))
    return gen.csr(inds)


@pytest.mark.parametrize("rows,cols", [(1023, 16), (1024, 17), (1025, 33), (3073, 49), (2048 * 9 + 5, 65)])
@pytest.mark.parametrize("tied", [0, 32, 33])
def test_panel_edges(ctx, rows, cols, tied):
    rng = np.random.default_rng(rows + tied)
    X = _tie_free(rng, rows, cols)
    order = rng.permutation(cols).astype(np.int32)
    half, more = rows // 2, rows // 2 + rows // 4
    X[:half, order] = np.sort(X[:half], axis=1)
    X[half:more, order] = -np.sort(-X[half:more], axis=1)
    # `tied` distinct pairs of the first chunk, on its last rows
    pairs = [(a, b) for a in range(cols) for b in range(a + 1, cols)]
    last = min(rows, 2048)
    for t, p in enumerate(rng.choice(len(pairs), size=min(tied, len(pairs)), replace=False)):
        a, b = pairs[p]
        X[last - 1 - t, a] = X[last - 1 - t, b]
    offs, cc = _population(rng, cols, order, 75)
    mat = ctx.upload(X)
    try:
        for shape in ((1, 1, 1), (1, 1, 9), (1, 2, 32), (1, 1, 64), (1, 3, 75)):
            ctx.set_launch_shape(1, shape[1], shape[2], ebic.STAGE_PAIRS, 0)
            for negative in (True, False):
                announce("panels", rows, cols, tied, shape, negative)
                got = gpu_eval(ctx, mat, offs, cc, negative=negative, masks=True)
                want = oracle_eval(X, offs, cc, negative=negative, masks=True)
                assert_same(got, want, f"rows={rows} cols={cols} tied={tied} {shape} negative={negative}")
    finally:
        ctx.set_launch_shape()
        ctx.release(mat)


def test_long_lists(ctx):
    """Enough items per list that blocks take them from the counters, with
    short lists in between on the same graph (the counters start over)."""
    import torch
    rng = np.random.default_rng(6)
    rows, cols = 60_001, 40
    X = _tie_free(rng, rows, cols)
    mat = ctx.upload(X)
    pops = [_population(rng, cols, rng.permutation(cols).astype(np.int32), n) for n in (700, 41, 650, 900)]
    want = [oracle_eval(X, o, c, masks=False) for o, c in pops]
    dev = [ctx.population(offsets=o, cols=c) for o, c in pops]
    try:
        ctx.set_launch_shape(1, 1, 1, ebic.STAGE_PAIRS, 0)  # an item per individual and panel
        for pick in ((0, 1, 2, 3), (1,), (3, 2, 0), (1,), (0, 1, 2, 3)):
            outs = [ctx.outputs(mat, dev[q].n) for q in pick]
            announce("long lists", pick)
            ctx.eval_batch([ctx.request(mat, dev[q], o) for q, o in zip(pick, outs)])
            torch.cuda.synchronize()
            for q, o in zip(pick, outs):
                assert_same((o[0].cpu().numpy(), o[1].cpu().numpy(), None, None), want[q], f"{pick} {q}")
    finally:
        ctx.set_launch_shape()
        ctx.release(mat)


@pytest.mark.parametrize("kind", ["finite", "infinite", "late"])
def test_order_words_of_special_values(ctx, kind):
    """The build compares by the sign of differences where no infinity has
    been staged: signed zeros, subnormal neighbours, differences that
    overflow, neighbouring floats; with infinities, from the first column on
    or in the last one only, by comparisons."""
    rng = np.random.default_rng(8)
    rows, cols = 2_300, 37
    big, tiny = np.finfo(np.float32).max, np.float32(1e-45)
    values = np.array([0.0, -0.0, tiny, -tiny, 2 * tiny, np.finfo(np.float32).tiny, big, -big, 1.0,
                       np.nextafter(np.float32(1), np.float32(2)), -1.0, 3e38], np.float32)
    X = _tie_free(rng, rows, cols)
    X[::7] = rng.choice(values, size=X[::7].shape)
    X[5, :5] = (1.0, np.nextafter(np.float32(1), np.float32(2)), -0.0, 0.0, tiny)
    if kind == "infinite":
        X[::5, ::3] = np.inf
        X[1::5, 1::4] = -np.inf
    elif kind == "late":
        X[::3, cols - 1] = np.inf
        X[1::9, cols - 2] = np.inf
    offs, cc = _population(rng, cols, rng.permutation(cols).astype(np.int32), 160)
    mat = ctx.upload(X)
    try:
        for negative in (True, False):
            announce("special order words", kind, negative)
            got = gpu_eval(ctx, mat, offs, cc, negative=negative, masks=True)
            assert_same(got, oracle_eval(X, offs, cc, negative=negative, masks=True), f"{kind} negative={negative}")
    finally:
        ctx.release(mat)
