"""Direct reads (the default past 512 columns) against the oracle, bit-exact:
row counts around the 4 rows of a lane, the 64-row padding and the 256-row
chunks (nine chunks: one past a multiple of eight), both missing-value modes
with the fill substituted on reading or kept as a copy, special values, with
and without negative trends and masks, individuals of one column to past the
window, repeats, invalid ones, and shapes down to one wave with more than the
64 individuals that it counts between two adds."""
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


def _population(rng, cols, order, n):
    inds = []
    for i in range(n):
        k = int(rng.integers(1, 31))
        c = rng.permutation(cols)[:k] if i % 3 else order[np.sort(rng.choice(order.size, min(k, order.size), replace=False))]
        c = [int(x) for x in c]
        if i % 9 == 0:
            c = [c[0], c[0]] + c
        if i % 11 == 0 and len(c) > 2:
            c = c[:2] + [c[1]] + c[2:]
        if i % 13 == 0:
            c = c[:1]
        if i % 17 == 0:
            c = c + [cols]  # invalid
        inds.append(np.asarray(c, np.int32))
    inds.append(np.asarray([], np.int32))
    return gen.csr(inds)


def _matrix(rng, rows, cols):
    X = np.round(rng.standard_normal((rows, cols)), 1).astype(np.float32)
    order = rng.permutation(cols)[:40]
    keep = np.arange(rows) % 3
    X[np.ix_(keep == 0, order)] = np.sort(X[np.ix_(keep == 0, order)], axis=1)   # chains that reach past the window
    X[np.ix_(keep == 1, order)] = -np.sort(-X[np.ix_(keep == 1, order)], axis=1)
    pick = rng.random(X.shape)
    X[pick < 0.01] = np.float32(-0.0)
    X[(pick >= 0.01) & (pick < 0.015)] = np.float32(np.inf)
    X[(pick >= 0.015) & (pick < 0.02)] = np.float32(-np.inf)
    X[(pick >= 0.02) & (pick < 0.03)] = np.float32(np.nan)
    return X, order


@pytest.mark.parametrize("rows", [1, 3, 63, 65, 255, 257, 8 * 256 + 66])
@pytest.mark.parametrize("keep", [False, True])
def test_direct_reads(ctx, rows, keep):
    rng = np.random.default_rng(rows)
    cols = 513 + rows % 7
    X, order = _matrix(rng, rows, cols)
    offs, cc = _population(rng, cols, order, 140)
    mat = ctx.upload(X, fill=0.25, keep_fill_copy=keep)
    try:
        assert ebic.ebic_plan_shape(ctx.handle, mat, offs.size - 1)[3] == ebic.STAGE_DIRECT
        for shape in (None, (1, 1), (1, 141), (16, 141), (3, 7)):
            if shape:
                ctx.set_launch_shape(1, shape[0], shape[1], ebic.STAGE_DIRECT, 0)
            for include in (False, True):
                for negative in (True, False):
                    announce("direct", rows, keep, shape, include, negative)
                    got = gpu_eval(ctx, mat, offs, cc, include=include, negative=negative, masks=True)
                    want = oracle_eval(X, offs, cc, include=include, negative=negative, masks=True, fill=0.25)
                    assert_same(got, want, f"rows={rows} shape={shape} include={include} negative={negative}")
    finally:
        ctx.set_launch_shape()
        ctx.release(mat)


def test_columns_past_four_gigabytes(ctx):
    """A matrix whose columns do not all start within 4 GB of the first takes
    64-bit addresses; compared with the oracle on the columns that are used."""
    import torch
    rows, cols = 1_100_003, 1_000
    g = torch.Generator(device="cuda").manual_seed(5)
    Xd = torch.empty(rows, cols, dtype=torch.float32, device="cuda").uniform_(-1, 1, generator=g)
    used = np.array([0, 1, 500, 975, 976, 977, 998, 999], np.int32)
    rng = np.random.default_rng(6)
    picks = [rng.permutation(used.size)[: int(rng.integers(1, used.size + 1))] for _ in range(40)]
    picks += [np.array([7]), np.array([0, 7]), np.arange(used.size)]
    X = Xd[:, torch.from_numpy(used.astype(np.int64)).cuda()].cpu().numpy()
    mat = ctx.upload(Xd)
    del Xd
    try:
        for negative in (True, False):
            announce("direct past 4 GB", rows, cols, negative)
            offs, cc = gen.csr([used[p] for p in picks])
            so, sc = gen.csr([p.astype(np.int32) for p in picks])
            got = gpu_eval(ctx, mat, offs, cc, negative=negative, masks=True)
            want = oracle_eval(np.ascontiguousarray(X), so, sc, negative=negative, masks=True)
            assert_same(got, want, f"{rows}x{cols} negative={negative}")
    finally:
        ctx.release(mat)
