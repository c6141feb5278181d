"""The one-kernel evaluation of matrices of few panels (its blocks of eight
individuals take every panel), bit-exact against the oracle at its edges:
one panel and up to several slices, the counts of individuals and panels
where the rule changes the slices or leaves for the two kernels, ragged last
steps, listed ties and more ties than are listed, missing values in both
modes, malformed individuals, a captured call replayed on changed inputs, and
calls of different sizes on two streams that take turns with the slices'
accumulators."""
import numpy as np
import pytest

from paper_1807_09932_amd import gen
from tests.gpu_common import announce, assert_same, gpu_eval, oracle_eval

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1807_09932_amd.ebic import Context
    c = Context(0)
    yield c
    c.close()


def _matrix(rng, rows, cols, kind):
    X = (np.argsort(rng.random((rows, cols)), axis=1) + rng.random((rows, 1))).astype(np.float32)
    order = rng.permutation(cols).astype(np.int32)
    X[: rows // 2, order] = np.sort(X[: rows // 2], axis=1)
    X[rows // 2: 3 * rows // 4, order] = -np.sort(-X[rows // 2: 3 * rows // 4], axis=1)
    if kind == "listed":
        for r in range(0, rows, 701):
            X[r, r % cols] = X[r, (r + 1) % cols]
    elif kind == "tied":
        X[::3] = np.round(X[::3] / 4)
    elif kind == "missing":
        X[rng.random(X.shape) < 0.002] = np.nan
    return X, order


def _population(rng, cols, order, n, malformed=False):
    inds = []
    for i in range(n):
        k = int(rng.integers(1, min(cols, 40) + 1))
        c = order[np.sort(rng.choice(cols, k, replace=False))] if i % 2 else rng.permutation(cols)[:k].astype(np.int32)
        if malformed and i % 5 == 0:
            c = c.copy()
            c[k // 2] = cols if i % 2 else -1
        if malformed and i % 7 == 0:
            c = c[:0]
        inds.append(c)
    return gen.csr(inds)


@pytest.mark.parametrize("rows,cols,n,kind", [
    (1, 9, 1, "plain"), (1024, 16, 7, "listed"), (1025, 17, 9, "tied"), (5_000, 41, 4_097, "listed"),
    (12_483, 30, 2_048, "plain"), (12_483, 30, 2_057, "listed"), (16_385, 25, 65, "missing"),
    (32_767, 33, 130, "listed"), (32_768, 12, 33, "tied"), (32_769, 12, 33, "plain"), (20_011, 64, 257, "missing"),
    (4_096, 20, 300, "listed"), (4_097, 20, 300, "tied"), (8_193, 20, 4_096, "plain"), (54_675, 20, 1_201, "listed"),
    (131_072, 15, 120, "tied"), (131_073, 15, 120, "missing"), (524_288, 9, 9, "listed"), (524_289, 9, 9, "plain")])
def test_few_panels(ctx, rows, cols, n, kind):
    rng = np.random.default_rng(rows + n)
    X, order = _matrix(rng, rows, cols, kind)
    offs, cc = _population(rng, cols, order, n, malformed=kind in ("listed", "missing"))
    mat = ctx.upload(X)
    masks = n <= 300
    try:
        for include in ((False, True) if kind == "missing" else (False,)):
            for negative in (True, False):
                announce("few panels", rows, cols, n, kind, include, negative)
                got = gpu_eval(ctx, mat, offs, cc, include=include, negative=negative, masks=masks)
                want = oracle_eval(X, offs, cc, include=include, negative=negative, masks=masks)
                assert_same(got, want, f"{rows}x{cols} n={n} {kind} include={include} negative={negative}")
    finally:
        ctx.release(mat)


def test_few_panels_captured(ctx):
    """A captured call writes its counts afresh on each replay."""
    import torch
    rng = np.random.default_rng(3)
    rows, cols, n = 7_001, 40, 99
    X, order = _matrix(rng, rows, cols, "listed")
    pops = [_population(rng, cols, order, n) for _ in range(3)]
    nnz = min(int(o[-1]) for o, _ in pops)
    pops = [(np.minimum(o, nnz).astype(np.int32), c[:nnz]) for o, c in pops]  # (the same buffers; some become empty)
    mat = ctx.upload(X)
    try:
        pop = ctx.population(offsets=pops[0][0], cols=pops[0][1])
        out = ctx.outputs(mat, n, True)
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            ctx.eval(mat, pop, out=out, stream=s)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            ctx.eval(mat, pop, out=out, stream=s)
        for o, c in pops * 2:
            pop.offsets.copy_(torch.from_numpy(o))
            pop.cols.copy_(torch.from_numpy(c))
            for t in out:
                t.fill_(-7)
            torch.cuda.synchronize()
            announce("few panels: replay")
            g.replay()
            torch.cuda.synchronize()
            got = tuple(t.cpu().numpy() for t in out)
            got = got[:2] + tuple(t.view(np.uint64) for t in got[2:])
            assert_same(got, oracle_eval(X, o, c), "replay")
    finally:
        ctx.release(mat)


def test_few_panels_in_turn(ctx):
    """Calls of different sizes one after the other, on two streams, with a
    captured one between: each call's counts start from zero."""
    import torch
    rng = np.random.default_rng(4)
    rows, cols = 6_001, 30
    X, order = _matrix(rng, rows, cols, "listed")
    sizes = (4_096, 8, 100, 4_000, 1, 333)
    pops = [_population(rng, cols, order, n, malformed=n > 50) for n in sizes]
    want = [oracle_eval(X, o, c, masks=False) for o, c in pops]
    mat = ctx.upload(X)
    try:
        dev = [ctx.population(offsets=o, cols=c) for o, c in pops]
        streams = [torch.cuda.Stream() for _ in range(2)]
        torch.cuda.synchronize()
        out = ctx.outputs(mat, sizes[2])
        ctx.eval(mat, dev[1])  # (what a first call builds cannot be built in a capture)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=streams[0]):
            ctx.eval(mat, dev[2], out=out, stream=streams[0])
        for turn in range(3):
            got = []
            for i in range(len(sizes)):
                for k, s in enumerate(streams):
                    q = (i * (k + 1) + turn) % len(sizes)
                    announce("few panels in turn", turn, k, sizes[q])
                    with torch.cuda.stream(s):
                        got.append((q, ctx.eval(mat, dev[q], stream=s)))
            torch.cuda.synchronize()
            for t in out[:2]:
                t.fill_(-7)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            for q, o in got + [(2, out)]:
                assert_same((o[0].cpu().numpy(), o[1].cpu().numpy(), None, None), want[q], f"turn {turn} {sizes[q]}")
    finally:
        ctx.release(mat)
