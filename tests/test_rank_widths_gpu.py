"""Rank codes of every kind at the widths where their kernels change: a
half-wave's columns in runs of 16, eight and four with what is left over, the
block's waves (four, eight, 16), single rows and ragged 32-row blocks, rows
with one tie in their first or last columns (the tie flags come from the sum
of a row's counts), infinities, signed zeros and missing cells."""
import numpy as np
import pytest

from paper_1807_09932_amd import ebic, gen
from tests.gpu_common import announce, assert_same, gpu_eval, oracle_eval

pytestmark = pytest.mark.gpu

SHAPES = {"bytes": (4, 8, 64, ebic.STAGE_BYTES), "halves": (2, 8, 64, ebic.STAGE_HALVES),
          "tens": (3, 8, 64, ebic.STAGE_T10), "fp16": (4, 8, 64, ebic.STAGE_CODES)}
MOST = {"bytes": 128, "halves": 384, "tens": 512, "fp16": 384}


@pytest.fixture(scope="module")
def ctx():
    from paper_1807_09932_amd.ebic import Context
    c = Context(0)
    yield c
    c.close()


def _case(rows, cols, missing):
    rng = np.random.default_rng(1000 * rows + cols)
    X = (np.argsort(rng.random((rows, cols)), axis=1) - cols // 2).astype(np.float32)
    order = rng.permutation(cols).astype(np.int32)
    X[::2, order] = np.sort(X[::2], axis=1)
    if cols > 3:
        X[rows // 2, cols - 1] = X[rows // 2, cols - 2]
        X[rows - 1, 0] = X[rows - 1, 1]
        X[rows // 3, [0, cols - 1]] = (np.inf, -np.inf)
        X[rows // 4, [0, 2]] = (0.0, -0.0)
    if missing:
        X[rng.random(X.shape) < 0.03] = np.nan
    inds = []
    for i in range(60):
        k = int(rng.integers(1, min(cols, 12) + 1))
        inds.append(order[np.sort(rng.choice(cols, k, replace=False))] if i % 2
                    else rng.permutation(cols)[:k].astype(np.int32))
    return X, gen.csr(inds)


@pytest.mark.parametrize("kind", sorted(SHAPES))
@pytest.mark.parametrize("rows,cols", [(1, 1), (31, 5), (33, 29), (65, 97), (193, 128), (577, 129), (1025, 193),
                                       (95, 320), (161, 321), (64, 384), (225, 385), (127, 512)])
def test_rank_widths(ctx, rows, cols, kind):
    if cols > MOST[kind] or (kind == "tens" and cols <= 128):
        cols = MOST[kind] - 1 if cols > MOST[kind] else cols + 128
    for missing in (False, True):
        X, (offs, cc) = _case(rows, cols, missing)
        mat = ctx.upload(X, fill=0.5, keep_fill_copy=True)
        try:
            ctx.set_launch_shape(*SHAPES[kind], 0)
            for include in (False, True) if missing else (False,):
                announce("rank widths", rows, cols, kind, missing, include)
                got = gpu_eval(ctx, mat, offs, cc, include=include)
                want = oracle_eval(X, offs, cc, include=include, fill=0.5)
                assert_same(got, want, f"{rows}x{cols} {kind} missing={missing} include={include}")
            assert ctx.stats(mat)["has_missing"] in (-1, int(missing and np.isnan(X).any()))
        finally:
            ctx.set_launch_shape()
            ctx.release(mat)
