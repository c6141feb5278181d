"""Uploads at the edges of their chunks (8 MB from host memory, a quarter of
that first, whole 1,536-row units where rank codes are made): exactly one
chunk, one row more, and more chunks than there are buffers, row-major,
strided and column-major, each bit-exact against the oracle with the codes
and the bitmaps, and with rows of the last chunk tied or missing."""
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


def _chunk(cols):
    unit = 1536 if cols <= 512 else 64
    return max(1, (8 << 20) // (4 * cols) // unit) * unit


@pytest.mark.parametrize("cols", [100, 200, 600])
@pytest.mark.parametrize("chunks,more", [(1, 0), (1, 1), (1.25, 0), (1.25, 31), (5.25, 0), (6.25, -1)])
@pytest.mark.parametrize("order", ["rows", "strided", "columns"])
def test_upload_chunks(ctx, cols, chunks, more, order):
    chunk = _chunk(cols)
    unit = 1536 if cols <= 512 else 64
    rows = int(chunks) * chunk + (chunk // 4 // unit * unit if chunks != int(chunks) else 0) + more
    rng = np.random.default_rng(rows + cols)
    X = rng.standard_normal((rows, cols)).astype(np.float32)
    X[rows - 1, 1] = X[rows - 1, 0]
    X[rows // 2, 2] = -999.0
    inds = [rng.permutation(cols)[: int(rng.integers(1, 5))].astype(np.int32) for _ in range(24)]
    inds += [np.array(c, np.int32) for c in ([0, 1], [1, 0], [2, 3], [3, 2])]
    offs, cc = gen.csr(inds)
    want = oracle_eval(X, offs, cc, include=True, sentinel=-999.0, fill=0.25)
    if order == "strided":
        wide = np.full((rows, cols + 3), 7.0, np.float32)
        wide[:, :cols] = X
        src = wide[:, :cols]
    else:
        src = np.asfortranarray(X) if order == "columns" else X
    announce("upload chunks", cols, rows, order)
    mat = ctx.upload(src, sentinel=-999.0, fill=0.25)
    try:
        shapes = [None]
        if order == "rows" and cols <= 512:
            shapes.append((4, 8, 64, ebic.STAGE_BYTES) if cols <= 128 else (3, 8, 64, ebic.STAGE_T10))
        for shape in shapes:
            if shape:
                ctx.set_launch_shape(*shape, 0)
            assert_same(gpu_eval(ctx, mat, offs, cc, include=True), want, f"{rows}x{cols} {order} {shape}")
        assert ctx.stats(mat)["has_missing"] == (1 if cols <= 512 else -1)
    finally:
        ctx.set_launch_shape()
        ctx.release(mat)
