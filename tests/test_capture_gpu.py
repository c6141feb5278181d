"""What a call under a stream capture cannot do, and how it leaves what it
touched: a layout built on first use is waited for before its memory goes, and
an upload is refused before anything joins the capture."""
import ctypes

import numpy as np
import pytest

from paper_1807_09932_amd import ebic, gen
from tests.gpu_common import announce, assert_same, gpu_eval, oracle_eval, to_np

pytestmark = pytest.mark.gpu

GLOBAL, THREAD_LOCAL, RELAXED = 0, 1, 2


class _Capture:
    """A capture through HIP itself (torch's allocator keeps out of it)."""

    def __init__(self, stream, mode):
        path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64.so" in line)
        self.hip, self.stream, self.mode = ctypes.CDLL(path), ctypes.c_void_p(stream.cuda_stream), mode

    def __enter__(self):
        assert self.hip.hipStreamBeginCapture(self.stream, self.mode) == 0
        return self

    def __exit__(self, *exc):
        graph = ctypes.c_void_p()
        self.status = self.hip.hipStreamEndCapture(self.stream, ctypes.byref(graph))
        if self.status == 0 and graph.value:
            self.hip.hipGraphDestroy(graph)
        self.hip.hipGetLastError()


def test_failed_first_use_is_waited_for():
    """The first evaluation of a matrix, in a capture: where the build of its
    bitmaps fails, it has ended before its memory goes back."""
    import torch
    rows, cols = 200_000, 300
    rng = np.random.default_rng(1)
    X = rng.random((rows, cols), dtype=np.float32)
    offs, cc = gen.csr([rng.permutation(cols)[:5].astype(np.int32) for _ in range(50)])
    size = cols * cols * -(-rows // 2048) * 256
    keep, seen, copy = {}, [], torch.zeros(size, dtype=torch.uint8, device="cuda")
    spare = [torch.zeros(2 * size, dtype=torch.uint8, device="cuda")]
    side, s = torch.cuda.Stream(), torch.cuda.Stream()
    torch.add(copy[:8], 0, out=copy[:8])

    def alloc(nbytes, _user):
        t = spare.pop() if nbytes > size // 2 and capturing and spare else torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
        keep[t.data_ptr()] = (t, nbytes)
        return t.data_ptr()

    def release(ptr, _user):
        if capturing and keep[ptr][1] > size // 2:
            c.hip.hipGetLastError()  # (of the wait that was refused)
            with torch.cuda.stream(side):
                torch.add(keep[ptr][0][:size], 0, out=copy)  # (what is there now, by a kernel)
            seen.append(keep[ptr][0])

    capturing = False
    ctx = ebic.Context(0, torch_allocator=False)
    try:
        hooks = ebic.ALLOC_FN(alloc), ebic.RELEASE_FN(release)
        ebic.ebic_set_allocator(ctx.handle, *hooks)
        mat = ctx.upload(X)
        pop = ctx.population(offsets=offs, cols=cc)
        out = ctx.outputs(mat, 50)
        torch.cuda.synchronize()
        announce("first use in a capture")
        capturing = True
        with _Capture(s, GLOBAL) as c:
            try:
                ctx.eval(mat, pop, out=out, stream=s)
                failed = False
            except ebic.EbicError:
                failed = True
        capturing = False
        torch.cuda.synchronize()
        if failed:
            assert len(seen) == 1
            assert bool((copy == seen[0][:size]).all())
        assert_same(gpu_eval(ctx, mat, offs, cc, masks=False), oracle_eval(X, offs, cc, masks=False), "afterwards")
    finally:
        ctx.close()


@pytest.mark.parametrize("where", ["host", "device"])
def test_upload_in_a_capture(where):
    """Refused as ever, with the capture left intact; uploads and first uses
    go on beside it and after it."""
    import torch
    rng = np.random.default_rng(2)
    X = rng.random((60_000, 150), dtype=np.float32)  # (36 MB: several chunks)
    offs, cc = gen.csr([rng.permutation(150)[:5].astype(np.int32) for _ in range(50)])
    want = oracle_eval(X, offs, cc, masks=False)
    src = torch.from_numpy(X).cuda() if where == "device" else X
    ctx, s, side = ebic.Context(0), torch.cuda.Stream(), torch.cuda.Stream()
    try:
        first = ctx.upload(X)  # (its bitmaps are not built yet)
        pop, out = ctx.population(offsets=offs, cols=cc), ctx.outputs(first, 50)
        torch.cuda.synchronize()
        announce("upload in a capture", where)
        with _Capture(s, RELAXED) as c:
            with pytest.raises(ebic.EbicError) as e:
                ctx.upload(src, stream=s)
            assert e.value.status == ebic.EBIC_EHIP
            ctx.eval(first, pop, out=out, stream=side)
        assert c.status == 0
        torch.cuda.synchronize()
        assert_same((to_np(out[0]), to_np(out[1]), None, None), want, "beside the capture")
        second = ctx.upload(src, stream=s)
        assert_same(gpu_eval(ctx, second, offs, cc, masks=False), want, "after it")
    finally:
        ctx.close()
