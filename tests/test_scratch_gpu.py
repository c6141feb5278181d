"""The device memory that calls on a stream share (headers, children's slots):
which calls keep out of it."""
import ctypes
import gc
import threading

import numpy as np
import pytest

from paper_1807_09932_amd import ebic, gen
from tests.gpu_common import announce, assert_same, oracle_eval, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture()
def ctx():
    from paper_1807_09932_amd.ebic import Context
    c = Context(0)
    yield c
    c.close()


@pytest.fixture(autouse=True)
def _no_garbage():
    """Device memory in reference cycles goes with the test that made it."""
    yield
    gc.collect()


class _Breeding:
    """A generation of n individuals and the buffers of the next one."""

    def __init__(self, ctx, n, seed, n_cols=120, k_max=30):
        import torch
        self.n, self.n_cols, self.k_max, self.seed = n, n_cols, k_max, seed
        ea = ebic.EA(n_cols, n, 2, k_max, seed=seed)
        offs, cols, _ = ea.population()
        self.params = ea.params
        ea.close()
        self.pop = ctx.population(offsets=offs, cols=cols)
        self.matched = torch.zeros(n, dtype=torch.int32, device=ctx.device)
        self.out = (torch.zeros(n + 1, dtype=torch.int32, device=ctx.device),
                    torch.zeros(n * k_max, dtype=torch.int32, device=ctx.device),
                    torch.zeros(1, dtype=torch.int32, device=ctx.device))

    def breed(self, ctx, stream):
        ctx.breed(self.params, 1, self.pop, self.matched, stream=stream, out=self.out)

    def set_counts(self, counts):
        import torch
        self.counts = counts
        self.matched.copy_(torch.from_numpy(counts))

    def check(self, what):
        ea = ebic.EA(self.n_cols, self.n, 2, self.k_max, seed=self.seed)
        best, _ = ea.step(self.counts)
        offs, cols, _ = ea.population()
        ea.close()
        got = to_np(self.out[0])
        assert int(self.out[2].cpu()[0]) == best, what
        assert np.array_equal(offs, got) and np.array_equal(cols, to_np(self.out[1])[: int(got[-1])]), what


def _graph_nodes(graph):
    """The number of nodes of a captured graph."""
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64.so" in line)
    n = ctypes.c_size_t(0)
    assert ctypes.CDLL(path).hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("n", [2, 800, 1024])
def test_captured_small_breeding_holds_no_scratch(ctx, n):
    """A captured breeding of up to 1,024 individuals is one kernel on the
    caller's buffers, though the stream has scratch: replays stay right when
    the scratch has been replaced, and beside calls that write it."""
    import torch
    rng = np.random.default_rng(n)
    b = _Breeding(ctx, n, seed=n)
    large = _Breeding(ctx, 5000, seed=5)
    s, other = torch.cuda.Stream(), torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        b.breed(ctx, s)
        s.synchronize()
        announce("capture with scratch in place", n)
        graph.capture_begin()
        b.breed(ctx, s)
        graph.capture_end()
    assert _graph_nodes(graph) == 1
    for rnd in range(3):
        b.set_counts(rng.integers(-1, 50, size=n).astype(np.int32))
        large.set_counts(rng.integers(-1, 50, size=5000).astype(np.int32))
        torch.cuda.synchronize()
        announce("replay beside a larger breeding", n, rnd)
        large.breed(ctx, s)  # (the first one replaces the scratch)
        with torch.cuda.stream(other):
            graph.replay()
        torch.cuda.synchronize()
        b.check(rnd)
        large.check(rnd)


class _Allocator:
    """Device memory from torch, counted; `make` changes what is returned."""

    def __init__(self, make=lambda address: address):
        import torch
        self.blocks, self.calls = {}, 0

        def alloc(nbytes, _user):
            self.calls += 1
            t = torch.empty(int(nbytes) + 256, dtype=torch.uint8, device="cuda")
            at = make(t.data_ptr())
            self.blocks[at] = t
            return at

        def release(ptr, _user):
            del self.blocks[ptr]

        self.alloc, self.release = ebic.ALLOC_FN(alloc), ebic.RELEASE_FN(release)


PER_THREAD = 2  # hipStreamPerThread


def test_small_breeding_on_the_per_thread_stream():
    """One handle stands for a stream of each thread: populations of up to
    1,024 keep out of the memory that is kept by handle."""
    import torch
    ctx = ebic.Context(0, torch_allocator=False)
    memory = _Allocator()
    try:
        ebic.ebic_set_allocator(ctx.handle, memory.alloc, memory.release)
        rng = np.random.default_rng(1)
        bs = [_Breeding(ctx, n, seed=n) for n in (700, 1024)]
        for b in bs:
            b.set_counts(rng.integers(-1, 50, size=b.n).astype(np.int32))
        torch.cuda.synchronize()

        def breed(b, times):
            for _ in range(times):
                ebic.ebic_ea_breed(ctx.handle, b.params, 1, b.n, b.pop.offsets.data_ptr(), b.pop.cols.data_ptr(),
                                   b.matched.data_ptr(), *(t.data_ptr() for t in b.out), PER_THREAD)
            # (a thread's stream goes with it: waited for by itself)
            torch.cuda.ExternalStream(PER_THREAD).synchronize()

        announce("per-thread stream, one thread")
        breed(bs[0], 1)
        assert memory.calls == 0
        bs[0].check("one thread")
        announce("per-thread stream, two threads")
        threads = [threading.Thread(target=breed, args=(b, 50)) for b in bs]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        for b in bs:
            b.check("two threads")
    finally:
        ctx.close()


@pytest.mark.parametrize("what", ["breeding", "evaluation"])
def test_captured_scratch_outlives_its_replacement(what):
    """The scratch that a captured call was given is not released when a
    larger call on the stream replaces it: replays write it."""
    import torch
    rng = np.random.default_rng(2)
    ctx = ebic.Context(0, torch_allocator=False)
    memory = _Allocator()
    try:
        ebic.ebic_set_allocator(ctx.handle, memory.alloc, memory.release)
        small, large = _Breeding(ctx, 1500, seed=3), _Breeding(ctx, 9000, seed=4)
        for b in (small, large):
            b.set_counts(rng.integers(-1, 50, size=b.n).astype(np.int32))
        if what == "evaluation":  # (40 panels and no accumulators: two kernels with the headers between them)
            X = rng.standard_normal((40_000, 20)).astype(np.float32)
            offs, cols = gen.csr([rng.permutation(20)[:k].astype(np.int32) for k in rng.integers(1, 12, size=100)])
            mat, pop = ctx.upload(X), ctx.population(offsets=offs, cols=cols)
            out = ctx.outputs(mat, 100)
            want = oracle_eval(X, offs, cols, masks=False)

        def call(s):
            if what == "evaluation":
                ctx.eval(mat, pop, out=out, stream=s)
            else:
                small.breed(ctx, s)

        s = torch.cuda.Stream()
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            call(s)  # (builds what a capture cannot)
            small.breed(ctx, s)
            s.synchronize()
            announce("capture", what)
            graph.capture_begin()
            call(s)
            graph.capture_end()
        held = set(memory.blocks)
        for rnd in range(3):
            for b in (small, large):
                b.set_counts(rng.integers(-1, 50, size=b.n).astype(np.int32))
            torch.cuda.synchronize()
            large.breed(ctx, s)  # (replaces the scratch the first time)
            assert held < set(memory.blocks)
            announce("replay on the replaced scratch", what, rnd)
            with torch.cuda.stream(s):
                graph.replay()
            torch.cuda.synchronize()
            large.check(rnd)
            if what == "evaluation":
                assert_same((to_np(out[0]), to_np(out[1]), None, None), want, "replay")
            else:
                small.check(rnd)
    finally:
        ctx.close()
    assert not memory.blocks


@pytest.mark.parametrize("why,make", [("unaligned memory", lambda address: address + 8), ("no memory", lambda _: None)])
def test_small_breeding_without_memory(why, make):
    """A population of up to 1,024 is bred whatever the allocator does."""
    import torch
    ctx = ebic.Context(0, torch_allocator=False)
    memory = _Allocator(make)
    try:
        ebic.ebic_set_allocator(ctx.handle, memory.alloc, memory.release)
        b = _Breeding(ctx, 600, seed=6)
        b.set_counts(np.random.default_rng(6).integers(-1, 50, size=600).astype(np.int32))
        announce("breeding without memory", why)
        b.breed(ctx, None)
        torch.cuda.synchronize()
        assert memory.calls >= 1
        b.check(why)
    finally:
        ctx.close()


def test_allocator_changes_after_a_small_breeding():
    """With no matrix resident the allocator may change; the scratch of a
    breeding that could do without goes back to the one that made it. One of a
    larger population stays in use."""
    import torch
    ctx = ebic.Context(0, torch_allocator=False)
    first, second = _Allocator(), _Allocator()
    rng = np.random.default_rng(7)
    try:
        ebic.ebic_set_allocator(ctx.handle, first.alloc, first.release)
        small, large = _Breeding(ctx, 1000, seed=8), _Breeding(ctx, 1500, seed=9)
        for b in (small, large):
            b.set_counts(rng.integers(-1, 50, size=b.n).astype(np.int32))
        for memory in (first, second):
            announce("breed, then change the allocator")
            small.breed(ctx, None)
            assert memory.calls == 1
            ebic.ebic_set_allocator(ctx.handle, second.alloc, second.release)
            assert not memory.blocks
            torch.cuda.synchronize()
            small.check("small")
        large.breed(ctx, None)
        with pytest.raises(ebic.EbicError) as e:
            ebic.ebic_set_allocator(ctx.handle, first.alloc, first.release)
        assert e.value.status == ebic.EBIC_EBUSY
        torch.cuda.synchronize()
        large.check("large")
    finally:
        ctx.close()
    assert first.calls == 1 and not second.blocks
