"""Device memory hooks for tests: count what the library holds, refuse chosen
allocations, or keep it within a budget (scan_set_allocator; the memory itself
comes from PyTorch's caching allocator)."""

from __future__ import annotations

import contextlib

import paper_2012_11188_amd as scan


class Hooks:
    def __init__(self):
        self.live = {}  # pointer -> bytes
        self.held = self.peak = self.calls = 0
        self.refuse = frozenset()  # allocation calls (numbered from 0) that get nothing
        self.budget = None         # most bytes held

    def start(self, refuse=(), budget=None):
        """Counts from here on; returns self."""
        self.calls, self.peak = 0, self.held
        self.refuse, self.budget = frozenset(refuse), budget
        return self

    def alloc(self, nbytes, stream, ctx):
        import torch

        call, self.calls = self.calls, self.calls + 1
        if call in self.refuse or (self.budget is not None and self.held + nbytes > self.budget):
            return None
        p = torch.cuda.caching_allocator_alloc(int(nbytes), torch.cuda.current_device(), int(stream or 0))
        self.live[p] = int(nbytes)
        self.held += int(nbytes)
        self.peak = max(self.peak, self.held)
        return p

    def release(self, ptr, nbytes, stream, ctx):
        import torch

        self.held -= self.live.pop(ptr)
        torch.cuda.caching_allocator_delete(ptr)


@contextlib.contextmanager
def hooks():
    """The library's allocations go through a Hooks while the block runs; what
    it made inside must be freed inside."""
    h = Hooks()
    scan._ready()
    fns = scan._ALLOC_FN(h.alloc), scan._RELEASE_FN(h.release)
    scan._check(scan.load_library().scan_set_allocator(fns[0], fns[1], None))
    try:
        yield h
    finally:
        scan.use_torch_allocator(True)
    assert not h.live
