"""block.merge_outputs takes what a loop over zip(outs, masks) takes: any iterables, up to the shorter one.  No GPU: the context
records what it is asked to do."""
import pytest
import torch

from paper_2302_02407_amd import block


class Recorder:
    N = 256

    def he_ptct_mac_rot(self, acc, cts, pts, galois, level, init=True):
        assert len(cts) == len(pts) == len(galois) and set(galois) <= {1} and init and acc.shape == (2, level + 1, self.N)
        self.terms = list(zip(cts, pts))
        return acc

    def he_rescale(self, ct, level, out):
        assert out.shape == (2, level, self.N)
        return out


class HostPool:
    def reset(self):
        pass

    def ct(self, level, N):
        return torch.empty((2, level + 1, N), dtype=torch.int64)


@pytest.mark.parametrize("outs,masks", [
    (lambda: ["a", "b", "c"], lambda: ["x", "y", "z"]),
    (lambda: (c for c in "abc"), lambda: (m for m in "xyz")),           # iterators
    (lambda: ["a", "b", "c", "d"], lambda: ["x", "y", "z"]),            # masks for the first three only
    (lambda: iter("abc"), lambda: list("xyzw")),
    (lambda: {"a": 0, "b": 0, "c": 0}.keys(), lambda: ("x", "y", "z")),  # sized, not a sequence
])
def test_merge_takes_any_iterables(outs, masks):
    ctx = Recorder()
    block.use_pool(HostPool())
    try:
        out = block.merge_outputs(ctx, outs(), masks(), 3)
    finally:
        block.use_pool(None)
    assert out.shape == (2, 3, 256) and ctx.terms == [("a", "x"), ("b", "y"), ("c", "z")]
