"""A load whose copy to the device fails gives its device memory back.  Host
only: without a GPU every copy fails, so memory from a caller's allocator
(here host memory) is all that is taken."""
import ctypes

import numpy as np
import pytest
import torch


@pytest.mark.skipif(torch.cuda.is_available(), reason="the copy succeeds on a GPU")
@pytest.mark.parametrize("n,bad", [(1000, False), (70_000, False), (70_000, True),
                                   (3_000_000, False)])
def test_failed_load_frees_its_memory(n, bad):
    import paper_1807_07691_amd as G
    held = {}

    def alloc(size, stream):
        buf = ctypes.create_string_buffer(size)
        held[ctypes.addressof(buf)] = buf
        return ctypes.addressof(buf)

    def free(p, size, stream):
        assert len(held.pop(p)) == size

    r = np.random.default_rng(n)
    s, p, o = (r.integers(0, hi, n).astype(np.int32) for hi in (50, 7, 50))
    if bad:
        o[n // 2] = 50
    with pytest.raises(G.GsmatError) as e:
        G.gsmat_load_triples(s, p, o, 50, 7, allocator=G.make_allocator(alloc, free))
    assert e.value.status == (G.GSMAT_EINVAL if bad else G.GSMAT_EHIP)
    assert not held
