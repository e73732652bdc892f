"""Read-outs into memory of every kind a C caller may pass."""
import ctypes as C

import numpy as np
import pytest

from paper_1507_07294_amd import mplb
from paper_1507_07294_amd import workloads as wl

pytestmark = pytest.mark.gpu


def test_read_into_page_locked_memory_equals_pageable():
    """Fields on both sides of the staging's limit (1.5 MB) and of the threads'
    (6 MB), at the start of a page-locked block and within it."""
    import torch

    for shape in ((57, 57, 57), (60, 60, 60), (96, 96, 96)):
        w = wl.static_droplet(n=8)
        w.shape, w.phi0 = shape, np.random.default_rng(5).uniform(-1, 1, shape[::-1])
        lt = mplb.from_workload(w, "f64")
        want = lt.read("phi")
        block = torch.full((lt.N + 1000,), 7.0, dtype=torch.float64, pin_memory=True)
        for at in (0, 999):
            block.fill_(7.0)
            out = block[at:at + lt.N]
            rc = mplb.lib().mplb_read(lt.handle, mplb.MPLB_PHI, C.cast(out.data_ptr(), C.POINTER(C.c_double)))
            assert rc == 0 and np.array_equal(out.numpy(), want.ravel())
            assert (block[:at] == 7.0).all() and (block[at + lt.N:] == 7.0).all()
        lt.destroy()
