"""Ordered scans beside a kernel that holds half of the compute units: they are exact, and through while it still holds them
(a workgroup that waited for one that cannot run yet would wait as long as the other kernel)."""
import ctypes as C
import os
import time

import numpy as np
import pytest

import oracle as orc

pytestmark = pytest.mark.gpu

SUB = 512
UNITS, HOLD_MS = 128, 20  # a scan takes well below a millisecond, also on the other half
LIB = os.path.join(os.path.dirname(os.path.abspath(__file__)), "toy_graph", "libtoy_graph.so")


class Holder:
    def __init__(self):
        import torch

        self.torch = torch
        self.call = C.CDLL(LIB).hold_units
        self.call.argtypes = [C.c_uint32, C.c_uint64, C.c_void_p, C.c_void_p]
        self.looks = torch.zeros(UNITS, dtype=torch.int32, device="cuda:0")
        self.end = torch.cuda.Event()
        # a stream that does not share a hardware queue with the default one
        for _ in range(8):
            self.stream = torch.cuda.Stream()
            self.begin(5)
            self.looks.sum()
            torch.cuda.current_stream().synchronize()
            apart = not self.end.query()
            torch.cuda.synchronize()
            if apart:
                return
        pytest.fail("no stream runs beside the default one")

    def begin(self, ms):
        rc = self.call(UNITS, ms * 100_000, self.looks.data_ptr(), self.stream.cuda_stream)
        assert rc == 0
        self.end.record(self.stream)
        time.sleep(0.001)


@pytest.fixture(scope="module")
def holder():
    return Holder()


@pytest.mark.parametrize("n_alloc", [300, 20000, 140000])  # level 0 alone, lines, nodes
@pytest.mark.parametrize("n", [40 * SUB + 3, 1500 * SUB, 3000 * SUB, 12000 * SUB + 511])
def test_scans_beside_a_kernel_that_holds_units(holder, n_alloc, n):
    import torch

    from tests.support import session
    from tests.test_gpu_flat_scan import table_of, words_of
    from tests.test_gpu_parity import oracle_rebase

    rng = np.random.default_rng(n_alloc + n)
    t = table_of(rng, n_alloc, "spread")
    words = words_of(rng, n, t, 0.25)
    new_base = rng.integers(0, 1 << 63, n_alloc, dtype=np.uint64)
    units = words.view(np.uint32)[1:]
    ref, cnt = orc.scan(words, t)
    ref4, cnt4 = orc.scan_stride4(units, t)
    out, _ = oracle_rebase(orc, words, t, new_base)
    for run, want in ((session.ScanRun(words, t, prepared=True), (ref, cnt, 0)),
                      (session.ScanStride4Run(units, t), (ref4, cnt4, 0)),
                      (session.ScanPointersRebaseRun(words, t, new_base, prepared=True), (ref, cnt, 0, out))):
        run.launch()  # (loads the kernels)
        torch.cuda.synchronize()
        holder.begin(HOLD_MS)
        run.launch()
        torch.cuda.current_stream().synchronize()
        early = not holder.end.query()
        got = run.result()
        for g, w in zip(got, want):
            assert np.array_equal(g, w), type(run).__name__
        assert early, type(run).__name__
