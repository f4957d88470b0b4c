"""Calls whose stream cannot be waited for (a capture is under way in the thread)
report an error; the pinned blocks that they leave behind are bounded, given back
by epi3.release(), and calls work as before afterwards."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2201_10956_amd import epi3
from synth import make_dataset

pytestmark = pytest.mark.gpu
THREAD_LOCAL = 1  # hipStreamCaptureModeThreadLocal


def hip():
    with open("/proc/self/maps") as f:
        return ctypes.CDLL(next(l.split()[-1] for l in f if "libamdhip64" in l))


def device_mappings():
    """Bytes of this process's mappings of the GPU's device files."""
    n = 0
    with open("/proc/self/maps") as f:
        for l in f:
            if "/dev/dri/" in l or "/dev/kfd" in l:
                a, b = l.split()[0].split("-")
                n += int(b, 16) - int(a, 16)
    return n


def test_blocks_left_behind():
    lib = hip()
    d = make_dataset(40, 700, 0.4, 0.05, 5)
    geno = torch.from_numpy(d.geno).cuda()
    ds = epi3.encode(geno, d.pheno)
    sc = epi3.Scanner(ds, 10)
    want = sc.run()
    side = torch.cuda.Stream()
    stream = ctypes.c_void_p()
    assert lib.hipStreamCreateWithFlags(ctypes.byref(stream), 1) == 0
    def works():
        return epi3.Scanner(epi3.encode(geno, d.pheno), 10).run().tobytes() == want.tobytes()

    def failing_calls(n):
        for x in range(n):
            assert lib.hipStreamBeginCapture(stream, THREAD_LOCAL) == 0
            with pytest.raises(epi3.Epi3Error):
                if x % 2:
                    sc.topk(stream=side)
                else:
                    epi3.encode(geno, d.pheno, into=ds, stream=side)
            graph = ctypes.c_void_p()
            assert lib.hipStreamEndCapture(stream, ctypes.byref(graph)) != 0
            lib.hipGetLastError()
            assert works()
        torch.cuda.synchronize()
        return device_mappings()

    before = failing_calls(40)  # (the runtime's own first mappings among them)
    assert failing_calls(100) - before <= 4 << 20
    assert works()
    epi3.release()
    after = device_mappings()
    assert before - after >= 8 << 20
    assert works()
    assert failing_calls(40) - before <= 4 << 20
    assert works()
    epi3.release()
    assert lib.hipStreamDestroy(stream) == 0
