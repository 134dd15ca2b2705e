"""The native launches release the interpreter lock during the library call, as a ctypes call
does: here a C function that sleeps stands for a launch that waits on a full queue."""
import ctypes
import threading
import time
import types

import pytest

from paper_2109_06976_amd import grid

pytestmark = pytest.mark.gpu


def test_other_threads_run_during_a_launch():
    import torch
    native = grid._native()
    usleep = ctypes.cast(ctypes.CDLL(None).usleep, ctypes.c_void_p).value
    # the first argument of a launch is the model's handle: 0.4 s in microseconds
    model = types.SimpleNamespace(_h=ctypes.c_void_p(400000))
    bufs = tuple(torch.zeros(1, device="cuda") for _ in range(2))
    ticks, stop = [], threading.Event()

    def tick():
        while not stop.is_set():
            ticks.append(time.monotonic())
            time.sleep(0.005)

    t = threading.Thread(target=tick)
    t.start()
    begin = time.monotonic()
    native.launch(usleep, model, 0, 1, bufs, (1, 1), None)
    end = time.monotonic()
    stop.set()
    t.join()
    assert end - begin >= 0.4
    # a thread that sleeps 5 ms between ticks; with the lock held it would tick at most twice
    assert sum(begin < x < end for x in ticks) >= 10
