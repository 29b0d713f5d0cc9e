"""The extension module of the online calls, as far as it goes without a device: arguments, errors, threads.  (Host tensors take a
call up to the current stream, which only a device has.)"""
import threading
import time

import pytest

from paper_2408_08554_amd import binding as B

torch = pytest.importorskip("torch")

FIELDS = B.ABQ_LAYOUT_FIELDS


def host(*shape, dtype=torch.uint8):
    return torch.zeros(shape, dtype=dtype)


def test_allocations_leave_other_threads_running():
    """A gigabyte of outputs, filled by torch's deterministic mode, takes long enough to see whether another thread stops meanwhile."""
    ticks, stop = [], threading.Event()

    def tick():
        while not stop.is_set():
            ticks.append(time.perf_counter())
            time.sleep(0.002)

    def allocate():
        t0 = time.perf_counter()
        with pytest.raises(RuntimeError):                       # K = 0, and no stream without a device
            B.abq_gemm(4, 8, 1 << 15, 1 << 14, 0, host(16), FIELDS, host(16), FIELDS)
        return t0, time.perf_counter()

    was = torch.are_deterministic_algorithms_enabled()
    torch.use_deterministic_algorithms(True)
    thread = threading.Thread(target=tick)
    try:
        thread.start()
        time.sleep(0.05)
        t0, t1 = allocate()
    finally:
        stop.set()
        thread.join()
        torch.use_deterministic_algorithms(was)
    # (one tick before the allocation and one behind it are possible with the GIL held all the while; freeing holds it)
    inside = [t for t in ticks if t0 < t < t1]
    assert len(inside) >= 6, (len(inside), t1 - t0)


def test_a_failed_allocation_is_an_exception():
    for _ in range(3):
        with pytest.raises(RuntimeError):
            B.abq_gemm(4, 8, 1 << 30, 1 << 30, 512, host(16), FIELDS, host(16), FIELDS)
        with pytest.raises(RuntimeError):
            B.abq_gemm_act_codes(4, 8, 1, -1, 512, host(1, 512), host(1), host(1), host(16), FIELDS)
