"""The native calls allocate their outputs without the interpreter's lock: where an allocation has to give cached memory back first, it waits
for the device, and may not stop every other Python thread meanwhile."""
import sys
import threading
import time

import pytest
import torch

from paper_2211_10438_amd import binding as sq

pytestmark = pytest.mark.gpu


def _codes(*shape):
    return torch.ones(shape, device="cuda", dtype=torch.int8)


def _linear():
    x, w, one = _codes(16384, 64), _codes(40960, 64), torch.ones(1, device="cuda")
    return lambda: sq.w8a8_linear(x, one, w, one, torch.float16)


def _linear_q8():
    x, w, one = _codes(32768, 64), _codes(40960, 64), torch.ones(1, device="cuda")
    return lambda: sq.w8a8_linear_q8(x, one, w, one, one, torch.float16)


def _bmm():
    a, b = _codes(1, 16384, 64), _codes(1, 40960, 64)
    return lambda: sq.w8a8_bmm(a, b, True, 1.0, torch.float16)


@pytest.mark.parametrize("make", [_linear, _linear_q8, _bmm])
def test_other_threads_run_while_an_allocation_waits(make):
    print(make.__name__, flush=True)
    sq.lib()
    assert sq._fast is not None
    call = make()  # 1.25 GiB of output
    square = torch.randn((8192, 8192), device="cuda").bfloat16()
    product = torch.empty_like(square)
    torch.matmul(square, square, out=product)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    device = torch.cuda.current_device()
    total = torch.cuda.get_device_properties(device).total_memory
    interval = sys.getswitchinterval()
    gap, last, stop = 0.0, time.perf_counter(), False

    def count():
        nonlocal gap, last
        while not stop:
            now = time.perf_counter()
            gap, last = max(gap, now - last), now

    other = threading.Thread(target=count)
    try:
        # room for the output only once the cached 1 GiB is given back, which waits for the products
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (3 << 29)) / total)
        torch.empty(1 << 30, dtype=torch.uint8, device="cuda")
        sys.setswitchinterval(1e-3)
        for _ in range(200):
            torch.matmul(square, square, out=product)
        other.start()
        time.sleep(0.005)
        gap, begun = 0.0, time.perf_counter()
        out = call()
        waited = time.perf_counter() - begun
        seen = gap
    finally:
        stop = True
        sys.setswitchinterval(interval)
        torch.cuda.set_per_process_memory_fraction(1.0)
        if other.ident is not None:
            other.join()
        torch.cuda.synchronize()
    del out
    torch.cuda.empty_cache()
    print(f"waited {waited * 1e3:.1f} ms, the other thread at most {seen * 1e3:.1f}", flush=True)
    assert waited > 0.03  # (the products take some 200 ms)
    assert seen < 0.5 * waited
