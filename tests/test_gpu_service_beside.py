"""Call-by-call heaps given up while a service kernel runs, with an installed
device allocator: nothing on that way may wait for the device to be idle."""
import threading
import time

import pytest

from paper_2405_07079_amd import hda

pytestmark = pytest.mark.gpu
pytest.importorskip("torch")


def test_heaps_are_given_up_beside_a_running_service():
    hda.use_torch_allocator()
    try:
        heaps = [hda.Heap(1 << 20, 64, k % 5) for k in range(200)]   # four pages of words
        assert all(h.alloc(100) == 0 for h in heaps)
        server = hda.Server(max_heaps=4, waves=16, max_seconds=30)
        took = []

        def give_up():
            t0 = time.perf_counter()
            for h in heaps:
                h.close()
            took.append(time.perf_counter() - t0)

        try:
            h = server.open(1 << 20, 64, 0)
            assert server.alloc(h, 64) == 0
            t = threading.Thread(target=give_up)
            t.start()
            t.join(10)
            print("case: 200 heaps given up beside a service in", took, "s", flush=True)
            assert took, "still waiting: for the service to stop"
            assert server.alloc(h, 64) == 64      # it runs on
        finally:
            server.stop()
            t.join(30)
    finally:
        hda.use_hip_allocator()
