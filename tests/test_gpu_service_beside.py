"""Call-by-call heaps given up while a service kernel runs, with an installed
device allocator: nothing on that way may wait for the device, or for the
service's hardware queue, to be idle."""
import threading
import time

import pytest

from paper_2405_07079_amd import hda

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_heaps_are_given_up_beside_a_running_service():
    """Several services in turn, each with another stream in use before it, so
    that one of them shares the hardware queue of the heaps' stream."""
    # (the binding installs torch's caching allocator, whose release does not wait)
    streams = []
    for rep in range(8):
        heaps = [hda.Heap(1 << 20, 64, k % 5) for k in range(200)]   # four pages of words
        assert all(h.alloc(100) == 0 for h in heaps)
        streams.append(torch.cuda.Stream())
        with torch.cuda.stream(streams[-1]):
            torch.zeros(8, device="cuda").add_(1)
        server = hda.Server(max_heaps=4, waves=16, max_seconds=30)
        took = []

        def give_up():
            t0 = time.perf_counter()
            for h in heaps:
                h.close()
            took.append(time.perf_counter() - t0)

        t = threading.Thread(target=give_up)
        try:
            h = server.open(1 << 20, 64, 0)
            assert server.alloc(h, 64) == 0
            t.start()
            t.join(5)
            print("case: 200 heaps given up beside service", rep, "in", took, "s", flush=True)
            assert took, "still waiting: for the service to stop"
            assert server.alloc(h, 64) == 64      # it runs on
        finally:
            server.stop()
            t.join(30)
