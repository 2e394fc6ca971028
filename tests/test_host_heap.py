"""The host code of the call-by-call heaps on the CPU (device memory is host
memory, a launch is an emulated wave): the pool of result words, which all
heaps share."""
import ctypes
import os
import shutil
import subprocess
import tempfile
import threading

import pytest

import emu

ALLOC = ctypes.CFUNCTYPE(ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p)
RELEASE = ctypes.CFUNCTYPE(None, ctypes.c_void_p, ctypes.c_void_p)
HOOK = ctypes.CFUNCTYPE(None)
HEAPS = 200          # more than three pages of words


@pytest.fixture(scope="module")
def lib():
    with tempfile.TemporaryDirectory() as d:
        for f in os.listdir(emu.CSRC):
            if f.endswith(".h") and f != "hda_wave.h" or f == "hda_heap.hip":
                shutil.copy(os.path.join(emu.CSRC, f), d)
        with open(os.path.join(d, "hda_wave.h"), "w") as f:
            f.write('#include "emu_wave.h"\n')
        shutil.copy(os.path.join(emu.HERE, "emu_host.cpp"), d)
        so = os.path.join(d, "emu_host.so")
        subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-pthread",
                               "-I", d, "-I", os.path.join(emu.HERE, "host"), "-I", emu.HERE,
                               "-I", os.path.join(emu.ROOT, "include"),
                               os.path.join(d, "emu_host.cpp"), "-o", so])
        L = ctypes.CDLL(so)
        L.hda_alloc.restype = ctypes.c_int64
        yield L


def create(L):
    h = ctypes.c_void_p()
    assert L.hda_heap_create(ctypes.c_uint64(1 << 16), ctypes.c_uint64(64), 0,
                             ctypes.c_uint32(64), ctypes.byref(h)) == 0
    return h


def test_words_are_apart_and_results_arrive(lib):
    heaps = [create(lib) for _ in range(HEAPS)]
    for k, h in enumerate(heaps):      # every heap has its own word and state
        assert lib.hda_alloc(h, ctypes.c_uint64(64 * (k % 7 + 1))) == 0
    for k, h in enumerate(heaps):
        assert lib.hda_alloc(h, ctypes.c_uint64(64)) == 64 * (k % 7 + 1)
        assert lib.hda_heap_destroy(h) == 0
    assert lib.emu_pages() == 1        # given back but for one


def test_no_heap_waits_for_the_device_in_an_installed_allocators_release(lib):
    """hipHostFree may wait for all work on the device, a running service
    included.  An installed allocator's release need not, so giving up heaps
    must not either: the pages stay for later heaps, and no more are made."""
    held, freed = {}, []

    @ALLOC
    def alloc(n, _):
        b = ctypes.create_string_buffer(n)
        held[ctypes.addressof(b)] = b
        return ctypes.addressof(b)

    @RELEASE
    def release(p, _):
        del held[p]

    hook = HOOK(lambda: freed.append(1))
    assert lib.hda_set_device_allocator(alloc, release, None) == 0
    lib.emu_set_on_host_free(hook)
    try:
        pages = None
        for _ in range(3):
            heaps = [create(lib) for _ in range(HEAPS)]
            pages = pages or lib.emu_pages()
            assert lib.emu_pages() == pages == (HEAPS + 63) // 64
            for h in heaps:
                assert lib.hda_heap_destroy(h) == 0
        assert not freed and not held
    finally:
        lib.emu_set_on_host_free(HOOK(0))
        assert lib.hda_set_device_allocator(ALLOC(0), RELEASE(0), None) == 0


def test_a_page_is_freed_outside_the_pools_lock(lib):
    """While one thread waits in hipHostFree, others create and use heaps."""
    done, stuck = [], []

    def other():
        h = create(lib)
        assert lib.hda_alloc(h, ctypes.c_uint64(64)) == 0
        done.append(h)

    @HOOK
    def hook():
        t = threading.Thread(target=other)
        t.start()
        t.join(20)
        if t.is_alive():
            stuck.append(t)

    heaps = [create(lib) for _ in range(HEAPS)]
    lib.emu_set_on_host_free(hook)
    try:
        for h in heaps:
            assert lib.hda_heap_destroy(h) == 0
            if stuck:
                break
        assert done and not stuck
    finally:
        lib.emu_set_on_host_free(HOOK(0))
        for t in stuck:
            t.join(20)
        for h in done:
            assert lib.hda_heap_destroy(h) == 0


def test_an_idle_heap_goes_without_a_wait_for_its_stream(lib):
    """Calls return when their result is released, after everything else they
    store: giving up the heap has nothing to wait for, where a wait would stand
    behind whatever kernel shares the stream's hardware queue."""
    h = create(lib)
    assert lib.hda_alloc(h, ctypes.c_uint64(64)) == 0
    assert lib.hda_free(h, ctypes.c_int64(0)) == 0
    waits = lib.emu_waits()
    assert lib.hda_heap_destroy(h) == 0
    assert lib.emu_waits() == waits
