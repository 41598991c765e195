"""Host logic of csrc/download.hip (the copies to pageable host memory), built for the host against a stand-in for the
runtime calls it makes (tests/hip_host): copies land only when something waits for them, and calls can
be made to fail or to wait."""
import ctypes as C
import os
import subprocess
import threading

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2203_04508_amd", "csrc")
MB = 1 << 20


@pytest.fixture()
def lib(tmp_path):
    so = str(tmp_path / "download_host.so")  # a library of its own for each test: the ring is a process-wide static
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-pthread", "-fno-gnu-unique", "-I", os.path.join(HERE, "hip_host"),
                           "-I", CSRC, "-x", "c++", os.path.join(HERE, "hip_host", "download_host.cpp"), "-o", so])
    L = C.CDLL(so)
    for f in ("t_in_flight", "t_ring_copies"):
        getattr(L, f).restype = C.c_int64
    L.t_download.argtypes = [C.c_int, C.c_void_p, C.c_void_p, C.c_int64]
    L.t_register.argtypes = [C.c_void_p, C.c_int]
    L.t_reset(0, -1, 0)
    return L


def arrays(n, seed=0):
    src = np.random.default_rng(seed).integers(0, 256, n, dtype=np.uint8)
    return src, np.zeros(n, np.uint8)


def copy(lib, k, dst, src):
    return lib.t_download(k, dst.ctypes.data, src.ctypes.data, dst.size)


def warm(lib, k=0):
    """the ring is in use: a copy large enough for it"""
    src, dst = arrays(128 * MB)
    assert copy(lib, k, dst, src) == 0 and np.array_equal(dst, src)


def test_whole(lib):
    lib.t_open(0, 0)
    warm(lib)
    for n in (4 * MB - 1, 4 * MB, 5 * MB + 3, 33 * MB + 7):
        src, dst = arrays(n, n)
        assert copy(lib, 0, dst, src) == 0 and np.array_equal(dst, src)
    lib.t_close()
    assert not lib.t_ring_there()


def test_a_failed_copy_leaves_nothing_in_flight(lib):
    """The ring's chunks that a failing copy had issued have landed before the next copy uses them."""
    lib.t_open(0, 0)
    warm(lib)
    src, dst = arrays(64 * MB, 1)
    lib.t_reset(0, 5, 0)
    assert copy(lib, 0, dst, src) != 0
    assert lib.t_in_flight() == 0
    lib.t_reset(0, -1, 0)
    assert copy(lib, 0, dst, src) == 0 and np.array_equal(dst, src)
    # where the stream cannot be waited for either, the ring is not used again
    lib.t_reset(0, 5, 1)
    assert copy(lib, 0, dst, src) != 0
    lib.t_drop()
    lib.t_reset(0, -1, 0)
    assert copy(lib, 0, dst, src) == 0 and np.array_equal(dst, src)
    assert lib.t_ring_copies() == 0
    lib.t_close()


def test_contexts_come_and_go_during_a_copy(lib):
    """Creating and destroying a context does not wait for another thread's copy."""
    lib.t_open(0, 0)
    warm(lib)
    src, dst = arrays(64 * MB, 2)
    lib.t_hold(1)
    rc = []
    a = threading.Thread(target=lambda: rc.append(copy(lib, 0, dst, src)))
    a.start()
    lib.t_wait_held()
    b = threading.Thread(target=lambda: (lib.t_open(1, 0), lib.t_close()))
    b.start()
    b.join(10.0)
    stuck = b.is_alive()
    lib.t_hold(0)
    a.join()
    b.join()
    assert not stuck
    assert rc == [0] and np.array_equal(dst, src)
    assert lib.t_ring_there()
    lib.t_close()
    assert not lib.t_ring_there()


@pytest.mark.parametrize("kind", [1, 2, 3], ids=["pinned", "device", "managed"])
def test_memory_the_runtime_knows_is_written_by_it(lib, kind):
    """A destination that is pinned (or no plain host memory at all) takes one copy, without the ring."""
    lib.t_open(0, 0)
    warm(lib)
    src, dst = arrays(64 * MB, 3)
    lib.t_register(dst.ctypes.data, kind)
    lib.t_reset(0, -1, 0)
    assert copy(lib, 0, dst, src) == 0 and np.array_equal(dst, src)
    assert lib.t_ring_copies() == 0
    lib.t_close()


def test_another_device_is_current(lib):
    """Events belong to the current device: a caller that has another one current takes the runtime's copy, and no
    ring is made for it."""
    lib.t_open(0, 0)
    src, dst = arrays(128 * MB, 4)
    lib.t_reset(1, -1, 0)
    assert copy(lib, 0, dst, src) == 0 and np.array_equal(dst, src)
    assert lib.t_ring_copies() == 0 and not lib.t_ring_there()
    lib.t_reset(0, -1, 0)
    warm(lib)
    assert lib.t_ring_copies() > 0
    lib.t_reset(1, -1, 0)
    assert copy(lib, 0, dst, src) == 0 and np.array_equal(dst, src)
    assert lib.t_ring_copies() == 0
    lib.t_close()


def test_the_ring_is_pinned_once_it_pays(lib):
    """A process that copies little never pays for the pinning; one that copies on does so once."""
    lib.t_open(0, 0)
    src, dst = arrays(12 * MB, 5)
    for k in range(6):
        lib.t_reset(0, -1, 0)
        assert copy(lib, 0, dst, src) == 0 and np.array_equal(dst, src)
        # 48 MB in all: the fourth copy reaches it
        assert bool(lib.t_ring_there()) == (k >= 3) and (lib.t_ring_copies() > 0) == (k >= 3), k
    lib.t_close()
    assert not lib.t_ring_there()
    lib.t_open(0, 0)
    assert copy(lib, 0, dst, src) == 0 and not lib.t_ring_there()
    lib.t_close()
