"""Copies to the host through the pinned ring (4 MB and more): whole, partial and last chunks, shorter than the
ring and longer, against the populations in the device arena; several threads and contexts at once (one takes
the ring, the others the runtime's copy), the ring's release with the last context and its return."""
import gc
import threading

import numpy as np
import pytest

from paper_2203_04508_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mcb():
    import torch  # before the library: both use the HIP runtime that torch brings

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_04508_amd import mcb as m

    m.load()
    return m


def lattice(mcb, dims, seed):
    import torch

    lat = mcb.Lattice(2, (*dims, 1), 1.0, 0.7 * W.CS_TC)
    lat.set_geometry(np.zeros((0, 8), np.int64))
    rng = np.random.default_rng(seed)
    lat.init_equilibrium(0.2 + 0.01 * rng.random(dims[0] * dims[1]))
    lat.step(2)
    lat.sync()
    f = lat.lat[: 72 * lat.N].view(torch.float64).view(9, lat.N).cpu().numpy()
    return lat, f


# 8 N bytes: just under 4 MB (the runtime's copy), just over, 2 whole chunks and a bit, more than the ring
@pytest.mark.parametrize("dims", [(724, 724), (1024, 512), (1021, 517), (1500, 1501)], ids=lambda d: f"{d[0]}x{d[1]}")
def test_copies_are_whole(mcb, dims):
    print(f"\n[case] download {dims}", flush=True)
    lat, f = lattice(mcb, dims, 1)
    assert np.array_equal(lat.get_f(), f)
    rho, v = lat.moments()
    assert np.abs(rho - f.sum(0)).max() < 1e-14 and np.isfinite(v).all()
    assert np.array_equal(lat.get_f(), f)
    lat.close()


def test_threads_and_release(mcb):
    print("\n[case] download from several threads", flush=True)
    gc.collect()
    lats = [lattice(mcb, (1021, 700 + 16 * k), k) for k in range(3)]
    bad = []

    def reader(lat, f):
        for _ in range(4):
            if not np.array_equal(lat.get_f(), f):
                bad.append(1)

    th = [threading.Thread(target=reader, args=x) for x in lats]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not bad
    for lat, _ in lats:
        lat.close()
    lat, f = lattice(mcb, (1021, 703), 9)  # after the last context of this test went
    assert np.array_equal(lat.get_f(), f)
    lat.close()
