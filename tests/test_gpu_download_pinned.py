"""Copies to the host into pinned and into plain arrays are the same, byte for byte."""
import numpy as np
import pytest

from paper_2203_04508_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_pinned_destination():
    import torch  # before the library: both use the HIP runtime that torch brings

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_04508_amd import mcb

    L = mcb.load()
    print("\n[case] copies into a pinned array", flush=True)
    n = 1021 * 703
    lat = mcb.Lattice(2, (1021, 703, 1), 1.0, 0.7 * W.CS_TC)
    lat.set_geometry(np.zeros((0, 8), np.int64))
    lat.init_equilibrium(0.2 + 0.01 * np.random.default_rng(1).random(n))
    lat.step(2)
    plain = lat.get_f()
    pinned = torch.zeros((9, n), dtype=torch.float64).pin_memory().numpy()
    assert L.mcb_get_f(lat.ctx, mcb._ptr(pinned)) == 0
    assert np.array_equal(plain, pinned)
    assert np.array_equal(lat.get_f(), plain)
    lat.close()
