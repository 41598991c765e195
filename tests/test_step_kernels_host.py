"""The kernels that bench.py names for a step are the ones the library's dispatch runs (no GPU: the rules are compared
with the sources that hold them)."""
import os
import re
import types

from paper_2203_04508_amd import roofline

CSRC = os.path.join(os.path.dirname(os.path.abspath(roofline.__file__)), "csrc")


def text(name):
    return open(os.path.join(CSRC, name)).read()


def test_names_follow_the_dispatch():
    assert int(re.search(r"TILE_BYTES = (\d+)", text("mcb_internal.h")).group(1)) == roofline.TILE_BYTES
    # D2Q9: tiles unless FP16, or past TILE_BYTES in the pseudopotential model; D3Q19: flat kernels unless FP16
    assert re.search(r"precision != MCB_F16S && \(cp \|\| 2 \* state_bytes\(c->p.precision, 9, c->g.N\) <= TILE_BYTES\)\)\s*"
                     r"return tile2d", text("step2d.hip"))
    assert re.search(r"if \(c->p.precision != MCB_F16S\) return flat3d", text("step3d.hip"))
    wl = lambda dim, n: types.SimpleNamespace(dim=dim, N=n, Q=9 if dim == 2 else 19)
    name = lambda dim, n, prec, model="pseudo": roofline.step_kernels(wl(dim, n), prec, model)
    assert name(2, 4096 ** 2, "f32s") == name(2, 1024 ** 2, "f16s") == name(2, 4096 ** 2, "f64") == "k_step2d"
    assert name(2, 1024 ** 2, "f32s") == name(2, 1531 * 1021, "f64") == "k_tile2d"
    last = roofline.TILE_BYTES // (2 * 9 * 8)
    assert name(2, last, "f64") == "k_tile2d" and name(2, last + 1, "f64") == "k_step2d"
    assert name(2, 4096 ** 2, "f64", "chempot") == name(2, 64, "f32s", "chempot") == "k_cptile (one step)"
    assert name(2, 4096 ** 2, "f16s", "chempot") == "k_cp_march (one step)"
    assert name(3, 64 ** 3, "f16s") == "k_rho3d + k_step3d (one step)"
    assert name(3, 64 ** 3, "f64") == name(3, 256 ** 3, "f32s") == "k_rho3f + k_psi3w + k_collide3f (one step)"
