"""Accuracy of the mirrored-pair kernel (complex64 matrix-core plans), far below
the form's gate: a lost part of the split or of a rotation shows here."""
import json
import math

import pytest

import oracle
from paper_2307_09226_amd import scenes
from gpu_util import errors

pytestmark = pytest.mark.gpu

TILES = ("64x128x4", "32x128x4", "32x128x8", "32x64x4", "32x64x8", "64x64x4", "64x64x8", "128x64x4", "32x128x8i",
         "32x64x8i", "64x64x8i")


def bound(chunk):
    """Twice the expected relative L2 error of a chunk of `chunk` pixels, in units
    u = 2^-24.  Sums in binary32: three products of 16 pixels a matrix
    instruction, taken as four roundings each, n = 12 chunk / 16 in all; the sum
    grows like a random walk, so its roundings (u / sqrt 3 of the sum so far)
    add up to sqrt(n / 2) u / sqrt 3.  Phasors: hardware sine and cosine, a rotation
    and the halves' product left out, 2^-22 each for F and D: 4 sqrt 2 u."""
    n = 12 * chunk / 16
    return 2.0 * 2.0 ** -24 * math.hypot(math.sqrt(n / 2 / 3), 4 * math.sqrt(2))


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("Ns,L,P", [(64, 33, 700), (127, 70, 1024), (129, 65, 2025), (255, 100, 1333), (256, 128, 2048)])
def test_far_below_the_gate(Ns, L, P, dtype):
    """Full cubes on every tile shape: complex64 (mirrored pairs) and, for
    comparison, complex128 plans (sample by sample)."""
    import torch
    from paper_2307_09226_amd import rs
    radar = scenes.radar_for(1, 2, Ns, L, Fs=10e6, Tb=40e-6)
    px = scenes.tiny_scene(300 + Ns, P, vmax=6.0)
    ref = oracle.cube(radar, px)
    d = rs.DevicePixels.from_host(px)
    for tile in TILES:
        plan = rs.rs_cube_plan(radar, rs.RS_FORM_MFMA_SPLIT16, dtype, max_pixels=P)
        rs.rs_plan_set_tile(plan, tile)
        desc = json.loads(plan.describe(P))
        cube = rs.new_cube(plan)
        rs.rs_beat_synthesize(plan, d, cube)
        torch.cuda.synchronize()
        rel, _ = errors(cube.cpu().numpy(), ref)
        lim = bound(min(P, desc["chunk_pixels"]))
        print(f"Ns={Ns} L={L} P={P} dtype={dtype} {tile}: chunks {desc['chunks']} relL2 {rel:.2e} bound {lim:.2e}", flush=True)
        assert rel <= lim, tile
        plan.close()
