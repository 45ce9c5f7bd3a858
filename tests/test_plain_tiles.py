"""Plain form at the edges of its tiles, mirrored pairs, steps and chunks, and
both direct forms where few pixels are cut into fine chunks."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2307_09226_amd import scenes
from gpu_util import GATE_MFMA, GATE_PLAIN_C128, errors, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Ns,L,P,model", [
    # 64x32 tile (one wave per SIMD), odd Ns (a sample that is its own mirror)
    (1, 1, 1, 0), (63, 32, 15, 0), (64, 33, 17, 16), (65, 31, 63, 0),
    # 128x64
    (127, 64, 65, 0), (128, 49, 255, 31), (129, 63, 257, 0),
    # 128x128, parameter blocks of 256 pixels, more than one chunk
    (128, 128, 511, 0), (255, 127, 513, 16), (257, 129, 1041, 15),
])
def test_tile_and_step_edges(Ns, L, P, model):
    """Full complex128 cubes against the oracle, within the form's gate."""
    from paper_2307_09226_amd import rs
    radar = dataclasses.replace(scenes.radar_for(1, 2, Ns, L, Fs=10e6, Tb=40e-6), model=model)
    px = scenes.tiny_scene(700 + Ns, P, vmax=6.0)
    if model & 16:
        px = scenes.block_strengths(px, L, seed=3)
    rel, mx = errors(synth(radar, px, rs.RS_FORM_FP64_DIRECT, rs.RS_C128), oracle.cube(radar, px))
    print(f"Ns={Ns} L={L} P={P} model={model}: relL2 {rel:.2e} maxabs {mx:.2e}")
    assert rel <= GATE_PLAIN_C128 and mx <= GATE_PLAIN_C128


@pytest.mark.parametrize("P", [1, 127, 128, 129, 1024, 2049, 4057])
def test_fine_chunks(P):
    """Few pixels in few tiles: the plan cuts them into chunks of down to 256
    (matrix-core form) or 64 (plain form) pixels; workspace as described, the
    cube within the gates, and a batch with the single call's bits."""
    import json
    import torch
    from paper_2307_09226_amd import rs
    radar = scenes.radar_for(1, 3, 100, 40, Fs=10e6, Tb=40e-6)
    px = scenes.tiny_scene(800 + P, P, vmax=6.0)
    ref = oracle.cube(radar, px)
    for form, dtype, gate in ((rs.RS_FORM_MFMA_SPLIT16, rs.RS_C64, GATE_MFMA),
                              (rs.RS_FORM_FP64_DIRECT, rs.RS_C128, GATE_PLAIN_C128)):
        plan = rs.rs_cube_plan(radar, form, dtype, max_pixels=P)
        desc = json.loads(plan.describe(P))
        assert desc["chunks"] * desc["chunk_pixels"] >= P > (desc["chunks"] - 1) * desc["chunk_pixels"]
        elem = 8 if dtype == rs.RS_C64 else 16
        need = desc["chunks"] * 3 * 100 * 40 * elem
        assert plan.workspace_bytes(P) == (need + 255) // 256 * 256 <= 16 << 20
        d = rs.DevicePixels.from_host(px)
        one, many = rs.new_cube(plan), rs.new_cube(plan, count=3)
        rs.rs_beat_synthesize(plan, d, one)
        rs.rs_beat_synthesize_batch(plan, [d, d, d], many)
        torch.cuda.synchronize()
        rel, mx = errors(one.cpu().numpy(), ref)
        assert rel <= gate and mx <= gate
        assert all(torch.equal(one, many[k]) for k in range(3))
        plan.close()
