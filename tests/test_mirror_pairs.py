"""Matrix-core form at the edges of its mirrored sample pairs, tiles and steps.

Fast time is taken from its middle, so an odd Ns has one sample that is its
own mirror; a tile holds 64, 128 or 256 pairs; pixels come in pairs, steps of
32 (16 in the 512-sample tiles), pairs of steps and parameter blocks of 256.
"""
import numpy as np
import pytest

import oracle
from paper_2307_09226_amd import scenes
from gpu_util import GATE_MFMA, errors, sample_indices, synth

pytestmark = pytest.mark.gpu


def _rs():
    from paper_2307_09226_amd import rs
    return rs


@pytest.mark.parametrize("Ns,L,P", [
    (1, 1, 1), (2, 3, 31), (3, 2, 33), (127, 5, 63), (128, 64, 64), (129, 65, 65),
    (255, 128, 255), (256, 129, 257), (257, 63, 511), (511, 9, 1025), (513, 33, 1056),
])
def test_pair_and_step_edges(Ns, L, P):
    """Full cubes against the oracle, within the form's gate: complex64
    (mirrored pairs) and complex128 (sample by sample) plans."""
    rs = _rs()
    radar = scenes.radar_for(1, 2, Ns, L, Fs=10e6, Tb=40e-6)
    px = scenes.tiny_scene(900 + Ns, P, vmax=6.0)
    ref = oracle.cube(radar, px)
    for dtype in (rs.RS_C64, rs.RS_C128):
        rel, mx = errors(synth(radar, px, rs.RS_FORM_MFMA_SPLIT16, dtype), ref)
        print(f"Ns={Ns} L={L} P={P} dtype={dtype}: relL2 {rel:.2e} maxabs {mx:.2e}")
        assert rel <= GATE_MFMA and mx <= GATE_MFMA


@pytest.mark.parametrize("model", [0, 16])
def test_complex128_tiles(model):
    """Every tile configuration of the complex128 plans' kernel: the full cube
    on ragged tiles, and the two schedules of an 8-wave shape bit for bit."""
    import dataclasses
    import torch
    rs = _rs()
    radar = dataclasses.replace(scenes.radar_for(2, 2, 130, 70, Fs=10e6, Tb=80e-6), model=model)
    px = scenes.tiny_scene(505, 1333, vmax=6.0)
    if model & 16:
        px = scenes.block_strengths(px, radar.L, seed=6)
    ref = oracle.cube(radar, px)
    d = rs.DevicePixels.from_host(px)
    first = {}
    for shape in ("64x128x4", "32x128x4", "32x128x8", "32x64x4", "32x64x8", "64x64x4", "64x64x8", "128x64x4",
                  "32x128x8i", "32x64x8i", "64x64x8i"):
        plan = rs.rs_cube_plan(radar, rs.RS_FORM_MFMA_SPLIT16, rs.RS_C128, max_pixels=px.P)
        rs.rs_plan_set_tile(plan, shape)
        cube = rs.new_cube(plan)
        rs.rs_beat_synthesize(plan, d, cube)
        torch.cuda.synchronize()
        rel, mx = errors(cube.cpu().numpy(), ref)
        assert rel <= GATE_MFMA and mx <= GATE_MFMA, shape
        assert torch.equal(cube, first.setdefault(shape.rstrip("i"), cube)), shape
        plan.close()


def test_session_mixes_both_kernels():
    """Requests of complex64 and complex128 plans of the same tile shape in
    one session: each cube has the bits of its own single call."""
    import torch
    rs = _rs()
    sess = rs.Session(hbm_budget=1 << 28, max_slots=4, slice_items=2)
    items = []
    for k, dtype in enumerate((rs.RS_C64, rs.RS_C128, rs.RS_C64, rs.RS_C128)):
        radar = scenes.radar_for(1, 3, 200, 100, Fs=10e6, Tb=40e-6)
        px = scenes.tiny_scene(970 + k, 4000 + 777 * k, vmax=6.0)
        plan = rs.rs_cube_plan(radar, rs.RS_FORM_MFMA_SPLIT16, dtype, max_pixels=px.P)
        rs.rs_plan_set_tile(plan, "32x128x8")
        d = rs.DevicePixels.from_host(px)
        alone, mixed = rs.new_cube(plan), rs.new_cube(plan)
        rs.rs_beat_synthesize(plan, d, alone)
        items.append((plan, d, alone, mixed))
    torch.cuda.synchronize()
    tickets = [sess.submit(plan, d, mixed) for plan, d, _, mixed in items]
    sess.drain()
    for t, (_, _, alone, mixed) in zip(tickets, items):
        assert sess.poll(t)[0] == rs.RS_REQ_DONE
        assert torch.equal(alone, mixed)
    sess.close()


@pytest.mark.parametrize("Ns,tile", [(129, "32x128x8"), (255, "32x64x8i"), (256, "32x64x4"), (513, "64x64x8")])
def test_parked_sums_keep_the_bits(Ns, tile):
    """A session that cuts a chunk into many segments (its raw cosine and sine
    sums parked in between) gives the bits of the single call."""
    import torch
    rs = _rs()
    radar = scenes.radar_for(1, 3, Ns, 70, Fs=10e6, Tb=40e-6)
    px = scenes.tiny_scene(950 + Ns, 40001, vmax=6.0)  # chunks of several 256-pixel blocks
    plan = rs.rs_cube_plan(radar, rs.RS_FORM_MFMA_SPLIT16, rs.RS_C64, max_pixels=px.P)
    rs.rs_plan_set_tile(plan, tile)
    d = rs.DevicePixels.from_host(px)
    alone, cut = rs.new_cube(plan), rs.new_cube(plan)
    rs.rs_beat_synthesize(plan, d, alone)
    torch.cuda.synchronize()
    sess = rs.Session(hbm_budget=1 << 28, max_slots=2, slice_items=1)
    t = sess.submit(plan, d, cut)
    sess.drain()
    assert sess.poll(t)[0] == rs.RS_REQ_DONE
    assert sess.stats()["launches"] > 1
    assert torch.equal(alone, cut)
    c, l, n = sample_indices(radar.cube_shape(), 400, seed=Ns)
    rel, _ = errors(alone.cpu().numpy()[c, l, n], oracle.entries(radar, px, c, l, n))
    assert rel <= GATE_MFMA
    sess.close()
    plan.close()


def test_lower_error_than_the_gate_by_far():
    """One chunk of 2,048 pixels: the rounding of the fp32 sums (2 chains of
    3 * 2048 / 16 additions of 2^-24 each, a random walk: 28 * 6e-8 = 1.7e-6)
    and of the phasors (2^-22 each) bounds the relative L2 error at 2e-6."""
    rs = _rs()
    radar = scenes.radar_for(8, 8, 128, 64, Fs=5e6, Tb=8 * 40e-6)
    px = scenes.scene_small(seed=4, grid=45, pedestrian=True)
    got = synth(radar, px, rs.RS_FORM_MFMA_SPLIT16, rs.RS_C128)
    rel, _ = errors(got, oracle.cube(radar, px))
    print(f"relL2 {rel:.2e}")
    assert rel <= 2e-6
