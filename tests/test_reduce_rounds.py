"""The plain form's reduction at the edges of its rounds of partial sums."""
import json

import pytest

import oracle
from paper_2307_09226_amd import scenes
from gpu_util import GATE_PLAIN_C128, errors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [1, 2, 7, 8, 9, 15, 16, 17, 23, 24, 25, 32, 33])
def test_chunk_counts(S):
    """Cubes of S chunks (128 pixels each, the last one ragged) against the
    oracle, within the form's gate."""
    import torch
    from paper_2307_09226_amd import rs
    radar = scenes.radar_for(1, 1, 37, 11, Fs=10e6, Tb=40e-6)
    P = 128 * S - 5
    px = scenes.tiny_scene(600 + S, P, vmax=6.0)
    plan = rs.rs_cube_plan(radar, rs.RS_FORM_FP64_DIRECT, rs.RS_C128, max_pixels=P)
    assert json.loads(plan.describe(P))["chunks"] == S
    cube = rs.new_cube(plan)
    rs.rs_beat_synthesize(plan, rs.DevicePixels.from_host(px), cube)
    torch.cuda.synchronize()
    rel, mx = errors(cube.cpu().numpy(), oracle.cube(radar, px))
    print(f"S={S}: relL2 {rel:.2e} maxabs {mx:.2e}")
    assert rel <= GATE_PLAIN_C128 and mx <= GATE_PLAIN_C128
    plan.close()
