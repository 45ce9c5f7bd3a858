"""Kept workspaces in a process of many streams and many plans."""
import pytest

from paper_2307_09226_amd import scenes

pytestmark = pytest.mark.gpu


def _free():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def _plan(P):
    from paper_2307_09226_amd import rs
    radar = scenes.radar_for(3, 4, 256, 128, Fs=10e6, Tb=120e-6)
    return rs.rs_cube_plan(radar, rs.RS_FORM_FP64_DIRECT, rs.RS_C64, max_pixels=P)


def _pixels(P):
    import torch
    from paper_2307_09226_amd import rs
    g = torch.Generator(device="cuda:0").manual_seed(P)
    x, y, z, a, v = (torch.rand(P, generator=g, device="cuda:0") for _ in range(5))
    return rs.DevicePixels(x * 4 - 2, y * 8 + 2, z, a, v * 2)


def test_a_stream_per_request():
    """40 streams, each used once: the cubes are right throughout and the plan
    holds no more than its bound."""
    import torch
    from paper_2307_09226_amd import rs
    plan, px = _plan(3000), _pixels(3000)
    want = rs.new_cube(plan)
    rs.rs_beat_synthesize(plan, px, want)
    cubes = [rs.new_cube(plan) for _ in range(40)]
    before = _free()
    for c in cubes:
        s = torch.cuda.Stream()
        rs.rs_beat_synthesize(plan, px, c, stream=s)
        s.synchronize()
    assert before - _free() <= 256 << 20
    assert all(torch.equal(c, want) for c in cubes)
    plan.close()


def test_many_plans_share_a_bound():
    """Twelve plans of 126 MiB each in turn hold at most 1 GiB together, and give
    it back when they go."""
    import torch
    from paper_2307_09226_amd import rs
    px = _pixels(65536)
    plans = [_plan(65536) for _ in range(12)]
    need = plans[0].workspace_bytes(65536)
    assert 12 * need > (1 << 30) + (64 << 20)
    want, cube = rs.new_cube(plans[0]), rs.new_cube(plans[0])
    before = _free()
    for k, plan in enumerate(plans):
        rs.rs_beat_synthesize(plan, px, cube if k else want)
        torch.cuda.synchronize()
        if k:
            assert torch.equal(cube, want)
    assert before - _free() <= (1 << 30) + (64 << 20)
    for plan in plans:
        plan.close()
    assert before - _free() <= 64 << 20
