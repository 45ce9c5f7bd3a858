"""Range-Doppler maps on both sides of the lines between the paths: few
channels (LDS Doppler pass), runs side by side of which the last group is
ragged, many frames, and the fused kernel at L = 32 and few channels."""
import pytest

from paper_2307_09226_amd import scenes
from test_rd_gpu import check_rd_frames
from test_rd_shapes import _cubes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,Ns,L,F,dtype", [
    (1, 64, 64, 300, 0), (1, 16, 16, 700, 1), (2, 128, 32, 40, 0), (2, 1024, 256, 1, 0),
    (3, 64, 16, 600, 0), (5, 32, 64, 2, 0), (4, 32, 16, 500, 1), (1, 256, 16, 130, 0), (3, 2048, 32, 3, 0),
    (1, 256, 32, 143, 0), (1, 256, 32, 144, 0), (3, 256, 32, 60, 1), (2, 256, 64, 47, 0), (2, 256, 64, 48, 0),
    (1, 256, 128, 96, 0),
])
def test_paths(N, Ns, L, F, dtype):
    """Frames at the ends and in between against the oracle, and the bits of the
    workspace form."""
    import torch
    from paper_2307_09226_amd import rs
    radar = scenes.radar_for(1, N, Ns, L, Fs=10e6, Tb=40e-6)
    plan = rs.rs_cube_plan(radar, rs.RS_FORM_MFMA_SPLIT16, dtype, max_pixels=16)
    cubes = _cubes(radar, F, dtype, 17 + Ns + L)
    frames = sorted({0, 1 % F, F // 3, F // 2, F - 2 if F > 1 else 0, F - 1})
    for skip in (True, False):
        check_rd_frames(radar, plan, cubes, frames, skip_static=skip)
    power, dtime, _ = rs.range_doppler(plan, cubes)
    p2, d2 = torch.empty_like(power), torch.empty_like(dtime)
    ws = torch.empty(rs.rs_range_doppler_workspace_bytes(plan, F, True), dtype=torch.uint8, device="cuda:0")
    rs.rs_range_doppler_ws(plan, cubes, True, p2, d2, None, ws)
    torch.cuda.synchronize()
    assert torch.equal(power, p2) and torch.equal(dtime, d2)
    plan.close()


@pytest.mark.parametrize("N,Ns,L,F", [(12, 256, 16, 641), (2, 1024, 64, 2049), (1, 256, 256, 4097)])
def test_rounds_of_frames(N, Ns, L, F):
    """One frame more than a round of the two passes holds (240 MiB of spectra at
    256 x 16, else 2 GiB): the frames at both ends of both rounds against the
    oracle, and a workspace that does not grow with the call."""
    import torch
    from paper_2307_09226_amd import rs
    radar = scenes.radar_for(1, N, Ns, L, Fs=10e6, Tb=40e-6)
    plan = rs.rs_cube_plan(radar, rs.RS_FORM_MFMA_SPLIT16, rs.RS_C64, max_pixels=16)
    need = {n: rs.rs_range_doppler_workspace_bytes(plan, n, True) for n in (F - 1, F, 50 * F)}
    for n in need:   # a round's spectra and maps, and every frame's maxima
        assert need[F - 1] <= need[n] <= need[F - 1] + n * (Ns * L // 256) * 8 + 256
    g = torch.Generator(device="cuda:0").manual_seed(F)
    cubes = torch.view_as_complex(torch.randn((F, N, L, Ns, 2), generator=g, device="cuda:0"))
    h = (F + 1) // 2
    check_rd_frames(radar, plan, cubes, [0, 1, h - 1, h, h + 1, F - 1], skip_static=True)
    plan.close()


@pytest.mark.parametrize("N,Ns,L,F", [(5, 512, 64, 1), (3, 64, 16, 600), (4, 256, 64, 24), (1, 64, 64, 3)])
def test_map_at_any_float(N, Ns, L, F):
    """A power map that starts at any float of a larger array (runs of channels,
    one run, the fused kernel, the LDS passes): the bits of an aligned one and
    nothing beside it."""
    import torch
    from paper_2307_09226_amd import rs
    radar = scenes.radar_for(1, N, Ns, L, Fs=10e6, Tb=40e-6)
    plan = rs.rs_cube_plan(radar, rs.RS_FORM_MFMA_SPLIT16, rs.RS_C64, max_pixels=16)
    g = torch.Generator(device="cuda:0").manual_seed(F)
    cubes = torch.view_as_complex(torch.randn((F, N, L, Ns, 2), generator=g, device="cuda:0"))
    want, dtime, _ = rs.range_doppler(plan, cubes)
    n = F * Ns * L
    for shift in (1, 2, 3):
        big = torch.full((n + 8,), -3.0, device="cuda:0")
        d2 = torch.empty_like(dtime)
        rs.rs_range_doppler(plan, cubes, True, big[shift:shift + n], d2)
        assert torch.equal(big[shift:shift + n], want.view(-1)) and torch.equal(d2, dtime)
        assert torch.all(big[:shift] == -3.0) and torch.all(big[shift + n:] == -3.0)
    plan.close()
