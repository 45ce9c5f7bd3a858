"""One workspace, sized for the largest call, serves every smaller one."""
import pytest

from paper_2307_09226_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,M,N,Ns,L,most,sizes", [
    # fewer pixels in more chunks: 256 against 247 and 250 of them
    ("mfma", 1, 1, 128, 64, 300000, [262144, 163841, 1, 0]),
    ("plain", 1, 1, 33, 17, 40000, [32768, 32767, 4096, 1]),
    ("plain", 2, 4, 64, 32, 40961, [32768, 4097, 0]),
    ("mfma", 3, 4, 256, 128, 65536, [21504, 21505, 4000]),
    ("nufft", 2, 2, 64, 32, 6001, [6000, 257, 1]),
])
def test_synthesis(form, M, N, Ns, L, most, sizes):
    import torch
    from paper_2307_09226_amd import rs
    radar = scenes.radar_for(M, N, Ns, L, Fs=10e6, Tb=M * 40e-6)
    f = dict(mfma=rs.RS_FORM_MFMA_SPLIT16, plain=rs.RS_FORM_FP64_DIRECT, nufft=rs.RS_FORM_NUFFT)[form]
    plan = rs.rs_cube_plan(radar, f, rs.RS_C64, max_pixels=most)
    ws = torch.empty(plan.workspace_bytes(most), dtype=torch.uint8, device="cuda:0")
    g = torch.Generator(device="cuda:0").manual_seed(7)
    x, y, z, a, v = (torch.rand(most, generator=g, device="cuda:0") for _ in range(5))
    for P in [most] + sizes:
        assert plan.workspace_bytes(P) <= ws.numel()
        px = rs.DevicePixels(x[:P] * 4 - 2, y[:P] * 8 + 2, z[:P], a[:P].contiguous(), v[:P] * 2)
        want, got = rs.new_cube(plan), rs.new_cube(plan)
        rs.rs_beat_synthesize(plan, px, want)
        rs.rs_beat_synthesize_ws(plan, px, got, ws)
        assert torch.equal(want, got), P
    plan.close()


@pytest.mark.parametrize("N,Ns,L,most,sizes", [
    # the fused kernel's partial maps for `most`, spectra for fewer frames
    (192, 256, 64, 40, [7, 3, 1]), (12, 256, 128, 100, [42, 15, 9, 1]), (1, 256, 32, 400, [143, 20]),
    (12, 512, 64, 30, [12, 5, 1]), (3, 64, 16, 90, [89, 31]),
])
def test_range_doppler(N, Ns, L, most, sizes):
    import torch
    from paper_2307_09226_amd import rs
    radar = scenes.radar_for(1, N, Ns, L, Fs=10e6, Tb=40e-6)
    plan = rs.rs_cube_plan(radar, rs.RS_FORM_MFMA_SPLIT16, rs.RS_C64, max_pixels=16)
    g = torch.Generator(device="cuda:0").manual_seed(most)
    cubes = torch.view_as_complex(torch.randn((most, N, L, Ns, 2), generator=g, device="cuda:0"))
    ws = torch.empty(rs.rs_range_doppler_workspace_bytes(plan, most, True), dtype=torch.uint8, device="cuda:0")
    for F in [most] + sizes:
        assert rs.rs_range_doppler_workspace_bytes(plan, F, True) <= ws.numel()
        want, dtime, _ = rs.range_doppler(plan, cubes[:F])
        got, d2 = torch.empty_like(want), torch.empty_like(dtime)
        rs.rs_range_doppler_ws(plan, cubes[:F], True, got, d2, None, ws)
        assert torch.equal(want, got) and torch.equal(dtime, d2), F
    plan.close()
