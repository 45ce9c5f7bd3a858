"""Range-Doppler maps at the edges of their paths: every factorisation of the
register FFTs, runs of channels that do not divide the channel count, the
lengths that stay on the LDS FFTs, and the fused kernel (many frames)."""
import dataclasses

import numpy as np
import pytest

from oracle import rd
from paper_2307_09226_amd import scenes
from test_rd_gpu import check_rd

pytestmark = pytest.mark.gpu


def _cubes(radar, F, dtype, seed):
    """Noise, a moving on-bin tone and a stronger static one, per frame."""
    import torch
    from paper_2307_09226_amd import rs
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    C, L, Ns = radar.cube_shape()
    x = torch.randn((F, C, L, Ns, 2), generator=g, dtype=torch.float64, device="cuda:0") * 0.1
    n = torch.arange(Ns, dtype=torch.float64, device="cuda:0")
    l = torch.arange(L, dtype=torch.float64, device="cuda:0")[:, None]
    x = torch.view_as_complex(x)
    for f in range(F):
        k, d = (3 + 5 * f) % Ns, 1 + f % max(1, L // 2 - 1)
        x[f] += torch.exp(2j * np.pi * (k * n / Ns - d * l / L)) + 2.0 * torch.exp(2j * np.pi * (7 % Ns) * n / Ns)
    return x.to(torch.complex128 if dtype == rs.RS_C128 else torch.complex64).contiguous()


@pytest.mark.parametrize("M,N,Ns,L,F,dtype", [
    # one, two and three factors of fast time; M = 1, 2, 4, 8, 16 of slow time
    (1, 3, 16, 16, 2, 0), (1, 5, 32, 32, 3, 1), (2, 2, 64, 64, 1, 0), (1, 7, 128, 128, 1, 1),
    (1, 3, 256, 256, 1, 0), (1, 3, 512, 16, 2, 0), (2, 4, 1024, 64, 1, 1), (1, 1, 1024, 256, 1, 0),
    # fewer range bins than a workgroup holds, runs side by side; 97 channels
    (1, 5, 16, 256, 1, 0), (1, 97, 64, 16, 1, 0), (1, 97, 16, 32, 2, 0), (1, 97, 512, 64, 1, 0),
    # the lengths on the LDS FFTs, alone and mixed with the register passes
    (1, 2, 8, 8, 2, 0), (1, 2, 2048, 32, 1, 0), (1, 2, 64, 512, 1, 0), (1, 2, 2, 1024, 1, 0), (1, 3, 4096, 4, 1, 1),
    # Ns 256 below and above the fused kernel's line
    (3, 4, 256, 128, 2, 0), (3, 4, 256, 128, 16, 0), (2, 4, 256, 64, 33, 1),
])
def test_shapes(M, N, Ns, L, F, dtype):
    """Power maps, peaks and Doppler rows against the oracle on the same
    cubes (check_rd), with and without the static bin; the workspace form gives
    the same bits."""
    import torch
    from paper_2307_09226_amd import rs
    radar = dataclasses.replace(scenes.radar_for(M, N, Ns, L, Fs=10e6, Tb=M * 40e-6))
    plan = rs.rs_cube_plan(radar, rs.RS_FORM_MFMA_SPLIT16, dtype, max_pixels=16)
    cubes = _cubes(radar, F, dtype, 17 + Ns + L)
    for skip in (True, False):
        check_rd(radar, plan, cubes, skip)
    power, dtime, _ = rs.range_doppler(plan, cubes)
    p2, d2 = torch.empty_like(power), torch.empty_like(dtime)
    ws = torch.empty(rs.rs_range_doppler_workspace_bytes(plan, F, True), dtype=torch.uint8, device="cuda:0")
    rs.rs_range_doppler_ws(plan, cubes, True, p2, d2, None, ws)
    torch.cuda.synchronize()
    assert torch.equal(power, p2) and torch.equal(dtime, d2)
    plan.close()
