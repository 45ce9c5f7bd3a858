"""Sessions whose budget is what small requests need."""
import pytest

from paper_2307_09226_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,Ns,L,P", [(1, 4, 128, 64, 4057), (3, 4, 256, 64, 4000), (2, 4, 128, 128, 9000)])
def test_budget_of_1024_pixel_chunks(M, N, Ns, L, P):
    """A budget of one partial cube per started 1,024 pixels, twice, serves two
    requests at a time, with the bits of the single call."""
    import torch
    from paper_2307_09226_amd import rs
    radar = scenes.radar_for(M, N, Ns, L, Fs=10e6, Tb=M * 40e-6)
    plan = rs.rs_cube_plan(radar, rs.RS_FORM_MFMA_SPLIT16, rs.RS_C64, max_pixels=P)
    need = (P + 1023) // 1024 * M * N * Ns * L * 8
    assert plan.workspace_bytes(P) <= need
    px = [rs.DevicePixels.from_host(scenes.tiny_scene(40 + k, P, vmax=6.0)) for k in range(4)]
    alone, served = ([rs.new_cube(plan) for _ in px] for _ in range(2))
    for p, c in zip(px, alone):
        rs.rs_beat_synthesize(plan, p, c)
    torch.cuda.synchronize()
    sess = rs.Session(hbm_budget=2 * need, max_slots=4)
    tickets = [sess.submit(plan, p, c) for p, c in zip(px, served)]
    sess.drain()
    assert all(sess.poll(t)[0] == rs.RS_REQ_DONE for t in tickets)
    assert sess.stats()["footprint_peak"] <= 2 * need
    sess.close()
    assert all(torch.equal(a, b) for a, b in zip(alone, served))
    plan.close()
