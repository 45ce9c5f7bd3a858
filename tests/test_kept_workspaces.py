"""Workspaces that the allocating calls keep with their plan."""
import threading

import pytest

from paper_2307_09226_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["mfma", "nufft"])
def test_streams_sizes_and_threads(form):
    """More streams than a plan keeps workspaces for, sizes that grow and
    shrink, and threads with a stream each: the bits of the call on a
    workspace of its own."""
    import torch
    from paper_2307_09226_amd import rs
    radar = scenes.radar_for(2, 2, 64, 32, Fs=10e6, Tb=40e-6)
    sizes = [33, 3000, 700, 6001, 1, 6001, 33]
    plan = rs.rs_cube_plan(radar, rs.RS_FORM_MFMA_SPLIT16 if form == "mfma" else rs.RS_FORM_NUFFT,
                           rs.RS_C64, max_pixels=max(sizes))
    px = [rs.DevicePixels.from_host(scenes.tiny_scene(70 + i, P, vmax=6.0)) for i, P in enumerate(sizes)]
    want = []
    for p, P in zip(px, sizes):
        cube = rs.new_cube(plan, "cuda:0")
        ws = torch.empty(max(plan.workspace_bytes(P), 1), dtype=torch.uint8, device="cuda:0")
        rs.rs_beat_synthesize_ws(plan, p, cube, ws)
        want.append(cube)
    torch.cuda.synchronize()

    streams = [torch.cuda.Stream() for _ in range(11)]
    got = []
    torch.cuda.synchronize()
    for k in range(3 * len(streams)):
        with torch.cuda.stream(streams[k % len(streams)]):
            cube = rs.new_cube(plan, "cuda:0")
        rs.rs_beat_synthesize(plan, px[k % len(px)], cube, stream=streams[k % len(streams)])
        got.append((k % len(px), cube))

    def work(t):
        for k in range(12):
            i = (k + t) % len(px)
            cube = cubes[t][k]
            rs.rs_beat_synthesize(plan, px[i], cube, stream=streams[t])
            got.append((i, cube))

    cubes = [[rs.new_cube(plan, "cuda:0") for _ in range(12)] for _ in range(4)]
    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert len(got) == 33 + 48
    for i, cube in got:
        assert torch.equal(cube, want[i])
    plan.close()


@pytest.mark.parametrize("form", ["mfma", "nufft"])
def test_captured_calls_keep_their_own_workspace(form):
    """A call captured after eager ones takes no kept workspace: replays
    between eager calls on other pixels give the bits of the eager call."""
    import torch
    from paper_2307_09226_amd import rs
    radar = scenes.radar_for(2, 2, 64, 32, Fs=10e6, Tb=40e-6)
    plan = rs.rs_cube_plan(radar, rs.RS_FORM_MFMA_SPLIT16 if form == "mfma" else rs.RS_FORM_NUFFT,
                           rs.RS_C64, max_pixels=6001)
    a, b = (rs.DevicePixels.from_host(scenes.tiny_scene(90 + i, P, vmax=6.0)) for i, P in enumerate((3000, 6001)))
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        want, cube, other = (rs.new_cube(plan, "cuda:0") for _ in range(3))
        rs.rs_beat_synthesize(plan, a, want, stream=s)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            rs.rs_beat_synthesize(plan, a, cube, stream=s)
        for _ in range(4):
            cube.zero_()
            rs.rs_beat_synthesize(plan, b, other, stream=s)
            g.replay()
            rs.rs_beat_synthesize(plan, b, other, stream=s)
            s.synchronize()
            assert torch.equal(cube, want)
    plan.close()
