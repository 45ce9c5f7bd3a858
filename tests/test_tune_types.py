"""The tile cache keeps the entries of complex64 and complex128 plans apart:
they run different kernels."""
import json

import pytest

from paper_2307_09226_amd import scenes

pytestmark = pytest.mark.gpu


def _tile(plan, P):
    d = json.loads(plan.describe(P))
    return f"{d['wave_rows']}x{d['tile_l']}x{d['waves']}"


def test_cache_entries_by_type(tmp_path):
    import torch
    from paper_2307_09226_amd import rs
    radar = scenes.radar_for(2, 2, 130, 70, Fs=10e6, Tb=80e-6)
    px = scenes.tiny_scene(506, 1333, vmax=6.0)
    d = rs.DevicePixels.from_host(px)
    key = "4 130 70 2048"

    def tuned(dtype, path):
        """(tile, whether anything was launched)"""
        plan = rs.rs_cube_plan(radar, rs.RS_FORM_MFMA_SPLIT16, dtype, max_pixels=px.P)
        cube = rs.new_cube(plan)
        cube.fill_(complex(3.0, -1.0))
        tile = rs.rs_plan_tune_cached(plan, d, cube, path, reps=1)
        torch.cuda.synchronize()
        assert _tile(plan, px.P) == tile.rstrip("i")
        plan.close()
        return tile, not bool(torch.all(cube == complex(3.0, -1.0)))

    # an entry of each type, in either order: each plan takes its own
    for k, lines in enumerate(([f"{key} 64x64x4", f"{key} 128x64x4 complex128"],
                               [f"{key} 128x64x4 complex128", f"{key} 64x64x4"])):
        path = str(tmp_path / f"both{k}.txt")
        with open(path, "w") as f:
            f.write("\n".join(lines) + "\n")
        assert tuned(rs.RS_C64, path) == ("64x64x4", False)
        assert tuned(rs.RS_C128, path) == ("128x64x4", False)
    # an entry of the other type alone is a miss, and the new entry is of its own type
    for dtype, line, tail in ((rs.RS_C64, f"{key} 128x64x4 complex128", ""), (rs.RS_C128, f"{key} 64x64x4", " complex128")):
        path = str(tmp_path / f"other{dtype}.txt")
        with open(path, "w") as f:
            f.write(line + "\n")
        tile, launched = tuned(dtype, path)
        assert launched
        assert open(path).read().splitlines() == [line, f"{key} {tile}{tail}"]
        assert tuned(dtype, path) == (tile, False)
