"""NUFFT spreading: the sort of a block's points by window column."""

import numpy as np
import pytest

from oracle import nufft as onufft
from paper_2307_09226_amd import scenes
from gpu_util import errors
from test_nufft_gpu import GATE_FP32, _synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [1, 31, 64, 65, 255, 256, 257])
@pytest.mark.parametrize("cols", [1, 2, 126, 129, 255, 258, 511, 514])
def test_columns_of_a_block(cols, P):
    """Points of one block over `cols` window columns (a thread counts two, a
    wavefront 128, a block at most 512), in random order, with whole groups in
    one column; every other scene in two Doppler groups (two sub-boxes).
    Within the float32 gate of the NUFFT oracle."""
    rng = np.random.default_rng(1000 * cols + P)
    z = np.zeros((1, 3))
    r = scenes.Radar(M=1, N=1, Ns=512, L=64, fc=77e9, mu=30e12, Fs=10e6, Tb=120e-6, tx=z, rx=z.copy())
    n1 = 1024
    cell = r.c0 * r.Fs / (2 * r.mu) / n1               # metres per grid column
    k = rng.integers(0, cols, P) if cols > 1 else np.zeros(P)
    k[: P // 4] = k[0]
    k[-1] = cols - 1
    rr = (40.3 + k + 0.4 * rng.uniform(size=P)) * cell
    f32 = lambda a: np.ascontiguousarray(a, dtype=np.float32)
    fast = (np.arange(P) % 3 == 0) & (cols % 2 == 0)
    px = scenes.Pixels(f32(rr), f32(np.zeros(P)), f32(np.zeros(P)), f32(rng.lognormal(0, 0.5, P)),
                       f32(np.where(fast, 5.0, 0.0)))
    rel, _ = errors(_synth(r, px, 1e-6), onufft.nufft_cube(r, px, 1e-6))
    print(f"cols={cols} P={P}: vs NUFFT oracle {rel:.2e}", flush=True)
    assert rel <= GATE_FP32
