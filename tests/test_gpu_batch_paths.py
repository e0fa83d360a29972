"""The kernels that the number of frames chooses between (a whole chip for few frames, a
workgroup a frame for many), at the sizes where their tiles end: each against the CPU oracle
with the tolerances of test_gpu_parity (bit-exact decisions, energies within 1e-5 of the
frame's largest)."""
import numpy as np
import pytest

from paper_1807_02752_amd import synth
from test_gpu_parity import compare_frame, run_gpu

pytestmark = pytest.mark.gpu


def _frames(kind, w, h, n):
    if kind == "random":     # every pixel an edge of some road row: rows far longer than a wave
        pair = [synth.degenerate("random", w, h, synth.FMT_U8, 32, seed=s) for s in range(2)]
        for _, d in pair:    # a road under the noise, so that the edges are on it
            d[:] = np.clip(np.arange(h)[:, None] * 30 // h, 0, 32)
    else:
        pair = [synth.make_scaled_c1(w, h, 48, seed=3, idx=s)[:2] for s in range(2)]
    g = np.stack([pair[i % 2][0] for i in range(n)])
    d = np.stack([pair[i % 2][1] for i in range(n)])
    return g, d


@pytest.mark.parametrize("kind,w,h,n", [
    ("road", 33, 20, 1), ("road", 238, 96, 2), ("road", 241, 97, 3), ("road", 479, 113, 1), ("road", 1290, 64, 1),
    ("random", 301, 75, 2), ("road", 320, 96, 192), ("road", 320, 96, 193), ("road", 129, 65, 384),
    ("road", 129, 65, 385), ("random", 150, 60, 193), ("random", 150, 60, 400), ("road", 1537, 72, 193),
])
def test_energies_by_frame_count(kind, w, h, n):
    g, d = _frames(kind, w, h, n)
    dm = 32 if kind == "random" else 48
    out = run_gpu(g, d, dm)
    for b in sorted({0, n // 2, n - 1}):
        compare_frame(out, b, g[b], d[b], dm)
