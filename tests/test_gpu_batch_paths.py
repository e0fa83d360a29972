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


@pytest.mark.parametrize("kind,w,h,kw", [
    # one wave of columns to its last, one and two more columns; several waves
    ("road", 319, 96, {}), ("road", 320, 96, {}), ("road", 321, 97, {}), ("road", 640, 80, {}), ("road", 643, 66, {}),
    # bands of one row, of three, and past the road
    ("road", 321, 96, {"chi": 0}), ("road", 257, 96, {"chi": 1}), ("road", 257, 96, {"chi": 400}),
    # narrower windows, and rows far longer than a wave
    ("road", 321, 64, {"tau_x_max": 0}), ("road", 321, 64, {"tau_x_max": 4, "lambda_x": 7}),
    ("random", 333, 61, {}), ("random", 300, 90, {"chi": 0}),
    # more edges than LDS stages: the rows past it read theirs from memory
    ("random", 1000, 400, {}),
])
def test_vpx_path_by_width_and_band(kind, w, h, kw):
    import oracle
    from paper_1807_02752_amd import ld
    g, d = _frames(kind, w, h, 2)
    dm = 32 if kind == "random" else 48
    out = run_gpu(g, d, dm, params=ld.params_default(**kw))
    for b in range(2):
        compare_frame(out, b, g[b], d[b], dm, params=oracle.default_params(**kw))


@pytest.mark.parametrize("w,h,n,kw", [
    # few and many frames a launch; point counts of every remainder of four; few samples, draws
    # that repeat an index (short frames), rounds cut off, no survivors, one round
    (96, 40, 512, {}), (96, 40, 513, {}), (129, 65, 2, {}), (129, 66, 2, {}), (129, 67, 2, {}), (129, 68, 2, {}),
    (64, 24, 3, {}), (64, 18, 3, {"n_hyp": 63}), (320, 96, 1, {"n_hyp": 1}), (320, 96, 2, {"n_hyp": 7, "max_rounds": 1}),
    (320, 97, 2, {"tr_x": 0.0, "tr_y": 0.0}), (321, 98, 2, {"tr_x": 1e9, "eps_num": 100}), (320, 99, 2, {"seed": 2 ** 40 + 5}),
])
def test_ransac_by_points_and_samples(w, h, n, kw):
    import oracle
    from paper_1807_02752_amd import ld
    g, d = _frames("road", w, h, n)
    out = run_gpu(g, d, 48, params=ld.params_default(**kw))
    out.pop("curves", None)     # a poor model's curves end at 1e5 columns, where FP32 itself is 4e-3 off
    for b in sorted({0, n // 2, n - 1}):
        compare_frame(out, b, g[b], d[b], 48, params=oracle.default_params(**kw))


@pytest.mark.parametrize("w,h,d_max,kw", [
    # rows of one wave to its last, one more, several waves; a step count of every kind of chunk
    (96, 127, 48, {}), (96, 128, 49, {}), (96, 129, 55, {}), (64, 257, 57, {}), (64, 385, 63, {}), (33, 20, 48, {}),
    # jump bounds of either register form, and past them
    (96, 130, 48, {"tau_y_max": 0}), (96, 130, 48, {"tau_y_max": 1}), (96, 131, 50, {"tau_y_max": 7, "lambda_y": 3}),
    (96, 255, 48, {"tau_y_max": 8}), (96, 255, 48, {"tau_y_max": 9}), (96, 130, 48, {"tau_y_max": 200}),
    (96, 130, 48, {"lambda_y": 1000}), (96, 130, 48, {"lambda_y": 0}),
    # a backtrace larger than LDS, and four rows a lane
    (64, 700, 600, {}), (64, 701, 1023, {}), (64, 2047, 64, {}), (32, 2049, 60, {}), (32, 2305, 57, {"tau_y_max": 8}),
])
def test_vdisp_path_by_rows_and_jumps(w, h, d_max, kw):
    import oracle
    from paper_1807_02752_amd import ld
    g, d = _frames("road", w, h, 2)
    out = run_gpu(g, d, d_max, params=ld.params_default(**kw))
    out.pop("curves", None)     # FP32, far outside the image for a poor model
    for b in range(2):
        compare_frame(out, b, g[b], d[b], d_max, params=oracle.default_params(**kw))


@pytest.mark.parametrize("h", [255, 256, 257, 513])
def test_curves_by_rows(h):
    # the curves leave in tiles of 256 rows
    g, d = _frames("road", 320, h, 2)
    out = run_gpu(g, d, 48)
    for b in range(2):
        r = compare_frame(out, b, g[b], d[b], 48)
        top = out["curves"][b, :, :r.v_end]
        assert np.isnan(top).all() and np.isnan(out["curves"][b, len(r.u_start):]).all()


@pytest.mark.parametrize("w,h,n", [(64, 41, 1), (64, 42, 3), (48, 39, 2458), (48, 40, 2457), (48, 42, 6700), (33, 44, 7100)])
def test_vdisp_histogram_by_frame_count(w, h, n):
    # four, eight and all rows a workgroup, with rows left over: counts of every row and disparity
    import torch
    from paper_1807_02752_amd import ld
    rng = np.random.default_rng(h)
    disp = rng.integers(0, 40, size=(n, h, w)).astype(np.uint8)
    det = ld.Detector(w, h, n, ld.LD_DISP_U8, 32)
    out = torch.full((n, h, 33), -1, dtype=torch.int32, device="cuda")
    det.vdisp(torch.from_numpy(disp).cuda(), vdisp_out=out)
    det.sync()
    got = out.cpu().numpy()
    det.close()
    for b in sorted({0, 1 % n, n // 2, n - 1}):
        want = np.stack([np.bincount(np.minimum(row[row > 0], 32), minlength=33) for row in disp[b]])
        assert np.array_equal(got[b], want), b


@pytest.mark.parametrize("w,h,n", [(257, 40, 51), (257, 41, 50), (130, 63, 130), (130, 64, 129), (64, 39, 1681), (64, 40, 1638)])
def test_edges_by_frame_count(w, h, n):
    # strips of two, four, eight and 32 rows, with and without rows left over
    g, d = _frames("road", w, h, n)
    out = run_gpu(g, d, 48)
    out.pop("curves", None)     # FP32, far outside the image for a poor model
    for b in sorted({0, n // 2, n - 1}):
        compare_frame(out, b, g[b], d[b], 48)


def _noise(w, h, d_max, every, seed=0):
    """A noise image over a plane: every pixel of one in `every` groups of eight columns."""
    g, d = synth.degenerate("random", w, h, synth.FMT_U8, 32, seed=seed)
    d[:] = np.arange(h)[:, None] * d_max // h
    g[:, (np.arange(w) // 8) % every != 0] = 90
    return g, d


@pytest.mark.parametrize("w,h,n,every,kw", [
    # rows of many edges, whose votes all the waves share: none, some and most of them staged; a few
    # more than a thread each, and several; bands of one row and past the road; narrower windows
    (641, 120, 2, 1, {}), (641, 121, 2, 2, {"chi": 0}), (1000, 90, 2, 1, {"chi": 400}), (1242, 60, 1, 2, {"tau_x_max": 3}),
    (641, 120, 600, 4, {}), (1242, 130, 2, 3, {"chi": 1}), (1930, 64, 1, 1, {"tau_x_max": 0}), (320, 96, 1030, 1, {}),
])
def test_vpx_votes_of_dense_rows(w, h, n, every, kw):
    import oracle
    from paper_1807_02752_amd import ld
    pair = [_noise(w, h, 120, every, s) for s in range(2)]
    g = np.stack([pair[i % 2][0] for i in range(n)])
    d = np.stack([pair[i % 2][1] for i in range(n)])
    out = run_gpu(g, d, 120, params=ld.params_default(**kw))
    out.pop("curves", None)     # FP32, far outside the image for a poor model
    for b in sorted({0, n // 2, n - 1}):
        compare_frame(out, b, g[b], d[b], 120, params=oracle.default_params(**kw))


def test_vpx_time_of_dense_rows():
    # with one wave keeping the counts a frame of noise took fifteen times as long as one with a
    # sixteenth of its edges, with the votes shared three times
    import torch
    from paper_1807_02752_amd import ld
    us = []
    for every in (1, 16):
        g, d = _noise(1920, 540, 200, every)
        det = ld.Detector(1920, 540, 1, ld.LD_DISP_U8, 200)
        g, d = torch.from_numpy(g[None]).cuda(), torch.from_numpy(d[None]).cuda()
        det.vdisp(d)
        det.vp_ransac(g, d)
        times = []
        for _ in range(5):
            det.profile(True)
            det.vp_ransac(g, d)
            det.sync()
            times.append(det.kernel_times()["k_vpx_fit"][0] * 1e3)
        us.append(min(times))
        det.close()
    assert us[0] < 6 * us[1], us


@pytest.mark.parametrize("w,h,every", [(641, 240, 5), (1242, 375, 8)])
def test_vpx_time_of_half_dense_rows(w, h, every):
    # rows of some 150 edges take 1.5 times as long as rows of a quarter of them, which one wave keeps
    # the counts of; 2 to 2.2 times while the shared votes waited for each read, or one wave kept these too
    import torch
    from paper_1807_02752_amd import ld
    us = []
    for k in (every, 32):
        g, d = _noise(w, h, 128, k)
        det = ld.Detector(w, h, 1, ld.LD_DISP_U8, 128)
        g, d = torch.from_numpy(g[None]).cuda(), torch.from_numpy(d[None]).cuda()
        det.vdisp(d)
        det.vp_ransac(g, d)
        times = []
        for _ in range(10):
            det.profile(True)
            det.vp_ransac(g, d)
            det.sync()
            times.append(det.kernel_times()["k_vpx_fit"][0] * 1e3)
        us.append(min(times))
        det.close()
    assert us[0] < 1.85 * us[1], us


@pytest.mark.parametrize("h,d_max,kw", [
    # the v-disparity DP in lockstep and, one disparity on, in turns: one wave, several, sixteen of either
    # number of rows a lane; steps of part of a chunk, a whole one and one more
    (128, 1, {}), (128, 4, {}), (128, 5, {}), (129, 8, {"tau_y_max": 8}), (300, 12, {}), (300, 13, {}), (720, 7, {"tau_y_max": 7}),
    (1080, 9, {}), (1080, 36, {}), (1080, 37, {}), (2048, 3, {}), (2048, 16, {"lambda_y": 0}), (2048, 64, {}), (2049, 8, {}),
    (2049, 36, {"tau_y_max": 3}), (2049, 37, {}), (4096, 2, {}), (4096, 17, {}), (4096, 64, {}), (4096, 65, {"tau_y_max": 8}),
])
def test_vdisp_path_of_tall_frames(h, d_max, kw):
    import oracle
    from paper_1807_02752_amd import ld
    pair = [_noise(40, h, d_max, 1, s) for s in range(2)]
    g, d = np.stack([p[0] for p in pair]), np.stack([p[1] for p in pair])
    rng = np.random.default_rng(h + d_max)
    d = np.where(rng.random(d.shape) < 0.4, rng.integers(0, d_max + 1, d.shape), d).astype(np.uint8)
    out = run_gpu(g, d, d_max, params=ld.params_default(**kw))
    out.pop("curves", None)     # FP32, far outside the image for a poor model
    for b in range(2):
        compare_frame(out, b, g[b], d[b], d_max, params=oracle.default_params(**kw))


@pytest.mark.parametrize("w,h,n", [(130, 63, 200), (257, 41, 180), (300, 64, 90), (64, 41, 4000), (64, 39, 8000), (64, 64, 4801)])
def test_edges_by_rows_of_waves(w, h, n):
    # strips of four, eight and 32 rows, with and without rows left over
    g, d = _frames("road", w, h, n)
    out = run_gpu(g, d, 48)
    out.pop("curves", None)     # FP32, far outside the image for a poor model
    for b in sorted({0, n // 2, n - 1}):
        compare_frame(out, b, g[b], d[b], 48)


@pytest.mark.parametrize("w,h,n", [
    # a workgroup a frame: 512 threads with three to eight columns each, 256 with two to six; widths that
    # fill the threads' columns, one more, and the largest
    (1025, 64, 193), (1242, 66, 193), (1536, 61, 384), (2048, 50, 193), (2049, 50, 193), (3072, 40, 193), (3073, 40, 193),
    (4096, 41, 193), (256, 70, 385), (257, 64, 385), (513, 64, 385), (769, 62, 385), (1024, 60, 385), (1280, 58, 385), (1281, 60, 385),
])
def test_energies_by_columns_a_thread(w, h, n):
    g, d = _frames("road", w, h, n)
    out = run_gpu(g, d, 48)
    out.pop("curves", None)     # FP32, far outside the image for a poor model
    for b in sorted({0, n // 2, n - 1}):
        compare_frame(out, b, g[b], d[b], 48)


@pytest.mark.parametrize("kind,w,h,few", [("road", 300, 96, 384), ("road", 1024, 64, 384), ("random", 320, 60, 384),
                                          ("road", 1100, 64, 192), ("road", 1600, 70, 192), ("random", 1242, 50, 192)])
def test_energies_same_bits_in_either_form(kind, w, h, few):
    # the most frames that take two launches, and one more: every sum is taken in the same order
    from paper_1807_02752_amd import ld
    import torch
    g, d = _frames(kind, w, h, few + 1)
    dm = 32 if kind == "random" else 48
    res = []
    for n in (few, few + 1):
        det = ld.Detector(w, h, n, ld.LD_DISP_U8, dm)
        gg, dd = torch.from_numpy(g[:n]).cuda(), torch.from_numpy(d[:n]).cuda()
        det.vdisp(dd)
        det.vp_ransac(gg, dd)
        det.lane_energy()
        det.sync()
        res.append(np.stack([det.read(ld.LD_STATE_ENERGY, b) for b in (0, 1, few // 2, few - 1)]))
        det.close()
    assert np.abs(res[0]).max() > 0
    assert np.array_equal(res[0], res[1])
