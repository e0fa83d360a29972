"""What the host decides before a launch (csrc/ld_launch.h holds it without HIP types), compiled
with g++ and run here."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run_host(tmp_path, body):
    """Lines that a program with `body` in its main prints."""
    src, exe = tmp_path / "p.cpp", tmp_path / "p"
    src.write_text('#include <algorithm>\n#include <cstdio>\n#include <thread>\n#include <vector>\n#include "ld_launch.h"\n' + body)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-pthread", "-Wall", "-Werror", "-I",
                           os.path.join(ROOT, "paper_1807_02752_amd", "csrc"), "-o", str(exe), str(src)])
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout.split("\n")[:-1]


def test_lds_limit_is_kept_by_kernel_and_gpu(tmp_path):
    # two instantiations of one template have the same type; a larger grant of the one, or on another
    # GPU, must not stand for the other's, and a refused size is asked for again
    out = run_host(tmp_path, r"""
template <int N> void kernel(int) {}
template <auto K> void ask(const char* name, int dev, size_t bytes, bool ok = true) {
    bool called = false;
    raise_lds<K>(dev, bytes, [&] { called = true; return ok; });
    std::printf("%s %d %zu %d\n", name, dev, bytes, called ? 1 : 0);
}
int main() {
    ask<kernel<1>>("a", 0, 100000);
    ask<kernel<2>>("b", 0, 71000);
    ask<kernel<1>>("a", 0, 71000);
    ask<kernel<1>>("a", 1, 71000);
    ask<kernel<2>>("b", 0, 90000, false);
    ask<kernel<2>>("b", 0, 90000);
    ask<kernel<2>>("b", 0, 90000);
    ask<kernel<2>>("b", 64, 1);
    ask<kernel<2>>("b", 64, 1);
    ask<kernel<2>>("b", -1, 1);
}
""")
    assert out == ["a 0 100000 1", "b 0 71000 1", "a 0 71000 0", "a 1 71000 1", "b 0 90000 1", "b 0 90000 1",
                   "b 0 90000 0", "b 64 1 1", "b 64 1 1", "b -1 1 1"]


def test_lds_limit_never_falls_between_threads(tmp_path):
    # the last size set is the largest one, whatever order the threads come in
    out = run_host(tmp_path, r"""
void kernel(int) {}
int main() {
    size_t last = 0;
    int falls = 0;
    std::vector<std::thread> ts;
    for (int t = 0; t < 8; ++t)
        ts.emplace_back([&, t] {
            for (size_t i = 0; i < 2000; ++i) {
                const size_t n = 1 + (i * 7919 + t * 104729) % 160000;
                raise_lds<kernel>(0, n, [&] { falls += n < last; last = n; return true; });
            }
        });
    for (auto& t : ts) t.join();
    size_t most = 0;
    for (size_t t = 0; t < 8; ++t)
        for (size_t i = 0; i < 2000; ++i) most = std::max(most, 1 + (i * 7919 + t * 104729) % 160000);
    std::printf("%d %d\n", falls, last == most);
}
""")
    assert out == ["0 1"]


# (width, block radius, d_max, propagation bound, pairs) and the form that was the fastest or within a few
# percent of it: strips of eight lanes (0), of four with 16 rows (1) or 8 (2), a pair a workgroup (3)
STEREO = [
    (64, 3, 48, 1, 1, 0), (64, 3, 48, 1, 64, 0), (64, 3, 48, 1, 96, 1), (64, 3, 48, 1, 128, 1), (64, 3, 48, 1, 256, 2), (64, 3, 48, 1, 512, 2),
    (160, 3, 48, 1, 192, 2), (160, 3, 48, 1, 256, 3), (160, 3, 48, 1, 384, 2), (160, 3, 48, 1, 512, 3),
    (320, 3, 64, 1, 128, 2), (320, 3, 64, 1, 192, 3), (320, 3, 64, 1, 400, 3), (320, 1, 64, 1, 192, 3), (320, 5, 64, 1, 192, 3),
    (640, 3, 64, 1, 96, 2), (640, 3, 64, 1, 160, 3), (640, 3, 64, 1, 192, 3),
    (1242, 3, 128, 1, 1, 0), (1242, 3, 128, 1, 8, 1), (1242, 3, 128, 1, 32, 2), (1242, 3, 128, 1, 109, 2), (1242, 3, 128, 1, 128, 3),
    (1242, 3, 128, 0, 64, 2), (1242, 3, 128, 0, 96, 3), (1242, 3, 255, 1, 64, 2), (1242, 3, 128, 1, 512, 3),
    (1920, 3, 128, 1, 96, 2), (1920, 3, 128, 1, 160, 3), (2048, 3, 128, 1, 96, 2), (2048, 3, 128, 1, 256, 3),
    (6, 3, 48, 1, 1, 3), (3, 1, 48, 1, 1, 3), (7, 3, 48, 1, 1, 0),
]


def test_stereo_form_by_width_and_pairs(tmp_path):
    # strips up to 2400 workgroups whatever the width made 192 to 400 pairs of 320 columns and 128 to 200
    # of 640 slower than the sweep
    calls = "".join(f"std::printf(\"%d\\n\", (int)stereo_form({w}, 60, {rho}, {dm}, {tau}, {n}));\n" for w, rho, dm, tau, n, _ in STEREO)
    out = run_host(tmp_path, "int main() {\n" + calls + "std::printf(\"%d\\n\", (int)stereo_form(64, 6, 3, 48, 1, 1));\n}\n")
    assert [(c[:-1], int(o)) for c, o in zip(STEREO, out)] == [(c[:-1], c[-1]) for c in STEREO]
    assert out[-1] == "3"


def test_stereo_strips_fit_lds(tmp_path):
    # whatever form is taken fits, and no form is refused for its size at the largest disparities
    out = run_host(tmp_path, r"""
int main() {
    size_t most = 0;
    for (int rho = 1; rho <= 5; ++rho)
        for (int E : {64, 128})
            for (int T : {8, 16}) most = std::max(most, stereo_strip_lds(rho, E, T, 255));
    std::printf("%d\n", most <= (size_t)kMaxLds);
}
""")
    assert out == ["1"]


def test_vdisp_dp_in_lockstep_by_rows(tmp_path):
    # (waves, d_max): tall frames of few disparities were slower in turns than before those
    cases = [(16, 1, 1), (16, 8, 1), (16, 24, 1), (16, 48, 1), (16, 128, 0), (9, 8, 1), (9, 64, 0), (6, 8, 1), (6, 48, 0), (3, 8, 1),
             (3, 48, 0), (3, 128, 0), (1, 48, 0), (2, 255, 0)]
    calls = "".join(f'std::printf("%d\\n", vdisp_lockstep({w}, {d}) ? 1 : 0);\n' for w, d, _ in cases)
    assert [int(x) for x in run_host(tmp_path, "int main() {\n" + calls + "}\n")] == [x for *_, x in cases]


def test_vpx_votes_staged_by_frames(tmp_path):
    # (width, height, waves, bytes beside, frames), frames a CU: the LDS of that many fits a CU, 1280 bytes
    # at a time, and is not given away where fewer would do
    cases = [(320, 96, 2, 5700, 1, 1), (320, 96, 2, 5700, 768, 3), (320, 96, 2, 5700, 1024, 4), (320, 96, 2, 5700, 1536, 6),
             (320, 96, 2, 5700, 2048, 8), (160, 120, 2, 5800, 1500, 6), (1242, 375, 5, 22800, 768, 3), (1242, 375, 5, 22800, 1024, 4),
             (1242, 375, 5, 22800, 2048, 4), (1920, 1080, 7, 36100, 256, 1), (1920, 1080, 7, 36100, 1024, 2), (4096, 700, 14, 71400, 600, 1)]
    calls = "".join(f'std::printf("%d\\n", vpx_staged_votes({w}, {h}, {nw}, {fx}, {n}));\n' for w, h, nw, fx, n, _ in cases)
    for (w, h, nw, fixed, n, per_cu), x in zip(cases, run_host(tmp_path, "int main() {\n" + calls + "}\n")):
        lds = -(-(fixed + 2 * int(x) + 512) // 1280) * 1280      # (the kernel's static arrays take 304)
        assert per_cu * lds <= 160 * 1024, (w, n, x)
        assert int(x) >= w * h or (per_cu + 1) * (lds + 1280 + 1024) > 160 * 1024, (w, n, x)


def test_energy_form_by_width_and_frames(tmp_path):
    # two launches (0), 512 threads a frame (1) or 256 (2), the fastest measured: one line at 192 frames for
    # every width made 193 to 384 frames of up to 512 columns slower than 256 threads had been
    cases = [(64, 1, 0), (64, 193, 0), (64, 384, 0), (64, 385, 2), (320, 320, 0), (512, 256, 0), (512, 384, 0), (512, 385, 2), (960, 384, 0),
             (1024, 384, 0), (1025, 193, 1), (1242, 192, 0), (1242, 193, 1), (1242, 384, 1), (1242, 385, 2), (1536, 1024, 2), (1537, 1024, 1),
             (1920, 192, 0), (1920, 193, 1), (4096, 1, 0), (4096, 500, 1)]
    calls = "".join(f'std::printf("%d\\n", (int)energy_form({w}, {n}));\n' for w, n, _ in cases)
    assert [int(x) for x in run_host(tmp_path, "int main() {\n" + calls + "}\n")] == [x for *_, x in cases]


def test_histogram_rows_by_width_and_frames(tmp_path):
    # rows a workgroup, within a few percent of the fastest measured: one line on the groups for every width
    # made some hundred narrow frames slower than 32 rows had been
    cases = [(64, 375, 256, 16), (64, 375, 1500, 32), (64, 64, 1, 4), (64, 64, 1024, 16), (160, 120, 1, 4), (160, 120, 256, 16), (160, 120, 2048, 32),
             (320, 96, 1, 4), (320, 96, 256, 8), (320, 96, 768, 16), (320, 96, 2048, 16), (641, 240, 256, 8), (641, 240, 2048, 16), (960, 300, 1, 4),
             (1242, 375, 1, 4), (1242, 375, 61, 4), (1242, 375, 512, 8), (1242, 375, 1024, 32), (1920, 1080, 1, 4), (1920, 1080, 256, 8),
             (4096, 700, 600, 32)]
    calls = "".join(f'std::printf("%d\\n", hist_rows({w}, {h}, {n}, 4, 32));\n' for w, h, n, _ in cases)
    out = run_host(tmp_path, "int main() {\n" + calls + 'std::printf("%d\\n", hist_rows(1242, 375, 1024, 4, 8));\n}\n')
    assert [int(x) for x in out] == [x for *_, x in cases] + [8]


def test_edge_rows_by_width_and_frames(tmp_path):
    # rows a workgroup by rows times waves: one line on the rows alone made 64 frames of 2560 x 720 and 64 to
    # 128 of 4000 x 400 slower than 32 rows had been
    cases = [(64, 1, 1, 2), (64, 1, 256, 4), (96, 2, 1, 2), (96, 2, 256, 8), (375, 5, 1, 2), (375, 5, 16, 4), (376, 5, 61, 8), (375, 5, 128, 8),
             (375, 5, 256, 32), (375, 5, 1024, 32), (1080, 8, 1, 2), (1080, 8, 4, 4), (1080, 8, 32, 8), (1080, 8, 64, 32), (720, 10, 64, 32),
             (400, 16, 4, 4), (400, 16, 32, 8), (400, 16, 64, 32), (400, 16, 128, 32)]
    calls = "".join(f'std::printf("%d\\n", edge_rows({h}, {nw}, {n}));\n' for h, nw, n, _ in cases)
    assert [int(x) for x in run_host(tmp_path, "int main() {\n" + calls + "}\n")] == [x for *_, x in cases]


def test_ransac_threads_by_frames(tmp_path):
    # 512 threads with two frames a CU were slower than 192 at every size, for short frames than before those
    body = "int main() { for (int n : {1, 256, 257, 384, 512, 513, 4096}) std::printf(\"%d\\n\", ransac_threads(n)); }\n"
    assert [int(x) for x in run_host(tmp_path, body)] == [512, 512, 192, 192, 192, 192, 192]
