// ld_launch.h -- what the host decides before a launch, without HIP types: the dynamic LDS that
// a kernel has been granted, and which form of a kernel a launch takes.  Not part of the C ABI.
#pragma once

#include <algorithm>
#include <atomic>
#include <cstddef>
#include <cstdint>
#include <mutex>

constexpr int kCUs = 256;              // compute units of one GPU
constexpr int kMaxLds = 160 * 1024;    // LDS bytes a workgroup may hold on gfx950
constexpr int kMaxDevices = 64;

// The dynamic LDS granted to one kernel on each GPU.
struct LdsGrants {
    std::mutex mu;
    std::atomic<size_t> bytes[kMaxDevices] = {};
};

// Raises the dynamic LDS limit of Kernel on `device` to `bytes` by set(), which says whether that
// worked, unless it is there already.  The record is the kernel's own (a template argument: two
// instantiations of one kernel template have the same type) and the GPU's, and set() runs under
// its lock, so that no thread lowers what another has just raised.
template <auto Kernel, typename Set>
void raise_lds(int device, size_t bytes, Set set) {
    static LdsGrants grants;
    if (device < 0 || device >= kMaxDevices) {
        (void)set();
        return;
    }
    std::atomic<size_t>& have = grants.bytes[device];
    if (bytes <= have.load(std::memory_order_acquire)) return;
    std::lock_guard<std::mutex> lock(grants.mu);
    if (bytes > have.load(std::memory_order_relaxed) && set()) have.store(bytes, std::memory_order_release);
}

// Whether the v-disparity DP of `waves` waves takes its steps in lockstep, a barrier a step, or in turns
// of eight steps, a wave a turn behind the one below it.  The turns to fill and drain that pipeline
// take as long as steps: us in turns and in lockstep, for 8, 24, 48 and 64 disparities, 375 rows (three
// waves) 11, 10; 14, 15; 28, 31; 29, 35; 720 (six) 15, 12; 17, 17; 22, 24; 37, 41; 1080 (nine) 18, 13; 21,
// 19; 26, 27; 30, 33; 2048 (sixteen) 27, 16; 30, 23; 38, 34; 42, 41; 4096 (sixteen, four rows a lane) 39, 20;
// 44, 32; 61, 50; 67, 62 (before the pipeline, a barrier and nine LDS reads a step, 4096 rows: 23, 40, 68, 86).
inline bool vdisp_lockstep(int waves, int d_max) { return d_max <= 4 * waves; }

// The largest LDS of a workgroup of which per_cu fit a CU: it is given out 1280 bytes at a time (with three
// equal shares of the 160 KiB the third found no place: 768 frames of 320 x 96 took 100 us, now 57).
inline size_t lds_share(int per_cu) { return (size_t)kMaxLds / per_cu / 1280 * 1280; }

// Vote columns (16 bits) that the V_px row DP stages in LDS, of `waves` waves a frame and `fixed` bytes
// beside them: what is left when a CU holds the frames that it is given (up to eight, and to seven waves
// a SIMD), fewer frames where that would not stage an edge on every 96 pixels (road scenes hold one on
// 55 to 170): a row that is not staged costs a load's latency, about two staged rows.  (With at
// most four frames a CU, 1536 frames of 320 x 96 took 124 us, now 79.)
inline int vpx_staged_votes(int W, int H, int waves, size_t fixed, int frames) {
    auto room = [&](int per_cu) -> size_t {
        const size_t share = lds_share(per_cu) - 1024;                 // 1 KiB: the static arrays
        return share > fixed ? (share - fixed) / 2 / 8 * 8 : 0;
    };
    const size_t px = (size_t)W * H;
    int per_cu = std::max(1, std::min(std::min(8, 28 / waves), (frames + kCUs - 1) / kCUs));
    while (per_cu > 1 && room(per_cu) < px / 96) --per_cu;
    return (int)std::min((px + 7) / 8 * 8, room(per_cu));
}

// Which form of the energies a launch takes: two launches over the whole chip (k_m1 and k_tracks), or one
// workgroup of 512 or of 256 threads a frame (k_energy); us of the step, 1242 x 375 and, after
// the slash, 1920 x 1080 frames with u16 disparity:
//   frames          1     61    128     192     256     384    512    1024
//   two launches  24/51   59   109/412 163/591 206/785  322   426     806
//   k_energy 512    -      -   189/602 194/614 198/617  257   262/914  515
//   k_energy 256  187/740 201  218/828 223/836 225/837  257   260/1047 388
// A frame's sweep is one workgroup with a barrier a row, so below about a workgroup per CU its
// time is its latency; the two launches use the whole chip for any number of frames but move M_1
// through memory (R W floats a frame, written and read), which costs more than the sweep the sooner
// the wider the frame is: from 192 frames, or from 384 up to 1024 columns (us at 384 frames, two
// launches, 512 and 256 threads: 64 x 64 28, 45, 38; 320 x 96 55, 63, 60; 512 x 160 84, 118, 98; 641 x
// 240 131, 189, 179; 960 x 300 227, 236, 243).  With one or two frames per CU the sweep of a wider
// frame is shortest with 512 threads (two waves a SIMD, edges loaded three rows ahead); with
// four, 256 threads issue less for the same columns.  Above 1536 columns 256 threads would own 8 and
// more columns each (192 VGPRs, two workgroups a CU): 512 threads there for every number of frames.
enum class EnergyForm { kTwoLaunches, kThreads512, kThreads256 };

inline EnergyForm energy_form(int W, int frames) {
    if (frames <= (W <= 1024 ? 384 : 192)) return EnergyForm::kTwoLaunches;
    return (frames <= 384 || W > 1536) ? EnergyForm::kThreads512 : EnergyForm::kThreads256;
}

// Rows a workgroup of the v-disparity histogram, from `group` (a load's rows) to `most`.  A group of rows is
// a load's latency and its LDS atomics, so few groups want one a workgroup; many want longer runs, whose
// counts leave as whole cache lines, the sooner the narrower the rows are; beyond 1024 columns the load takes
// longer and runs of 16 rows were the slowest.  us at 4, 8, 16 and 32 rows, u8 disparity:
//   64 x 375      64 frames 13, 12, 11, 14   256 32, 26, 24, 26   512 57, 44, 40, 41   1500 173, 130, 117, 108
//   160 x 120     64 8, 8, 9, 12             512 25, 22, 22, 22   1024 46, 36, 36, 37   2048 87, 68, 68, 65
//   320 x 96      64 8, 9, 11, 16            256 18, 16, 16, 19   1024 50, 43, 39, 42   2048 93, 76, 68, 69
//   641 x 240     64 17, 18, 19, 25          256 44, 42, 43, 51   512 80, 72, 72, 87    2048 289, 256, 244, 300
//   1242 x 375    1 8, 11, 17, 30            128 51, 50, 57, 61   512 172, 160, 188, 187   (f32, 1024 frames 470, 480, 443 at 4, 8 and 32)
//   1920 x 1080   1 10, 15, 25, 44           64 95, 95, 101, 113  256 340, 323, 326, 336
inline int hist_rows(int W, int H, int frames, int group, int most) {
    const int64_t groups = (int64_t)frames * ((H + group - 1) / group);
    int rows = 8 * group;
    if (groups <= (int64_t)9 * W) rows = group;
    else if (groups <= (W < 1024 ? (int64_t)36 * W : 72 * 1024)) rows = 2 * group;
    else if (W < 1024 && (W >= 256 || groups <= 48 * 1024)) rows = 4 * group;
    return std::min(rows, most);
}

// Rows a workgroup of the edges, `waves` waves wide.  Its time is a chain of rows and of the disparities
// gathered for them, and each strip loads two rows more than it takes, so the line is one on rows times
// waves.  us at 2, 4, 8 and 32 rows:
//   1242 x 375 (5 waves)    1 frame 7, 9, 12, 27   16 17, 14, 15, 31   128 79, 61, 49, 58   256 153, 114, 87, 90   1024 590, 426, 312, 285
//   320 x 96 (2)            64 10, 10, 12, 23      256 22, 18, 16, 27  1024 64, 48, 42, 39
//   641 x 240 (3)           64 18, 16, 16, 27      512 100, 75, 61, 78 1024 190, 139, 109, 135
//   1920 x 1080 (8)         4 16, 14, 13, 25       32 83, 61, 47, 53   64 158, 114, 82, 80
//   4000 x 400 (16)         4 16, 15, 13, 30       16 44, 37, 29, 31   32 81, 65, 52, 54    64 163, 126, 94, 81   128 317, 241, 180, 143
inline int edge_rows(int H, int waves, int frames) {
    const int64_t all = (int64_t)frames * H * waves;
    return all <= 10 * 1024 ? 2 : all <= 40 * 1024 ? 4 : all <= 300 * 1024 ? 8 : 32;
}

// Threads a frame of the V_px RANSAC: eight waves while every frame has a CU to itself, else three, so that a
// CU's frames share it evenly.  us with 192 and 512 threads: 1242 x 375, one frame 29, 27; 256 frames 78, 68; 320
// 89, 93; 512 89, 108; 1280 x 720, 256 frames 127, 105; 384 131, 133; 320 x 96, 1 to 256 frames 18, 19; 384 20, 33.
inline int ransac_threads(int frames) { return frames <= kCUs ? 512 : 192; }

// LDS of a stereo strip of E columns and T rows
inline size_t stereo_strip_lds(int rho, int E, int T, int d_max) {
    const size_t rows = (size_t)T + 2 * rho, own = (size_t)(E + 2 * rho + 3 + 8) / 4;
    const size_t other = (size_t)(E + 255 + 2 * rho + 3 + 8) / 4, wb = (size_t)E + d_max, cols = E + wb + 4 * rho;
    return 4 * rows * (own + other) + (size_t)T * (wb + E) * 12 + 2 * cols * 8 + 2 * 4 * (size_t)(E + 2) + 64;
}

// The form that a launch of the stereo maps takes: strips of eight or four lanes a pixel, of 16 or 8
// rows, or one workgroup that sweeps a pair (kSweep).
//
// The sweep's time hardly depends on the number of pairs up to one a CU; the strips spread a pair over
// the chip but work on their halo again.  Eight lanes a pixel have the shortest row and the most
// halo (30 of 64 columns), so they are taken while all workgroups of a row block run at once, four
// after that, and blocks of eight rows (two or three workgroups fit a CU, less halo) from there on, until
// their work passes the sweep's.  ms for 1, 8, 16, 32, 96 and 128 pairs of 1242 x 375:
//   8 lanes, 64 columns, 16 rows    0.68  1.35  2.08
//   4 lanes, 128 columns, 16 rows   0.84  0.86  1.63  3.10
//   4 lanes, 128 columns, 8 rows    0.91  0.95  1.23  1.58  3.92  4.89
//   a pair a workgroup              4.64  4.68  4.74  4.80  4.82  4.83
// Where the last two meet is a matter of the width: a launch of the strips costs by its workgroups (0.55
// us each for a round of 15 launches), a sweep by its columns and by the rounds of 256 pairs
// (ms for 120 rows, 8-row strips and sweep: 64 wide, 512 pairs 0.52, 0.87; 160 wide, 160 and 256 pairs
// 0.41, 0.46 and 0.55, 0.46; 320 wide, 128 and 192 pairs 0.42, 0.56 and 0.64, 0.56; 640 wide, 96 and
// 160 pairs 0.64, 0.76 and 0.96, 0.77; 960 wide, 96 and 160 pairs 1.04, 1.28 and 1.62, 1.30; 1920
// wide, 96 and 160 pairs 1.80, 2.45 and 2.96, 2.47), so the limit is one on workgroups that grows with
// the width, three quarters of it without a propagation bound, where the sweep has fewer candidates a
// pixel to wait for (96 pairs of 1242 columns: 1.07, 0.92).
enum class StereoForm { kStrip8, kStrip4, kStrip4Short, kSweep };

inline StereoForm stereo_form(int W, int H, int rho, int d_max, int tau, int64_t pairs) {
    if (W <= 2 * rho || W < 4 || H <= 2 * rho) return StereoForm::kSweep;   // (no block, or no word a row)
    auto fits = [&](int E, int T, int64_t most) {
        const int use = E - 2 * (T - 1);
        return stereo_strip_lds(rho, E, T, d_max) <= (size_t)kMaxLds &&
               (int64_t)((W + use - 1) / use) * 2 * pairs <= most;
    };
    if (fits(64, 16, kCUs)) return StereoForm::kStrip8;
    if (fits(128, 16, kCUs)) return StereoForm::kStrip4;
    const int64_t most = std::max(960, 2 * W) * ((pairs + kCUs - 1) / kCUs);
    if (fits(128, 8, tau == 0 ? most * 3 / 4 : most)) return StereoForm::kStrip4Short;
    return StereoForm::kSweep;
}
