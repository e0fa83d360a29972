// ld.hip -- MI355X (gfx950) kernels and C ABI of the lane-detection hot path.
//
// Method: Fan & Dahnoun, "Real-Time Stereo Vision-Based Lane Detection System"
// (arXiv 1807.02752), Sec. 2.2-2.4.  One launch of each kernel processes a whole batch of
// frames; per-pixel steps are spread over many workgroups per frame, the serial steps
// (dynamic programming, RANSAC, row sweeps) run one workgroup per frame out of LDS.
//
//   k_vdisp_hist   S1   v-disparity histogram (LDS bins, wave-aggregated atomics)
//   k_vdisp_fit    S2-3 DP on the v-disparity map, RANSAC road profile, V_py, road rows
//   k_edges        S4-5 Sobel on road rows, road mask, V_px vote column per edge
//   k_vpx_fit      S6-7 sliding band accumulator, row DP
//   k_vpx_ransac   S8   RANSAC V_px, track tables
//   k_energy       S9-12 w_g, M_0, M_1 row ring, candidate-by-row energy accumulation; for few
//                  frames in two launches over the whole chip:
//   k_m1           S9-11 w_g, M_0, M_1 in tiles, k_tracks S12 a candidate a lane
//   k_peaks        S13  minima, threshold, suppression, lane curves
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <algorithm>
#include <cstring>
#include <new>
#include <mutex>
#include <vector>
#include <type_traits>

#include "ld_device.h"
#include "ld_internal.h"

using namespace ldk;

namespace {

struct FitRes {
    int32_t ok, flags, center, kshift, rounds, n_surv;
    double coef[5];
    double raw[5];
};
static_assert(sizeof(FitRes) == sizeof(ld_fit), "FitRes must mirror ld_fit");

struct FrameInfo {
    int32_t flags, v_h, v_end, n_my, n_edges, n_votes, R, n_mx;
};

constexpr int kMaxRounds = 64;
constexpr int kBig = 0x3FFFFFFF;

// Device view of a frame object: sizes, parameters and the scratch carried between steps.
struct Dev {
    int W, H, D1, W2, half, fmt, d_max, B;
    int hist_rows;      // rows binned by one histogram workgroup, at most
    int Hm;             // row stride of myT: H rounded up to 32, so a histogram workgroup's rows
                        // of one disparity fill whole 128-byte lines
    ld_params P;
    int32_t* myT;       // B x D1 x Hm  v-disparity counts, transposed (m_y(d, .) contiguous)
    uint8_t* back_y;    // B x D1 x H   v-disparity DP backtrace (tau)
    int32_t* my_pts;    // B x 2 x D1   DP path points with votes: rows, then disparities
    FitRes* fit;        // B x 2        beta, gamma
    FrameInfo* info;    // B
    double* tab;        // B x 6 x H    f, f', V_py, V_px, A_v, B_v
    int32_t* rowcnt;    // B x H        road edges per row
    ld_edge* edges;     // B x H x W    per-row edge buckets
    int8_t* back_x;     // B x H x ceil(2W/8) x 4 B   backtrace of the windowed search (k_vpx_window), 4-bit tie ranks
    int32_t* mxpath;    // B x H        row-DP path columns
    double* energy;     // B x 2W
    int32_t* trace;     // B x 2 x 3 x kMaxRounds
    float* qbuf;        // B x H x W    in turn: the row DP's backtrace, two words for every ten columns of 2W at
                        // the start of a row's W words (k_vpx_fit; read to its end there); then, from the
                        // edges, G_x w_g of every road edge in bucket order (k_energy) or M_1 (k_m1)
    uint32_t* rbound;   // B x H x 2    raw disparity interval of the road test per row
    uint8_t* lbits;     // B x 4 x 16 x W   network decisions on the bands (pruned search)
    int32_t* prune;     // B x 16       pruned-search state (LD_STATE_PRUNE layout)
    uint8_t* cmask;     // B x 2W       candidate mask of the pruned search
    double* seedg;      // B x 5        RANSAC hypothesis 0 of the pruned search (raw basis)
    const int32_t* nact;   // nullable device count: frames b >= *nact of a launch are skipped
    // nullable: run only the frames whose fallback bits prune[b][1] & only_bits are
    // non-zero (only_set = 1) or zero (only_set = 0)
    const int32_t* only;
    int only_bits, only_set;
};

constexpr int kPruneWords = 16;
constexpr int kFbPlainVpx = 1, kFbPlainEnergy = 2, kFbNoSeed = 4, kFbTouch = 8;

__device__ __forceinline__ bool frame_masked(const Dev& d, int b) {
    if (d.nact != nullptr && b >= *d.nact) return true;
    if (d.only != nullptr && (((d.only[b * kPruneWords + 1] & d.only_bits) != 0) != (d.only_set != 0))) return true;
    return false;
}

// ------------------------------------------------------------------------------------------
// Block-wide helpers (any multiple of 64 threads up to 1024)
__device__ __forceinline__ int nwaves() { return blockDim.x / kWave; }

__device__ __forceinline__ int block_max_i32(int x, int* red) {
    x = wave_max_i32(x);
    int w = threadIdx.x / kWave;
    __syncthreads();
    if (lane_id() == 0) red[w] = x;
    __syncthreads();
    int r = red[0];
    for (int i = 1; i < nwaves(); ++i) r = max(r, red[i]);
    return r;
}

__device__ __forceinline__ int block_min_i32(int x, int* red) {
    x = wave_min_i32(x);
    int w = threadIdx.x / kWave;
    __syncthreads();
    if (lane_id() == 0) red[w] = x;
    __syncthreads();
    int r = red[0];
    for (int i = 1; i < nwaves(); ++i) r = min(r, red[i]);
    return r;
}

__device__ __forceinline__ int block_sum_i32(int x, int* red) {
    x = wave_sum_i32(x);
    int w = threadIdx.x / kWave;
    __syncthreads();
    if (lane_id() == 0) red[w] = x;
    __syncthreads();
    int r = 0;
    for (int i = 0; i < nwaves(); ++i) r += red[i];
    return r;
}

// (value, index) argmin over the block, ties to the smaller index
__device__ __forceinline__ void block_argmin_i64(int64_t& v, int& i, int64_t* rv, int* ri) {
    wave_argmin_i64(v, i);
    int w = threadIdx.x / kWave;
    __syncthreads();
    if (lane_id() == 0) { rv[w] = v; ri[w] = i; }
    __syncthreads();
    v = rv[0];
    i = ri[0];
    for (int k = 1; k < nwaves(); ++k)
        if (rv[k] < v || (rv[k] == v && ri[k] < i)) { v = rv[k]; i = ri[k]; }
}

// ------------------------------------------------------------------------------------------
// RANSAC (Alg. "beta/gamma estimation with the assist of RANSAC").  Each round scores up to
// 64 random samples of DEG+1 points, one per lane of wave 0, and the points are split over
// the waves of the workgroup for the inlier count; the best sample's outliers are removed by a
// stable ballot compaction; the loop ends when the inliers reach eps of the round's points.
// The final model is refitted on the survivors from exact 128-bit moments.
//
// A round is a chain of one wave's latency (samples and fits) and of FP64 issue (the counts:
// 64 samples x the points x 16 operations).  So the random words of the next round, which depend
// on no result, are formed by other waves beside this round's fits; the points move with the
// compaction, so a count reads them four at a time with no index between; the best sample is
// found by every wave for itself; and a fit sums in int64 whatever fits there.  A round of a
// 1242 x 375 frame's V_px took 13.5 us (words 2.4, fit 2.5, counts 7.5 over three waves) and takes
// 6.2 (words and draw 0.9, fit 1.8, counts 2.0 over eight); k_vpx_ransac 87 -> 44 us.
struct RansacShared {
    double models[kMaxHyp][5];
    int mvalid[kMaxHyp];            // 0 invalid, 1 fitted (s basis), 2 caller seed (raw basis)
    int counts[kMaxWaves][kMaxHyp];
    uint64_t words[2][8][kMaxHyp];  // random words of this round and the next
    int wsum[2][kMaxWaves];
    int red[kMaxWaves];
    i128 mred[kMaxWaves][14];
    double mom[14];
};

// Model values are Horner sums in (x - off) * scale: the s basis, or x itself for a caller seed.
template <int DEG>
__device__ __forceinline__ bool is_inlier(const double* m, int off, double scale, int x, int y, double tr) {
    const double a = (double)(x - off) * scale;
    double f = m[DEG];
#pragma unroll
    for (int p = DEG - 1; p >= 0; --p) f = f * a + m[p];
    const double res = (double)y - f;
    return res * res < tr;
}

// maximum over the wave, in every lane
__device__ __forceinline__ int wave_max_dpp(int x) {
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0xB1, 0xF, 0xF, false));     // quad_perm 1 0 3 2
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x4E, 0xF, 0xF, false));     // quad_perm 2 3 0 1
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x141, 0xF, 0xF, false));    // row_half_mirror
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x140, 0xF, 0xF, false));    // row_mirror: rows of 16 done
    return max(max(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
               max(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}

// X, Y: the points (16-byte aligned, lengths rounded up to 4, as X2 and Y2, which take the
// survivors in turn); both pairs are overwritten.
template <int DEG>
__device__ void ransac_block(int* X, int* Y, int n0, int* X2, int* Y2, uint32_t* bitmap, int bitmap_words,
                             RansacShared& S, double tr, const ld_params& P, uint64_t key1, uint64_t ctr0, int stage,
                             const double* seed_raw, FitRes* out, int* trace) {
    constexpr int s = DEG + 1, kBlocks = (s + 3) / 4, NM = Moments<DEG>::kCount;
    const int t = threadIdx.x, lane = lane_id(), wave = t / kWave, nw = nwaves(), nt = blockDim.x;
    FitRes res;
    res.ok = 0; res.flags = 0; res.center = 0; res.kshift = 0; res.rounds = 0; res.n_surv = 0;
    for (int p = 0; p < 5; ++p) { res.coef[p] = 0.0; res.raw[p] = 0.0; }
    if (n0 < s) {
        if (t == 0) { res.flags = 1; *out = res; }
        __syncthreads();
        return;
    }
    const int n_hyp = min(P.n_hyp, kMaxHyp);
    auto philox = [&](int r, int blk) {
        return philox4x64_10(ctr0, ((uint64_t)stage << 32) | (uint64_t)(uint32_t)r, (uint64_t)lane, (uint64_t)blk, P.seed,
                             key1);
    };
    // the first random words of round r, a block of four a wave
    auto draw = [&](int r) {
        for (int blk = 0; blk < kBlocks; ++blk)
            if (wave == (1 + blk) % nw) {
                const U64x4 w = philox(r, blk);
#pragma unroll
                for (int q = 0; q < 4; ++q) S.words[r & 1][4 * blk + q][lane] = w.w[q];
            }
    };
    draw(0);
    int xmn = 0x7fffffff, xmx = -0x7fffffff;
    for (int j = t; j < n0; j += nt) { xmn = min(xmn, X[j]); xmx = max(xmx, X[j]); }
    xmn = block_min_i32(xmn, S.red);
    xmx = block_max_i32(xmx, S.red);
    const int center = (xmn + xmx) >> 1;
    const int wmax = max(xmx - center, center - xmn);
    int k = 0;
    while ((1 << k) < wmax) ++k;
    res.center = center;
    res.kshift = k;
    const double scale = ldexp(1.0, -k);
    const int need = max(s, (n0 + 9) / 10);
    int n_cur = n0;
    bool converged = false;
    int r = 0;
    for (; r < P.max_rounds; ++r) {
        // ---- phase A: one sample + fit per hypothesis (wave 0)
        if (t < n_hyp) {
            double model[5] = {0, 0, 0, 0, 0};
            int kind = 0;
            if (t == 0 && seed_raw != nullptr && !isnan(seed_raw[0])) {   // a NaN seed means none
                for (int p = 0; p <= DEG; ++p) model[p] = seed_raw[p];
                kind = 2;
            } else {
                // draw indices until s distinct ones; the picks stay in registers (every
                // array index below is static after unrolling)
                int pick[s];
#pragma unroll
                for (int e = 0; e < s; ++e) pick[e] = -1;
                int got = 0;
                auto next = [&](uint64_t w) {
                    const int ix = (int)__umul64hi(w, (uint64_t)n_cur);
                    bool dup = false;
#pragma unroll
                    for (int e = 0; e < s; ++e) dup = dup || (e < got && pick[e] == ix);
                    const bool take = got < s && !dup;
#pragma unroll
                    for (int e = 0; e < s; ++e) pick[e] = (take && e == got) ? ix : pick[e];
                    got += take ? 1 : 0;
                };
#pragma unroll
                for (int q = 0; q < s; ++q) next(S.words[r & 1][q][lane]);
                if (got < s) {
                    for (int q = s; q < 4 * kBlocks; ++q) next(S.words[r & 1][q][lane]);
                    for (int blk = kBlocks; blk < 16 && got < s; ++blk) {
                        const U64x4 w = philox(r, blk);
#pragma unroll
                        for (int q = 0; q < 4; ++q) next(w.w[q]);
                    }
                }
                if (got == s) {
                    int px[s], py[s];
#pragma unroll
                    for (int e = 0; e < s; ++e) { px[e] = X[pick[e]]; py[e] = Y[pick[e]]; }
                    bool distinct = true;
#pragma unroll
                    for (int e = 1; e < s; ++e)
#pragma unroll
                        for (int f = 0; f < e; ++f) distinct = distinct && (px[f] != px[e]);
                    if (distinct) {
                        Moments<DEG> M;
                        moments_zero<DEG>(M);
#pragma unroll
                        for (int e = 0; e < s; ++e) moments_add<DEG>(M, px[e], py[e], center);
                        double mom[NM];
#pragma unroll
                        for (int i = 0; i < NM; ++i) mom[i] = moment_f64<DEG>(M, i);
                        kind = solve_moments<DEG>(mom, k, model) ? 1 : 0;
                    }
                }
            }
            for (int p = 0; p < 5; ++p) S.models[t][p] = model[p];
            S.mvalid[t] = kind;
        }
        if (r + 1 < P.max_rounds) draw(r + 1);
        __syncthreads();
        // ---- phase B: inlier counts, hypothesis = lane, points split over the waves by fours
        {
            int cnt = -1;
            if (lane < n_hyp && S.mvalid[lane] != 0) {
                double m[DEG + 1];
#pragma unroll
                for (int p = 0; p <= DEG; ++p) m[p] = S.models[lane][p];
                const bool raw = S.mvalid[lane] == 2;
                const int off = raw ? 0 : center;
                const double sc = raw ? 1.0 : scale;
                cnt = 0;
#pragma unroll 2
                for (int j = 4 * wave; j < n_cur; j += 4 * nw) {
                    const int4 x = *reinterpret_cast<const int4*>(X + j), y = *reinterpret_cast<const int4*>(Y + j);
                    const bool i0 = is_inlier<DEG>(m, off, sc, x.x, y.x, tr), i1 = is_inlier<DEG>(m, off, sc, x.y, y.y, tr);
                    const bool i2 = is_inlier<DEG>(m, off, sc, x.z, y.z, tr), i3 = is_inlier<DEG>(m, off, sc, x.w, y.w, tr);
                    cnt += (i0 ? 1 : 0) + ((i1 & (j + 1 < n_cur)) ? 1 : 0) + ((i2 & (j + 2 < n_cur)) ? 1 : 0) +
                           ((i3 & (j + 3 < n_cur)) ? 1 : 0);
                }
            }
            S.counts[wave][lane] = cnt;
        }
        __syncthreads();
        // ---- phase C: best hypothesis (most inliers, lowest index), each wave for itself
        int tot = -1;
        if (S.counts[0][lane] >= 0) {
            tot = 0;
            for (int w = 0; w < nw; ++w) tot += S.counts[w][lane];
        }
        const int key = wave_max_dpp(tot < 0 ? -1 : tot * kMaxHyp + (kMaxHyp - 1 - lane));
        const int best_h = key < 0 ? -1 : kMaxHyp - 1 - key % kMaxHyp, best_n = key < 0 ? -1 : key / kMaxHyp;
        if (trace && t == 0) { trace[3 * r] = best_h; trace[3 * r + 1] = best_n; trace[3 * r + 2] = n_cur; }
        if (best_h < 0 || best_n < need) { ++r; break; }
        // ---- phase D: keep the inliers of the best sample, in order
        {
            double m[DEG + 1];
#pragma unroll
            for (int p = 0; p <= DEG; ++p) m[p] = S.models[best_h][p];
            const bool raw = S.mvalid[best_h] == 2;
            const int off = raw ? 0 : center;
            const double sc = raw ? 1.0 : scale;
            int base = 0;
            for (int c0 = 0, par = 0; c0 < n_cur; c0 += nt, par ^= 1) {
                const int j = c0 + t;
                int x = 0, y = 0;
                bool pred = false;
                if (j < n_cur) {
                    x = X[j];
                    y = Y[j];
                    pred = is_inlier<DEG>(m, off, sc, x, y, tr);
                }
                const uint64_t bal = __ballot(pred);
                if (lane == 0) S.wsum[par][wave] = __popcll(bal);
                __syncthreads();
                int o = base + __popcll(bal & lanes_below());
                for (int w = 0; w < nw; ++w) {
                    const int c = S.wsum[par][w];
                    o += w < wave ? c : 0;
                    base += c;
                }
                if (pred) { X2[o] = x; Y2[o] = y; }
            }
        }
        const bool done = (int64_t)P.eps_den * best_n >= (int64_t)P.eps_num * n_cur;
        int* tmp = X; X = X2; X2 = tmp;
        tmp = Y; Y = Y2; Y2 = tmp;
        n_cur = best_n;
        __syncthreads();
        if (done) { converged = true; ++r; break; }
    }
    res.rounds = r;
    res.flags = converged ? 0 : 1;
    res.n_surv = n_cur;
    // ---- final fit on the survivors: distinct abscissae, exact moments, solve
    for (int i = t; i < bitmap_words; i += nt) bitmap[i] = 0u;
    __syncthreads();
    Moments<DEG> M;
    moments_zero<DEG>(M);
    for (int j = t; j < n_cur; j += nt) {                   // (at most 4096 points over 192 threads)
        const int x = X[j];
        atomicOr(&bitmap[x >> 5], 1u << (x & 31));
        moments_add<DEG>(M, x, Y[j], center);
    }
    i128 v[DEG == 2 ? 8 : 16];
    static_assert(NM == 8 || NM == 14, "moments");
#pragma unroll
    for (int i = 0; i < NM; ++i) v[i] = moment_i128<DEG>(M, i);
    if constexpr (NM == 14) v[14] = v[15] = 0;
    const i128 mine = wave_sums_i128(v);
    if (lane < NM) S.mred[wave][lane] = mine;
    __syncthreads();
    int pc = 0;
    for (int i = t; i < bitmap_words; i += nt) pc += __popc(bitmap[i]);
    if (t < NM) {
        i128 sum = S.mred[0][t];
        for (int w = 1; w < nw; ++w) sum += S.mred[w][t];
        S.mom[t] = i128_to_f64(sum);
    }
    const int distinct = block_sum_i32(pc, S.red);          // (its barriers order S.mom too)
    if (t == 0) {
        if (distinct >= s) {
            double mom[NM];
#pragma unroll
            for (int i = 0; i < NM; ++i) mom[i] = S.mom[i];
            if (solve_moments<DEG>(mom, k, res.coef)) {
                res.ok = 1;
                to_raw<DEG>(res.coef, center, k, res.raw);
            }
        }
        *out = res;
    }
    __syncthreads();
}

// ------------------------------------------------------------------------------------------
// S1: v-disparity histogram m_y(d, v) (Sec. 2.2).  A workgroup bins hist_rows rows of one
// frame into LDS; within a wave, the lanes that share the first active lane's bin are merged
// by ballot into one LDS atomic and the other lanes add directly (a road row puts most
// pixels into one or two bins, so one merge removes most of the same-address traffic; merging
// two or three bins this way measured slower).  Rows
// are taken four at a time, and the raw values of the next four rows are loaded while the
// current four are binned, so a wave always has a group of loads in flight.  The counts
// leave transposed, hist_rows consecutive rows per disparity.
constexpr int kHistGroup = 4;
constexpr int kHistMerge = 1;

template <int FMT> struct RawPixel { using T = uint8_t; };
template <> struct RawPixel<LD_DISP_F32> { using T = float; };
template <> struct RawPixel<LD_DISP_U16Q4> { using T = uint16_t; };

// Bin of one raw disparity value; false for the invalid ones (0 in the integer formats,
// non-positive or non-finite in F32), so a load masked to 0 is never counted.
template <int FMT>
__device__ __forceinline__ bool disp_bin(typename RawPixel<FMT>::T x, int d_max, int& bin) {
    if (FMT == LD_DISP_U8) {
        bin = min((int)x, d_max);
        return x != 0;
    } else if (FMT == LD_DISP_F32) {
        if (!(isfinite((float)x) && (float)x > 0.0f)) return false;
        double b = floor((double)x + 0.5);
        bin = b > (double)d_max ? d_max : (int)b;
        return true;
    } else {
        bin = min(((int)x + 8) >> 4, d_max);
        return x != 0;
    }
}

template <int FMT, int NPT>
__device__ __forceinline__ void hist_load(const typename RawPixel<FMT>::T* base, int64_t pitch_px, int W, int t,
                                          int g, int rows, typename RawPixel<FMT>::T (&dst)[kHistGroup][NPT]) {
#pragma unroll
    for (int r = 0; r < kHistGroup; ++r) {
        const typename RawPixel<FMT>::T* row = base + (int64_t)min(g + r, rows - 1) * pitch_px;
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int u = t + k * kBlock;
            dst[r][k] = (g + r < rows && u < W) ? row[u] : typename RawPixel<FMT>::T(0);
        }
    }
}

template <int FMT, int NPT>
__global__ __launch_bounds__(kBlock) void k_vdisp_hist(Dev d, const uint8_t* disp, int64_t pitch, int32_t* vdisp_out) {
    using Raw = typename RawPixel<FMT>::T;
    extern __shared__ int hist[];   // hist_rows x D1
    const int hr = d.hist_rows;
    const int b = blockIdx.y, v0 = blockIdx.x * hr, t = threadIdx.x, lane = lane_id();
    if (frame_masked(d, b)) return;
    const int D1 = d.D1, W = d.W, H = d.H;
    const int rows = min(hr, H - v0);
    const Raw* base = reinterpret_cast<const Raw*>(disp + ((int64_t)b * H + v0) * pitch);
    const int64_t pitch_px = pitch / (int64_t)sizeof(Raw);
    Raw nxt[kHistGroup][NPT];
    hist_load<FMT, NPT>(base, pitch_px, W, t, 0, rows, nxt);
    for (int i = t; i < hr * D1; i += kBlock) hist[i] = 0;
    __syncthreads();
    for (int g = 0; g < rows; g += kHistGroup) {
        int bins[kHistGroup][NPT];
        bool ok[kHistGroup][NPT];
#pragma unroll
        for (int r = 0; r < kHistGroup; ++r)
#pragma unroll
            for (int k = 0; k < NPT; ++k) {
                bins[r][k] = 0;
                ok[r][k] = disp_bin<FMT>(nxt[r][k], d.d_max, bins[r][k]);
            }
        if (g + kHistGroup < rows) hist_load<FMT, NPT>(base, pitch_px, W, t, g + kHistGroup, rows, nxt);
#pragma unroll
        for (int r = 0; r < kHistGroup; ++r) {
#pragma unroll
            for (int k = 0; k < NPT; ++k) {
                bool pend = ok[r][k];
                const int bin = bins[r][k];
                int* hrow = hist + (g + r) * D1;
                uint64_t act = __ballot(pend);
                // up to kHistMerge distinct bins of the wave are merged, each into one atomic
                // by its first lane; the lanes left over (many distinct bins) add one each
#pragma unroll
                for (int it = 0; it < kHistMerge; ++it) {
                    if (act == 0) break;
                    const int leader = __ffsll((unsigned long long)act) - 1;
                    const int b0 = __builtin_amdgcn_readlane(bin, leader);   // uniform: no LDS round trip
                    const bool same = pend && bin == b0;
                    const uint64_t m = __ballot(same);
                    if (lane == leader) atomicAdd(&hrow[b0], __popcll(m));
                    pend = pend && !same;
                    act &= ~m;
                }
                if (act != 0 && pend) atomicAdd(&hrow[bin], 1);
            }
        }
    }
    __syncthreads();
    for (int i = t; i < rows * D1; i += kBlock) {
        const int dd = i / rows, r = i % rows;
        d.myT[((int64_t)b * D1 + dd) * d.Hm + v0 + r] = hist[r * D1 + dd];
    }
    if (vdisp_out) {
        for (int i = t; i < rows * D1; i += kBlock) {
            const int r = i / D1, dd = i % D1;
            vdisp_out[((int64_t)b * H + v0 + r) * D1 + dd] = hist[r * D1 + dd];
        }
    }
}

// ------------------------------------------------------------------------------------------
// S2 + S3: DP on the v-disparity map (Eq. vpy_estimation), RANSAC road profile beta
// (Alg. "beta estimation"), tables f, f', V_py (Eq. vpy_equation) and the road rows.  One
// workgroup per frame.

// The road test of Sec. 2.3.1, valid(raw) and |D(raw) - f| <= varpi in FP64, as an interval
// of raw pixel values.  D is non-decreasing in the raw value over the valid values (u8:
// 1..255, u16: 1..65535, f32: the bit patterns of positive finite floats) and the rounded
// difference D - f is non-decreasing in D, so the passing raw values form one interval
// [lo, hi]; both ends are found by bisection on the same FP64 predicate.  Every invalid raw
// value (0, negative, infinite or NaN floats) lies outside it.  lo > hi when it is empty.
__device__ __forceinline__ double raw_to_d(int fmt, uint32_t r) {
    if (fmt == LD_DISP_U8) return (double)r;
    if (fmt == LD_DISP_U16Q4) return (double)r / 16.0;
    return (double)__uint_as_float(r);
}

__device__ __forceinline__ uint32_t d_to_raw(int fmt, double x) {           // about; 0 for x <= 0
    x = fmin(fmax(x, 0.0), 3.0e38);
    if (fmt == LD_DISP_F32) return __float_as_uint((float)x);
    return (uint32_t)fmin(fmt == LD_DISP_U8 ? x : x * 16.0, 65535.0);
}

// The bisections start from two values either side of the rounded end f -+ varpi where the
// predicate confirms them (always but for extreme f), so they take 2 steps instead of up to 31:
// the tables of a 375-row frame took 6.4 us of k_vdisp_fit's time and take 1.9.
__device__ void road_interval(int fmt, double f, double varpi, uint32_t& lo, uint32_t& hi) {
    const uint32_t top = fmt == LD_DISP_U8 ? 255u : (fmt == LD_DISP_U16Q4 ? 65535u : 0x7F7FFFFFu);
    lo = 1u;
    hi = 0u;
    auto above = [&](uint32_t r) { return raw_to_d(fmt, r) - f >= -varpi; };
    auto below = [&](uint32_t r) { return raw_to_d(fmt, r) - f <= varpi; };
    // smallest r with D(r) - f >= -varpi
    if (!above(top)) return;
    uint32_t a = 1u, z = top;
    if (!above(a)) {
        const uint32_t g = d_to_raw(fmt, f - varpi);
        if (g > 3u && g - 2u < z && !above(g - 2u)) a = g - 2u;
        if (g < top - 2u && g + 2u > a && above(g + 2u)) z = g + 2u;
        while (z - a > 1u) {            // predicate false at a, true at z
            const uint32_t m = a + (z - a) / 2u;
            if (above(m)) z = m; else a = m;
        }
        a = z;
    }
    // largest r with D(r) - f <= varpi
    if (!below(1u)) return;
    uint32_t x = 1u, y = top;
    if (!below(y)) {
        const uint32_t g = d_to_raw(fmt, f + varpi);
        if (g > 3u && g - 2u < y && below(g - 2u)) x = g - 2u;
        if (g < top - 2u && g + 2u > x && !below(g + 2u)) y = g + 2u;
        while (y - x > 1u) {            // predicate true at x, false at y
            const uint32_t m = x + (y - x) / 2u;
            if (below(m)) x = m; else y = m;
        }
    } else {
        x = y;
    }
    lo = a;
    hi = x;
}

constexpr int kVdTau = 8;                  // largest tau of the DP in registers
constexpr int kVdSteps = 8;                // its steps a chunk: a word of 4-bit backtraces a row
constexpr int kVdRows = 4;                 // rows per thread in the DP of wider jumps
constexpr int kVdWalk = 32;                // its steps of the backtrace staged in LDS per walk chunk
constexpr int kVdWalkCols = 257;           // staged rows per step (covers kVdWalk steps of tau_max)
constexpr int kVdPadKey = 0x3FFFFFF0;      // padding key: above any real key, and twice it fits int32

// rows a lane of the DP in registers, and its waves (0 where it does not apply)
__host__ __device__ __forceinline__ int vdisp_lane_rows(int H) { return H <= 2 * kWave * kMaxWaves ? 2 : 4; }
__host__ __device__ __forceinline__ int vdisp_dp_waves(int H, int tau_max) {
    const int n = (H + kWave * vdisp_lane_rows(H) - 1) / (kWave * vdisp_lane_rows(H));
    return tau_max <= kVdTau && n <= kMaxWaves ? n : 0;
}
// words of its backtrace, and of the boundary rows that its waves hand on
__host__ __device__ __forceinline__ int vdisp_back_words(int H, int d_max) { return (d_max + kVdSteps - 1) / kVdSteps * H; }
__host__ __device__ __forceinline__ int vdisp_seam_words(int waves) { return (waves + 1) * 2 * kVdSteps * 8; }

// The DP over jumps of at most TM <= kVdTau rows.  A row needs itself and the TM rows below, so
// with R rows a lane (two, or four past 2048 rows) the window comes from the next lanes by wave
// shifts, and a wave needs
// nothing but the eight topmost rows of the wave below it, before each step: those go
// through LDS a chunk of steps at a time, and wave w works on a chunk one turn after wave w + 1 did,
// so a turn of kVdSteps steps has one barrier.  Where the waves' turns to fill and drain that would
// outlast the steps (many rows, few disparities), LOCK has all waves take the same step instead,
// with a barrier a step.  The keys are packed: the key of jump tau is
// (E(v + tau) + lambda tau) << 4 | tau; the minimum is the smallest cost, and among equal
// costs the smallest tau (the strict-< scan over tau = 0, 1, ...).  Rows past H - 1 hold the
// padding key.  The votes of the chunk after this one are loaded ahead; bw is the
// backtrace (bits 4 j of word (chunk, row): step 8 chunk + j; step i is disparity d_max - 1 - i).
// E0 receives the last row's keys.
//
// Bound: a wave's issue, about 45 instructions a step, and their chain.  A barrier and nine LDS
// reads a row a step took 0.50 us a step at 375 rows and 0.70 at 1080; this takes 0.13 and 0.25
// (the boundary rows of a step are read a step ahead).
template <int TM, int R, bool LOCK>
__device__ __forceinline__ void vdisp_dp(const int32_t* myT, int Hm, int H, int d_max, int lam, int tau_max, int nwdp,
                                         uint32_t* bw, int* seam, int* E0) {
    const int t = threadIdx.x, lane = lane_id(), wave = t / kWave, nt = blockDim.x;
    for (int i = t; i < 2 * kVdSteps * 8; i += nt) seam[nwdp * 2 * kVdSteps * 8 + i] = kVdPadKey;   // below the last wave
    const int v = (wave * kWave + lane) * R;                     // this lane's rows v .. v + R - 1
    const int vc = min(v, Hm - R);                               // (Hm is a multiple of 32)
    const int chunks = (d_max + kVdSteps - 1) / kVdSteps;
    int addc[TM + 1];
#pragma unroll
    for (int tau = 1; tau <= TM; ++tau) addc[tau] = tau <= tau_max ? 16 * lam * tau + tau : kVdPadKey;
    struct alignas(4 * R) Rows { int x[R]; };
    Rows e, nxt[kVdSteps];
    auto column = [&](int dd) __attribute__((always_inline)) {
        return *reinterpret_cast<const Rows*>(myT + (int64_t)dd * Hm + vc);
    };
    auto load = [&](int c) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < kVdSteps; ++j) nxt[j] = column(max(d_max - 1 - (c * kVdSteps + j), 0));
    };
    if (wave < nwdp) {
        e = column(d_max);
#pragma unroll
        for (int i = 0; i < R; ++i) e.x[i] = v + i < H ? -e.x[i] * 16 : kVdPadKey;
        load(0);
    }
    __syncthreads();
    // the votes and backtraces of a chunk, and a step on: old holds the wave below's rows
    Rows m[kVdSteps];
    uint32_t back[R];
    auto begin = [&](int c) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < kVdSteps; ++j)
#pragma unroll
            for (int i = 0; i < R; ++i) m[j].x[i] = v + i < H ? nxt[j].x[i] * 16 : 0;
        load(min(c + 1, chunks - 1));
#pragma unroll
        for (int i = 0; i < R; ++i) back[i] = 0;
    };
    auto advance = [&](int j, const int (&old)[8]) __attribute__((always_inline)) {
        // rows v .. v + R - 1 + TM: those past its own are the next lane's, by a shift whose last
        // lane takes the wave below's
        int w[R + TM];
#pragma unroll
        for (int i = 0; i < R; ++i) w[i] = e.x[i];
#pragma unroll
        for (int i = 0; i < TM; ++i) w[R + i] = __builtin_amdgcn_update_dpp(old[i], w[i], 0x130, 0xF, 0xF, false);
#pragma unroll
        for (int i = 0; i < R; ++i) {
            int k = w[i];
#pragma unroll
            for (int tau = 1; tau <= TM; ++tau) k = min(k, w[i + tau] + addc[tau]);
            back[i] = (back[i] >> 4) | ((uint32_t)k << 28);
            e.x[i] = (k & -16) - m[j].x[i];
        }
    };
    auto end = [&](int c, int n) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < R; ++i)
            if (v + i < H) bw[(int64_t)c * H + v + i] = back[i] >> (4 * (kVdSteps - n));
    };
    for (int turn = 0; turn < chunks + nwdp - 1 && !LOCK; ++turn) {
        const int c = turn - (nwdp - 1 - wave);
        if (wave < nwdp && c >= 0 && c < chunks) {
            begin(c);
            const int4* below = reinterpret_cast<const int4*>(seam + ((wave + 1) * 2 + (c & 1)) * kVdSteps * 8);
            Rows* mine = reinterpret_cast<Rows*>(seam + (wave * 2 + (c & 1)) * kVdSteps * 8);
            const int n = min(kVdSteps, d_max - c * kVdSteps);
            int4 pn = below[0], qn = below[1];
            auto step = [&](int j) __attribute__((always_inline)) {
                const int old[8] = {pn.x, pn.y, pn.z, pn.w, qn.x, qn.y, qn.z, qn.w};
                if (j + 1 < kVdSteps) {                          // the next step's, ahead of its use
                    pn = below[2 * j + 2];
                    qn = below[2 * j + 3];
                }
                if (lane < 8 / R) mine[8 / R * j + lane] = e;
                advance(j, old);
            };
            if (n == kVdSteps) {
#pragma unroll
                for (int j = 0; j < kVdSteps; ++j) step(j);
            } else {
#pragma unroll
                for (int j = 0; j < kVdSteps; ++j)
                    if (j < n) step(j);
            }
            end(c, n);
        }
        __syncthreads();
    }
    for (int c = 0; c < chunks && LOCK; ++c) {
        const int n = min(kVdSteps, d_max - c * kVdSteps);
        if (wave < nwdp) begin(c);
#pragma unroll
        for (int j = 0; j < kVdSteps; ++j)
            if (j < n) {                                         // (the rows by step parity)
                if (wave < nwdp && lane < 8 / R) reinterpret_cast<Rows*>(seam + (wave * 2 + (j & 1)) * kVdSteps * 8)[lane] = e;
                __syncthreads();
                if (wave < nwdp) {
                    const int4* below = reinterpret_cast<const int4*>(seam + ((wave + 1) * 2 + (j & 1)) * kVdSteps * 8);
                    const int4 p = below[0], q = below[1];
                    const int old[8] = {p.x, p.y, p.z, p.w, q.x, q.y, q.z, q.w};
                    advance(j, old);
                }
            }
        if (wave < nwdp) end(c, n);
    }
    if (wave < nwdp) {
#pragma unroll
        for (int i = 0; i < R; ++i)
            if (v + i < H) E0[v + i] = e.x[i];
    }
    __syncthreads();
}

__global__ __launch_bounds__(1024) void k_vdisp_fit(Dev d, const uint64_t* stream_ids, const int64_t* frame_idx,
                                                    double* beta_out, int back_in_lds, int lockstep) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int64_t rv[kMaxWaves];
    __shared__ int ri[kMaxWaves];
    __shared__ int s_n, s_v;
    const int b = blockIdx.x, t = threadIdx.x, nt = blockDim.x;
    if (frame_masked(d, b)) return;
    const int H = d.H, D1 = d.D1, d_max = d.d_max;
    const int D4 = (D1 + 3) / 4 * 4;
    int* PX = reinterpret_cast<int*>(smem);
    int* PY = PX + D4;
    int* cur = PY + D4;
    int* cur2 = cur + D4;
    uint32_t* bitmap = reinterpret_cast<uint32_t*>(cur2 + D4);
    const int bm_words = (H + 31) / 32;
    int* E0 = reinterpret_cast<int*>(bitmap + (bm_words + 3) / 4 * 4);
    // the RANSAC's memory, before that the DP's
    int* const region = E0 + (H + 3) / 4 * 4;
    RansacShared& S = *reinterpret_cast<RansacShared*>(region);
    const int Hm = d.Hm;
    const int32_t* myT = d.myT + (int64_t)b * D1 * Hm;
    const int tau_max = d.P.tau_y_max, lam = d.P.lambda_y;
    for (int v = t; v < H; v += nt) d.rowcnt[(int64_t)b * H + v] = 0;
    const int nwdp = vdisp_dp_waves(H, tau_max);
    // the row of the smallest E at disparity 0 (ties to the smaller row), every thread's
    auto first_row = [&](const int* E) {
        int64_t bv = INT64_MAX;
        int bi = 0x7fffffff;
        for (int v = t; v < H; v += nt)
            if ((int64_t)E[v] < bv) { bv = E[v]; bi = v; }
        block_argmin_i64(bv, bi, rv, ri);
        return bi;
    };
    if (nwdp > 0) {
        int* seam = region;
        uint32_t* lback = reinterpret_cast<uint32_t*>(seam + vdisp_seam_words(nwdp));
        uint32_t* gback = reinterpret_cast<uint32_t*>(d.back_y + (((int64_t)b * D1 * H + 3) & ~(int64_t)3));
        uint32_t* bw = back_in_lds ? lback : gback;
        auto dp = [&](auto lock) __attribute__((always_inline)) {
            constexpr bool L = decltype(lock)::value;
            if (vdisp_lane_rows(H) > 2) vdisp_dp<8, 4, L>(myT, Hm, H, d_max, lam, tau_max, nwdp, bw, seam, E0);
            else if (tau_max <= 6) vdisp_dp<6, 2, L>(myT, Hm, H, d_max, lam, tau_max, nwdp, bw, seam, E0);
            else vdisp_dp<8, 2, L>(myT, Hm, H, d_max, lam, tau_max, nwdp, bw, seam, E0);
        };
        if (__builtin_expect(!lockstep, 1)) dp(std::false_type{}); else dp(std::true_type{});
        const int v0 = __builtin_amdgcn_readfirstlane(first_row(E0));
        // The walk, by wave 0: disparities from 0 are the last step and down, so a chunk's words of the
        // 64 rows from the path's present one hold its next eight steps (tau <= 8), a lane a row.
        if (t < kWave) {
            int v = v0, dd = 0;
            for (int c = (d_max - 1) / kVdSteps; c >= 0; --c) {
                const int n = min(kVdSteps, d_max - c * kVdSteps), base = v;
                const int word = (int)bw[(int64_t)c * H + min(base + t, H - 1)];
                int keep = 0;
                auto step = [&](int j, int at) __attribute__((always_inline)) {
                    keep = t == at ? v : keep;
                    v += (__builtin_amdgcn_readlane(word, v - base) >> (4 * j)) & 15;
                };
                if (n == kVdSteps) {
#pragma unroll
                    for (int j = kVdSteps - 1; j >= 0; --j) step(j, kVdSteps - 1 - j);
                } else {
                    for (int j = n - 1; j >= 0; --j) step(j, n - 1 - j);
                }
                if (t < n) cur[dd + t] = keep;
                dd += n;
            }
            if (t == 0) cur[d_max] = v;
        }
        __syncthreads();
    } else {
        // jumps past 8 rows: the row before and this one in LDS, a barrier a step
        int* E1 = region;
        uint8_t* win = reinterpret_cast<uint8_t*>(E1 + H);       // kVdWalk x kVdWalkCols
        uint8_t* back = d.back_y + (int64_t)b * D1 * H;
        for (int v = t; v < H; v += nt) E0[v] = -myT[(int64_t)d_max * Hm + v];
        // the column m_y(d, .) of the next DP step is loaded while the current one is computed
        int nxt[kVdRows];
#pragma unroll
        for (int k = 0; k < kVdRows; ++k) nxt[k] = myT[(int64_t)(d_max - 1) * Hm + min(t + k * nt, H - 1)];
        __syncthreads();
        int* Ec = E0;
        int* En = E1;
        for (int dd = d_max - 1; dd >= 0; --dd) {
            int m[kVdRows];
#pragma unroll
            for (int k = 0; k < kVdRows; ++k) {
                m[k] = nxt[k];
                nxt[k] = myT[(int64_t)max(dd - 1, 0) * Hm + min(t + k * nt, H - 1)];
            }
#pragma unroll
            for (int k = 0; k < kVdRows; ++k) {
                const int v = t + k * nt;
                if (v >= H) continue;
                int best = Ec[v], bt = 0;
                for (int tau = 1; tau <= tau_max && v + tau <= H - 1; ++tau) {
                    const int c = Ec[v + tau] + lam * tau;
                    if (c < best) { best = c; bt = tau; }
                }
                En[v] = best - m[k];
                back[(int64_t)dd * H + v] = (uint8_t)bt;
            }
            __syncthreads();
            int* tmp = Ec; Ec = En; En = tmp;
        }
        const int bi = first_row(Ec);
        // backtrace: stage the rows the path can reach in the next kVdWalk steps, then one thread
        // follows it (the path moves down by at most tau_max rows per step)
        const int steps = max(1, min(kVdWalk, (kVdWalkCols - 1) / max(1, tau_max)));
        if (t == 0) s_v = bi;
        __syncthreads();
        for (int d0 = 0; d0 <= d_max; d0 += steps) {
            const int v0 = s_v;
            const int nst = min(steps, d_max - d0);               // steps with a backtrace entry
            const int ncols = min(H - v0, tau_max * steps + 1);
            for (int i = t; i < nst * ncols; i += nt) {
                const int r = i / ncols, c = i % ncols;
                win[r * kVdWalkCols + c] = back[(int64_t)(d0 + r) * H + v0 + c];
            }
            __syncthreads();
            if (t == 0) {
                int v = v0;
                const int last = min(d0 + steps - 1, d_max);
                for (int dd = d0; dd <= last; ++dd) {
                    cur[dd] = v;                                    // row of disparity dd on the path
                    if (dd < d_max) v += win[(dd - d0) * kVdWalkCols + (v - v0)];
                }
                s_v = v;
            }
            __syncthreads();
        }
    }
    // keep the path points that carry votes, in order of disparity (stable ballot compaction)
    {
        const int lane = lane_id(), wave = t / kWave, nw = nwaves();
        int base = 0;
        for (int c0 = 0; c0 <= d_max; c0 += nt) {
            const int dd = c0 + t;
            const bool pred = dd <= d_max && myT[(int64_t)dd * Hm + cur[dd]] > 0;
            const uint64_t bal = __ballot(pred);
            if (lane == 0) S.wsum[0][wave] = __popcll(bal);
            __syncthreads();
            int off = base, tot = 0;
            for (int w = 0; w < nw; ++w) {
                if (w < wave) off += S.wsum[0][w];
                tot += S.wsum[0][w];
            }
            if (pred) {
                const int o = off + __popcll(bal & lanes_below());
                PX[o] = cur[dd];
                PY[o] = dd;
            }
            base += tot;
            __syncthreads();
        }
        if (t == 0) s_n = base;
        __syncthreads();
    }
    const int n_my = s_n;
    for (int i = t; i < n_my; i += nt) {
        d.my_pts[(int64_t)b * 2 * D1 + i] = PX[i];
        d.my_pts[(int64_t)b * 2 * D1 + D1 + i] = PY[i];
    }
    const uint64_t sid = stream_ids ? stream_ids[b] : 0ull;
    const uint64_t fid = frame_idx ? (uint64_t)frame_idx[b] : (uint64_t)b;
    FitRes* fit = d.fit + 2 * b;
    ransac_block<2>(PX, PY, n_my, cur, cur2, bitmap, bm_words, S, d.P.tr_y, d.P, sid, fid, 0, nullptr, fit,
                    d.trace + (int64_t)b * 6 * kMaxRounds);
    // tables and road rows
    const FitRes& beta = *fit;
    const int ok = beta.ok;
    double* tf = d.tab + (int64_t)b * 6 * H;
    double* tfp = tf + H;
    double* tvpy = tf + 2 * H;
    double* tvpx = tf + 3 * H;
    const double nan = __longlong_as_double(0x7ff8000000000000LL);
    int bad = -1;
    if (ok) {
        const double sc = ldexp(1.0, -beta.kshift);
        for (int v = t; v < H; v += nt) {
            double s = (double)(v - beta.center) * sc;
            double fv = beta.coef[2];
            fv = fv * s + beta.coef[1];
            fv = fv * s + beta.coef[0];
            double tt = 2.0 * beta.coef[2];
            double dv = (beta.coef[1] + tt * s) * sc;
            tf[v] = fv;
            tfp[v] = dv;
            tvpy[v] = (double)v - fv / dv;
            tvpx[v] = nan;
            if (!(fv > 0.0 && dv > 0.0)) bad = max(bad, v);
            uint32_t lo, hi;
            road_interval(d.fmt, fv, d.P.varpi, lo, hi);
            d.rbound[((int64_t)b * H + v) * 2] = lo;
            d.rbound[((int64_t)b * H + v) * 2 + 1] = hi;
        }
    } else {
        for (int v = t; v < H; v += nt) { tf[v] = nan; tfp[v] = nan; tvpy[v] = nan; tvpx[v] = nan; }
    }
    bad = block_max_i32(bad, S.red);
    if (t == 0) {
        FrameInfo fi;
        fi.flags = (beta.flags & 1) ? LD_FLAG_NOCONS_Y : 0;
        fi.v_h = ok ? bad + 1 : H;
        fi.R = H - fi.v_h;
        if (!ok || fi.R < 8) fi.flags |= LD_FLAG_NOROAD;
        fi.v_end = H;
        fi.n_my = n_my;
        fi.n_edges = 0;
        fi.n_votes = 0;
        fi.n_mx = 0;
        d.info[b] = fi;
        if (beta_out) {
            for (int p = 0; p < 3; ++p) beta_out[3 * b + p] = ok ? beta.raw[p] : nan;
        }
    }
}

// ------------------------------------------------------------------------------------------
// S4 + S5: Sobel gradient on the road rows, edge test, road mask (Sec. 2.3.1) and the V_px
// vote of every road edge (Eq. sparse_vpx_estimation with the gradient read as the edge
// slope).
//
// A workgroup takes up to kEdgeStrip rows of one frame across its whole width: wave w owns the 256
// columns from 256 w, four consecutive columns per lane, and walks the rows down.  A row is
// loaded as one aligned dword per lane (plus the dwords left and right of the wave's span for
// its first and last lane); the six bytes a lane needs (columns ub-1 .. ub+4) come from its own
// dword and its neighbours' by DPP lane shifts.  The loads go through a buffer resource bounded
// by the frame's rows, so a dword outside the frame reads as 0 and is never fetched (those
// bytes feed no result: the gradient is only taken at 1 <= u <= W-2, 1 <= v <= H-2).  Rows go
// in groups of three, the loads of the next group issued before the current one is worked on.
// Only the grey image is streamed: the edge test needs no disparity.  The edge pixels of a
// wave are queued in LDS and, in batches of 64, each lane gathers the raw disparity of one
// queued pixel, applies the road test (an integer compare against the row's raw interval),
// takes the vote column and appends the record to its row's bucket (LDS slot counters of the
// strip, so every bucket of the strip, and its count, is written by this workgroup alone and
// nothing carries over from an earlier call).
template <int N> using IntC = std::integral_constant<int, N>;

constexpr int kEdgeStrip = 32;                        // rows per workgroup (edge_rows), at most
constexpr int kEdgeCols = 4 * kWave;                  // columns per wave
constexpr int kEdgeQueue = 512;                       // queued edge pixels per wave
constexpr int kEdgeFlushAt = kEdgeQueue - kEdgeCols;  // a row queues at most kEdgeCols
static_assert(sizeof(ld_edge) == 8, "an edge record is written as one 8-byte store");

template <int FMT>
__device__ __forceinline__ uint32_t disp_raw(const uint8_t* row, int u) {
    if (FMT == LD_DISP_U8) return row[u];
    if (FMT == LD_DISP_F32) return reinterpret_cast<const uint32_t*>(row)[u];
    return reinterpret_cast<const uint16_t*>(row)[u];
}

// Vote column of an edge: floor(x + 0.5) with x = u + (tt * gy) / gx in IEEE FP64, each
// operation rounded as written.  The quotient is first taken as p * (1/gx) with the
// reciprocal refined by two Newton steps and one residual correction, which is within an ulp
// or two of the rounded quotient; the floor of x + 0.5 can differ from the exact one only
// when x + 0.5 lies within a few ulps of an integer, and there (and for non-finite values)
// the rounded division is taken.  Returns the bin or -1 when the column is outside
// [-half, W2 - half).
__device__ __forceinline__ int vote_bin(double tt, int gy, int gx, int u, int half, int W2) {
    const double p = tt * (double)gy;
    const double g = (double)gx;
    double r = __builtin_amdgcn_rcp(g);
    r = fma(r, fma(-g, r, 1.0), r);
    r = fma(r, fma(-g, r, 1.0), r);
    double q = p * r;
    q = fma(fma(-g, q, p), r, q);
    double y = ((double)u + q) + 0.5;
    double bf = floor(y);
    const double fr = y - bf;
    if (!(fr >= 0x1p-30 && fr <= 1.0 - 0x1p-30)) bf = floor(((double)u + p / g) + 0.5);
    return (bf >= -(double)half && bf < (double)(W2 - half)) ? (int)bf + half : -1;
}

__device__ __forceinline__ uint32_t dpp_from_prev(uint32_t x) {   // lane l gets lane l-1's x
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x138, 0xF, 0xF, false);
}
__device__ __forceinline__ uint32_t dpp_from_next(uint32_t x) {   // lane l gets lane l+1's x
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x130, 0xF, 0xF, false);
}

template <int FMT>
__global__ __launch_bounds__(1024) void k_edges(Dev d, const uint8_t* grey, int64_t gpitch, const uint8_t* disp,
                                                int64_t dpitch, int strip) {
    extern __shared__ __attribute__((aligned(16))) unsigned char esm[];   // strip tables, then the wave queues
    const int b = blockIdx.y, s0 = blockIdx.x * strip;
    if (frame_masked(d, b)) return;
    const int W = d.W, H = d.H, t = threadIdx.x, lane = lane_id(), wave = t / kWave;
    const int rows = min(strip, H - s0);
    double* svpy = reinterpret_cast<double*>(esm);                      // V_py of the strip's rows
    uint32_t* sbnd = reinterpret_cast<uint32_t*>(svpy + kEdgeStrip);    // raw road interval per row
    int* scnt = reinterpret_cast<int*>(sbnd + 2 * kEdgeStrip);          // edges per row
    uint2* queue = reinterpret_cast<uint2*>(scnt + kEdgeStrip) + wave * kEdgeQueue;
    const FrameInfo fi = d.info[b];
    const bool road = !(fi.flags & LD_FLAG_NOROAD);
    if (t < kEdgeStrip) {
        scnt[t] = 0;
        if (road && t < rows) {
            const int64_t v = (int64_t)b * H + s0 + t;
            svpy[t] = d.tab[(int64_t)b * 6 * H + 2 * H + s0 + t];
            sbnd[2 * t] = d.rbound[2 * v];
            sbnd[2 * t + 1] = d.rbound[2 * v + 1];
        }
    }
    __syncthreads();
    const int vs = max(max(s0, road ? fi.v_h : H), 1), ve = min(s0 + rows - 1, H - 2);
    const int ub = wave * kEdgeCols + 4 * lane;
    if (vs <= ve) {
        // the frame's rows through a buffer resource: base aligned down to a dword, records up
        // to the end of the frame's last row rounded up to a dword
        const uintptr_t fbase = (uintptr_t)(grey + (int64_t)b * H * gpitch);
        const uintptr_t abase = fbase & ~(uintptr_t)3;
        const int nrec = (int)((((fbase + (uintptr_t)((int64_t)H * gpitch)) + 3) & ~(uintptr_t)3) - abase);
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(abase), 0, nrec, 0x00020000);
        // every lane issues both loads; the extra one is fetched only by the first and last
        // lane (the others give an offset past the records, which reads 0 without a fetch)
        const int xoff = lane == 0 ? -4 : (lane == kWave - 1 ? 4 : INT32_MIN);
        struct RowD { uint32_t own, ext; };
        auto load_row = [&](int v) -> RowD {
            const uintptr_t ra = fbase + (uintptr_t)((int64_t)min(max(v, 0), H - 1) * gpitch);
            const int off = (int)((ra & ~(uintptr_t)3) - abase) + ub;
            RowD r;
            r.own = __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0);
            r.ext = __builtin_amdgcn_raw_buffer_load_b32(rs, xoff == INT32_MIN ? INT32_MIN : off + xoff, 0, 0);
            return r;
        };
        // columns ub-1 .. ub+4 of row v
        auto unpack = [&](const RowD& r, int v, int* x) {
            const uint32_t sh = (uint32_t)((fbase + (uintptr_t)((int64_t)min(max(v, 0), H - 1) * gpitch)) & 3);
            uint32_t dp = dpp_from_prev(r.own), dn = dpp_from_next(r.own);
            if (lane == 0) dp = r.ext;
            if (lane == kWave - 1) dn = r.ext;
            const uint32_t mid = __builtin_amdgcn_alignbyte(dn, r.own, sh);   // ub .. ub+3
            const uint32_t lft = __builtin_amdgcn_alignbyte(r.own, dp, 3u);   // ub-sh-1 .. ub-sh+2
            x[0] = (int)((lft >> (8u * sh)) & 255u);
#pragma unroll
            for (int k = 0; k < 4; ++k) x[k + 1] = (int)((mid >> (8 * k)) & 255u);
            x[5] = (int)((dn >> (8u * sh)) & 255u);
        };
        const int t2 = d.P.edge_t * d.P.edge_t;
        bool colok[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) colok[k] = ub + k >= 1 && ub + k <= W - 2;
        int qn = 0;
        const uint8_t* dframe = disp + (int64_t)b * H * dpitch;
        ld_edge* eframe = d.edges + (int64_t)b * H * W;
        auto flush = [&]() {
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            for (int i0 = 0; i0 < qn; i0 += kWave) {
                const int i = i0 + lane;
                if (i < qn) {
                    const uint2 e = queue[i];
                    const int u = (int)(e.x & 0xffffu), r = (int)(e.y >> 16);
                    const int gx = (int)(int16_t)(e.x >> 16), gy = (int)(int16_t)(e.y & 0xffffu);
                    const int v = s0 + r;
                    const uint32_t raw = disp_raw<FMT>(dframe + (int64_t)v * dpitch, u);
                    if (raw >= sbnd[2 * r] && raw <= sbnd[2 * r + 1]) {
                        const int bin = gx != 0 ? vote_bin((double)v - svpy[r], gy, gx, u, d.half, d.W2) : -1;
                        const int slot = atomicAdd(&scnt[r], 1);
                        reinterpret_cast<uint2*>(eframe + (int64_t)v * W)[slot] =
                            make_uint2(e.x, (uint32_t)(uint16_t)gy | ((uint32_t)(uint16_t)bin << 16));
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            qn = 0;
        };
        // Ring of three unpacked rows (rotated by renaming: at the step of phase P, rows v-1 and
        // v sit in U[(P+2)%3] and U[P], and row v+1 is unpacked into U[(P+1)%3]) and two sets of
        // three rows of loads: a group of steps consumes one set, whose loads were issued a
        // whole group earlier, after issuing the other set's loads for the next group.  Steps
        // past the strip's last row compute masked rows.
        int U[3][6];
        RowD LA[3], LB[3];
        LA[0] = load_row(vs - 1);
        LA[1] = load_row(vs);
        unpack(LA[0], vs - 1, U[2]);
        unpack(LA[1], vs, U[0]);
        LA[0] = load_row(vs + 1);
        LA[1] = load_row(vs + 2);
        LA[2] = load_row(vs + 3);
        int v = vs;
        auto step = [&](auto Pc, const RowD& row_next) {
            constexpr int P = decltype(Pc)::value;
            constexpr int A = (P + 2) % 3, M = P % 3, C = (P + 1) % 3;
            const bool rowok = v <= ve;
            unpack(row_next, v + 1, U[C]);
            int S[6], T[6];
#pragma unroll
            for (int j = 0; j < 6; ++j) {
                S[j] = U[A][j] + 2 * U[M][j] + U[C][j];
                T[j] = U[C][j] - U[A][j];
            }
            uint64_t bal[4];
            int gxk[4], gyk[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                gxk[k] = S[k + 2] - S[k];
                gyk[k] = T[k] + 2 * T[k + 1] + T[k + 2];
                const int m2 = __mul24(gxk[k], gxk[k]) + __mul24(gyk[k], gyk[k]);
                bal[k] = __ballot(colok[k] & rowok & (m2 > t2));
            }
            if ((bal[0] | bal[1] | bal[2] | bal[3]) != 0) {
                int off = qn;
                const uint32_t rv = (uint32_t)(v - s0) << 16;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (bal[k] != 0) {
                        if ((bal[k] >> lane) & 1ull)
                            queue[off + __popcll(bal[k] & lanes_below())] =
                                make_uint2((uint32_t)(ub + k) | ((uint32_t)gxk[k] << 16),
                                           ((uint32_t)gyk[k] & 0xffffu) | rv);
                        off += __popcll(bal[k]);
                    }
                }
                qn = off;
                if (qn >= kEdgeFlushAt) flush();
            }
            ++v;
        };
        while (v <= ve) {
#pragma unroll
            for (int j = 0; j < 3; ++j) LB[j] = load_row(v + 4 + j);
            step(IntC<0>{}, LA[0]);
            step(IntC<1>{}, LA[1]);
            step(IntC<2>{}, LA[2]);
            if (v > ve) break;
#pragma unroll
            for (int j = 0; j < 3; ++j) LA[j] = load_row(v + 4 + j);
            step(IntC<3>{}, LB[0]);
            step(IntC<4>{}, LB[1]);
            step(IntC<5>{}, LB[2]);
        }
        flush();
    }
    __syncthreads();
    if (t < rows) d.rowcnt[(int64_t)b * H + s0 + t] = scnt[t];
}

// ------------------------------------------------------------------------------------------
// S6 + S7 + S8: band accumulator m_x (Alg. "Dense V_px accumulation", a band of 2 chi + 1 rows
// clipped to the road), DP path over the 2W vote columns (Eq. dense_vpx_estimation), RANSAC
// quartic gamma (Alg. "gamma estimation"), V_px table (Eq. vpx_estimation) and the
// coefficients of the lane track of Eq. lane_visualisation.  One workgroup per frame.
//
// DP step.  The value E + lambda|tau| and the tie rank of tau in the scan order
// 0, -1, +1, -2, +2, ... (0..10) are packed into one key (value << 4 | rank): the minimum key
// is the minimum value with the first tau of the scan order, which is exactly the
// first-strict-minimum rule.  With Sh = E << 4 the key of tau = -a is
// Sh(c') - (16 lambda + 2) c' + ((16 lambda + 2) c - 1) and of tau = +a is
// Sh(c') + (16 lambda + 2) c' - (16 lambda + 2) c (c' = c + tau), so each side is a plain
// minimum of a per-column term over a window, plus a per-c constant.  The rank (4 bits) is
// the backtrace.
constexpr int kDpRun = 8;            // columns of a backtrace word of the windowed search
constexpr int kFitWalk = 8;          // rows of the backtrace per register chunk of the walk

// tau of rank r, plus 8, in bits 4r .. 4r+3 for r = 0 .. 10
constexpr uint64_t kRankTau = [] {
    uint64_t x = 0;
    for (int r = 0; r <= 10; ++r) x |= (uint64_t)((r == 0 ? 0 : ((r & 1) ? -((r + 1) >> 1) : (r >> 1))) + 8) << (4 * r);
    return x;
}();

// S8: RANSAC of the quartic through the path points (PX = rows, PY = u columns), V_px and the
// track tables, frame info.
__device__ void vpx_fit_tail(Dev& d, int b, FrameInfo fi, int* PX, int* PY, int* cur, int* cur2, uint32_t* bitmap,
                             int bm_words, RansacShared& S, const uint64_t* stream_ids, const int64_t* frame_idx,
                             const double* seed, double* vp_out) {
    const int t = threadIdx.x, nt = blockDim.x;
    const int H = d.H, v_max = H - 1, v_h = fi.v_h, R = v_max - v_h + 1;
    double* tf = d.tab + (int64_t)b * 6 * H;
    double* tvpy = tf + 2 * H;
    double* tvpx = tf + 3 * H;
    double* tA = tf + 4 * H;
    double* tB = tf + 5 * H;
    const double nan = __longlong_as_double(0x7ff8000000000000LL);
    const uint64_t sid = stream_ids ? stream_ids[b] : 0ull;
    const uint64_t fid = frame_idx ? (uint64_t)frame_idx[b] : (uint64_t)b;
    FitRes* fit = d.fit + 2 * b + 1;
    ransac_block<4>(PX, PY, R, cur, cur2, bitmap, bm_words, S, d.P.tr_x, d.P, sid, fid, 1,
                    seed, fit,
                    d.trace + (int64_t)b * 6 * kMaxRounds + 3 * kMaxRounds);
    const FitRes& g = *fit;
    int bad = v_h - 1;
    if (g.ok) {
        for (int v = t; v < H; v += nt)
            tvpx[v] = (v >= v_h) ? eval_s<4>(g.coef, g.center, g.kshift, v) : nan;
    }
    __syncthreads();
    if (g.ok) {
        for (int v = v_h + t; v <= v_max - 1; v += nt) {
            const double den = (double)(v + 1) - tvpy[v + 1];
            if (!(den > 0.0)) {
                bad = max(bad, v);
            } else {
                tA[v] = tvpx[v + 1] / den;
                tB[v] = ((double)v - tvpy[v + 1]) / den;
            }
        }
    }
    bad = block_max_i32(bad, S.red);
    if (t == 0) {
        fi.flags |= (g.flags & 1) ? LD_FLAG_NOCONS_X : 0;
        if (!g.ok) fi.flags |= LD_FLAG_NOVP;
        fi.v_end = g.ok ? bad + 1 : H;
        fi.n_mx = R;
        d.info[b] = fi;
    }
    if (vp_out) {
        for (int v = t; v < H; v += nt) {
            const bool road = v >= v_h && g.ok;
            vp_out[((int64_t)b * H + v) * 2] = road ? tvpx[v] : nan;
            vp_out[((int64_t)b * H + v) * 2 + 1] = v >= v_h ? tvpy[v] : nan;
        }
    }
}

// The workgroup's first vpx_fit_waves(2W) waves own kFitCols consecutive columns a thread and keep
// their DP row (E << 4) in registers; the five columns either side come from the neighbouring
// lanes by wave shifts, and at a wave's ends from the neighbouring wave through LDS.  The vote
// columns of the road rows are staged in LDS first (rows past stage_cap read their edges from
// memory).  One more wave keeps the band's counts, one LDS row of them for the rows of each
// parity: while a row is worked on from its parity's counts, the other parity's move on by the
// two rows that enter and the two that leave.  So a row has one barrier, its window and minima
// touch no LDS, and nothing in it waits for memory (with the votes read from memory a row ahead,
// a row took 1.1 us for any number of columns and waves).
//
// What bounds it: one frame alone, a row's chain of barrier, seam and count reads (about 300
// cycles) and its 200 operations; many frames, the operations issued, about 13 a column.  Ten
// columns a thread make four waves of 1242 wide frames, one a SIMD; 4, 6, 8, 12 and 16 were
// slower alone and with 1024 frames.
//
// Registers for seven waves a SIMD (the backtrace walk has two chunks in flight for that): at 79
// VGPRs and 106 SGPRs the fourth five-wave frame of a CU found no place in half of the processes,
// and 1024 frames of 1242 x 375 took 290 us in one and 400 to 440 in the next; now 300 in each.
// 1242 x 375, one frame 218 -> 138 us, 1024 frames 410 -> 300 us; 1920 x 1080, one frame 660 -> 480
// us, 256 frames 705 -> 518 us.
constexpr int kFitCols = 10;         // columns a thread
constexpr int kSeam = 8;             // LDS words of one end of a wave's row (five used)
constexpr int kNoVote = 0xFFFF;      // a staged edge without a vote column

constexpr bool back_rows_fit() {     // the backtrace's words of a row in the even ones of its W words
    for (int W = 8; W <= 4096; ++W)
        if (2 * ((2 * W + kFitCols - 1) / kFitCols) > W / 2 * 2) return false;
    return true;
}
static_assert(back_rows_fit(), "the row DP's backtrace fits the q buffer's rows");

__host__ __device__ constexpr int vpx_fit_waves(int W2) { return (W2 + kFitCols * kWave - 1) / (kFitCols * kWave); }

__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(7))) void k_vpx_fit(Dev d, int stage_cap) {
    constexpr int K = kFitCols;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ int64_t rv[kMaxWaves + 1];
    __shared__ int ri[kMaxWaves + 1];
    __shared__ int red[kMaxWaves + 1];
    const int b = blockIdx.x, t = threadIdx.x, nt = blockDim.x, lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(t / kWave), nw = nwaves() - 1;   // nw: the waves that own columns
    if (frame_masked(d, b)) return;
    const int H = d.H, W = d.W, W2 = d.W2, v_max = H - 1;
    FrameInfo fi = d.info[b];
    for (int v = t; v < H; v += nt) d.mxpath[(int64_t)b * H + v] = -1;
    if (fi.flags & LD_FLAG_NOROAD) return;
    const int v_h = __builtin_amdgcn_readfirstlane(fi.v_h), R = v_max - v_h + 1, chi = d.P.chi;
    const int WP = nw * kWave * K;                             // columns of one row of counts
    int* hist = reinterpret_cast<int*>(smem);                  // 2 x WP, by row parity: 16 x the band's votes
    int* seam = reinterpret_cast<int*>(hist + 2 * WP);         // 2 x (nw + 2) x 2 x kSeam: the columns either side of a wave
    int* roff = seam + 2 * (nw + 2) * 2 * kSeam;               // R + 1: edges on the road rows above
    uint16_t* wb = reinterpret_cast<uint16_t*>(roff + H + 1);  // stage_cap vote columns
    const ld_edge* fedges = d.edges + (int64_t)b * H * W;
    for (int r = t; r < R; r += nt) roff[r + 1] = d.rowcnt[(int64_t)b * H + v_h + r];
    for (int i = t; i < 2 * WP; i += nt) hist[i] = 0;
    for (int i = t; i < 2 * (nw + 2) * 2 * kSeam; i += nt) seam[i] = kBig;
    // staging: a wave takes kStageRows rows at a time, their first 64 edges in flight at once
    constexpr int kStageRows = 16;
    int c[kStageRows];
    auto load_rows = [&](int r0) {
#pragma unroll
        for (int j = 0; j < kStageRows; ++j)
            c[j] = fedges[(int64_t)(v_h + min(r0 + j, R - 1)) * W + min(lane, W - 1)].bin;
    };
    load_rows(wave * kStageRows);
    __syncthreads();
    if (wave == 0) {                                           // inclusive prefix, 64 rows a scan
        int carry = 0;
        for (int base = 0; base < R; base += kWave) {
            int x = base + lane < R ? roff[base + lane + 1] : 0;
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const int y = __shfl_up(x, o, kWave);
                if (lane >= o) x += y;
            }
            if (base + lane < R) roff[base + lane + 1] = carry + x;
            carry += __shfl(x, kWave - 1, kWave);
        }
        if (lane == 0) roff[0] = 0;
    }
    __syncthreads();
    // A frame with many edges would wait for the one wave that keeps the counts, which moves each vote
    // twice (once for either parity) and reads what is not staged from memory: there all the waves
    // share the votes of one row of counts, with a second barrier a row, and nothing is staged.  An
    // edge that is not staged counts as five, and the line lies the higher the more waves meet at that
    // barrier; with one of columns, two share the votes and so gain little (us, one wave and shared, by
    // edges a row and of them not staged; 320 x 96, one: 121, 0: 96, 91; 176, 0: 127, 127; 1024 frames 155,
    // 176; 287, 110: 304, 199; 512 x 160, two: 96, 0: 144, 138; 512 frames 157, 173; 141, 0: 199, 172;
    // 641 x 240, three: 89, 0: 177, 207; 143, 0: 258, 208; 1024 frames 61, 13: 312, 380; 71, 23: 376, 382; 1242 x
    // 375, four: 89, 0: 270, 326; 116, 0: 318, 327; 179, 0: 442, 323; 1024 frames 26, 3: 290, 365; 44, 21: 654, 628;
    // 89, 66: 875, 640; 1536 x 400, five: 107, 0: 339, 426; 143, 0: 413, 432; 1024 frames 53, 22: 1065, 997; 1920 x
    // 1080, six: 71, 12: 1020, 1158; 89, 31: 1218, 1145; 1778, 1720: 11400, 2290; 2560 x 400, eight: 124, 0: 348,
    // 458; 512 frames 88, 42: 696, 678; 4096 x 256, thirteen: 197, 15: 353, 424; 287, 105: 530, 425; there every thread
    // kept counts before: 1242 wide 413, 1024 frames 750, 1920 x 1080 1230 to 2750).
    const int dense = nw == 1 ? 200 : max(120, 28 * nw);
    const bool shared_votes = __builtin_expect(roff[R] + 4 * max(roff[R] - stage_cap, 0) > dense * R, 0);
    int nv = 0;   // votes that landed in a column
    for (int r0 = wave * kStageRows; r0 < R && !shared_votes; r0 += (nw + 1) * kStageRows) {
        const int mine = roff[min(r0 + lane, R)];              // lane l: the offset of row r0 + l
#pragma unroll
        for (int j = 0; j < kStageRows; ++j) {
            const int r = r0 + j, o = __builtin_amdgcn_readlane(mine, j), n = __builtin_amdgcn_readlane(mine, j + 1) - o;
            const bool fits = o + n <= stage_cap;              // (rows past the last have n = 0)
            if (lane < n) {
                nv += c[j] >= 0 ? 1 : 0;
                if (fits) wb[o + lane] = (uint16_t)c[j];       // -1 is kNoVote
            }
            if (n > kWave)
                for (int i = lane + kWave; i < n; i += kWave) {
                    const int bin = fedges[(int64_t)(v_h + r) * W + i].bin;
                    nv += bin >= 0 ? 1 : 0;
                    if (fits) wb[o + i] = (uint16_t)bin;
                }
        }
        load_rows(r0 + (nw + 1) * kStageRows);
    }
    __syncthreads();
    // one vote enters (x = 1) or leaves (-1) the counts
    auto vote = [&](int* to, int bin, int x) {
        if (bin != kNoVote) atomicAdd(&to[bin], 16 * x);
    };
    // votes of edges i, i + 64, ... < n of a run, four of them read at a time
    auto vote_run = [&](int* to, auto bin_at, int i, int n, int x) {
        for (; i < n; i += 4 * kWave) {
            int bin[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) bin[q] = i + q * kWave < n ? bin_at(i + q * kWave) : kNoVote;
#pragma unroll
            for (int q = 0; q < 4; ++q) vote(to, bin[q], x);
        }
    };
    // a road row's edge in memory
    auto edge_of = [&](int r, int i) -> int { return (uint16_t)fedges[(int64_t)(v_h + r) * W + i].bin; };
    // the votes of road rows r0 .. r1
    auto vote_rows = [&](int* to, int r0, int r1, int x) {
        for (int r = r0; r <= r1; ++r) {
            const int o = roff[r], n = roff[r + 1] - o;
            if (o + n <= stage_cap)
                for (int i = lane; i < n; i += kWave) vote(to, wb[o + i], x);
            else vote_run(to, [&](int i) { return edge_of(r, i); }, lane, n, x);
        }
    };
    // the bands of the two lowest rows (road rows R - 1 and R - 2)
    for (int r = max(R - 1 - chi, 0) + wave; r < R && !shared_votes; r += nw + 1) vote_rows(hist + (v_max & 1) * WP, r, r, 1);
    for (int r = max(R - 2 - chi, 0) + wave; r <= min(R - 2 + chi, R - 1) && !shared_votes; r += nw + 1)
        vote_rows(hist + ((v_max & 1) ^ 1) * WP, r, r, 1);
    // Shared votes: from the band of road row r + 1 to that of row r, one row enters and one leaves
    // (rows outside the road hold nothing).  A thread's first edge of either is read a row ahead, as
    // soon as the one before has been counted and into the same register, so that no wave waits for
    // a copy of a load in flight (read before it, and compared when read: 1242 x 375 with 179 edges a
    // row 449 us, now 323, 1920 x 1080 with 271 1532, now 1158); the others two of either row at a
    // time.  The loops are the workgroup's, so that the votes are counted a wave at a time
    // (nvs) and take no register.
    int nvs = 0, na = 0, nl = 0, enters = kNoVote, leaves = kNoVote;
    auto edges_of = [&](int r) { return r >= 0 && r < R ? __builtin_amdgcn_readfirstlane(roff[r + 1] - roff[r]) : 0; };
    auto ahead = [&](int ra, int rl) __attribute__((always_inline)) {
        na = edges_of(ra);
        nl = edges_of(rl);
        enters = t < na ? edge_of(ra, t) : kNoVote;
        leaves = t < nl ? edge_of(rl, t) : kNoVote;
    };
    auto move = [&](int a, int l) __attribute__((always_inline)) {
        vote(hist, a, 1);
        vote(hist, l, -1);
        nvs += __popcll(__ballot(a != kNoVote));
    };
    auto move_band = [&](int ra, int rl) __attribute__((always_inline)) {
        move(enters, leaves);
        for (int i0 = nt; i0 < max(na, nl); i0 += 2 * nt) {
            int a[2], l[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int i = i0 + q * nt + t;
                a[q] = i < na ? edge_of(ra, i) : kNoVote;
                l[q] = i < nl ? edge_of(rl, i) : kNoVote;
            }
#pragma unroll
            for (int q = 0; q < 2; ++q) move(a[q], l[q]);
        }
        ahead(ra - 1, rl - 1);
    };
    if (__builtin_expect(shared_votes, 0)) {
        ahead(R - 1, R);
        for (int r = R - 1; r >= max(R - 1 - chi, 0); --r) move_band(r, R + 1);
        ahead(R - 2 - chi, R - 1 + chi);
    }
    // backtrace: the ranks of a thread's columns in two words, at the start of the q buffer's row
    // of W words (rounded down to an even one, so perhaps from the last word of the frame before, where no
    // backtrace lies)
    const int L = (W2 + K - 1) / K;                            // threads with a column
    uint2* back = reinterpret_cast<uint2*>(d.qbuf + ((int64_t)b * H * W & ~(int64_t)1));
    const int64_t pitch = W / 2;
    const int c0 = t * K;
    int S[K];
    if (__builtin_expect(wave == nw && shared_votes, 0)) {
        __syncthreads();                                       // row v_max
        for (int r = R - 2; r >= 0; --r) {
            __syncthreads();
            move_band(r - chi, r + chi + 1);
            __syncthreads();
        }
    } else if (wave == nw) {
        // While row v is worked on from the counts of its parity, those of the other parity go
        // from the band of row v + 1 to that of v - 1: rows v - 1 - chi and v - chi enter, v + chi and
        // v + 1 + chi leave (with chi = 0 one each), two runs of staged edges.  Lane l holds
        // both runs (offset, count; -1 when not all staged) of iteration 64 m + l; their first
        // 128 entries are read a row ahead.
        int oA = 0, nA = 0, oR = 0, nR = 0;
        const int two = chi > 0 ? 1 : 0;
        auto heads = [&](int it0) {
            const int r = R - 1 - it0 - lane;                  // road row of iteration it0 + lane
            const int a0 = max(r - 1 - chi, 0), a1 = r - 1 - chi + two, l0 = r + 1 + chi - two, l1 = min(r + 1 + chi, R - 1);
            nA = nR = 0;
            if (r >= 1 && a1 >= 0) {
                oA = roff[a0];
                nA = roff[a1 + 1] - oA;
                if (oA + nA > stage_cap) nA = -1;
            }
            if (r >= 1 && l0 <= l1) {
                oR = roff[l0];
                nR = roff[l1 + 1] - oR;
                if (oR + nR > stage_cap) nR = -1;
            }
        };
        auto own = [&](int o, int n, int i) -> int { return i < n ? wb[o + i] : kNoVote; };
        int cA, cR, bA[2], bR[2];
        auto next = [&](int it) {
            const int l = it & (kWave - 1);
            const int fA = __builtin_amdgcn_readlane(oA, l), fR = __builtin_amdgcn_readlane(oR, l);
            cA = __builtin_amdgcn_readlane(nA, l);
            cR = __builtin_amdgcn_readlane(nR, l);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                bA[j] = own(fA, cA, lane + j * kWave);
                bR[j] = own(fR, cR, lane + j * kWave);
            }
        };
        heads(0);
        next(1);
        __builtin_amdgcn_s_setprio(3);                         // the others wait for this wave at each row
        __syncthreads();                                       // row v_max
        for (int it = 1; it < R; ++it) {
            const int r = R - 1 - it;
            __syncthreads();
            int* to = hist + ((v_max - it - 1) & 1) * WP;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                vote(to, bA[j], 1);
                vote(to, bR[j], -1);
            }
            if (r >= 1) {
                // runs past 128 edges or not staged (rare)
                const int fA = __builtin_amdgcn_readlane(oA, it & (kWave - 1)), fR = __builtin_amdgcn_readlane(oR, it & (kWave - 1));
                for (int i = lane + 2 * kWave; i < cA; i += kWave) vote(to, wb[fA + i], 1);
                for (int i = lane + 2 * kWave; i < cR; i += kWave) vote(to, wb[fR + i], -1);
                if (cA < 0) vote_rows(to, max(r - 1 - chi, 0), r - 1 - chi + two, 1);
                if (cR < 0) vote_rows(to, r + 1 + chi - two, min(r + 1 + chi, R - 1), -1);
            }
            if (((it + 1) & (kWave - 1)) == 0) heads(it + 1);
            next(it + 1);
        }
    } else {
        const int tau_max = d.P.tau_x_max;
        const int slope = 16 * d.P.lambda_x + 2;
        const int* own0 = hist + t * K;
        const int seam_par = (nw + 2) * 2 * kSeam;
        // the first lane reads the columns before the wave, the last lane those after it
        const int* get0 = seam + (wave + 1) * 2 * kSeam + (lane == kWave - 1 ? kSeam : 0);
        int* put0 = seam + (lane == 0 ? wave * 2 * kSeam + kSeam : (wave + 2) * 2 * kSeam);
        auto counts = [&](int par, int (&h)[K]) {
            static_assert(K % 2 == 0, "counts are read by twos");
            const int2* p = reinterpret_cast<const int2*>(own0 + par * WP);
#pragma unroll
            for (int q = 0; q < K / 2; ++q) {
                const int2 x = p[q];
                h[2 * q] = x.x; h[2 * q + 1] = x.y;
            }
        };
        // the wave's first and last five columns, for the row that parity `par` reads
        auto put_seams = [&](int par) {
            if (lane == 0 || lane == kWave - 1) {
                int x[5];
#pragma unroll
                for (int j = 0; j < 5; ++j) x[j] = lane == 0 ? S[j] : S[K - 5 + j];
                int* s = put0 + par * seam_par;
                *reinterpret_cast<int4*>(s) = make_int4(x[0], x[1], x[2], x[3]);
                s[4] = x[4];
            }
        };
        // One row: TL[j] = S(c0 - 5 + j) - slope (j - 5) for tau < 0, TR for tau > 0, the offset of
        // a term from its column taken against the thread's first column; the minima over five
        // consecutive entries share their middle three.  Instantiated for the full window
        // (tau_max = 5) and for a narrower one, and for the wave that holds the last column, whose
        // columns past it keep the padding value.
        auto row = [&](auto full, auto last, auto shared, int par, int v) __attribute__((always_inline)) {
            constexpr bool kFull = decltype(full)::value, kLast = decltype(last)::value;
            int w[K + 10];
            int h[K];
            {
                const int* sg = get0 + par * seam_par;
                const int4 g4 = *reinterpret_cast<const int4*>(sg);
                const int g[5] = {g4.x, g4.y, g4.z, g4.w, sg[4]};
                counts(decltype(shared)::value ? 0 : par, h);
#pragma unroll
                for (int j = 0; j < 5; ++j) {
                    w[j] = __builtin_amdgcn_update_dpp(g[j], S[K - 5 + j], 0x138, 0xF, 0xF, false);      // lane - 1
                    w[K + 5 + j] = __builtin_amdgcn_update_dpp(g[j], S[j], 0x130, 0xF, 0xF, false);      // lane + 1
                }
            }
#pragma unroll
            for (int k = 0; k < K; ++k) w[k + 5] = S[k];
            int lm[K], rm[K];
            if constexpr (kFull) {
                int TL[K + 4], TR[K + 4];
#pragma unroll
                for (int j = 0; j < K + 4; ++j) {
                    TL[j] = w[j] - slope * (j - 5);
                    TR[j] = w[j + 6] + slope * (j + 1);
                }
                auto min5 = [](auto n, const int* T, int* m) { // m[k] = min T[k .. k + 4], k = 0 .. n - 1
                    const int x = min(min(T[2], T[3]), T[4]);
                    m[0] = min(min(T[0], T[1]), x);
                    m[1] = min(min(T[1], x), T[5]);
                    if constexpr (decltype(n)::value == 4) {
                        m[2] = min(min(x, T[5]), T[6]);
                        m[3] = min(min(T[3], T[4]), min(min(T[5], T[6]), T[7]));
                    }
                };
                static_assert(K == 10, "the minima of ten columns");
                min5(IntC<4>{}, TL, lm); min5(IntC<4>{}, TL + 4, lm + 4); min5(IntC<2>{}, TL + 8, lm + 8);
                min5(IntC<4>{}, TR, rm); min5(IntC<4>{}, TR + 4, rm + 4); min5(IntC<2>{}, TR + 8, rm + 8);
            } else {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    lm[k] = kBig; rm[k] = kBig;
#pragma unroll
                    for (int a = 1; a <= 5; ++a)
                        if (a <= tau_max) {
                            lm[k] = min(lm[k], w[k + 5 - a] - slope * (k - a));
                            rm[k] = min(rm[k], w[k + 5 + a] + slope * (k + a));
                        }
                }
            }
            uint32_t word[2] = {0, 0};
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int key = min(min(w[k + 5], lm[k] + (slope * k - 1)), rm[k] - slope * k);
                const int e = (key & -16) - h[k];              // (E_min - votes) << 4
                S[k] = !kLast || c0 + k < W2 ? e : kBig;
                word[k / 8] = __builtin_amdgcn_alignbit((uint32_t)key, word[k / 8], 4);   // enters from the top
            }
            if (!kLast || c0 < W2) (back + v * pitch)[t] = make_uint2(word[0], word[1]);
            put_seams(par ^ 1);
        };
        auto rows = [&](auto full, auto last, auto shared) __attribute__((always_inline)) {
            constexpr bool kShared = decltype(shared)::value;
            __syncthreads();                                   // row v_max: its counts alone
            int h[K];
            counts(kShared ? 0 : v_max & 1, h);
#pragma unroll
            for (int k = 0; k < K; ++k) S[k] = c0 + k < W2 ? -h[k] : kBig;
            put_seams((v_max & 1) ^ 1);
            int v = v_max - 1;
            if constexpr (kShared) {
                for (; v >= v_h; --v) {
                    __syncthreads();                           // every wave has read the counts
                    move_band(v - v_h - chi, v - v_h + chi + 1);
                    __syncthreads();
                    row(full, last, shared, v & 1, v);
                }
                return;
            }
            if (v >= v_h && (v & 1) == 0) {
                __syncthreads();
                row(full, last, shared, 0, v);
                --v;
            }
            for (; v >= v_h; v -= 2) {                         // v is odd here
                __syncthreads();
                row(full, last, shared, 1, v);
                if (v - 1 < v_h) break;
                __syncthreads();
                row(full, last, shared, 0, v - 1);
            }
        };
        // (the common forms first in the code: behind the shared ones they took 3% longer)
        if (!shared_votes && tau_max == 5 && (wave + 1) * K * kWave <= W2) rows(std::true_type{}, std::false_type{}, std::false_type{});
        else if (!shared_votes && tau_max == 5) rows(std::true_type{}, std::true_type{}, std::false_type{});
        else if (!shared_votes) rows(std::false_type{}, std::true_type{}, std::false_type{});
        else if (tau_max == 5) rows(std::true_type{}, std::true_type{}, std::true_type{});
        else rows(std::false_type{}, std::true_type{}, std::true_type{});
    }
    int64_t bvv = INT64_MAX;
    int bi = 0x7fffffff;
    if (wave < nw) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (c0 + k < W2 && (int64_t)(S[k] >> 4) < bvv) { bvv = S[k] >> 4; bi = c0 + k; }
    }
    block_argmin_i64(bvv, bi, rv, ri);
    // backtrace, by wave 0: lane l holds the ranks of thread w0 + l of each of kFitWalk rows (64
    // threads, 64 K columns); the column is wave-uniform, so a step is a readlane and a few scalar
    // operations.  kAhead chunks of rows are in flight beside the one that is walked: the path
    // moves at most 5 columns a row, so the words centred on a chunk's start column, 32 K to
    // either side, cover it up to the end of the last of them.
    if (t < kWave) {
        constexpr int kAhead = 2;
        static_assert(5 * (kAhead + 1) * kFitWalk + K <= 32 * K, "a chunk's words cover the path");
        const int l = t;
        int c = __builtin_amdgcn_readfirstlane(bi);
        struct Chunk { uint2 w[kFitWalk]; int w0; };
        auto load_chunk = [&](int v0, Chunk& q) {
            q.w0 = max(0, min(c / K - 32, L - kWave));
            const int wi = min(q.w0 + l, L - 1);
#pragma unroll
            for (int r = 0; r < kFitWalk; ++r)                 // rows v < v_max hold an entry
                q.w[r] = back[max(min(v0 + r, v_max - 1), 0) * pitch + wi];
        };
        // the rank of a thread's column k: eight in the first word, the rest at the second's top
        auto rank_of = [](const uint2& w, int lane_of, int k) -> int {
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)w.x, lane_of);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)w.y, lane_of);
            return (int)((k < 8 ? lo >> (4 * k) : hi >> (4 * (k + 8 - K))) & 15u);
        };
        auto walk = [&](int v0, const Chunk& q) {
            int pv = 0;
            auto step = [&](int r) {
                const int g = c / K;
                c += (int)((kRankTau >> (4 * rank_of(q.w[r], g - q.w0, c - g * K))) & 15u) - 8;
            };
            if (v0 + kFitWalk <= v_max) {                      // every row of the chunk has an entry
#pragma unroll
                for (int r = 0; r < kFitWalk; ++r) {
                    pv = l == r ? c : pv;
                    step(r);
                }
            } else {
#pragma unroll
                for (int r = 0; r < kFitWalk; ++r) {
                    if (v0 + r > v_max) break;
                    pv = l == r ? c : pv;
                    if (v0 + r < v_max) step(r);
                }
            }
            if (l < kFitWalk && v0 + l <= v_max) d.mxpath[(int64_t)b * H + v0 + l] = pv;
        };
        Chunk q[kAhead + 1];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) load_chunk(v_h + i * kFitWalk, q[i]);
        for (int v0 = v_h; v0 <= v_max; v0 += (kAhead + 1) * kFitWalk) {
#pragma unroll
            for (int i = 0; i <= kAhead; ++i) {
                load_chunk(v0 + (i + kAhead) * kFitWalk, q[(i + kAhead) % (kAhead + 1)]);
                walk(v0 + i * kFitWalk, q[i]);
            }
        }
    }
    nv = block_sum_i32(nv + (lane == 0 ? nvs : 0), red);
    if (t == 0) {
        fi.n_edges = roff[R];
        fi.n_votes = nv;
        d.info[b] = fi;
    }
}

// S8 for every frame: RANSAC of the quartic through the row-DP path (read back from the path
// columns), V_px and the track tables.  One workgroup per frame (ransac_threads).  Hypothesis 0:
// the seed of the narrowed search for the frames that kept one (pruned = 1), otherwise the
// caller's seed rows.
__global__ __launch_bounds__(512) void k_vpx_ransac(Dev d, const uint64_t* stream_ids, const int64_t* frame_idx,
                                                    const double* seed_gamma, int pruned, double* vp_out) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ RansacShared S;
    const int b = blockIdx.x, t = threadIdx.x, nt = blockDim.x;
    if (frame_masked(d, b)) return;
    const int H = d.H, v_max = H - 1;
    const FrameInfo fi = d.info[b];
    double* tf = d.tab + (int64_t)b * 6 * H;
    for (int v = t; v < H; v += nt) {
        tf[4 * H + v] = 0.0;
        tf[5 * H + v] = 0.0;
    }
    if (fi.flags & LD_FLAG_NOROAD) {
        const double nan = __longlong_as_double(0x7ff8000000000000LL);
        if (vp_out)
            for (int v = t; v < H; v += nt) {
                vp_out[((int64_t)b * H + v) * 2] = nan;
                vp_out[((int64_t)b * H + v) * 2 + 1] = nan;
            }
        return;
    }
    const int v_h = fi.v_h;
    const int H4 = (H + 3) / 4 * 4;
    int* PX = reinterpret_cast<int*>(smem);
    int* PY = PX + H4;
    int* cur = PY + H4;
    int* cur2 = cur + H4;
    uint32_t* bitmap = reinterpret_cast<uint32_t*>(cur2 + H4);
    const int bm_words = (H + 31) / 32;
    for (int v = v_h + t; v <= v_max; v += nt) {
        PX[v - v_h] = v;
        PY[v - v_h] = d.mxpath[(int64_t)b * H + v] - d.half;
    }
    __syncthreads();
    // hypothesis 0: the narrowed search's own seed when it has one (no fallback, a seed line
    // drawn), else the caller's seed (NaN first coefficient or NULL: none)
    const double* seed = seed_gamma ? seed_gamma + 5 * (int64_t)b : nullptr;
    if (pruned && !(d.prune[(int64_t)b * kPruneWords + 1] & kFbPlainVpx) && !isnan(d.seedg[5 * (int64_t)b]))
        seed = d.seedg + 5 * (int64_t)b;
    vpx_fit_tail(d, b, fi, PX, PY, cur, cur2, bitmap, bm_words, S, stream_ids, frame_idx, seed, vp_out);
}

// ------------------------------------------------------------------------------------------
// S9 - S12: piecewise weight w_g (Eq. sigma_g), q = G_x w_g, M_0 (box of 3 columns x 7 rows),
// M_1 = Sobel-x of M_0 (Alg. "Lane position validation"), and the energy of every candidate
// along its track (Eq. lane_energy, Eq. lane_visualisation).
//
// One workgroup of BT threads per frame.  First q is computed for every road edge (each wave a
// group of rows) into a per-edge buffer.  Then the road rows are swept upwards.  At the step of row v every
// thread pushes its NC columns (consecutive when NC is odd, a stride coprime with the LDS
// banks; else t, t + BT, ...) of the dense q row v-4 (scattered into LDS during the previous
// step) into a 9-row register ring (rows v-4..v+4) and forms V(x, v) = sum_y s_y C(x, v+y),
// C = vertical 7-row sums, with the zero padding of M_0 outside the image (a uniform branch:
// rows strictly inside take both neighbours without a select), while the edges of row v-5 are
// scattered into the other q row; after the step's one barrier the column owners form
// M_1(u, v) = sum_{dx} V(u+1+dx) - sum_{dx} V(u-1+dx) (terms outside the image dropped, on the
// few edge lanes only; consecutive columns share their three-column sums) into one of two LDS
// rows, and every candidate adds M_1 at its track column of row v+1.  The q, V and M_1 rows are
// double-buffered by row parity, so one barrier per row orders every write before its reads.
// Rows are padded to the NC * BT columns the threads own (the columns past W hold zeros), so
// the column loops carry no bounds test.  The row loop is unrolled nine times so that the ring
// rotates by renaming registers instead of moving them.
// mode 0 / 1: G_x w_g with the exponent as printed / squared; mode 2: the prior work's vote
// |grad| cos(theta_e - theta_Vp) = t . (p - V_p) / |p - V_p| = -dot / |r|, in FP64 (no gate)
__device__ __forceinline__ float edge_q(const ld_edge& ed, int r, double vx, double vy, float inv_sg2, int sq) {
    const double tx = (double)(-ed.gy), ty = (double)ed.gx;
    const double rx = vx - (double)ed.u, ry = vy - (double)r;
    const double dot = tx * rx + ty * ry;
    const double tt = tx * tx + ty * ty;
    const double rr = rx * rx + ry * ry;
    if (sq == 2) return rr > 0.0 ? (float)(-dot / sqrt(rr)) : 0.0f;
    if (!(dot * dot >= (0.75 * tt) * rr)) return 0.0f;
    const double cr = tx * ry - ty * rx;
    const float delta = atan2f((float)fabs(cr), (float)fabs(dot));
    const float p = delta * (float)(36.0 / 3.14159265358979323846);
    const float w = sq ? expf(-(p * p) * inv_sg2) : expf(-p * inv_sg2);
    return (float)ed.gx * w;
}

template <int NC, int NT, int BT, int PD>
__global__ __launch_bounds__(BT) void k_energy(Dev d, const uint8_t* cand_mask, float* energy_out, int stage_off) {
    extern __shared__ __attribute__((aligned(16))) float fsm[];
    const int b = blockIdx.x, t = threadIdx.x, lane = lane_id(), wave = t / kWave;
    if (frame_masked(d, b)) return;
    const int W = d.W, H = d.H, W2 = d.W2, v_max = H - 1;
    const FrameInfo fi = d.info[b];
    double* Eout = d.energy + (int64_t)b * W2;
    if (fi.flags & (LD_FLAG_NOROAD | LD_FLAG_NOVP)) {
        for (int i = t; i < W2; i += BT) {
            Eout[i] = 0.0;
            if (energy_out) energy_out[(int64_t)b * W2 + i] = 0.0f;
        }
        return;
    }
    constexpr int WP = NC * BT;  // columns owned by the threads (>= W)
    // a thread owns NC consecutive columns when NC is odd (a stride coprime with the LDS banks),
    // else columns t, t + BT, ...
    constexpr bool kConsec = NC % 2 == 1;
    auto col = [&](int k) { return kConsec ? t * NC + k : t + k * BT; };
    // by row parity: dense q rows; V rows, column u at u + 2 (two zero columns each side); M_1
    // rows (entries >= W stay 0)
    auto qb = [&](int par) -> float* { return fsm + par * WP; };
    auto Vp = [&](int par) -> float* { return fsm + 2 * WP + par * (WP + 4); };
    auto mb = [&](int par) -> float* { return fsm + 4 * WP + 8 + par * (WP + 1); };
    const double* tf = d.tab + (int64_t)b * 6 * H;
    const double* tvpy = tf + 2 * H;
    const double* tvpx = tf + 3 * H;
    const double* tA = tf + 4 * H;
    const double* tB = tf + 5 * H;
    const int v_h = fi.v_h, v_end = fi.v_end;
    const float inv_sg2 = (float)(1.0 / (d.P.sigma_g * d.P.sigma_g));
    const int sq = d.P.vote ? 2 : d.P.weight_squared;
    const ld_edge* edges = d.edges + (int64_t)b * H * W;
    float* qbuf = d.qbuf + (int64_t)b * H * W;
    const int32_t* rowcnt = d.rowcnt + (int64_t)b * H;

    // q of every road edge: a wave takes kQRows rows at a time and loads two edge slots per
    // lane (i = lane, lane + 64) of each, every load of the group issued before any q is
    // formed (clamped to the row's W slots; the counts mask them); longer rows go on in a loop
    constexpr int kQRows = 4;
    for (int r0 = v_h + wave * kQRows; r0 <= v_max; r0 += (BT / kWave) * kQRows) {
        int cnt[kQRows];
        double vx[kQRows], vy[kQRows];
        ld_edge e0[kQRows], e1[kQRows];
#pragma unroll
        for (int j = 0; j < kQRows; ++j) {
            const int r = min(r0 + j, v_max);
            cnt[j] = r0 + j <= v_max ? rowcnt[r] : 0;
            vx[j] = tvpx[r];
            vy[j] = tvpy[r];
            e0[j] = edges[(int64_t)r * W + min(lane, W - 1)];
            e1[j] = edges[(int64_t)r * W + min(lane + kWave, W - 1)];
        }
#pragma unroll
        for (int j = 0; j < kQRows; ++j) {
            const int r = r0 + j;
            if (lane < cnt[j]) qbuf[(int64_t)r * W + lane] = edge_q(e0[j], r, vx[j], vy[j], inv_sg2, sq);
            if (lane + kWave < cnt[j]) qbuf[(int64_t)r * W + lane + kWave] = edge_q(e1[j], r, vx[j], vy[j], inv_sg2, sq);
            for (int i = lane + 2 * kWave; i < cnt[j]; i += kWave)
                qbuf[(int64_t)r * W + i] = edge_q(edges[(int64_t)r * W + i], r, vx[j], vy[j], inv_sg2, sq);
        }
    }
    for (int i = t; i < 6 * WP + 10; i += BT) fsm[i] = 0.0f;
    // the track coefficients and edge counts of the swept rows, in LDS when they fit (stage_off
    // > 0): a row's scalar loads would otherwise be waited for at its barrier
    double2* sAB = reinterpret_cast<double2*>(fsm + stage_off);
    int* scnt = reinterpret_cast<int*>(sAB + H);
    const bool staged = stage_off > 0;
    if (staged)
        for (int r = v_h + t; r <= v_max; r += BT) {
            sAB[r] = r < v_max ? make_double2(tA[r], tB[r]) : make_double2(0.0, 1.0);
            scnt[r] = rowcnt[r];
        }
    float ring[NC][9];
#pragma unroll
    for (int k = 0; k < NC; ++k)
#pragma unroll
        for (int j = 0; j < 9; ++j) ring[k][j] = 0.0f;
    double uu[NT], ee[NT];
    bool live[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        const int i = t + k * BT;
        uu[k] = (double)(i - d.half);
        ee[k] = 0.0;
        live[k] = i < W2 && (cand_mask == nullptr || cand_mask[(int64_t)b * W2 + i] != 0);
    }
    __syncthreads();

    // the next PD rows to scatter: each thread's first edge of row r waits in slot
    // (v_max - r) mod PD, loaded PD steps ahead (from a clamped, always valid index; the row's
    // count masks it when it is used)
    int nx_u[PD];
    float nx_q[PD];
    auto count = [&](int r) -> int {
        if (r < v_h || r > v_max) return 0;
        return staged ? scnt[r] : rowcnt[r];
    };
    auto prefetch = [&](auto slot, int r) {
        constexpr int K = decltype(slot)::value;
        const int rr = min(max(r, 0), v_max), i = min(t, W - 1);
        nx_u[K] = edges[(int64_t)rr * W + i].u;
        nx_q[K] = qbuf[(int64_t)rr * W + i];
    };
    auto scatter = [&](auto slot, int r, float* q) {
        constexpr int K = decltype(slot)::value;
        const int n = count(r);
        if (t < n) q[nx_u[K]] = nx_q[K];
        for (int i = t + BT; i < n; i += BT)
            q[edges[(int64_t)r * W + i].u] = qbuf[(int64_t)r * W + i];
    };
    // slot S of the ring takes the newest row; reads and re-zeroes the owned columns of q
    auto push = [&](auto Sc, float* q) {
        constexpr int S = decltype(Sc)::value;
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const int u = col(k);
            ring[k][S] = q[u];
            q[u] = 0.0f;
        }
    };
    // the track of every live candidate moves to row w and adds M_1(col, w); a track outside
    // the image (or a dead candidate) reads the zero entry W (ee is never -0, so adding +0
    // leaves it unchanged).  The tracks are finite (A_v, B_v are finite on the swept rows);
    // the conversion saturates, so the unsigned compare also rejects x < 0 and huge x.
    // A_w, B_w are loaded one step before their row's turn (fma(1, u, 0) = u for w = v_max).
    double cA = 0.0, cB = 1.0;
    auto coef = [&](int w) {
        if (staged) {
            const double2 ab = sAB[w];
            cA = ab.x;
            cB = ab.y;
        } else {
            const bool upd = w < v_max;
            cA = upd ? tA[w] : 0.0;
            cB = upd ? tB[w] : 1.0;
        }
    };
    auto candidates = [&](const float* m1row) {
        const double A = cA, Bc = cB;
#pragma unroll
        for (int k = 0; k < NT; ++k) {
            uu[k] = fma(Bc, uu[k], A);
            const int c = (int)floor(uu[k] + 0.5);
            const bool in = live[k] & ((unsigned)c < (unsigned)W);   // no branch: both are computed
            ee[k] += (double)m1row[in ? c : W];
        }
    };
    // rows v_max .. v_max-3 enter slots 0, 8, 7, 6; rows below the image stay zero; row
    // v_max-4 waits in its q row for the first step
    auto enter = [&](auto kc, auto Sc) {                  // row v_max - k
        constexpr int K = decltype(kc)::value;
        scatter(IntC<K % PD>{}, v_max - K, qb((v_max - K) & 1));
        prefetch(IntC<K % PD>{}, v_max - K - PD);
        __syncthreads();
        if constexpr (K < 4) push(Sc, qb((v_max - K) & 1));
    };
    prefetch(IntC<0>{}, v_max);
    if constexpr (PD > 1) prefetch(IntC<1 % PD>{}, v_max - 1);
    if constexpr (PD > 2) prefetch(IntC<2 % PD>{}, v_max - 2);
    enter(IntC<0>{}, IntC<0>{});
    enter(IntC<1>{}, IntC<8>{});
    enter(IntC<2>{}, IntC<7>{});
    enter(IntC<3>{}, IntC<6>{});
    enter(IntC<4>{}, IntC<5>{});
    int v = v_max;
    // one row: newest ring slot S holds row v-4, slot (S + j) % 9 row v-4+j
    auto step = [&](auto Sc) -> bool {
        constexpr int S = decltype(Sc)::value;
        if (v < v_end) return false;
        const int par = v & 1;
        push(Sc, qb(par));               // row v - 4 (same parity as v)
        const bool up = v >= 1, dn = v + 1 <= v_max;   // M_0 is zero outside the image rows
        // (uniform over the workgroup: the rows strictly inside the image take both terms
        // without a per-column select)
        auto vcol = [&](auto both) {
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                const int u = col(k);
                float r[9];
#pragma unroll
                for (int j = 0; j < 9; ++j) r[j] = ring[k][(S + j) % 9];
                const float s5 = (((r[2] + r[3]) + r[4]) + r[5]) + r[6];
                const float cm1 = (r[0] + r[1]) + s5;   // C(v-1): rows v-4..v+2
                const float c0 = (r[1] + s5) + r[7];    // C(v):   rows v-3..v+3
                const float cp1 = (s5 + r[7]) + r[8];   // C(v+1): rows v-2..v+4
                float V = 2.0f * c0;
                if constexpr (decltype(both)::value) {
                    V += cm1;
                    V += cp1;
                } else {
                    V += up ? cm1 : 0.0f;
                    V += dn ? cp1 : 0.0f;
                }
                Vp(par)[u + 2] = V;
            }
        };
        if (up && dn) vcol(std::bool_constant<true>{}); else vcol(std::bool_constant<false>{});
        // row v - 5 (v = v_max - (5 - S) modulo 9, and PD divides 9)
        scatter(IntC<(10 - S) % PD>{}, v - 5, qb(par ^ 1));
        prefetch(IntC<(10 - S) % PD>{}, v - 5 - PD);
        __syncthreads();
        float* mrow = mb(par);
        const float* vr = Vp(par);
        // the three-column sums (the one over columns u-2 .. u, M_0 at u-1, is the one over
        // u .. u+2, M_0 at u+1, of the column two to the left: shared by consecutive columns)
        float g1[NC], g2[NC];
        if constexpr (kConsec) {
            float vv[NC + 4], T3[NC + 2];
#pragma unroll
            for (int j = 0; j < NC + 4; ++j) vv[j] = vr[t * NC + j];
#pragma unroll
            for (int j = 0; j < NC + 2; ++j) T3[j] = (vv[j] + vv[j + 1]) + vv[j + 2];
#pragma unroll
            for (int k = 0; k < NC; ++k) { g1[k] = T3[k + 2]; g2[k] = T3[k]; }
        } else {
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                const int u = col(k);
                g1[k] = (vr[u + 2] + vr[u + 3]) + vr[u + 4];
                g2[k] = (vr[u] + vr[u + 1]) + vr[u + 2];
            }
        }
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const int u = col(k);
            float m1 = g1[k] - g2[k];
            // the columns at the image edges and past it (a few lanes of a few waves)
            if (u < 1 || u >= W - 1) m1 = u < W ? (u + 1 <= W - 1 ? g1[k] : 0.0f) - (u >= 1 ? g2[k] : 0.0f) : 0.0f;
            mrow[u] = m1;
        }
        if (v < v_max) candidates(mb(par ^ 1));   // row v + 1
        coef(v);                       // for this row's candidates in the next step
        --v;
        return true;
    };
    while (step(IntC<5>{}) && step(IntC<4>{}) && step(IntC<3>{}) && step(IntC<2>{}) && step(IntC<1>{}) &&
           step(IntC<0>{}) && step(IntC<8>{}) && step(IntC<7>{}) && step(IntC<6>{})) {
    }
    if (v_end <= v_max) {
        __syncthreads();
        candidates(mb(v_end & 1));
    }
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        const int i = t + k * BT;
        if (i < W2) {
            Eout[i] = ee[k];
            if (energy_out) energy_out[(int64_t)b * W2 + i] = (float)ee[k];
        }
    }
}

// The same energies by two launches, for few frames (energy_form): k_m1 forms M_1 of every
// track row (in the q buffer, which is a frame's size), k_tracks follows the tracks, a candidate
// a thread.  Every sum is taken in the order of k_energy, so the energies are the same bits.
// Neither has a chain over the rows with a barrier a row: 1242 x 375, one frame, 187 us by
// k_energy, 4 + 15 us by these two.
//
// k_m1: a workgroup takes kM1Rows rows of M_1 and kM1Waves x kM1Cols columns.  The edges on
// those rows and four more either side are listed (a row has few in these columns, so q formed
// row by row would run mostly empty waves), their q scattered into a dense LDS tile; then each
// wave takes 64 columns (two of halo either side) down the tile with its rows of q in registers,
// the neighbours' V by wave shifts, so no V is stored.  A wave without an edge in its columns
// writes zeros.  Bound by its loads' latency (info, then edges; five workgroups a CU by LDS) and
// the M_1 write: 256 frames 0.27 GB in 128 us.
constexpr int kM1Rows = 16, kM1Cols = 60, kM1Waves = 4;
constexpr int kM1Halo = 4;                                   // rows of q above and below
constexpr int kM1List = 1024;                                // listed edges of a tile
constexpr int kM1Span = kM1Waves * kM1Cols + 4;              // columns of the LDS tile

__device__ __forceinline__ float wave_next0(float x) {       // lane l + 1's x, 0 on lane 63
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x130, 0xF, 0xF, true));
}
__device__ __forceinline__ float wave_prev0(float x) {       // lane l - 1's x, 0 on lane 0
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x138, 0xF, 0xF, true));
}

__global__ __launch_bounds__(kM1Waves * kWave) void k_m1(Dev d) {
    constexpr int kTileRows = kM1Rows + 2 * kM1Halo, kT = kM1Waves * kWave;
    __shared__ __attribute__((aligned(16))) float q[kTileRows][kM1Span];
    __shared__ uint2 list[kM1List];
    __shared__ double sv[kTileRows][2];
    __shared__ int act[kM1Waves], s_n;
    const int b = blockIdx.z, t = threadIdx.x, lane = lane_id(), wave = t / kWave;
    if (frame_masked(d, b)) return;
    const FrameInfo fi = d.info[b];
    if (fi.flags & (LD_FLAG_NOROAD | LD_FLAG_NOVP)) return;
    const int W = d.W, H = d.H, v_max = H - 1, v_h = fi.v_h;
    const int v0 = fi.v_end + blockIdx.y * kM1Rows, u0 = blockIdx.x * (kM1Waves * kM1Cols) - 2;
    if (v0 > v_max) return;
    // the wave's rows of the tile: the counts and the first 64 edges of each in flight at once
    constexpr int kPer = (kTileRows + kM1Waves - 1) / kM1Waves;
    const ld_edge* edges = d.edges + (int64_t)b * H * W;
    int cnt[kPer];
    uint2 e0[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int r = v0 - kM1Halo + wave + j * kM1Waves, rc = min(max(r, 0), v_max);
        cnt[j] = d.rowcnt[(int64_t)b * H + rc];
        e0[j] = reinterpret_cast<const uint2*>(edges + (int64_t)rc * W)[min(lane, W - 1)];
        if (r != rc || r < v_h || wave + j * kM1Waves >= kTileRows) cnt[j] = 0;
    }
    static_assert(kTileRows * kM1Span % 4 == 0, "the tile is cleared by 16-byte stores");
    for (int i = t; i < kTileRows * kM1Span / 4; i += kT) reinterpret_cast<float4*>(&q[0][0])[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (t < kM1Waves) act[t] = 0;
    if (t == 0) s_n = 0;
    if (t < kTileRows) {
        const double* tv = d.tab + (int64_t)b * 6 * H + 2 * H + min(max(v0 - kM1Halo + t, 0), v_max);
        sv[t][0] = tv[H];      // V_px
        sv[t][1] = tv[0];      // V_py
    }
    __syncthreads();
    const float inv_sg2 = (float)(1.0 / (d.P.sigma_g * d.P.sigma_g));
    const int sq = d.P.vote ? 2 : d.P.weight_squared;
    auto place = [&](uint2 w, int row) {
        ld_edge e;
        e.u = (int16_t)(w.x & 0xFFFFu);
        e.gx = (int16_t)(w.x >> 16);
        e.gy = (int16_t)(w.y & 0xFFFFu);
        e.bin = 0;
        const int x = e.u - u0;
        q[row][x] = edge_q(e, v0 - kM1Halo + row, sv[row][0], sv[row][1], inv_sg2, sq);
        const int k = x / kM1Cols;                            // columns 60 k .. 60 k + 63 belong to wave k
        if (k < kM1Waves) act[k] = 1;
        if (x % kM1Cols < 4 && k > 0) act[k - 1] = 1;
    };
    // the tile's edges are listed first, so that q is formed by full waves (a row holds few of
    // this tile's columns); the edges past the list's end are placed at once
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int row = wave + j * kM1Waves;
        for (int i0 = 0; i0 < cnt[j]; i0 += kWave) {
            uint2 e = e0[j];
            if (i0 > 0) e = reinterpret_cast<const uint2*>(edges + (int64_t)(v0 - kM1Halo + row) * W)[min(i0 + lane, W - 1)];
            const int x = (int)(int16_t)(e.x & 0xFFFFu) - u0;
            const bool on = i0 + lane < cnt[j] && (unsigned)x < (unsigned)kM1Span;
            const uint64_t m = __ballot(on);
            if (m != 0) {
                int base = 0;
                if (lane == 0) base = atomicAdd(&s_n, __popcll(m));
                const int slot = __builtin_amdgcn_readfirstlane(base) + __popcll(m & lanes_below());
                e.y = (e.y & 0xFFFFu) | ((uint32_t)row << 16);
                if (on && slot < kM1List) list[slot] = e;
                else if (on) place(e, row);
            }
        }
    }
    __syncthreads();
    const int n = min(s_n, kM1List);
    for (int i = t; i < n; i += kT) {
        const uint2 e = list[i];
        place(e, (int)(e.y >> 16));
    }
    __syncthreads();
    const int u = u0 + wave * kM1Cols + lane;                 // lanes 2 .. 61 write their column
    const bool mine = lane >= 2 && lane < 2 + kM1Cols && u < W;
    float* out = d.qbuf + (int64_t)b * H * W + u;
    const int rows = min(kM1Rows, v_max - v0 + 1);
    if (!act[wave]) {
        if (mine)
            for (int i = 0; i < rows; ++i) out[(int64_t)(v0 + i) * W] = 0.0f;
        return;
    }
    float r[kTileRows];
#pragma unroll
    for (int j = 0; j < kTileRows; ++j) r[j] = q[j][wave * kM1Cols + lane];
#pragma unroll
    for (int i = 0; i < kM1Rows; ++i) {
        const int v = v0 + i;
        if (v > v_max) break;
        const float s5 = (((r[i + 2] + r[i + 3]) + r[i + 4]) + r[i + 5]) + r[i + 6];
        const float cm1 = (r[i] + r[i + 1]) + s5;
        const float c0 = (r[i + 1] + s5) + r[i + 7];
        const float cp1 = (s5 + r[i + 7]) + r[i + 8];
        float V = 2.0f * c0;
        V += v >= 1 ? cm1 : 0.0f;
        V += v + 1 <= v_max ? cp1 : 0.0f;
        const float n1 = wave_next0(V), g1 = (V + n1) + wave_next0(n1);   // V(u) + V(u+1) + V(u+2)
        const float g2 = wave_prev0(wave_prev0(g1));                       // V(u-2) + V(u-1) + V(u)
        float m1 = g1 - g2;
        if (u < 1 || u >= W - 1) m1 = (u + 1 <= W - 1 ? g1 : 0.0f) - (u >= 1 ? g2 : 0.0f);
        if (mine) out[(int64_t)v * W] = m1;
    }
}

// k_tracks: one candidate a thread, one wave a workgroup (a frame spreads over 2W / 64 of them).
// The columns of kTrackRows rows are found first, then their M_1 loads are issued together and
// added in row order, the next rows' columns and loads going on meanwhile.  A row is read through
// a buffer resource that ends with it, so a column outside the image reads 0.  Issue bound with
// many frames (1024: 245 us, about ten operations a row and candidate), with few by the chain of
// 13 groups of loads (one frame 15 us).
constexpr int kTrackRows = 16;

__global__ __launch_bounds__(kWave) void k_tracks(Dev d, const uint8_t* cand_mask, float* energy_out) {
    const int b = blockIdx.y, i = blockIdx.x * kWave + threadIdx.x;
    if (frame_masked(d, b)) return;
    const int W = d.W, H = d.H, W2 = d.W2, v_max = H - 1;
    const FrameInfo fi = d.info[b];
    const bool in = i < W2;
    const bool live = in && (cand_mask == nullptr || cand_mask[(int64_t)b * W2 + i] != 0);
    double ee = 0.0;
    if (!(fi.flags & (LD_FLAG_NOROAD | LD_FLAG_NOVP)) && __any(live)) {
        const int v_end = __builtin_amdgcn_readfirstlane(fi.v_end);
        const double* __restrict__ tA = d.tab + (int64_t)b * 6 * H + 4 * H;
        const double* __restrict__ tB = tA + H;
        float* base = d.qbuf + (int64_t)b * H * W;
        double uu = (double)(i - d.half);
        // rows top .. top - kTrackRows + 1; with tail set some of them lie below v_end or all do:
        // nothing is read there and 0 is added
        auto fetch = [&](auto tail, int top, float (&m)[kTrackRows]) {
            constexpr bool kTail = decltype(tail)::value;
            double A[kTrackRows], B[kTrackRows];
#pragma unroll
            for (int j = 0; j < kTrackRows; ++j) {
                const int v = kTail ? max(top - j, 0) : top - j;
                A[j] = tA[v];
                B[j] = tB[v];
            }
#pragma unroll
            for (int j = 0; j < kTrackRows; ++j) {
                const int v = top - j, row = (kTail ? max(v, v_end) : v) * W;
                uu = fma(B[j], uu, A[j]);
                const unsigned c = min((unsigned)(int)floor(uu + 0.5), (unsigned)W);
                const __amdgpu_buffer_rsrc_t rs =
                    __builtin_amdgcn_make_buffer_rsrc(base, 0, !kTail || v >= v_end ? (row + W) * 4 : 0, 0x00020000);
                m[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)(c * 4u), row * 4, 0));
            }
        };
        auto fetch_at = [&](int top, float (&m)[kTrackRows]) {
            if (top - kTrackRows + 1 >= v_end) fetch(std::false_type{}, top, m);
            else fetch(std::true_type{}, top, m);
        };
        auto add = [&](const float (&m)[kTrackRows]) {
#pragma unroll
            for (int j = 0; j < kTrackRows; ++j) ee += (double)m[j];
        };
        // row v_max: the start column itself
        {
            const int c = i - d.half;
            ee = (unsigned)c < (unsigned)W ? (double)base[v_max * W + c] : 0.0;
        }
        float ma[kTrackRows], mb[kTrackRows];
        fetch_at(v_max - 1, ma);
        for (int v = v_max - 1; v >= v_end; v -= 2 * kTrackRows) {
            fetch_at(v - kTrackRows, mb);
            add(ma);
            fetch_at(v - 2 * kTrackRows, ma);
            add(mb);
        }
    }
    if (in) {
        if (!live) ee = 0.0;
        d.energy[(int64_t)b * W2 + i] = ee;
        if (energy_out) energy_out[(int64_t)b * W2 + i] = (float)ee;
    }
}

// ------------------------------------------------------------------------------------------
// S13: strict local minima of the energies, below rho * (deepest energy); greedy suppression
// of minima within d_nms of a deeper accepted one; lane curves by iterating the track.
constexpr int kCurveRows = 256, kCurveStride = kCurveRows + 1;
constexpr size_t kCurveLds = kCurveRows * 16 + sizeof(float) * LD_MAX_LANES * kCurveStride;

__global__ __launch_bounds__(kBlock) void k_peaks(Dev d, ld_lanes* lanes_out, float* curves_out) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int64_t rv[kMaxWaves];
    __shared__ int ri[kMaxWaves];
    __shared__ double dred[kMaxWaves];
    __shared__ int acc[LD_MAX_LANES];
    __shared__ int s_nacc;
    const int b = blockIdx.x, t = threadIdx.x;
    if (frame_masked(d, b)) return;
    const int W2 = d.W2, H = d.H, v_max = H - 1;
    const FrameInfo fi = d.info[b];
    const double* E = d.energy + (int64_t)b * W2;
    uint8_t* alive = smem;   // W2
    const double* tA = d.tab + (int64_t)b * 6 * H + 4 * H;
    const double* tB = tA + H;
    double mn = INFINITY;
    for (int i = t; i < W2; i += kBlock) mn = fmin(mn, E[i]);
    for (int o = 32; o > 0; o >>= 1) mn = fmin(mn, __shfl_xor(mn, o, kWave));
    if (lane_id() == 0) dred[t / kWave] = mn;
    __syncthreads();
    mn = dred[0];
    for (int w = 1; w < nwaves(); ++w) mn = fmin(mn, dred[w]);
    const bool any = !(fi.flags & (LD_FLAG_NOROAD | LD_FLAG_NOVP)) && mn < 0.0;
    const double thr = d.P.rho_lpv * mn;
    for (int i = t; i < W2; i += kBlock) {
        bool a = any && i >= 1 && i + 1 < W2 && E[i] < E[i - 1] && E[i] < E[i + 1] && E[i] < thr;
        alive[i] = a ? 1 : 0;
    }
    if (t == 0) s_nacc = 0;
    __syncthreads();
    const int dn = d.P.d_nms > 0 ? d.P.d_nms : max(8, d.W / 64);
    for (int it = 0; it < LD_MAX_LANES; ++it) {
        // argmin over the alive minima by (E, i); E is compared through its order-preserving
        // 64-bit image so that ties fall to the smaller index
        int64_t key = INT64_MAX;
        int idx = 0x7fffffff;
        for (int i = t; i < W2; i += kBlock)
            if (alive[i]) {
                const int64_t bits = __double_as_longlong(E[i]);
                const int64_t k = bits >= 0 ? bits : (bits ^ 0x7fffffffffffffffLL);
                if (k < key || (k == key && i < idx)) { key = k; idx = i; }
            }
        block_argmin_i64(key, idx, rv, ri);
        if (idx == 0x7fffffff) break;
        if (t == 0) acc[s_nacc++] = idx;
        for (int i = t; i < W2; i += kBlock)
            if (alive[i] && abs(i - idx) <= dn) alive[i] = 0;
        __syncthreads();
    }
    __syncthreads();
    const int n = s_nacc;
    if (t == 0) {
        for (int i = 1; i < n; ++i) {
            int x = acc[i], j = i - 1;
            while (j >= 0 && acc[j] > x) { acc[j + 1] = acc[j]; --j; }
            acc[j + 1] = x;
        }
        ld_lanes L;
        L.n = n;
        L.flags = fi.flags;
        L.v_h = fi.v_h;
        L.v_end = fi.v_end;
        for (int l = 0; l < LD_MAX_LANES; ++l) {
            L.u_start[l] = l < n ? acc[l] - d.half : 0;
            L.energy[l] = l < n ? (float)E[acc[l]] : 0.0f;
        }
        lanes_out[b] = L;
    }
    __syncthreads();
    if (curves_out) {
        float* cv = curves_out + (int64_t)b * LD_MAX_LANES * H;
        const float fnan = __int_as_float(0x7fc00000);
        // A curve is a chain of one fma a row, a lane each.  The rows' coefficients are staged in LDS and the
        // columns leave through it, kCurveRows rows at a time, so that the chain waits for LDS only
        // (loads and stores of memory in it took k_peaks 107 us for a 1920 x 1080 frame; now 40).
        double2* ab = reinterpret_cast<double2*>(smem);
        float* cu = reinterpret_cast<float*>(ab + kCurveRows);          // [lane][row]
        double u = t < n ? (double)(acc[t] - d.half) : 0.0;
        for (int v1 = v_max; v1 >= 0; v1 -= kCurveRows) {               // rows v1 and up to kCurveRows - 1 above
            const int rows = min(kCurveRows, v1 + 1), swept = min(rows, max(v1 - fi.v_end + 1, 0));
            for (int i = t; i < swept; i += kBlock)
                ab[i] = v1 - i < v_max ? make_double2(tA[v1 - i], tB[v1 - i]) : make_double2(0.0, 1.0);
            __syncthreads();
            if (t < n) {
                int i = 0;
                for (; i + 8 <= swept; i += 8) {
                    double2 c[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) c[k] = ab[i + k];
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        u = fma(c[k].y, u, c[k].x);
                        cu[t * kCurveStride + i + k] = (float)u;
                    }
                }
                for (; i < swept; ++i) {
                    u = fma(ab[i].y, u, ab[i].x);
                    cu[t * kCurveStride + i] = (float)u;
                }
            }
            __syncthreads();
            for (int i = t; i < LD_MAX_LANES * rows; i += kBlock) {
                const int l = i / rows, r = rows - 1 - (i - l * rows);  // (upwards in memory)
                cv[(int64_t)l * H + v1 - r] = l < n && r < swept ? cu[l * kCurveStride + r] : fnan;
            }
            __syncthreads();
        }
    }
}

// ------------------------------------------------------------------------------------------
// Pruned search (learned part, not in the paper).  The network's decisions on a few bands of
// road rows (lbits) select the edges that lie on lane markings; their V_px vote columns give a
// seed for the V_px path, the DP then runs inside a window around the seed, and the tracks of
// the candidates through the bands decide which candidates are scored.  Any sign that the
// narrowed search may differ from the full one sends the frame back to the full search.
__device__ __forceinline__ int band_top(const Dev& d, int v_h, int nb, int k) { return ldi_band_top(v_h, d.H, nb, k); }

// Seed: per-band histograms of the vote columns of marking edges; pooled argmax c_s; window;
// RANSAC hypothesis 0 (line through the lowest and the highest band estimates).  One workgroup
// per frame; LDS 2 x 2W ints.
__global__ __launch_bounds__(kBlock) void k_seed(Dev d, int nb, int delta, int min_votes, int seed_ransac) {
    extern __shared__ int hs[];
    __shared__ int64_t rv[kMaxWaves];
    __shared__ int ri[kMaxWaves];
    __shared__ int red[kMaxWaves];
    const int b = blockIdx.x, t = threadIdx.x;
    if (frame_masked(d, b)) return;
    const int W = d.W, W2 = d.W2, H = d.H;
    const FrameInfo fi = d.info[b];
    int32_t* pr = d.prune + (int64_t)b * kPruneWords;
    double* sg = d.seedg + (int64_t)b * 5;
    int* hb = hs;          // band histogram
    int* hp = hs + W2;     // pooled histogram
    for (int i = t; i < 2 * W2; i += kBlock) hs[i] = 0;
    int est[LDI_MAX_BANDS], cnt[LDI_MAX_BANDS];
    for (int k = 0; k < LDI_MAX_BANDS; ++k) { est[k] = -1; cnt[k] = 0; }
    const bool road = !(fi.flags & LD_FLAG_NOROAD);
    const ld_edge* fe = d.edges + (int64_t)b * H * W;
    const uint8_t* lb = d.lbits + (int64_t)b * LDI_MAX_BANDS * LDI_BAND_ROWS * W;
    __syncthreads();
    for (int k = 0; k < nb && road; ++k) {
        const int top = band_top(d, fi.v_h, nb, k);
        if (top < 0) break;
        for (int r = 0; r < LDI_BAND_ROWS; ++r) {
            const int v = top + r, n = d.rowcnt[(int64_t)b * H + v];
            for (int i = t; i < n; i += kBlock) {
                const ld_edge e = fe[(int64_t)v * W + i];
                if (e.bin >= 0 && lb[(k * LDI_BAND_ROWS + r) * W + e.u]) {
                    atomicAdd(&hb[e.bin], 1);
                    atomicAdd(&hp[e.bin], 1);
                }
            }
        }
        __syncthreads();
        int64_t key = INT64_MAX;
        int bi = 0x7fffffff, tot = 0;
        for (int c = t; c < W2; c += kBlock) {
            const int h = hb[c];
            tot += h;
            if (h > 0 && -(int64_t)h < key) { key = -(int64_t)h; bi = c; }
            hb[c] = 0;
        }
        tot = block_sum_i32(tot, red);
        block_argmin_i64(key, bi, rv, ri);
        est[k] = tot > 0 ? bi : -1;
        cnt[k] = tot;
    }
    int64_t key = INT64_MAX;
    int bi = 0x7fffffff, tot = 0;
    for (int c = t; c < W2; c += kBlock) {
        const int h = hp[c];
        tot += h;
        if (h > 0 && -(int64_t)h < key) { key = -(int64_t)h; bi = c; }
    }
    tot = block_sum_i32(tot, red);
    block_argmin_i64(key, bi, rv, ri);
    if (t == 0) {
        int fb = 0, cs = -1, lo = 0, hi = -1;
        if (!road || tot < min_votes) {
            fb = kFbPlainVpx | kFbNoSeed;
        } else {
            cs = bi;
            lo = max(0, cs - delta);
            hi = min(W2 - 1, cs + delta);
            if (W < 128) fb = kFbPlainVpx | kFbNoSeed;   // the window backtrace needs 128 B per row
        }
        // hypothesis 0: line through the lowest and the highest band with min_votes votes
        int klo = -1, khi = -1;
        for (int k = 0; k < nb; ++k)
            if (cnt[k] >= min_votes) { if (klo < 0) klo = k; khi = k; }
        for (int p = 0; p < 5; ++p) sg[p] = 0.0;
        if (cs >= 0 && seed_ransac) {
            if (klo >= 0 && khi != klo) {
                const double v0 = (double)(band_top(d, fi.v_h, nb, klo) + 8), v1 = (double)(band_top(d, fi.v_h, nb, khi) + 8);
                const double u0 = (double)(est[klo] - d.half), u1 = (double)(est[khi] - d.half);
                const double g1 = (u1 - u0) / (v1 - v0);
                sg[1] = g1;
                sg[0] = u0 - g1 * v0;
            } else {
                sg[0] = (double)((klo >= 0 ? est[klo] : cs) - d.half);
            }
        } else {
            sg[0] = __longlong_as_double(0x7ff8000000000000LL);   // no seed
        }
        pr[0] = nb; pr[1] = fb; pr[2] = cs; pr[3] = lo; pr[4] = hi; pr[5] = tot;
        for (int k = 0; k < 4; ++k) { pr[6 + k] = est[k]; pr[10 + k] = cnt[k]; }
        pr[14] = 0; pr[15] = 0;
    }
}

// Windowed V_px search: band accumulator and row DP on columns lo..hi only (transitions
// leaving the window are not allowed), the same tie order as the full DP, backtrace, a check
// that the path never reaches an inner edge of the window.  One wave per frame: lane l keeps
// window columns 4l .. 4l+3 (16 E of the previous row and the column counts) in registers and
// takes the neighbours' values from lanes l-2 .. l+2 by DPP wave shifts, so a row needs no
// barrier; the band deltas of a row go through LDS atomics, from the road rows' vote columns
// staged in LDS before the sweep; the backtrace (the rank of tau, 4 bits per column,
// 128 B per row) goes to the frame's backtrace buffer and is walked 32 rows at a time from
// registers.  Needs W >= 128 (the buffer holds W bytes per row); narrower frames use the full
// search.
constexpr int kWalkChunk = 32;

__device__ __forceinline__ int shfl_i(int x, int src) { return __shfl(x, src, kWave); }
__device__ __forceinline__ int min3_i(int a, int b, int c) { return min(min(a, b), c); }
// x of lane l - 1 (kBig on lane 0) and of lane l + 1 (kBig on lane 63): DPP wave shifts by one
__device__ __forceinline__ int lane_prev(int x) { return __builtin_amdgcn_update_dpp(kBig, x, 0x138, 0xF, 0xF, false); }
__device__ __forceinline__ int lane_next(int x) { return __builtin_amdgcn_update_dpp(kBig, x, 0x130, 0xF, 0xF, false); }
// the same shifts filling with 0 (lane 0, lane 63)
__device__ __forceinline__ int lane_prev0(int x) { return __builtin_amdgcn_update_dpp(0, x, 0x138, 0xF, 0xF, true); }
__device__ __forceinline__ int lane_next0(int x) { return __builtin_amdgcn_update_dpp(0, x, 0x130, 0xF, 0xF, true); }
constexpr int kBig16 = 0x3FFFFFF0;

__global__ __launch_bounds__(256) void k_vpx_window(Dev d, int stage_cap, int wave_bytes, int nframes) {
    extern __shared__ unsigned char smem_all[];
    // blockDim.x / 64 frames per workgroup, one per wave with its own LDS slice: the waves of
    // a workgroup go to different SIMDs, so a batch of four frames per CU runs one wave per SIMD
    // the frame's values are wave-uniform: kept in scalar registers, so every loop below
    // branches on scalars
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int b = (int)blockIdx.x * (int)(blockDim.x / kWave) + wv, l = lane_id();
    if (b >= nframes || frame_masked(d, b)) return;
    unsigned char* smem = smem_all + (size_t)wv * wave_bytes;
    int32_t* pr = d.prune + (int64_t)b * kPruneWords;
    if (__builtin_amdgcn_readfirstlane(pr[1]) & kFbPlainVpx) return;
    const int H = d.H, W2 = d.W2, v_max = H - 1;
    FrameInfo fi = d.info[b];
    for (int v = l; v < H; v += kWave) d.mxpath[(int64_t)b * H + v] = -1;
    const int v_h = __builtin_amdgcn_readfirstlane(fi.v_h), chi = d.P.chi, R = v_max - v_h + 1;
    const int lo = __builtin_amdgcn_readfirstlane(pr[3]), hi = __builtin_amdgcn_readfirstlane(pr[4]);
    const int win = hi - lo + 1;
    int* dlt = reinterpret_cast<int*>(smem);                 // 256 band deltas of a row + 64 lane sinks
    int* cntL = dlt + 256 + kWave;                            // H
    int* path = cntL + H;                                     // H + 1 (the last: touch flag)
    int* roff = path + H + 1;                                 // R + 1 <= H + 1
    uint8_t* wb = reinterpret_cast<uint8_t*>(roff + H + 1);               // stage_cap bytes
    uint16_t* back = reinterpret_cast<uint16_t*>(d.back_x) + (int64_t)b * H * ((W2 + kDpRun - 1) / kDpRun) * 2;
    const ld_edge* fe = d.edges + (int64_t)b * H * d.W;
    // the road rows' edge counts (the search reads no other row), eight loads per lane in
    // flight before the first is stored
    for (int base = 0; base < R; base += 8 * kWave) {
        int cn[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) cn[k] = d.rowcnt[(int64_t)b * H + v_h + min(base + k * kWave + l, R - 1)];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (base + k * kWave + l < R) cntL[v_h + base + k * kWave + l] = cn[k];
    }
    for (int i = l; i < 256; i += kWave) dlt[i] = 0;
    {   // exclusive prefix of the road rows' edge counts, 64 rows per wave scan
        int carry = 0;
        for (int base = 0; base < R; base += kWave) {
            const int own = base + l < R ? cntL[v_h + base + l] : 0;
            int x = own;
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const int y = __shfl_up(x, o, kWave);
                if (l >= o) x += y;
            }
            if (base + l < R) roff[base + l] = carry + x - own;
            carry += __shfl(x, kWave - 1, kWave);
        }
        if (l == 0) roff[R] = carry;
    }
    const int ne = __builtin_amdgcn_readfirstlane(roff[R]);
    // window offset of every road edge's vote column (255: outside the window or no vote),
    // loaded eight rows at a time with every load of the group in flight
    const bool staged = ne <= stage_cap;
    auto woff = [&](int c) -> uint8_t { return (c >= lo && c <= hi) ? (uint8_t)(c - lo) : (uint8_t)255; };
    int nv = 0;
    if (staged) {
        // Groups of 16 rows, two in flight while a third is written to LDS: lane l loads the
        // vote columns of entries l and l + 64 of every row of a group (the window search needs
        // W >= 128, so both lie in the row's slots; entries past the row's count and rows past
        // v_max, read as row v_max, are loaded and not used).  The two register sets are
        // written in turn, so no copy waits on loads in flight.  Lane l holds the count and
        // offset (offset << 16 | count) of row v_h + 64 m + l of the current 64-row chunk m.
        uint8_t* junk = reinterpret_cast<uint8_t*>(dlt + 256 + l);   // stores of lanes without an entry
        const int ng = (R + 15) / 16;
        auto load_group = [&](int g, int (&c)[16][2]) {
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const ld_edge* row = fe + (int64_t)min(v_h + 16 * g + k, v_max) * d.W;
                c[k][0] = row[l].bin;
                c[k][1] = row[l + kWave].bin;
            }
        };
        int desc = 0;
        auto store_group = [&](int g, const int (&c)[16][2]) {
            if ((g & 3) == 0) {
                const int r = 16 * g + l;
                desc = r < R ? (roff[r] << 16 | cntL[v_h + r]) : 0;
            }
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int r = 16 * g + k;
                if (r >= R) break;
                const int rd = __builtin_amdgcn_readlane(desc, r & 63);
                const int n = rd & 0xFFFF, o = rd >> 16;
                const bool e0 = l < n, e1 = l + kWave < n;
                nv += (e0 && c[k][0] >= 0 ? 1 : 0) + (e1 && c[k][1] >= 0 ? 1 : 0);
                *(e0 ? wb + o + l : junk) = woff(c[k][0]);
                *(e1 ? wb + o + l + kWave : junk) = woff(c[k][1]);
                if (n > 2 * kWave) {                 // long rows: 8 loads in flight
                    const int v = v_h + r;
                    for (int i0 = l + 2 * kWave; i0 < n; i0 += 8 * kWave) {
                        int cc[8];
#pragma unroll
                        for (int j = 0; j < 8; ++j) {
                            const int i = i0 + j * kWave;
                            cc[j] = i < n ? fe[(int64_t)v * d.W + i].bin : -1;
                        }
#pragma unroll
                        for (int j = 0; j < 8; ++j) {
                            const int i = i0 + j * kWave;
                            if (i < n) {
                                nv += cc[j] >= 0 ? 1 : 0;
                                wb[o + i] = woff(cc[j]);
                            }
                        }
                    }
                }
            }
        };
        int ca[16][2], cb[16][2];
        load_group(0, ca);
        load_group(1, cb);
        for (int g = 0; g < ng; g += 2) {
            store_group(g, ca);
            load_group(g + 2, ca);
            if (g + 1 < ng) store_group(g + 1, cb);
            load_group(g + 3, cb);
        }
    } else {
        for (int v = v_h; v <= v_max; ++v)
            for (int i = l; i < cntL[v]; i += kWave) nv += fe[(int64_t)v * d.W + i].bin >= 0 ? 1 : 0;
    }
    // band rows entering (sign +1) or leaving (-1) the accumulator
    auto apply = [&](int r, int sign) {
        const int n = cntL[r];
        const int o = staged ? roff[r - v_h] : 0;
        for (int base = 0; base < n; base += kWave) {
            const int i = base + l;
            int key = -1;
            if (i < n) {
                if (staged) {
                    const int c = wb[o + i];
                    key = c != 255 ? c : -1;
                } else {
                    const int c = fe[(int64_t)r * d.W + i].bin;
                    key = (c >= lo && c <= hi) ? c - lo : -1;
                }
            }
            if (key >= 0) atomicAdd(&dlt[key], sign);
        }
    };
    for (int r = max(v_max - chi, v_h); r <= v_max; ++r) apply(r, 16);
    // S = 16 E of the own columns (kBig16 outside the window), H = 16 x the column's band count
    // (the deltas are applied in units of 16); the registers hold S - kBig16, so the columns
    // outside the window and beyond the wave's ends are 0 and the wave shifts fill with 0.
    // kBig16 is a multiple of 16, so the rank bits and the update below are unchanged by the
    // offset, and it exceeds every reachable |16 E|.  A candidate from column c + tau costs
    // S(c + tau) + slope |tau| - [tau < 0] with slope = 16 lambda + 2, i.e. 16 (E + lambda |tau|)
    // plus the rank of tau in the tie order 0, -1, +1, -2, +2, ..., so one min picks the cost
    // and the tie; offsets are taken relative to the lane's first column 4l.
    int Hc[4], S[4];
    bool inw[4];
    {
        const int4 q = *reinterpret_cast<const int4*>(dlt + 4 * l);
        Hc[0] = q.x; Hc[1] = q.y; Hc[2] = q.z; Hc[3] = q.w;
        *reinterpret_cast<int4*>(dlt + 4 * l) = make_int4(0, 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        inw[j] = 4 * l + j < win;
        S[j] = inw[j] ? -Hc[j] - kBig16 : 0;
    }
    const int tau_max = d.P.tau_x_max, slope = 16 * d.P.lambda_x + 2;
    // one row of the DP from the previous row's S and this row's H (returns the 4-bit ranks)
    auto dp_row = [&]() -> uint32_t {
        // w[p] = S of column 4l - 5 + p of the previous row (p = 0 .. 13)
        int w[14];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            w[1 + j] = lane_prev0(S[j]);
            w[5 + j] = S[j];
            w[9 + j] = lane_next0(S[j]);
        }
        w[0] = lane_prev0(w[4]);
        w[13] = lane_next0(w[9]);
        int lm[4], rm[4];
        if (tau_max == 5) {
            // TL[p] = w[p] + slope (5 - p) for p = 0 .. 7 and TR[p] = w[p] + slope (p - 5) for
            // p = 6 .. 13; the minima over five consecutive entries share their middle terms
            int TL[8], TR[8];
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                TL[p] = w[p] + slope * (5 - p);
                TR[p] = w[p + 6] + slope * (p + 1);
            }
            const int cl = min3_i(TL[2], TL[3], TL[4]);
            lm[0] = min3_i(TL[0], TL[1], cl);
            lm[1] = min3_i(TL[1], cl, TL[5]);
            lm[2] = min3_i(cl, TL[5], TL[6]);
            lm[3] = min3_i(TL[3], TL[4], min3_i(TL[5], TL[6], TL[7]));
            const int cr = min3_i(TR[2], TR[3], TR[4]);
            rm[0] = min3_i(TR[0], TR[1], cr);
            rm[1] = min3_i(TR[1], cr, TR[5]);
            rm[2] = min3_i(cr, TR[5], TR[6]);
            rm[3] = min3_i(TR[3], TR[4], min3_i(TR[5], TR[6], TR[7]));
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                lm[j] = 0; rm[j] = 0;
#pragma unroll
                for (int a = 1; a <= 5; ++a)
                    if (a <= tau_max) {
                        lm[j] = min(lm[j], w[j + 5 - a] + slope * (a - j));
                        rm[j] = min(rm[j], w[j + 5 + a] + slope * (a + j));
                    }
            }
        }
        uint32_t bits = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int key = min3_i(w[5 + j], lm[j] + (slope * j - 1), rm[j] - slope * j);
            S[j] = inw[j] ? (key & ~15) - Hc[j] : 0;
            bits |= (uint32_t)(key & 15) << (4 * j);
        }
        return bits;
    };
    auto take_deltas = [&]() {
        // the wave's LDS operations complete in order: the deltas are final here
        const int4 q = *reinterpret_cast<const int4*>(dlt + 4 * l);
        *reinterpret_cast<int4*>(dlt + 4 * l) = make_int4(0, 0, 0, 0);
        Hc[0] += q.x; Hc[1] += q.y; Hc[2] += q.z; Hc[3] += q.w;
    };
    if (staged) {
        // Row v (v = v_max - 1 - t) adds the votes of row v - chi and removes those of row
        // v + chi + 1.  Lane l holds the two lists' heads (offset << 16 | count) of row
        // t0 + l of the current 64-row chunk, taken by readlane; the own entries of the next
        // row's lists are read while the current row is computed.  Lanes without an entry
        // add to their own sink word.
        int* sink = dlt + 256 + l;
        auto heads = [&](int t0, int& hA, int& hR) {
            const int v = v_max - 1 - t0 - l, ra = v - chi, rr = v + chi + 1;
            hA = (v >= v_h && ra >= v_h) ? (roff[ra - v_h] << 16 | cntL[ra]) : 0;
            hR = (v >= v_h && rr <= v_max) ? (roff[rr - v_h] << 16 | cntL[rr]) : 0;
        };
        auto own_slot = [&](int hd) -> int* {
            const int n = hd & 0xFFFF, o = hd >> 16;
            const int c = wb[l < n ? o + l : 0];
            return (l < n && c != 255) ? dlt + c : sink;
        };
        int hA, hR;
        heads(0, hA, hR);
        int* pA = own_slot(__builtin_amdgcn_readlane(hA, 0));
        int* pR = own_slot(__builtin_amdgcn_readlane(hR, 0));
        for (int t = 0; t < R - 1; ++t) {
            const int v = v_max - 1 - t;
            const int cA = __builtin_amdgcn_readlane(hA, t & 63), cR = __builtin_amdgcn_readlane(hR, t & 63);
            atomicAdd(pA, 16);
            atomicAdd(pR, -16);
            const int nA = cA & 0xFFFF, nR = cR & 0xFFFF;
            for (int i0 = kWave; i0 < max(nA, nR); i0 += kWave) {     // long lists
                const int i = i0 + l;
                const int ca = i < nA ? wb[(cA >> 16) + i] : 255;
                const int cr = i < nR ? wb[(cR >> 16) + i] : 255;
                atomicAdd(ca != 255 ? dlt + ca : sink, 16);
                atomicAdd(cr != 255 ? dlt + cr : sink, -16);
            }
            if (((t + 1) & 63) == 0) heads(t + 1, hA, hR);
            pA = own_slot(__builtin_amdgcn_readlane(hA, (t + 1) & 63));
            pR = own_slot(__builtin_amdgcn_readlane(hR, (t + 1) & 63));
            take_deltas();
            back[(int64_t)(v - v_h) * kWave + l] = (uint16_t)dp_row();
        }
    } else {
        for (int v = v_max - 1; v >= v_h; --v) {
            if (v - chi >= v_h) apply(v - chi, 16);
            if (v + chi + 1 <= v_max) apply(v + chi + 1, -16);
            take_deltas();
            back[(int64_t)(v - v_h) * kWave + l] = (uint16_t)dp_row();
        }
    }
    // start column: argmin over the window of E at v_h, ties to the smaller column
    int64_t bv = INT64_MAX;
    int bc = 0x7fffffff;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (4 * l + j < win && (int64_t)(S[j] >> 4) < bv) { bv = S[j] >> 4; bc = 4 * l + j; }
    wave_argmin_i64(bv, bc);
    __threadfence_block();   // the backtrace stores are complete before the wave reads them back
    // Walk: the backtrace words of kWalkChunk rows in registers (lane l holds columns
    // 4l .. 4l+3 of each row) with the next chunk in flight; the column is wave-uniform, so a
    // step is a readlane and a few scalar operations.  Lane r keeps the path of row v0 + r.
    int c = __builtin_amdgcn_readfirstlane(bc), touch = 0;
    auto load_chunk = [&](int v0, uint32_t (&dst)[kWalkChunk]) {
#pragma unroll
        for (int r = 0; r < kWalkChunk; ++r) {
            const int v = min(v0 + r, v_max - 1);          // rows v < v_max hold an entry
            dst[r] = back[(int64_t)max(v - v_h, 0) * kWave + l];
        }
    };
    auto walk_chunk = [&](int v0, const uint32_t (&bk)[kWalkChunk]) {
        int pv = 0;
#pragma unroll
        for (int r = 0; r < kWalkChunk; ++r) {
            const int v = v0 + r;
            if (v <= v_max) {
                if (l == r) pv = lo + c;
                if (v < v_max) {
                    const uint32_t word = __builtin_amdgcn_readlane(bk[r], c >> 2);
                    const int rank = (int)((word >> (4 * (c & 3))) & 15u);
                    c += (int)((kRankTau >> (4 * rank)) & 15u) - 8;
                }
            }
        }
        if (l < kWalkChunk && v0 + l <= v_max) path[v0 + l] = pv;
    };
    // two chunks in flight, the register sets written in turn (row loads are clamped, so
    // every chunk is a full set of loads)
    uint32_t ba[kWalkChunk], bb[kWalkChunk];
    load_chunk(v_h, ba);
    load_chunk(v_h + kWalkChunk, bb);
    for (int v0 = v_h; v0 <= v_max; v0 += 2 * kWalkChunk) {
        walk_chunk(v0, ba);
        load_chunk(v0 + 2 * kWalkChunk, ba);
        if (v0 + kWalkChunk <= v_max) walk_chunk(v0 + kWalkChunk, bb);
        load_chunk(v0 + 3 * kWalkChunk, bb);
    }
    // the path touches an inner edge of the window (a column the window cut off could have
    // been reached): the frame goes back to the full search
    for (int v = v_h + l; v <= v_max; v += kWave) {
        const int pc = path[v];
        if ((lo > 0 && pc == lo) || (hi < W2 - 1 && pc == hi)) touch = 1;
    }
    touch = __any(touch) ? 1 : 0;
    nv = wave_sum_i32(nv);
    if (touch) {
        if (l == 0) pr[1] |= kFbPlainVpx | kFbTouch;
        return;
    }
    for (int v = v_h + l; v <= v_max; v += kWave) d.mxpath[(int64_t)b * H + v] = path[v];
    if (l == 0) {
        fi.n_edges = ne;
        fi.n_votes = nv;
        d.info[b] = fi;
    }
}

// Candidate mask: candidate i is kept when its track meets a marking pixel on a band row, then
// dilated.  Frames on the plain V_px search keep every candidate.  One workgroup per frame.
__global__ __launch_bounds__(kBlock) void k_cand_mask(Dev d, int nb, int dilate) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double ta[LDI_MAX_BANDS * LDI_BAND_ROWS], tb[LDI_MAX_BANDS * LDI_BAND_ROWS];
    __shared__ int red[kMaxWaves];
    const int b = blockIdx.x, t = threadIdx.x;
    if (frame_masked(d, b)) return;
    const int W = d.W, W2 = d.W2, H = d.H, v_max = H - 1;
    int32_t* pr = d.prune + (int64_t)b * kPruneWords;
    uint8_t* cm = d.cmask + (int64_t)b * W2;
    const FrameInfo fi = d.info[b];
    if ((pr[1] & kFbPlainVpx) || (fi.flags & (LD_FLAG_NOROAD | LD_FLAG_NOVP)) || dilate < 0) {
        for (int i = t; i < W2; i += kBlock) cm[i] = 1;
        if (t == 0) pr[14] = W2;
        return;
    }
    const int wpr = (W + 31) / 32;
    uint32_t* bits = reinterpret_cast<uint32_t*>(smem);            // nb x 16 x wpr
    uint8_t* hit = reinterpret_cast<uint8_t*>(bits + nb * LDI_BAND_ROWS * wpr);   // W2
    const uint8_t* lb = d.lbits + (int64_t)b * LDI_MAX_BANDS * LDI_BAND_ROWS * W;
    for (int w = t; w < nb * LDI_BAND_ROWS * wpr; w += kBlock) {
        const int row = w / wpr, c0 = (w % wpr) * 32;
        uint32_t x = 0;
        for (int j = 0; j < 32 && c0 + j < W; ++j) x |= (lb[row * W + c0 + j] ? 1u : 0u) << j;
        bits[w] = x;
    }
    const double* tA = d.tab + (int64_t)b * 6 * H + 4 * H;
    const double* tB = tA + H;
    const int v_end = fi.v_end;
    const int top_hi = band_top(d, fi.v_h, nb, nb - 1);
    if (t == 0) {
        double a = 1.0, c = 0.0;
        for (int v = v_max; v >= top_hi; --v) {
            if (v < v_max) {
                a = tB[v] * a;
                c = fma(tB[v], c, tA[v]);
            }
            for (int k = 0; k < nb; ++k) {
                const int r = v - band_top(d, fi.v_h, nb, k);
                if (r >= 0 && r < LDI_BAND_ROWS) { ta[k * LDI_BAND_ROWS + r] = a; tb[k * LDI_BAND_ROWS + r] = c; }
            }
        }
    }
    __syncthreads();
    for (int i = t; i < W2; i += kBlock) {
        const double us = (double)(i - d.half);
        uint8_t h = 0;
        for (int k = 0; k < nb && !h; ++k) {
            const int top = band_top(d, fi.v_h, nb, k);
            for (int r = 0; r < LDI_BAND_ROWS; ++r) {
                if (top + r < v_end) continue;
                const double x = fma(ta[k * LDI_BAND_ROWS + r], us, tb[k * LDI_BAND_ROWS + r]) + 0.5;
                if (x >= 0.0 && x < (double)W) {
                    const int col = (int)floor(x);
                    if ((bits[(k * LDI_BAND_ROWS + r) * wpr + (col >> 5)] >> (col & 31)) & 1u) { h = 1; break; }
                }
            }
        }
        hit[i] = h;
    }
    __syncthreads();
    int kept = 0;
    for (int i = t; i < W2; i += kBlock) {
        uint8_t k = 0;
        for (int j = max(0, i - dilate); j <= min(W2 - 1, i + dilate); ++j) k |= hit[j];
        cm[i] = k;
        kept += k;
    }
    kept = block_sum_i32(kept, red);
    if (t == 0) pr[14] = kept;
}

// After the masked energies and peaks: a frame on the narrowed search falls back to the full
// energies when it found no lane or a lane sits next to a pruned candidate.  Marks
// LD_FLAG_FALLBACK on every frame that used any part of the full search.
__global__ void k_lane_check(Dev d, ld_lanes* lanes, int nframes, int pruning) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nframes || frame_masked(d, b)) return;
    int32_t* pr = d.prune + (int64_t)b * kPruneWords;
    const uint8_t* cm = d.cmask + (int64_t)b * d.W2;
    int fb = pr[1];
    const FrameInfo fi = d.info[b];
    if (!pruning) pr[14] = d.W2;        // candidates kept: all
    if (pruning && !(fb & kFbPlainVpx) && !(fi.flags & (LD_FLAG_NOROAD | LD_FLAG_NOVP))) {
        const int n = lanes[b].n;
        bool bad = n == 0;
        for (int l = 0; l < n; ++l) {
            const int i = lanes[b].u_start[l] + d.half;
            bad = bad || cm[i - 1] == 0 || cm[i + 1] == 0;
        }
        if (bad) fb |= kFbPlainEnergy;
    }
    pr[1] = fb;
    if (fb & (kFbPlainVpx | kFbPlainEnergy)) {
        d.info[b].flags = fi.flags | LD_FLAG_FALLBACK;
        lanes[b].flags |= LD_FLAG_FALLBACK;
    }
}

}  // namespace

// ==========================================================================================
// Host side: frame objects and the C ABI.
// k_vdisp_hist, k_vdisp_fit, k_edges, k_vpx_fit, k_energy, k_peaks, then the pruned search:
// k_cnn_fwd, k_seed, k_vpx_window, k_cand_mask + k_lane_check, then k_vpx_ransac
constexpr int kNumKernels = 11;

struct ProfEvent {
    int kernel;
    hipEvent_t start, stop;
};

struct ld_frame_s {
    Dev d;
    bool prof = false;                  // bracket every kernel launch with HIP events
    std::vector<ProfEvent> pending;     // recorded, not yet read
    std::vector<ProfEvent> pool;        // reusable event pairs
    double acc_ms[kNumKernels] = {};
    int64_t calls[kNumKernels] = {};
    int batch;          // allocated frames
    int active;         // frames processed by the next calls
    void* mem;          // one device allocation holding all scratch
    size_t mem_bytes;
    int device;
    hipStream_t last;
    int stage;          // 0 nothing, 1 vdisp done, 2 vp done, 3 energy done
    int bands;          // bands of the last network decisions (0 none since the last ld_vdisp)
};

namespace {

size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

int elem_size(int fmt) { return fmt == LD_DISP_U8 ? 1 : (fmt == LD_DISP_F32 ? 4 : 2); }

bool aligned(const void* p, size_t a) { return ((uintptr_t)p % a) == 0; }

ld_status launch_ok() { return hipGetLastError() == hipSuccess ? LD_OK : LD_E_HIP; }

// Optional per-kernel timing: an event pair on the launch stream around one kernel.
struct ProfScope {
    ld_frame f;
    int kernel;
    hipStream_t st;
    ProfEvent ev;
    bool on;
    ProfScope(ld_frame f_, int k, hipStream_t s) : f(f_), kernel(k), st(s), on(f_->prof) {
        if (!on) return;
        if (f->pool.empty()) {
            ProfEvent e;
            e.kernel = 0;
            if (hipEventCreate(&e.start) != hipSuccess || hipEventCreate(&e.stop) != hipSuccess) { on = false; return; }
            f->pool.push_back(e);
        }
        ev = f->pool.back();
        f->pool.pop_back();
        ev.kernel = kernel;
        (void)hipEventRecord(ev.start, st);
    }
    ~ProfScope() {
        if (!on) return;
        (void)hipEventRecord(ev.stop, st);
        f->pending.push_back(ev);
    }
};

int vdisp_fit_threads(const Dev& d) {
    const int waves = vdisp_dp_waves(d.H, d.P.tau_y_max);
    if (waves > 0) return std::max(256, waves * kWave);
    return std::min(1024, std::max(256, ((d.H + kVdRows - 1) / kVdRows + 63) / 64 * 64));
}

// LDS of k_vdisp_fit; the register DP's backtrace only if it fits (and then *in_lds = 1)
size_t vdisp_fit_lds(const Dev& d, int* in_lds) {
    const size_t H4 = ((size_t)d.H + 3) / 4 * 4, bm4 = (((size_t)d.H + 31) / 32 + 3) / 4 * 4;
    size_t words = 4 * (((size_t)d.D1 + 3) / 4 * 4) + bm4 + H4;
    const int waves = vdisp_dp_waves(d.H, d.P.tau_y_max);
    size_t region = 4 * (size_t)d.H + (size_t)kVdWalk * kVdWalkCols;
    *in_lds = 0;
    if (waves > 0) {
        region = 4 * (size_t)vdisp_seam_words(waves);
        const size_t back = 4 * (size_t)vdisp_back_words(d.H, d.d_max);
        if (4 * words + region + back <= 160 * 1024 - 512) {    // (512: the kernel's other LDS)
            *in_lds = 1;
            region += back;
        }
    }
    return 4 * words + std::max(region, sizeof(RansacShared));
}

// LDS of k_vpx_fit without the staged vote columns
size_t vpx_fit_lds(const Dev& d) {
    const int nw = vpx_fit_waves(d.W2);
    return sizeof(int) * ((size_t)nw * kWave * kFitCols * 2 + 2 * (size_t)(nw + 2) * 2 * kSeam + (size_t)d.H + 1);
}

size_t edges_lds(int nwaves) {
    return (sizeof(double) + 3 * sizeof(uint32_t)) * kEdgeStrip + sizeof(uint2) * kEdgeQueue * (size_t)nwaves;
}

size_t energy_lds(int columns) { return sizeof(float) * (6 * (size_t)columns + 10); }

constexpr int kRegions = 18;

// Byte offsets and sizes of the regions of one frame object's device allocation.
size_t frame_layout(int width, int height, int batch, int d_max, size_t* off, size_t* sz) {
    const size_t B = (size_t)batch, H = (size_t)height, W = (size_t)width, D1 = (size_t)d_max + 1, W2 = 2 * (size_t)width;
    const size_t s[kRegions] = {
        B * D1 * ((H + 31) / 32 * 32) * 4,   // myT (rows padded to 32)
        B * D1 * H,                     // back_y
        B * 2 * D1 * 4,                 // my_pts
        B * 2 * sizeof(FitRes),         // fit
        B * sizeof(FrameInfo),          // info
        B * 6 * H * 8,                  // tab
        B * H * 4,                      // rowcnt
        B * H * W * sizeof(ld_edge),    // edges
        B * H * ((W2 + kDpRun - 1) / kDpRun) * 4,   // back_x (4 bits per column)
        B * H * 4,                      // mxpath
        B * W2 * 8,                     // energy
        B * 6 * kMaxRounds * 4,         // trace
        B * H * W * 4,                  // qbuf
        B * H * 2 * 4,                  // rbound
        B * LDI_MAX_BANDS * LDI_BAND_ROWS * W,   // lbits
        B * kPruneWords * 4,            // prune
        B * W2,                         // cmask
        B * 5 * 8,                      // seedg
    };
    size_t o = 0;
    for (int i = 0; i < kRegions; ++i) {
        sz[i] = s[i];
        off[i] = o;
        o += align_up(s[i]);
    }
    return o;
}

ld_status check_params(const ld_params& p) {
    if (p.chi < 0 || p.tau_y_max < 0 || p.tau_y_max > 255 || p.tau_x_max < 0 || p.tau_x_max > 5) return LD_E_INVAL;
    if (p.lambda_y < 0 || p.lambda_x < 0 || p.lambda_y > 1000 || p.lambda_x > 1000) return LD_E_INVAL;
    if (p.n_hyp < 1 || p.n_hyp > kMaxHyp || p.max_rounds < 1 || p.max_rounds > kMaxRounds) return LD_E_INVAL;
    if (p.eps_num < 0 || p.eps_den < 1 || p.edge_t < 0 || p.edge_t > 46340) return LD_E_INVAL;
    if (p.nu != 1 || p.varsigma != 3) return LD_E_INVAL;    // the kernels are built for the paper's box
    if (!(p.sigma_g > 0.0) || !(p.tr_x >= 0.0) || !(p.tr_y >= 0.0) || !(p.varpi >= 0.0)) return LD_E_INVAL;
    if (p.d_nms < 0 || (p.weight_squared != 0 && p.weight_squared != 1) || (p.vote != 0 && p.vote != 1))
        return LD_E_INVAL;
    return LD_OK;
}

// Point the scratch fields of d at the regions of one allocation laid out by frame_layout.
void bind_regions(Dev& d, char* base, const size_t* off) {
    d.myT = reinterpret_cast<int32_t*>(base + off[0]);
    d.back_y = reinterpret_cast<uint8_t*>(base + off[1]);
    d.my_pts = reinterpret_cast<int32_t*>(base + off[2]);
    d.fit = reinterpret_cast<FitRes*>(base + off[3]);
    d.info = reinterpret_cast<FrameInfo*>(base + off[4]);
    d.tab = reinterpret_cast<double*>(base + off[5]);
    d.rowcnt = reinterpret_cast<int32_t*>(base + off[6]);
    d.edges = reinterpret_cast<ld_edge*>(base + off[7]);
    d.back_x = reinterpret_cast<int8_t*>(base + off[8]);
    d.mxpath = reinterpret_cast<int32_t*>(base + off[9]);
    d.energy = reinterpret_cast<double*>(base + off[10]);
    d.trace = reinterpret_cast<int32_t*>(base + off[11]);
    d.qbuf = reinterpret_cast<float*>(base + off[12]);
    d.rbound = reinterpret_cast<uint32_t*>(base + off[13]);
    d.lbits = reinterpret_cast<uint8_t*>(base + off[14]);
    d.prune = reinterpret_cast<int32_t*>(base + off[15]);
    d.cmask = reinterpret_cast<uint8_t*>(base + off[16]);
    d.seedg = reinterpret_cast<double*>(base + off[17]);
    d.nact = nullptr;
    d.only = nullptr;
    d.only_bits = 0;
    d.only_set = 0;
}

// Sizes, parameters and derived launch constants of a frame object (no device memory).
ld_status init_dev(Dev& d, int32_t width, int32_t height, int32_t batch, int32_t fmt, int32_t d_max,
                   const ld_params* p) {
    if (width < 8 || width > 4096 || height < 8 || height > 4096 || batch < 1 || batch > 65535) return LD_E_INVAL;
    if (fmt < 0 || fmt > 2 || d_max < 1 || d_max > 1023) return LD_E_INVAL;
    ld_params P;
    ld_params_default(&P);
    if (p) P = *p;
    if (check_params(P) != LD_OK) return LD_E_INVAL;
    // the row DP keeps (E << 4 | rank) in int32: E >= -width * height * (2 chi + 1)
    if ((int64_t)width * height * (2 * (int64_t)P.chi + 1) + 5 * (int64_t)P.lambda_x >= ((int64_t)1 << 27)) return LD_E_INVAL;
    d.W = width; d.H = height; d.D1 = d_max + 1; d.W2 = 2 * width; d.half = width / 2; d.fmt = fmt;
    d.d_max = d_max; d.B = batch; d.P = P;
    d.hist_rows = std::max(kHistGroup, std::min(32, (8192 / d.D1) / kHistGroup * kHistGroup));
    d.Hm = (height + 31) / 32 * 32;
    return LD_OK;
}

template <int FMT>
void launch_hist(int npt, dim3 g, size_t lds, hipStream_t st, const Dev& d, const uint8_t* dp, int64_t pitch,
                 int32_t* out) {
    if (npt <= 1) hipLaunchKernelGGL((k_vdisp_hist<FMT, 1>), g, dim3(kBlock), lds, st, d, dp, pitch, out);
    else if (npt <= 2) hipLaunchKernelGGL((k_vdisp_hist<FMT, 2>), g, dim3(kBlock), lds, st, d, dp, pitch, out);
    else if (npt <= 4) hipLaunchKernelGGL((k_vdisp_hist<FMT, 4>), g, dim3(kBlock), lds, st, d, dp, pitch, out);
    else if (npt <= 5) hipLaunchKernelGGL((k_vdisp_hist<FMT, 5>), g, dim3(kBlock), lds, st, d, dp, pitch, out);
    else if (npt <= 8) hipLaunchKernelGGL((k_vdisp_hist<FMT, 8>), g, dim3(kBlock), lds, st, d, dp, pitch, out);
    else hipLaunchKernelGGL((k_vdisp_hist<FMT, 16>), g, dim3(kBlock), lds, st, d, dp, pitch, out);
}

// S1 for the active frames of f
ld_status run_hist(ld_frame f, const void* disp, int64_t pitch, int32_t* vdisp_out, hipStream_t st) {
    Dev d = f->d;
    d.hist_rows = hist_rows(d.W, d.H, f->active, kHistGroup, d.hist_rows);
    dim3 g1((d.H + d.hist_rows - 1) / d.hist_rows, f->active);
    const size_t l1 = sizeof(int) * d.hist_rows * d.D1;
    const uint8_t* dp = static_cast<const uint8_t*>(disp);
    ProfScope ps(f, 0, st);
    const int npt = (d.W + kBlock - 1) / kBlock;
    if (d.fmt == LD_DISP_U8) launch_hist<LD_DISP_U8>(npt, g1, l1, st, d, dp, pitch, vdisp_out);
    else if (d.fmt == LD_DISP_F32) launch_hist<LD_DISP_F32>(npt, g1, l1, st, d, dp, pitch, vdisp_out);
    else launch_hist<LD_DISP_U16Q4>(npt, g1, l1, st, d, dp, pitch, vdisp_out);
    return launch_ok();
}

// S2-S3 for the active frames of f
ld_status run_vdisp_fit(ld_frame f, const uint64_t* sid, const int64_t* fidx, double* beta_out, hipStream_t st) {
    Dev& d = f->d;
    int in_lds;
    const int lock = vdisp_lockstep(vdisp_dp_waves(d.H, d.P.tau_y_max), d.d_max) ? 1 : 0;
    const size_t l2 = vdisp_fit_lds(d, &in_lds);
    allow_lds<k_vdisp_fit>(l2);
    {
        ProfScope ps(f, 1, st);
        hipLaunchKernelGGL(k_vdisp_fit, dim3(f->active), dim3(vdisp_fit_threads(d)), l2, st, d, sid, fidx, beta_out,
                           in_lds, lock);
    }
    return launch_ok();
}

ld_status run_vdisp(ld_frame f, const void* disp, int64_t pitch, const uint64_t* sid, const int64_t* fidx,
                    int32_t* vdisp_out, double* beta_out, hipStream_t st) {
    const ld_status s = run_hist(f, disp, pitch, vdisp_out, st);
    return s == LD_OK ? run_vdisp_fit(f, sid, fidx, beta_out, st) : s;
}

ld_status run_edges(ld_frame f, const uint8_t* grey, int64_t gp, const void* disp, int64_t dpt, hipStream_t st) {
    Dev& d = f->d;
    const int nw = (d.W + kEdgeCols - 1) / kEdgeCols;
    const int strip = edge_rows(d.H, nw, f->active);
    const dim3 g3((d.H + strip - 1) / strip, f->active);
    const size_t lds = edges_lds(nw);
    const uint8_t* dp = static_cast<const uint8_t*>(disp);
    ProfScope ps(f, 2, st);
    if (d.fmt == LD_DISP_U8) {
        allow_lds<k_edges<LD_DISP_U8>>(lds);
        hipLaunchKernelGGL(k_edges<LD_DISP_U8>, g3, dim3(nw * kWave), lds, st, d, grey, gp, dp, dpt, strip);
    } else if (d.fmt == LD_DISP_F32) {
        allow_lds<k_edges<LD_DISP_F32>>(lds);
        hipLaunchKernelGGL(k_edges<LD_DISP_F32>, g3, dim3(nw * kWave), lds, st, d, grey, gp, dp, dpt, strip);
    } else {
        allow_lds<k_edges<LD_DISP_U16Q4>>(lds);
        hipLaunchKernelGGL(k_edges<LD_DISP_U16Q4>, g3, dim3(nw * kWave), lds, st, d, grey, gp, dp, dpt, strip);
    }
    return launch_ok();
}

// the full band accumulator and row DP of S6-S7 for the frames that `d` selects
ld_status run_vpx_dp(ld_frame f, const Dev& d, hipStream_t st) {
    const size_t fixed = vpx_fit_lds(d);
    const int nt = kWave * (vpx_fit_waves(d.W2) + 1);
    const int cap = vpx_staged_votes(d.W, d.H, nt / kWave, fixed, f->active);
    const size_t l4 = fixed + sizeof(uint16_t) * (size_t)cap;
    ProfScope ps(f, 3, st);
    allow_lds<k_vpx_fit>(l4);
    hipLaunchKernelGGL(k_vpx_fit, dim3(f->active), dim3(nt), l4, st, d, cap);
    return launch_ok();
}

// S8 for every active frame
ld_status run_vpx_ransac(ld_frame f, const uint64_t* sid, const int64_t* fidx, const double* seed_gamma, int pruned,
                         double* vp_out, hipStream_t st) {
    const Dev& d = f->d;
    const size_t l = sizeof(int) * 4 * (((size_t)d.H + 3) / 4 * 4) + sizeof(uint32_t) * ((d.H + 31) / 32);
    allow_lds<k_vpx_ransac>(l);
    ProfScope ps(f, 10, st);
    const int nt = ransac_threads(f->active);
    hipLaunchKernelGGL(k_vpx_ransac, dim3(f->active), dim3(nt), l, st, d, sid, fidx, seed_gamma, pruned, vp_out);
    return launch_ok();
}

ld_status run_vp(ld_frame f, const uint8_t* grey, int64_t gp, const void* disp, int64_t dpt, const uint64_t* sid,
                 const int64_t* fidx, const double* seed_gamma, double* vp_out, hipStream_t st) {
    ld_status s = run_edges(f, grey, gp, disp, dpt, st);
    if (s == LD_OK) s = run_vpx_dp(f, f->d, st);
    if (s == LD_OK) s = run_vpx_ransac(f, sid, fidx, seed_gamma, 0, vp_out, st);
    return s;
}

template <int NC, int NT, int BT, int PD>
void launch_energy(ld_frame f, const Dev& d, const uint8_t* mask, float* eout, hipStream_t st) {
    static_assert(9 % PD == 0, "the unrolled sweep rotates the prefetch slots by renaming");
    const size_t base = (energy_lds(NC * BT) + 15) / 16 * 16, rows = (size_t)d.H * (sizeof(double) * 2 + sizeof(int));
    const bool staged = base + rows <= (size_t)kMaxLds;
    const size_t l = staged ? base + rows : base;
    allow_lds<k_energy<NC, NT, BT, PD>>(l);
    hipLaunchKernelGGL((k_energy<NC, NT, BT, PD>), dim3(f->active), dim3(BT), l, st, d, mask, eout,
                       staged ? (int)(base / sizeof(float)) : 0);
}

ld_status run_energy(ld_frame f, const uint8_t* mask, float* eout, hipStream_t st, const Dev* dsel = nullptr) {
    ProfScope ps(f, 4, st);
    const Dev& d = dsel ? *dsel : f->d;
    const EnergyForm form = energy_form(d.W, f->active);
    if (form == EnergyForm::kTwoLaunches) {
        const int cols = kM1Waves * kM1Cols;
        const dim3 g1((d.W + cols - 1) / cols, (d.H + kM1Rows - 1) / kM1Rows, f->active);
        hipLaunchKernelGGL(k_m1, g1, dim3(kM1Waves * kWave), 0, st, d);
        hipLaunchKernelGGL(k_tracks, dim3((d.W2 + kWave - 1) / kWave, f->active), dim3(kWave), 0, st, d, mask, eout);
        return launch_ok();
    }
    if (form == EnergyForm::kThreads512) {                   // (more than 1024 columns)
        const int nc = (d.W + 511) / 512;
        if (nc <= 3) launch_energy<3, 6, 512, 3>(f, d, mask, eout, st);
        else if (nc <= 4) launch_energy<4, 8, 512, 3>(f, d, mask, eout, st);
        else if (nc <= 6) launch_energy<6, 12, 512, 3>(f, d, mask, eout, st);
        else launch_energy<8, 16, 512, 3>(f, d, mask, eout, st);
        return launch_ok();
    }
    const int nc = (d.W + kBlock - 1) / kBlock;
    if (nc <= 1) launch_energy<1, 2, kBlock, 1>(f, d, mask, eout, st);
    else if (nc <= 2) launch_energy<2, 4, kBlock, 1>(f, d, mask, eout, st);
    else if (nc <= 3) launch_energy<3, 6, kBlock, 1>(f, d, mask, eout, st);
    else if (nc <= 4) launch_energy<4, 8, kBlock, 1>(f, d, mask, eout, st);
    else if (nc <= 5) launch_energy<5, 10, kBlock, 1>(f, d, mask, eout, st);
    else launch_energy<6, 12, kBlock, 1>(f, d, mask, eout, st);
    return launch_ok();
}

ld_status run_peaks(ld_frame f, ld_lanes* lanes, float* curves, hipStream_t st, const Dev* dsel = nullptr) {
    ProfScope ps(f, 5, st);
    const Dev& d = dsel ? *dsel : f->d;
    const size_t l = curves ? std::max((size_t)d.W2, kCurveLds) : (size_t)d.W2;
    hipLaunchKernelGGL(k_peaks, dim3(f->active), dim3(kBlock), l, st, d, lanes, curves);
    return launch_ok();
}

ld_status check_images(ld_frame f, const uint8_t* grey, int64_t gp, const void* disp, int64_t dpt) {
    const Dev& d = f->d;
    const int es = elem_size(d.fmt);
    if (disp == nullptr || dpt < (int64_t)d.W * es || dpt % es != 0 || !aligned(disp, es)) return LD_E_INVAL;
    // the edge kernel addresses a frame's grey rows with 32-bit offsets
    if (grey != nullptr && (gp < d.W || (int64_t)d.H * gp > (int64_t)INT32_MAX - 4096)) return LD_E_INVAL;
    return LD_OK;
}

// Every step of ld_detect on the active frames of f, on one stream.
ld_status detect_all(ld_frame f, const uint8_t* grey, int64_t gp, const void* disp, int64_t dpt,
                     const uint64_t* sid, const int64_t* fidx, ld_lanes* lanes, float* curves, hipStream_t st) {
    f->last = st;
    ld_status s = run_vdisp(f, disp, dpt, sid, fidx, nullptr, nullptr, st);
    if (s == LD_OK) s = run_vp(f, grey, gp, disp, dpt, sid, fidx, nullptr, nullptr, st);
    if (s == LD_OK) s = run_energy(f, nullptr, nullptr, st);
    if (s == LD_OK) s = run_peaks(f, lanes, curves, st);
    f->stage = s == LD_OK ? 3 : 0;
    f->bands = 0;
    return s;
}

}  // namespace

// Scratch of ld_detect_noalloc: a fixed device array, one copy per GPU for the life of the
// process.  Host code never uses the name `scratch` as an address: the device address of each
// GPU's copy is taken once per device with hipGetSymbolAddress (that device current) and kept
// in scratch_ptr.  Every ld_detect_noalloc call on a GPU uses that GPU's copy, so calls that
// overlap on one GPU (different streams or threads without ordering) race on it.
constexpr size_t kNoAllocBytes = LD_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

namespace {

std::mutex scratch_mu;
char* scratch_ptr[kMaxDevices] = {};

// The current device's copy of the scratch array (set up on the first call on that device).
ld_status noalloc_scratch(char** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return LD_E_HIP;
    if (dev < 0 || dev >= kMaxDevices) return LD_E_INVAL;
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (scratch_ptr[dev] == nullptr) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) {
            (void)hipGetLastError();
            return LD_E_HIP;
        }
        scratch_ptr[dev] = static_cast<char*>(ptr);
    }
    *out = scratch_ptr[dev];
    return LD_OK;
}

}  // namespace

extern "C" {

void ld_params_default(ld_params* p) {
    if (!p) return;
    p->chi = 25; p->tau_y_max = 6; p->tau_x_max = 5; p->lambda_y = 1; p->lambda_x = 1;
    p->tr_y = 4.0; p->tr_x = 16.0; p->eps_num = 99; p->eps_den = 100; p->varpi = 3.0;
    p->edge_t = 100; p->sigma_g = 3.5; p->nu = 1; p->varsigma = 3; p->n_hyp = 64; p->max_rounds = 16;
    p->rho_lpv = 0.25; p->d_nms = 0; p->weight_squared = 0; p->vote = 0; p->seed = 0;
}

const char* ld_status_string(ld_status s) {
    switch (s) {
        case LD_OK: return "ok";
        case LD_E_INVAL: return "invalid argument";
        case LD_E_NOMEM: return "out of device memory";
        case LD_E_HIP: return "HIP runtime error";
        case LD_E_STATE: return "step called out of order";
        case LD_E_BUSY: return "queue full, retry later";
    }
    return "unknown status";
}

ld_status ld_frame_create(int32_t width, int32_t height, int32_t batch, int32_t fmt, int32_t d_max,
                          const ld_params* p, ld_frame* out) {
    if (!out) return LD_E_INVAL;
    *out = nullptr;
    Dev d0{};
    if (init_dev(d0, width, height, batch, fmt, d_max, p) != LD_OK) return LD_E_INVAL;
    ld_frame f = new (std::nothrow) ld_frame_s();
    if (!f) return LD_E_NOMEM;
    Dev& d = f->d;
    d = d0;
    size_t off[kRegions], sz[kRegions];
    const size_t o = frame_layout(width, height, batch, d_max, off, sz);

    if (hipGetDevice(&f->device) != hipSuccess) { delete f; return LD_E_HIP; }
    if (hipMalloc(&f->mem, o) != hipSuccess) { (void)hipGetLastError(); delete f; return LD_E_NOMEM; }
    f->mem_bytes = o;
    bind_regions(d, static_cast<char*>(f->mem), off);
    // small state starts zeroed so that introspection of an unprocessed frame is defined
    if (hipMemset(d.info, 0, sz[4]) != hipSuccess || hipMemset(d.trace, 0xff, sz[11]) != hipSuccess ||
        hipMemset(d.fit, 0, sz[3]) != hipSuccess || hipMemset(d.prune, 0, sz[15]) != hipSuccess ||
        hipMemset(d.lbits, 0, sz[14]) != hipSuccess || hipMemset(d.cmask, 1, sz[16]) != hipSuccess ||
        hipDeviceSynchronize() != hipSuccess) {
        (void)hipFree(f->mem);
        delete f;
        return LD_E_HIP;
    }
    f->batch = batch;
    f->active = batch;
    f->last = nullptr;
    f->stage = 0;
    f->bands = 0;
    *out = f;
    return LD_OK;
}

ld_status ld_frame_destroy(ld_frame f) {
    if (!f) return LD_OK;
    ld_status s = LD_OK;
    if (hipStreamSynchronize(f->last) != hipSuccess) s = LD_E_HIP;
    for (auto& e : f->pending) { (void)hipEventDestroy(e.start); (void)hipEventDestroy(e.stop); }
    for (auto& e : f->pool) { (void)hipEventDestroy(e.start); (void)hipEventDestroy(e.stop); }
    if (hipFree(f->mem) != hipSuccess) s = LD_E_HIP;
    delete f;
    return s;
}

ld_status ld_frame_set_active(ld_frame f, int32_t n) {
    if (!f || n < 1 || n > f->batch) return LD_E_INVAL;
    f->active = n;
    return LD_OK;
}

ld_status ld_vdisp(ld_frame f, const void* disp, int64_t disp_pitch, const uint64_t* stream_ids,
                   const int64_t* frame_idx, int32_t* vdisp_out, double* beta_out, void* hip_stream) {
    LdRange rr_("ld_vdisp");
    if (!f) return LD_E_INVAL;
    if (check_images(f, nullptr, 0, disp, disp_pitch) != LD_OK) return LD_E_INVAL;
    if ((stream_ids && !aligned(stream_ids, 8)) || (frame_idx && !aligned(frame_idx, 8))) return LD_E_INVAL;
    if ((vdisp_out && !aligned(vdisp_out, 4)) || (beta_out && !aligned(beta_out, 8))) return LD_E_INVAL;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    ld_status s = run_vdisp(f, disp, disp_pitch, stream_ids, frame_idx, vdisp_out, beta_out, st);
    f->last = st;
    if (s == LD_OK) f->stage = 1;
    f->bands = 0;
    return s;
}

ld_status ld_vp_ransac(ld_frame f, const uint8_t* grey, int64_t grey_pitch, const void* disp, int64_t disp_pitch,
                       const uint64_t* stream_ids, const int64_t* frame_idx, const double* seed_gamma,
                       double* vp_out, void* hip_stream) {
    LdRange rr_("ld_vp_ransac");
    if (!f) return LD_E_INVAL;
    if (!grey || check_images(f, grey, grey_pitch, disp, disp_pitch) != LD_OK) return LD_E_INVAL;
    if ((stream_ids && !aligned(stream_ids, 8)) || (frame_idx && !aligned(frame_idx, 8))) return LD_E_INVAL;
    if ((seed_gamma && !aligned(seed_gamma, 8)) || (vp_out && !aligned(vp_out, 8))) return LD_E_INVAL;
    if (f->stage < 1) return LD_E_STATE;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    ld_status s = run_vp(f, grey, grey_pitch, disp, disp_pitch, stream_ids, frame_idx, seed_gamma, vp_out, st);
    f->last = st;
    if (s == LD_OK) f->stage = 2;
    return s;
}

ld_status ld_lane_energy(ld_frame f, const uint8_t* cand_mask, float* energy_out, void* hip_stream) {
    LdRange rr_("ld_lane_energy");
    if (!f) return LD_E_INVAL;
    if (energy_out && !aligned(energy_out, 4)) return LD_E_INVAL;
    if (f->stage < 2) return LD_E_STATE;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    ld_status s = run_energy(f, cand_mask, energy_out, st);
    f->last = st;
    if (s == LD_OK) f->stage = 3;
    return s;
}

ld_status ld_peaks(ld_frame f, ld_lanes* lanes_out, float* curves_out, void* hip_stream) {
    LdRange rr_("ld_peaks");
    if (!f || !lanes_out || !aligned(lanes_out, 4)) return LD_E_INVAL;
    if (curves_out && !aligned(curves_out, 4)) return LD_E_INVAL;
    if (f->stage < 3) return LD_E_STATE;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    ld_status s = run_peaks(f, lanes_out, curves_out, st);
    f->last = st;
    return s;
}

ld_status ld_detect(ld_frame f, const uint8_t* grey, int64_t grey_pitch, const void* disp, int64_t disp_pitch,
                    const uint64_t* stream_ids, const int64_t* frame_idx, ld_lanes* lanes_out, float* curves_out,
                    void* hip_stream) {
    LdRange rr_("ld_detect");
    if (!f || !lanes_out || !aligned(lanes_out, 4)) return LD_E_INVAL;
    if (!grey || check_images(f, grey, grey_pitch, disp, disp_pitch) != LD_OK) return LD_E_INVAL;
    if ((stream_ids && !aligned(stream_ids, 8)) || (frame_idx && !aligned(frame_idx, 8))) return LD_E_INVAL;
    if (curves_out && !aligned(curves_out, 4)) return LD_E_INVAL;
    return detect_all(f, grey, grey_pitch, disp, disp_pitch, stream_ids, frame_idx, lanes_out, curves_out,
                      static_cast<hipStream_t>(hip_stream));
}

ld_status ld_detect_noalloc(int32_t width, int32_t height, int32_t batch, int32_t fmt, int32_t d_max,
                            const ld_params* p, const uint8_t* grey, int64_t grey_pitch, const void* disp,
                            int64_t disp_pitch, const uint64_t* stream_ids, const int64_t* frame_idx,
                            ld_lanes* lanes_out, float* curves_out, void* hip_stream) {
    LdRange rr_("ld_detect_noalloc");
    ld_frame_s fr;                      // host state on the stack; prof stays off (no event pool)
    if (init_dev(fr.d, width, height, batch, fmt, d_max, p) != LD_OK) return LD_E_INVAL;
    if (!lanes_out || !aligned(lanes_out, 4)) return LD_E_INVAL;
    if (!grey || check_images(&fr, grey, grey_pitch, disp, disp_pitch) != LD_OK) return LD_E_INVAL;
    if ((stream_ids && !aligned(stream_ids, 8)) || (frame_idx && !aligned(frame_idx, 8))) return LD_E_INVAL;
    if (curves_out && !aligned(curves_out, 4)) return LD_E_INVAL;
    size_t off[kRegions], sz[kRegions];
    if (frame_layout(width, height, batch, d_max, off, sz) > kNoAllocBytes) return LD_E_NOMEM;
    char* base = nullptr;
    const ld_status s = noalloc_scratch(&base);
    if (s != LD_OK) return s;
    bind_regions(fr.d, base, off);
    fr.batch = batch;
    fr.active = batch;
    fr.mem = nullptr;
    fr.mem_bytes = 0;
    (void)hipGetDevice(&fr.device);
    return detect_all(&fr, grey, grey_pitch, disp, disp_pitch, stream_ids, frame_idx, lanes_out, curves_out,
                      static_cast<hipStream_t>(hip_stream));
}

ld_status ld_detect_pruned(ld_frame f, ld_cnn n, const uint8_t* grey, int64_t grey_pitch, const void* disp,
                           int64_t disp_pitch, const uint64_t* stream_ids, const int64_t* frame_idx,
                           const double* seed_gamma, ld_lanes* lanes_out, float* curves_out, void* hip_stream) {
    LdRange rr_("ld_detect_pruned");
    if (!f || !n || !lanes_out || !aligned(lanes_out, 4)) return LD_E_INVAL;
    if (seed_gamma && !aligned(seed_gamma, 8)) return LD_E_INVAL;
    if (!grey || check_images(f, grey, grey_pitch, disp, disp_pitch) != LD_OK) return LD_E_INVAL;
    if ((stream_ids && !aligned(stream_ids, 8)) || (frame_idx && !aligned(frame_idx, 8))) return LD_E_INVAL;
    if (curves_out && !aligned(curves_out, 4)) return LD_E_INVAL;
    const ld_cnn_config* c = ldi_cnn_config(n);
    if (!c || !(f->d.P.varpi > 0.0)) return LD_E_INVAL;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    f->last = st;
    Dev& d = f->d;
    const int nb = c->n_bands;
    ld_status s = run_vdisp(f, disp, disp_pitch, stream_ids, frame_idx, nullptr, nullptr, st);
    f->stage = s == LD_OK ? 1 : 0;
    f->bands = 0;
    // the edges first: without the candidate mask the network decisions are read only at voting
    // road edges of the band rows, so the network skips the column tiles that hold none
    if (s == LD_OK) s = run_edges(f, grey, grey_pitch, disp, disp_pitch, st);
    if (s == LD_OK) {
        ProfScope ps(f, 6, st);
        s = ldi_cnn_bits(n, f, grey, grey_pitch, disp, disp_pitch, nullptr, c->dilate < 0 ? 1 : 0, st);
    }
    if (s == LD_OK) {
        ProfScope ps(f, 7, st);
        const size_t ls = sizeof(int) * 2 * (size_t)d.W2;
        allow_lds<k_seed>(ls);
        hipLaunchKernelGGL(k_seed, dim3(f->active), dim3(kBlock), ls, st, d, nb, c->delta_x, c->min_votes,
                           c->seed_ransac);
        s = launch_ok();
    }
    if (s == LD_OK) {
        ProfScope ps(f, 8, st);
        const int cap = std::min(16384, std::max(4096, 16 * d.W));   // staged road edges (bytes)
        const size_t lw = sizeof(int) * (256 + kWave + 3 * (size_t)d.H + 2) + cap;
        const int wave_bytes = (int)((lw + 15) / 16 * 16);
        const int fpw = std::max(1, std::min(4, kMaxLds / wave_bytes));   // frames per workgroup
        allow_lds<k_vpx_window>((size_t)fpw * wave_bytes);
        hipLaunchKernelGGL(k_vpx_window, dim3((f->active + fpw - 1) / fpw), dim3(kWave * fpw), (size_t)fpw * wave_bytes,
                           st, d, cap, wave_bytes, f->active);
        s = launch_ok();
    }
    Dev full = d;                       // frames sent back to the full V_px search
    full.only = d.prune;
    full.only_bits = kFbPlainVpx;
    full.only_set = 1;
    if (s == LD_OK) s = run_vpx_dp(f, full, st);
    if (s == LD_OK) s = run_vpx_ransac(f, stream_ids, frame_idx, seed_gamma, 1, nullptr, st);
    // without candidate pruning every candidate is kept: no mask, and no frame is sent back
    // to the full energies
    const bool pruning = c->dilate >= 0;
    if (s == LD_OK && pruning) {
        ProfScope ps(f, 9, st);
        const size_t lm = sizeof(uint32_t) * nb * LDI_BAND_ROWS * (size_t)((d.W + 31) / 32) + (size_t)d.W2;
        allow_lds<k_cand_mask>(lm);
        hipLaunchKernelGGL(k_cand_mask, dim3(f->active), dim3(kBlock), lm, st, d, nb, c->dilate);
        s = launch_ok();
    }
    if (s == LD_OK) s = run_energy(f, pruning ? d.cmask : nullptr, nullptr, st);
    if (s == LD_OK) s = run_peaks(f, lanes_out, curves_out, st);
    if (s == LD_OK) {
        ProfScope ps(f, 9, st);
        hipLaunchKernelGGL(k_lane_check, dim3((f->active + 63) / 64), dim3(64), 0, st, d, lanes_out, f->active,
                           pruning ? 1 : 0);
        s = launch_ok();
    }
    Dev again = d;                      // frames sent back to the full energies
    again.only = d.prune;
    again.only_bits = kFbPlainEnergy;
    again.only_set = 1;
    if (s == LD_OK && pruning) s = run_energy(f, nullptr, nullptr, st, &again);
    if (s == LD_OK && pruning) s = run_peaks(f, lanes_out, curves_out, st, &again);
    f->stage = s == LD_OK ? 3 : 0;
    if (s == LD_OK) f->bands = nb;
    return s;
}

ld_status ld_sync(ld_frame f) {
    if (!f) return LD_E_INVAL;
    return hipStreamSynchronize(f->last) == hipSuccess ? LD_OK : LD_E_HIP;
}

ld_status ld_frame_profile(ld_frame f, int32_t enable) {
    if (!f) return LD_E_INVAL;
    if (hipStreamSynchronize(f->last) != hipSuccess) return LD_E_HIP;
    for (auto& e : f->pending) f->pool.push_back(e);
    f->pending.clear();
    for (int k = 0; k < kNumKernels; ++k) { f->acc_ms[k] = 0.0; f->calls[k] = 0; }
    f->prof = enable != 0;
    return LD_OK;
}

ld_status ld_frame_kernel_times(ld_frame f, double* ms_out, int64_t* calls_out, int32_t n) {
    if (!f || !ms_out || n < 1) return LD_E_INVAL;
    ld_status s = LD_OK;
    for (auto& e : f->pending) {
        float ms = 0.0f;
        if (hipEventSynchronize(e.stop) != hipSuccess || hipEventElapsedTime(&ms, e.start, e.stop) != hipSuccess) {
            s = LD_E_HIP;
        } else {
            f->acc_ms[e.kernel] += ms;
            f->calls[e.kernel] += 1;
        }
        f->pool.push_back(e);
    }
    f->pending.clear();
    for (int k = 0; k < n && k < kNumKernels; ++k) {
        ms_out[k] = f->acc_ms[k];
        if (calls_out) calls_out[k] = f->calls[k];
    }
    return s;
}

ld_status ld_frame_read(ld_frame f, int32_t what, int32_t b, void* dst, int64_t bytes, void* hip_stream) {
    if (!f || !dst || b < 0 || b >= f->batch) return LD_E_INVAL;
    const Dev& d = f->d;
    const void* src = nullptr;
    size_t n = 0;
    switch (what) {
        case LD_STATE_INFO: src = d.info + b; n = sizeof(FrameInfo); break;
        case LD_STATE_MY_PATH: src = d.my_pts + (size_t)b * 2 * d.D1; n = sizeof(int32_t) * 2 * d.D1; break;
        case LD_STATE_BETA: src = d.fit + 2 * (size_t)b; n = sizeof(FitRes); break;
        case LD_STATE_GAMMA: src = d.fit + 2 * (size_t)b + 1; n = sizeof(FitRes); break;
        case LD_STATE_TABLES: src = d.tab + (size_t)b * 6 * d.H; n = sizeof(double) * 6 * d.H; break;
        case LD_STATE_ROWCOUNT: src = d.rowcnt + (size_t)b * d.H; n = sizeof(int32_t) * d.H; break;
        case LD_STATE_EDGES: src = d.edges + (size_t)b * d.H * d.W; n = sizeof(ld_edge) * d.H * d.W; break;
        case LD_STATE_MX_PATH: src = d.mxpath + (size_t)b * d.H; n = sizeof(int32_t) * d.H; break;
        case LD_STATE_ENERGY: src = d.energy + (size_t)b * d.W2; n = sizeof(double) * d.W2; break;
        case LD_STATE_TRACE: src = d.trace + (size_t)b * 6 * kMaxRounds; n = sizeof(int32_t) * 6 * kMaxRounds; break;
        case LD_STATE_LANE_BITS:
            src = d.lbits + (size_t)b * LDI_MAX_BANDS * LDI_BAND_ROWS * d.W;
            n = (size_t)LDI_MAX_BANDS * LDI_BAND_ROWS * d.W;
            break;
        case LD_STATE_PRUNE: src = d.prune + (size_t)b * kPruneWords; n = sizeof(int32_t) * kPruneWords; break;
        case LD_STATE_CAND_MASK: src = d.cmask + (size_t)b * d.W2; n = (size_t)d.W2; break;
        default: return LD_E_INVAL;
    }
    if (bytes < (int64_t)n) return LD_E_INVAL;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    return hipMemcpyAsync(dst, src, n, hipMemcpyDefault, st) == hipSuccess ? LD_OK : LD_E_HIP;
}

}  // extern "C"

// ==========================================================================================
// Internal hooks for the serving layer (ld_server.hip); not part of the C ABI.
ld_status ldi_frame_bind_count(ld_frame f, const int32_t* d_count) {
    if (!f) return LD_E_INVAL;
    f->d.nact = d_count;
    return LD_OK;
}

const ld_fit* ldi_frame_fits(ld_frame f) { return f ? reinterpret_cast<const ld_fit*>(f->d.fit) : nullptr; }

ld_status ldi_frame_get_view(ld_frame f, ldi_frame_view* v) {
    if (!f || !v) return LD_E_INVAL;
    const Dev& d = f->d;
    v->W = d.W; v->H = d.H; v->fmt = d.fmt; v->d_max = d.d_max; v->batch = f->batch; v->active = f->active;
    v->stage = f->stage;
    v->varpi = d.P.varpi;
    v->tab = d.tab;
    v->info = reinterpret_cast<const int32_t*>(d.info);
    v->lane_bits = d.lbits;
    v->nact = d.nact;
    v->edges = d.edges;
    v->rowcnt = d.rowcnt;
    return LD_OK;
}

ld_status ldi_frame_set_last(ld_frame f, void* stream) {
    if (!f) return LD_E_INVAL;
    f->last = static_cast<hipStream_t>(stream);
    return LD_OK;
}

ld_status ldi_frame_mark_bands(ld_frame f, int32_t n_bands, void* stream) {
    if (!f) return LD_E_INVAL;
    f->bands = n_bands;
    f->last = static_cast<hipStream_t>(stream);
    return LD_OK;
}

size_t ldi_frame_bytes(int32_t width, int32_t height, int32_t batch, int32_t d_max) {
    size_t off[kRegions], sz[kRegions];
    return frame_layout(width, height, batch, d_max, off, sz);
}
