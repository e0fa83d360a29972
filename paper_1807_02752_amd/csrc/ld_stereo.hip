// ld_stereo.hip -- disparity maps of rectified stereo pairs (Sec. 2.1): NCC block matching on
// memorised block statistics (Eq. ncc_1 with Eq. sigma_l_1 / sigma_r_1), search range
// propagation from the bottom row up (Eq. srp, Alg. "SRP-based disparity map estimation") and the
// left-right consistency check (Alg. "LRC check").
//
// Definitions (the same on the CPU check): a pixel is matched only when its (2 rho + 1)^2 block
// lies in the image, 0 meaning "no match", candidates 1..d_max whose other block lies in the
// image too.  With S, Q the block sum and sum of squares, P the sum of products of the two
// blocks and n the block size, the cost is (n P - S_a S_b) / (sqrt(n Q_a - S_a^2) sqrt(n Q_b -
// S_b^2)): integers exactly, the quotient in FP64 in that order; a flat block (n Q = S^2) is not
// scored; the largest cost wins, ties to the smaller disparity.  Row v searches the union of
// [l - tau, l + tau] over the matched neighbours u-1..u+1 of row v+1 with l > 0, else 1..d_max.
// The right map is the same search with the roles of the images swapped (the other block at
// x + d); the check keeps l(u) when |l(u) - l_right(u - l(u))| <= tr.
//
// Layout: one workgroup per frame sweeps the rows from the bottom, its two halves the left and
// the right map in step; each half keeps the statistics of its own image, which the other half
// reads as its partner's, so an image's ring, column sums, block sums and variances are formed
// once for both maps.  The 2 rho + 1 image rows of both images sit in LDS rings (one new row
// per step into the slot of the row that leaves, fetched from HBM while the row before it is
// matched), stored word-interleaved (word g of all slots together) so that a block's words are
// constant offsets from one address; the sum of products takes the rows in slot order for both
// blocks, which leaves it unchanged.  The
// column sums over the ring follow each new row incrementally, the block sums of a row come
// from the column sums four columns a thread, and the block variances are kept per column as
// integers with their FP32 reciprocal roots.  A candidate costs its 2 rho + 1 rows of byte dot
// products and one FP32 multiplication (the own block's root is the same for all of a pixel's
// candidates); the quotient in FP64 is formed only for two candidates whose FP32 values are
// within 2e-6 of each other, some ten times the rounding of those (1 ulp of the root, half of the
// conversion and of the product), so the choice is the FP64 one.  The FP64 division and roots of
// every candidate were a tenth of the sweep (512 pairs of 1242 x 375: 11.0 -> 9.9 ms).  A pixel
// with a matched neighbour below scores its few propagated candidates (up to three runs) in one
// loop of its own lane; a pixel without one (every pixel of the first row) searches all of
// 1..d_max, which would hold up the 63 other lanes of its wave, so such pixels are queued: many
// (the first row) are taken one a lane, few one a wave with a candidate per lane and a reduction
// over the wave.  The propagation makes
// the rows of a frame sequential; frames are independent workgroups.  Launches of few frames
// (stereo_form; up to 112 of 1242 x 375) take the same maps in strips of columns and blocks of rows,
// k_stereo_strip, a launch per block of rows (1 pair: 5.15 -> 0.68 ms, 32: 5.3 -> 1.6 ms).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>

#include "ld.h"
#include "ld_internal.h"

namespace {

constexpr int kT = 512;        // sweep threads per map: a workgroup holds both maps of a frame, 16 waves
constexpr int kWaves = kT / 64;
constexpr int kRowWords = 2;   // words of a new row per thread and image: widths up to 4 kT kRowWords
constexpr int kPad = 8;        // zero columns on both sides of the column sums (block sums four at a time)
constexpr int kTL = 320;       // consistency check threads (a 1242-pixel row in one workgroup)
constexpr int kLrcPx = 4;      // consistency check pixels a thread
constexpr int kLrcRows = 8;    // consistency check rows a workgroup
constexpr int kNone = 1 << 20; // an absent neighbour in the sorted propagation bounds

__host__ __device__ constexpr size_t round16(size_t x) { return (x + 15) / 16 * 16; }

size_t stereo_lds(int W, int rho) {
    const size_t Wp = (size_t)(W + 3) / 4 * 4;
    const size_t rows = 2 * (size_t)rho + 1;
    return round16(2 * rows * Wp)                      // image rings (u8)
           + 4 * sizeof(int32_t) * (Wp + 2 * kPad)     // column sums S, Q of both images
           + 2 * sizeof(int32_t) * Wp                  // block sums S of both images
           + 4 * sizeof(int32_t) * Wp                  // block variances and their reciprocal roots, both images
           + 4 * Wp                                    // disparities of the previous and the current row, both maps
           + 2 * sizeof(uint16_t) * Wp + 16;           // queues of full-range pixels and their lengths, both maps
}

// The best candidate so far: its FP32 cost without the own block's factor, its exact numerator and
// its disparity (0: none).
struct Best {
    float f = -3.0e38f;
    int num = 0, d = 0;
};

// The union of [l - tau, l + tau] over the matched neighbours (l > 0) within 1 .. d_max, as up to
// three disjoint runs in increasing order (an empty one has b < a).
struct Runs { int a0, b0, a1, b1, a2, b2; };
__device__ __forceinline__ Runs runs_of(int l0, int l1, int l2, int tau, int d_max) {
    int s0 = l0 ? l0 : kNone, s1 = l1 ? l1 : kNone, s2 = l2 ? l2 : kNone;
    {   // s0 <= s1 <= s2
        const int a = min(s0, s1), c = max(s0, s1);
        const int hi3 = max(c, s2), mid = min(c, s2);
        s0 = min(a, mid); s1 = max(a, mid); s2 = hi3;
    }
    // (written as selects: a wave's lanes take every path)
    Runs r{max(s0 - tau, 1), min(s0 + tau, d_max), 1, 0, 1, 0};
    {
        const int lo = s1 - tau, hi = min(s1 + tau, d_max);
        const bool in = s1 < kNone, join = lo <= r.b0 + 1, own = in && !join;
        r.b0 = in && join ? max(r.b0, hi) : r.b0;
        r.a1 = own ? lo : 1;
        r.b1 = own ? hi : 0;
    }
    {
        const int lo = s2 - tau, hi = min(s2 + tau, d_max);
        const bool in = s2 < kNone, two = r.b1 >= r.a1, join = lo <= (two ? r.b1 : r.b0) + 1;
        const bool own = in && !join;
        r.b0 = in && join && !two ? max(r.b0, hi) : r.b0;
        r.b1 = in && join && two ? max(r.b1, hi) : r.b1;
        r.a2 = own && two ? lo : 1;
        r.b2 = own && two ? hi : 0;
        r.a1 = own && !two ? lo : r.a1;
        r.b1 = own && !two ? hi : r.b1;
    }
    return r;
}

template <int RHO>
__global__ __launch_bounds__(2 * kT) void k_stereo(const uint8_t* left, int64_t lp, const uint8_t* right, int64_t rp,
                                               int W, int H, const int32_t* nact, int nframes, int d_max, int tau,
                                               uint8_t* lf, uint8_t* rt) {
    constexpr int K = 2 * RHO + 1, N = K * K;
    constexpr int NW = (K + 3) / 4;                                   // words of a block row
    constexpr uint32_t kLastMask = (K % 4 == 0) ? 0xFFFFFFFFu : ((1u << (8 * (K % 4))) - 1u);
    constexpr int kC = (RHO + 3) / 4;                                 // column-sum quads either side
    extern __shared__ __align__(16) unsigned char smem[];
    // NW words holding bytes o .. o + 4 NW - 1 of the row in slot j of a ring whose word g of
    // slot j is word g K + j (the words past a row's last byte lie in the LDS allocation, their
    // bytes are cleared or unused)
    auto fetch = [&](const uint32_t* ring, int j, int o, uint32_t (&w)[NW]) {
        const uint32_t* r = ring + (o >> 2) * K + j;
        const uint32_t s = (uint32_t)(o & 3);
        uint32_t x[NW + 1];
#pragma unroll
        for (int k = 0; k <= NW; ++k) x[k] = r[k * K];
#pragma unroll
        for (int k = 0; k < NW; ++k) w[k] = __builtin_amdgcn_alignbyte(x[k + 1], x[k], s);
    };
    const int b = blockIdx.x, t = threadIdx.x;
    const int nf = nact != nullptr ? min(*nact, nframes) : nframes;
    if (b >= nf) return;
    // the workgroup's first half sweeps the left map (own image left, blocks of the right image
    // at u - d), the second the right map (own image right, blocks of the left image at u + d);
    // each half keeps the ring, column sums, block sums and variances of its own image, which
    // the other half reads as the partner's
    const int m = t / kT, tm = t % kT;
    const uint8_t* ga = (m == 0 ? left + (int64_t)b * H * lp : right + (int64_t)b * H * rp);
    const int64_t pa = m == 0 ? lp : rp;
    uint8_t* out = (m == 0 ? lf : rt) + (int64_t)b * H * W;
    const int sgn = m == 0 ? -1 : 0;                              // x = u + (d ^ sgn) - sgn
    const int Wp = (W + 3) / 4 * 4, Wq = Wp / 4;
    uint32_t* ring0 = reinterpret_cast<uint32_t*>(smem);
    uint32_t* ring1 = ring0 + K * Wq;
    int32_t* colS0 = reinterpret_cast<int32_t*>(smem + round16(2 * (size_t)K * Wp)) + kPad;
    int32_t* colQ0 = colS0 + Wp + 2 * kPad;
    int32_t* colS1 = colQ0 + Wp + 2 * kPad;
    int32_t* colQ1 = colS1 + Wp + 2 * kPad;
    int32_t* S0 = colQ1 + Wp + kPad;
    int32_t* S1 = S0 + Wp;
    float* rq0 = reinterpret_cast<float*>(S1 + Wp);    // 1 / sqrt(n Q - S^2); 0 where no block fits or it is flat
    float* rq1 = rq0 + Wp;
    int32_t* var0 = reinterpret_cast<int32_t*>(rq1 + Wp);   // n Q - S^2
    int32_t* var1 = var0 + Wp;
    uint8_t* pc = reinterpret_cast<uint8_t*>(var1 + Wp);
    uint16_t* queues = reinterpret_cast<uint16_t*>(pc + 4 * Wp);
    int* qns = reinterpret_cast<int*>(queues + 2 * Wp);
    uint32_t* ringA = m == 0 ? ring0 : ring1;
    uint32_t* ringB = m == 0 ? ring1 : ring0;
    uint8_t* ringA8 = reinterpret_cast<uint8_t*>(ringA);
    int32_t* colS_a = m == 0 ? colS0 : colS1;
    int32_t* colQ_a = m == 0 ? colQ0 : colQ1;
    int32_t* S_a = m == 0 ? S0 : S1;
    const int32_t* S_b = m == 0 ? S1 : S0;
    float* rq_a = m == 0 ? rq0 : rq1;
    const float* rq_b = m == 0 ? rq1 : rq0;
    int32_t* var_a = m == 0 ? var0 : var1;
    const int32_t* var_b = m == 0 ? var1 : var0;
    uint8_t* prev = pc + (2 * m) * Wp;
    uint8_t* cur = pc + (2 * m + 1) * Wp;
    uint16_t* queue = queues + m * Wp;
    int* qn = qns + m;
    // rows outside the matched band are 0 (every row when no block fits)
    const bool none = W < K || H < K;
    for (int v = 0; v < H; ++v) {
        if (!none && v >= RHO && v <= H - 1 - RHO) continue;
        for (int u = tm; u < W; u += kT) out[(int64_t)v * W + u] = 0;
    }
    if (none) return;
    // the first 2 rho + 1 rows of the own image (slot v mod K), bytes past the width cleared;
    // its column sums
    const int vb = H - 1 - RHO;
    for (int v = vb - RHO; v <= vb + RHO; ++v) {
        const int slot = v % K;
        for (int u = tm; u < Wp; u += kT) ringA8[((u >> 2) * K + slot) * 4 + (u & 3)] = u < W ? ga[(int64_t)v * pa + u] : 0;
    }
    for (int i = tm; i < kPad; i += kT) {
        colS_a[-1 - i] = colQ_a[-1 - i] = 0;
        colS_a[Wp + i] = colQ_a[Wp + i] = 0;
    }
    if (tm == 0) *qn = 0;
    __syncthreads();
    for (int u = tm; u < Wp; u += kT) {
        int sa = 0, qa = 0;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int x = ringA8[((u >> 2) * K + j) * 4 + (u & 3)];
            sa += x; qa += x * x;
        }
        colS_a[u] = sa; colQ_a[u] = qa;
    }
    // the FP64 cost of a candidate (num its numerator, xc its column)
    auto cost = [&](int num, int va, int xc) -> double {
        return (double)num / (sqrt((double)va) * sqrt((double)var_b[xc]));
    };
    // the candidate of disparity d for the pixel at u against the best so far (b.d = 0: none); ties
    // go to the smaller d.  The numerator n P - S_a S_b is exact in 32 bits (each product below
    // 2^30 for rho <= 5); a candidate whose block leaves the image or is flat is scored at a
    // stand-in position and not taken.  The cost decides by its FP64 value, but is compared by
    // an FP32 one first, num rounded times the reciprocal root of the variance (v_rsq_f32,
    // within an ulp): that is within 4e-7 of the true ratio (the own block's factor left out), so
    // two candidates further apart than 2e-6 of the larger are in the order of their FP64
    // costs, and only the others take the two square roots and the division.
    auto score = [&](const uint32_t (&A)[K][NW], int u, int Sa, int d, Best& b) {
        const int x = u + (d ^ sgn) - sgn;
        const bool inr = (unsigned)(x - RHO) <= (unsigned)(W - 1 - 2 * RHO);
        const int xc = inr ? x : RHO;
        const float rb = rq_b[xc];
        uint32_t P = 0;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            uint32_t Bw[NW];
            fetch(ringB, j, xc - RHO, Bw);
#pragma unroll
            for (int k = 0; k < NW; ++k) P = __builtin_amdgcn_udot4(A[j][k], Bw[k], P, false);
        }
        const int num = __mul24(N, (int)P) - __mul24(Sa, S_b[xc]);
        const float f = (float)num * rb;
        const float g = f - b.f, tol = fmaxf(fabsf(f), fabsf(b.f)) * 2.0e-6f;
        const bool on = inr & (rb > 0.0f);
        bool take = on & (g > tol);
        if (on & (fabsf(g) <= tol)) {
            const int va = var_a[u];
            const double c = cost(num, va, xc), bc = cost(b.num, va, u + (b.d ^ sgn) - sgn);
            take = c > bc || (c == bc && d < b.d);
        }
        b.f = take ? f : b.f;
        b.num = take ? num : b.num;
        b.d = take ? d : b.d;
    };
    auto own_block = [&](int u, uint32_t (&A)[K][NW]) {
#pragma unroll
        for (int j = 0; j < K; ++j) {
            fetch(ringA, j, u - RHO, A[j]);
            A[j][NW - 1] &= kLastMask;        // the bytes past the block are cleared
        }
    };
    for (int v = vb; v >= RHO; --v) {
        const bool more = v > RHO;             // a row v - rho - 1 follows
        const int vlo = v - RHO;
        __syncthreads();
        // block sums, variances n Q - S^2 and their reciprocal roots of the own image, four
        // columns a thread (root 0 where no block fits)
        for (int g = tm; g < Wq; g += kT) {
            int cs[2][4 * (2 * kC + 1)];
            const int32_t* arr[2] = {colS_a, colQ_a};
#pragma unroll
            for (int a = 0; a < 2; ++a) {
#pragma unroll
                for (int c = -kC; c <= kC; ++c) {
                    const int4 q = *reinterpret_cast<const int4*>(arr[a] + 4 * (g + c));
                    cs[a][4 * (c + kC) + 0] = q.x; cs[a][4 * (c + kC) + 1] = q.y;
                    cs[a][4 * (c + kC) + 2] = q.z; cs[a][4 * (c + kC) + 3] = q.w;
                }
            }
            int bs[2][4];
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                int s_ = 0;
#pragma unroll
                for (int mm = -RHO; mm <= RHO; ++mm) s_ += cs[a][4 * kC + mm];
                bs[a][0] = s_;
#pragma unroll
                for (int i = 1; i < 4; ++i) {
                    s_ += cs[a][4 * kC + i + RHO] - cs[a][4 * kC + i - 1 - RHO];
                    bs[a][i] = s_;
                }
            }
            int4 oa, ov;
            float4 orq;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int u = 4 * g + i;
                const bool fits = u >= RHO && u <= W - 1 - RHO;
                const int va = N * bs[1][i] - bs[0][i] * bs[0][i];
                (&oa.x)[i] = fits ? bs[0][i] : 0;
                (&ov.x)[i] = va;
                (&orq.x)[i] = fits && va > 0 ? __builtin_amdgcn_rsqf((float)va) : 0.0f;
            }
            *reinterpret_cast<int4*>(S_a + 4 * g) = oa;
            *reinterpret_cast<int4*>(var_a + 4 * g) = ov;
            *reinterpret_cast<float4*>(rq_a + 4 * g) = orq;
        }
        __syncthreads();
        // the own image's next row from HBM while this one is matched: four bytes a word for
        // words tm and tm + kT, byte loads at clamped positions (their values are masked when
        // the words are put together), so that nothing waits for them before the row is done
        uint32_t ra[kRowWords][4];
        {
            const uint8_t* pa0 = ga + (int64_t)(more ? vlo - 1 : vlo) * pa;
#pragma unroll
            for (int k = 0; k < kRowWords; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i) ra[k][i] = pa0[min(4 * (tm + k * kT) + i, W - 1)];
        }
        // pixels with a matched neighbour below: the union of [l - tau, l + tau] over those
        // neighbours, in increasing d, in the pixel's own lane; the others are queued
        const bool first = v == vb;
        for (int u = tm; u < W; u += kT) {
            Best best;
            if (u >= RHO && u <= W - 1 - RHO && rq_a[u] > 0.0f) {
                int l0 = 0, l1 = 0, l2 = 0;
                if (!first) {
                    l0 = u - 1 >= RHO ? prev[u - 1] : 0;
                    l1 = prev[u];
                    l2 = u + 1 <= W - 1 - RHO ? prev[u + 1] : 0;
                }
                if ((l0 | l1 | l2) == 0) {
                    queue[atomicAdd(qn, 1)] = (uint16_t)u;
                } else {
                    Runs r = runs_of(l0, l1, l2, tau, d_max);
                    uint32_t A[K][NW];
                    own_block(u, A);
                    const int Sa = S_a[u];
                    // one loop over all the candidates (a lane's runs follow each other
                    // without waiting for the other lanes' runs to end)
                    const int n = (r.b0 - r.a0 + 1) + max(r.b1 - r.a1 + 1, 0) + max(r.b2 - r.a2 + 1, 0);
                    int d = r.a0, e = r.b0;
                    for (int k = 0; k < n; ++k) {
                        score(A, u, Sa, d, best);
                        const bool nx = d == e;
                        d = nx ? r.a1 : d + 1;
                        e = nx ? r.b1 : e;
                        r.a1 = nx ? r.a2 : r.a1;
                        r.b1 = nx ? r.b2 : r.b1;
                    }
                }
            }
            cur[u] = (uint8_t)best.d;
        }
        __syncthreads();
        // queued pixels: many (the first row) one a lane over all of 1..d_max; few one a wave,
        // candidates 1 + lane, 65 + lane, ..., then the best (largest cost, then smallest d)
        // over the wave.  Both halves take the barrier when either map queued any.
        const int nq = *qn;
        if (qns[0] > 0 || qns[1] > 0) {
            if (nq >= kT / 2) {
                for (int q = tm; q < nq; q += kT) {
                    const int u = queue[q];
                    uint32_t A[K][NW];
                    own_block(u, A);
                    const int Sa = S_a[u];
                    Best best;
                    for (int d = 1; d <= d_max; ++d) score(A, u, Sa, d, best);
                    cur[u] = (uint8_t)best.d;
                }
            } else if (nq > 0) {
                const int wv = tm >> 6, lane = tm & 63;
                for (int q = wv; q < nq; q += kWaves) {
                    const int u = queue[q];
                    uint32_t A[K][NW];
                    own_block(u, A);
                    const int Sa = S_a[u];
                    Best b;
                    for (int d = 1 + lane; d <= d_max; d += 64) score(A, u, Sa, d, b);
                    int best = b.d;
                    double bc = best != 0 ? cost(b.num, var_a[u], u + (best ^ sgn) - sgn) : -__builtin_inf();
#pragma unroll
                    for (int off = 32; off >= 1; off >>= 1) {
                        const double oc = __shfl_xor(bc, off);
                        const int od = __shfl_xor(best, off);
                        if (od != 0 && (best == 0 || oc > bc || (oc == bc && od < best))) { best = od; bc = oc; }
                    }
                    if (lane == 0) cur[u] = (uint8_t)best;
                }
            }
            __syncthreads();
        }
        // the own image's next row replaces row v + rho in its ring and column sums; the row out
        if (more) {
            const int slot = (v + RHO) % K;
#pragma unroll
            for (int k = 0; k < kRowWords; ++k) {
                const int g = tm + k * kT;
                if (g >= Wq) continue;
                uint32_t na = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (4 * g + i < W) na |= ra[k][i] << (8 * i);
                const uint32_t oa = ringA[g * K + slot];
                ringA[g * K + slot] = na;
                int4 s1 = *reinterpret_cast<int4*>(colS_a + 4 * g), q1 = *reinterpret_cast<int4*>(colQ_a + 4 * g);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int xn = (na >> (8 * i)) & 0xFF, xo = (oa >> (8 * i)) & 0xFF;
                    (&s1.x)[i] += xn - xo; (&q1.x)[i] += xn * xn - xo * xo;
                }
                *reinterpret_cast<int4*>(colS_a + 4 * g) = s1; *reinterpret_cast<int4*>(colQ_a + 4 * g) = q1;
            }
        }
        for (int u = tm; u < W; u += kT) out[(int64_t)v * W + u] = cur[u];
        if (tm == 0) *qn = 0;
        uint8_t* tmp = prev; prev = cur; cur = tmp;
    }
}

// ------------------------------------------------------------------------------------------
// The same maps for few pairs.  One workgroup a frame leaves all but a few CUs idle, so a launch
// takes T rows of every frame and map, a workgroup E columns of them: a row needs the row
// below one column further on either side, so of the E columns 2 (T - 1) are worked on again by
// the neighbours, and the lowest row's neighbours come from the map that the launch before
// wrote.  LP lanes share a pixel's candidates.  The image rows of both images and the block
// statistics of the T rows are formed in LDS first, so a row of the sweep has one barrier.  A
// row's time, about 1.2 us, is its chain: neighbours, range, one candidate a lane (14 dot
// products on 14 pairs of LDS words), the best over the lanes, barrier; the statistics and image
// rows take about 5 us a launch.
template <int RHO, int LP, int E, int T>
struct Strip {
    static constexpr int K = 2 * RHO + 1, N = K * K, NT = E * LP, kUse = E - 2 * (T - 1), kRows = T + 2 * RHO;
    static constexpr int kA = (E + 2 * RHO + 3 + 8) / 4;             // words of a row of the own image
    static constexpr int kB = (E + 255 + 2 * RHO + 3 + 8) / 4;       // and of the other one
    static_assert(kUse > 0 && T % 2 == 0, "columns left after the halo; pairs of words aligned behind T rows");
};

template <int RHO, int LP, int E, int T>
__global__ __launch_bounds__(E* LP) void k_stereo_strip(const uint8_t* left, int64_t lp, const uint8_t* right,
                                                        int64_t rp, int W, int H, const int32_t* nact, int nframes,
                                                        int d_max, int tau, uint8_t* lf, uint8_t* rt, int v_start) {
    using G = Strip<RHO, LP, E, T>;
    constexpr int K = G::K, N = G::N, NT = G::NT, NW = (K + 3) / 4;
    constexpr uint32_t kLastMask = (K % 4 == 0) ? 0xFFFFFFFFu : ((1u << (8 * (K % 4))) - 1u);
    extern __shared__ __align__(16) unsigned char smem[];
    const int b = blockIdx.z, m = blockIdx.y, t = threadIdx.x;
    const int nf = nact != nullptr ? min(*nact, nframes) : nframes;
    if (b >= nf) return;
    const uint8_t* ga = (m == 0 ? left + (int64_t)b * H * lp : right + (int64_t)b * H * rp);
    const uint8_t* gb = (m == 0 ? right + (int64_t)b * H * rp : left + (int64_t)b * H * lp);
    const int64_t pa = m == 0 ? lp : rp, pb = m == 0 ? rp : lp;
    uint8_t* out = (m == 0 ? lf : rt) + (int64_t)b * H * W;
    const int sgn = m == 0 ? -1 : 0;                                  // x = u + (d ^ sgn) - sgn
    const int vb = H - 1 - RHO, rows = min(T, v_start - RHO + 1);
    const int x0 = blockIdx.x * G::kUse, ub = x0 - (T - 1);           // the columns written; the first worked on
    // rows outside the matched band are 0
    const int xe = min(x0 + G::kUse, W);
    if (v_start == vb)
        for (int v = vb + 1; v < H; ++v)
            for (int u = x0 + t; u < xe; u += NT) out[(int64_t)v * W + u] = 0;
    if (v_start - rows < RHO)
        for (int v = 0; v < RHO; ++v)
            for (int u = x0 + t; u < xe; u += NT) out[(int64_t)v * W + u] = 0;
    const int wb = E + d_max;                                         // other columns xb0 .. xb0 + wb - 1
    const int xb0 = m == 0 ? ub - d_max : ub;
    uint32_t* ta = reinterpret_cast<uint32_t*>(smem);                 // rows v_start + rho - r, columns ca ..
    uint32_t* tb = ta + G::kRows * G::kA;                             // columns cb ..
    int32_t* Sb = reinterpret_cast<int32_t*>(tb + G::kRows * G::kB);  // T x wb: block sums, variances, reciprocal roots
    int32_t* vrb = Sb + T * wb;
    float* rqb = reinterpret_cast<float*>(vrb + T * wb);
    int32_t* Sa = reinterpret_cast<int32_t*>(rqb + T * wb);           // T x E
    int32_t* vra = Sa + T * E;
    float* rqa = reinterpret_cast<float*>(vra + T * E);
    const int na = E + 2 * RHO, nb = wb + 2 * RHO;                    // columns with vertical sums
    int2* col = reinterpret_cast<int2*>(rqa + T * E);   // 2 x (na + nb): sum and sum of squares
    int* prev = reinterpret_cast<int*>(col + 2 * (na + nb));          // 2 x (E + 2)
    const int ca = (ub - RHO) & ~3, cb = (xb0 - RHO) & ~3;
    // image rows (0 outside the image)
    auto stage = [&](uint32_t* to, int stride, const uint8_t* g, int64_t pitch, int c0, int ncols) {
        const int wn = (ncols + 3) / 4;
        for (int i = t; i < G::kRows * wn; i += NT) {
            const int r = i / wn, w = i - r * wn, v = v_start + RHO - r, x = c0 + 4 * w;
            // four bytes from x on, moved to where they belong at the image's sides
            const int xc = min(max(x, 0), W - 4), sh = x - xc;
            uint32_t q;
            __builtin_memcpy(&q, g + (int64_t)max(v, 0) * pitch + xc, 4);
            q = sh < 0 ? (sh > -4 ? q << (-8 * sh) : 0u) : (sh < 4 ? q >> (8 * sh) : 0u);
            to[r * stride + w] = q;
        }
    };
    stage(ta, G::kA, ga, pa, ca, ub + E + RHO - ca);
    stage(tb, G::kB, gb, pb, cb, xb0 + wb + RHO - cb);
    for (int i = t; i < E + 2; i += NT) {                             // the row below: columns ub - 1 .. ub + E
        const int u = ub - 1 + i;
        prev[i] = v_start != vb && u >= 0 && u < W ? out[(int64_t)(v_start + 1) * W + u] : 0;
        prev[E + 2 + i] = 0;
    }
    __syncthreads();
    // block statistics row by row: each thread slides the vertical sums of its columns, then forms
    // the sums over 2 rho + 1 of them
    {
        constexpr int kCols = (2 * E + 255 + 4 * RHO + NT - 1) / NT;
        int cs[kCols], cq[kCols];
        const uint8_t* src[kCols];
        int step[kCols];
#pragma unroll
        for (int k = 0; k < kCols; ++k) {
            const int i = t + k * NT;
            const bool own = i < na;
            src[k] = reinterpret_cast<const uint8_t*>(own ? ta : tb) + (own ? ub - RHO - ca + i : xb0 - RHO - cb + min(i - na, nb - 1));
            step[k] = 4 * (own ? G::kA : G::kB);
            cs[k] = cq[k] = 0;
#pragma unroll
            for (int j = 0; j < K - 1; ++j) {
                const int x = src[k][j * step[k]];
                cs[k] += x;
                cq[k] += x * x;
            }
        }
        for (int r = 0; r < rows; ++r) {
            int2* c = col + (r & 1) * (na + nb);
#pragma unroll
            for (int k = 0; k < kCols; ++k) {
                const int i = t + k * NT, x = src[k][(r + K - 1) * step[k]], y = src[k][r * step[k]];
                cs[k] += x;
                cq[k] += x * x;
                if (i < na + nb) c[i] = make_int2(cs[k], cq[k]);
                cs[k] -= y;
                cq[k] -= y * y;
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kCols; ++k) {
                const int i = t + k * NT;
                if (i >= E + wb) continue;
                const bool own = i < E;
                const int2* p = c + (own ? i : na + (i - E));
                int sum = 0, sq = 0;
#pragma unroll
                for (int j = 0; j < K; ++j) { sum += p[j].x; sq += p[j].y; }
                const int u = own ? ub + i : xb0 + (i - E);
                const bool fits = u >= RHO && u <= W - 1 - RHO;
                const int var = N * sq - sum * sum;
                const float rq = fits && var > 0 ? __builtin_amdgcn_rsqf((float)var) : 0.0f;
                if (own) { Sa[r * E + i] = sum; vra[r * E + i] = var; rqa[r * E + i] = rq; }
                else { Sb[r * wb + i - E] = sum; vrb[r * wb + i - E] = var; rqb[r * wb + i - E] = rq; }
            }
        }
    }
    __syncthreads();
    const int p = t / LP, sub = t % LP, u = ub + p;
    for (int r = 0; r < rows; ++r) {
        const int v = v_start - r;
        const int* pv = prev + (r & 1) * (E + 2);
        int* cur = prev + ((r & 1) ^ 1) * (E + 2);
        const int32_t* S = Sb + r * wb;
        const int32_t* vr = vrb + r * wb;
        const float* rq = rqb + r * wb;
        Best best;
        // the better of two, as in the frame sweep: by the FP32 values unless they are close
        auto keep = [&](const Best& q, bool on) {
            const float g = q.f - best.f, tol = fmaxf(fabsf(q.f), fabsf(best.f)) * 2.0e-6f;
            bool take = on & (g > tol);
            if (on & (fabsf(g) <= tol)) {
                int va = vra[r * E + p];
                asm volatile("" : "+v"(va));                 // (its square root stays in this branch)
                auto cost = [&](const Best& z) -> double {
                    return (double)z.num / (sqrt((double)va) * sqrt((double)vr[u + (z.d ^ sgn) - sgn - xb0]));
                };
                const double c = cost(q), bc = cost(best);
                take = c > bc || (c == bc && q.d < best.d);
            }
            best.f = take ? q.f : best.f;
            best.num = take ? q.num : best.num;
            best.d = take ? q.d : best.d;
        };
        if (rqa[r * E + p] > 0.0f) {
            int l0 = pv[p], l1 = pv[p + 1], l2 = pv[p + 2];
            l0 = u - 1 >= RHO ? l0 : 0;
            l2 = u + 1 <= W - 1 - RHO ? l2 : 0;
            uint32_t A[K][NW];
            {
                const int o = u - RHO - ca;
                const uint32_t* w = ta + r * G::kA + (o >> 2);
#pragma unroll
                for (int j = 0; j < K; ++j) {
#pragma unroll
                    for (int k = 0; k < NW; ++k) A[j][k] = __builtin_amdgcn_alignbyte(w[j * G::kA + k + 1], w[j * G::kA + k], (uint32_t)(o & 3));
                    A[j][NW - 1] &= kLastMask;
                }
            }
            const int sa = Sa[r * E + p];
            const bool all = (l0 | l1 | l2) == 0;            // no matched neighbour: 1 .. d_max
            Runs q = runs_of(all ? 1 : l0, l1, l2, tau, d_max);
            q.b0 = all ? d_max : q.b0;
            const int n0 = q.b0 - q.a0 + 1, n1 = n0 + max(q.b1 - q.a1 + 1, 0), n2 = n1 + max(q.b2 - q.a2 + 1, 0);
            for (int k = sub; k < n2; k += LP) {
                int d = k + q.a0;
                d = k >= n0 ? k + q.a1 - n0 : d;
                d = k >= n1 ? k + q.a2 - n1 : d;
                const int xi = min(max(u + (d ^ sgn) - sgn - xb0, 0), wb - 1);   // a column's place in the statistics
                const float rb = rq[xi];
                const int sb = S[xi], o = xi + xb0 - RHO - cb;
                const uint32_t* w = tb + r * G::kB + (o >> 2);
                uint32_t P = 0;
#pragma unroll
                for (int j = 0; j < K; ++j)
#pragma unroll
                    for (int i = 0; i < NW; ++i)
                        P = __builtin_amdgcn_udot4(A[j][i], __builtin_amdgcn_alignbyte(w[j * G::kB + i + 1], w[j * G::kB + i], (uint32_t)(o & 3)), P, false);
                Best c;
                c.num = __mul24(N, (int)P) - __mul24(sa, sb);
                c.f = (float)c.num * rb;
                c.d = d;
                keep(c, rb > 0.0f);                          // 0: the block leaves the image or is flat
            }
        }
        // the best of the pixel's lanes: pairs, quads, then (both quads of eight lanes each hold
        // one value) the mirror of eight
        static_assert(LP == 4 || LP == 8, "lanes a pixel");
        auto merge = [&](auto ctl) {
            constexpr int C = decltype(ctl)::value;
            Best c;
            c.f = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(best.f), C, 0xF, 0xF, true));
            c.num = __builtin_amdgcn_update_dpp(0, best.num, C, 0xF, 0xF, true);
            c.d = __builtin_amdgcn_update_dpp(0, best.d, C, 0xF, 0xF, true);
            keep(c, (c.d != 0) & (c.d != best.d));
        };
        merge(std::integral_constant<int, 0xB1>{});                            // quad_perm 1 0 3 2
        merge(std::integral_constant<int, 0x4E>{});                            // quad_perm 2 3 0 1
        if constexpr (LP == 8) merge(std::integral_constant<int, 0x141>{});    // row_half_mirror
        if (sub == 0) {
            cur[p + 1] = best.d;
            if (p >= T - 1 && p < T - 1 + G::kUse && u < W) out[(int64_t)v * W + u] = (uint8_t)best.d;
        }
        __syncthreads();
    }
}

// l(u) = l_left(u) unless it is 0, u - l(u) < 0 or |l(u) - l_right(u - l(u))| > tr.  A workgroup
// takes kLrcRows rows of a frame (grid: row groups, frames), kLrcPx consecutive pixels a thread.
template <int PX>
__global__ __launch_bounds__(kTL) void k_lrc(const uint8_t* lf, const uint8_t* rt, int W, int H, const int32_t* nact,
                                            int nframes, int tr, uint8_t* out, int64_t op) {
    const int b = blockIdx.y;
    const int nf = nact != nullptr ? min(*nact, nframes) : nframes;
    if (b >= nf) return;
    for (int v = blockIdx.x * kLrcRows; v < min(H, (int)(blockIdx.x + 1) * kLrcRows); ++v) {
        const uint8_t* L = lf + ((int64_t)b * H + v) * W;
        const uint8_t* R = rt + ((int64_t)b * H + v) * W;
        uint8_t* O = out + ((int64_t)b * H + v) * op;
        for (int u0 = threadIdx.x * PX; u0 < W; u0 += kTL * PX) {
            uint8_t l[PX];
#pragma unroll
            for (int k = 0; k < PX; ++k) l[k] = L[min(u0 + k, W - 1)];
#pragma unroll
            for (int k = 0; k < PX; ++k) {
                const int u = u0 + k, lk = l[k];
                if (u >= W) break;
                int o = 0;
                if (lk > 0 && u - lk >= 0 && abs(lk - (int)R[u - lk]) <= tr) o = lk;
                O[u] = (uint8_t)o;
            }
        }
    }
}

// The same check over the maps as one flat array when the left map and the output are whole
// words apart and the output rows are contiguous: a thread loads a word of four disparities,
// gathers their right-map partners (same row: u - l >= 0) and stores a word.
__global__ __launch_bounds__(256) void k_lrc_words(const uint8_t* lf, const uint8_t* rt, int W, int64_t HW,
                                                  const int32_t* nact, int nframes, int tr, uint8_t* out) {
    const int nf = nact != nullptr ? min(*nact, nframes) : nframes;
    const int64_t total = (int64_t)nf * HW;
    const int64_t p0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (p0 >= total) return;
    const int64_t row = p0 / W;
    int u = (int)(p0 - row * W);
    if (p0 + 4 <= total) {
        const uint32_t w = *reinterpret_cast<const uint32_t*>(lf + p0);
        uint32_t o = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int l = (int)((w >> (8 * i)) & 0xFFu);
            const int ui = u + i < W ? u + i : u + i - W;     // a word spans at most two rows
            if (l > 0 && ui - l >= 0 && abs(l - (int)rt[p0 + i - l]) <= tr) o |= (uint32_t)l << (8 * i);
        }
        *reinterpret_cast<uint32_t*>(out + p0) = o;
    } else {
        for (int64_t p = p0; p < total; ++p, ++u) {      // the last few bytes
            if (u == W) u = 0;
            const int l = lf[p];
            out[p] = (l > 0 && u - l >= 0 && abs(l - (int)rt[p - l]) <= tr) ? (uint8_t)l : 0;
        }
    }
}

template <int RHO, int LP, int E, int T>
void launch_strips(const uint8_t* left, int64_t lp, const uint8_t* right, int64_t rp, const ldi_frame_view& V, int tau,
                   uint8_t* lf, uint8_t* rt, hipStream_t st) {
    using G = Strip<RHO, LP, E, T>;
    const size_t lds = stereo_strip_lds(RHO, E, T, V.d_max);
    allow_lds<k_stereo_strip<RHO, LP, E, T>>(lds);
    const dim3 grid((V.W + G::kUse - 1) / G::kUse, 2, V.active);
    for (int v = V.H - 1 - RHO; v >= RHO; v -= T)
        hipLaunchKernelGGL((k_stereo_strip<RHO, LP, E, T>), grid, dim3(G::NT), lds, st, left, lp, right, rp, V.W, V.H,
                           V.nact, V.active, V.d_max, tau, lf, rt, v);
}

template <int RHO>
void launch(const uint8_t* left, int64_t lp, const uint8_t* right, int64_t rp, const ldi_frame_view& V, int tau,
            uint8_t* lf, uint8_t* rt, hipStream_t st) {
    switch (stereo_form(V.W, V.H, RHO, V.d_max, tau, V.active)) {
        case StereoForm::kStrip8: return launch_strips<RHO, 8, 64, 16>(left, lp, right, rp, V, tau, lf, rt, st);
        case StereoForm::kStrip4: return launch_strips<RHO, 4, 128, 16>(left, lp, right, rp, V, tau, lf, rt, st);
        case StereoForm::kStrip4Short: return launch_strips<RHO, 4, 128, 8>(left, lp, right, rp, V, tau, lf, rt, st);
        case StereoForm::kSweep: break;
    }
    const size_t lds = stereo_lds(V.W, RHO);
    allow_lds<k_stereo<RHO>>(lds);
    hipLaunchKernelGGL(k_stereo<RHO>, dim3(V.active), dim3(2 * kT), lds, st, left, lp, right, rp, V.W, V.H, V.nact,
                       V.active, V.d_max, tau, lf, rt);
}

}  // namespace

extern "C" ld_status ld_stereo(ld_frame f, const uint8_t* left, int64_t left_pitch, const uint8_t* right,
                               int64_t right_pitch, int32_t rho, int32_t tau, int32_t tr_lrc, uint8_t* disp_out,
                               int64_t disp_pitch, uint8_t* disp_lf, uint8_t* disp_rt, void* hip_stream) {
    LdRange rr_("ld_stereo");
    ldi_frame_view V;
    if (!f || !left || !right || !disp_out || !disp_lf || !disp_rt || ldi_frame_get_view(f, &V) != LD_OK)
        return LD_E_INVAL;
    if (rho < 1 || rho > 5 || tau < 0 || tau > 255 || tr_lrc < 0 || V.d_max > 255) return LD_E_INVAL;
    if (left_pitch < V.W || right_pitch < V.W || disp_pitch < V.W) return LD_E_INVAL;
    if (stereo_lds(V.W, rho) > 160 * 1024 || V.W > 4 * kT * kRowWords) return LD_E_INVAL;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (V.active > 0) {
        switch (rho) {
            case 1: launch<1>(left, left_pitch, right, right_pitch, V, tau, disp_lf, disp_rt, st); break;
            case 2: launch<2>(left, left_pitch, right, right_pitch, V, tau, disp_lf, disp_rt, st); break;
            case 3: launch<3>(left, left_pitch, right, right_pitch, V, tau, disp_lf, disp_rt, st); break;
            case 4: launch<4>(left, left_pitch, right, right_pitch, V, tau, disp_lf, disp_rt, st); break;
            default: launch<5>(left, left_pitch, right, right_pitch, V, tau, disp_lf, disp_rt, st); break;
        }
        const int64_t HW = (int64_t)V.W * V.H;
        if (disp_pitch == V.W && ((uintptr_t)disp_lf & 3) == 0 && ((uintptr_t)disp_out & 3) == 0) {
            const int64_t words = (V.active * HW + 3) / 4;
            hipLaunchKernelGGL(k_lrc_words, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, st, disp_lf, disp_rt,
                               V.W, HW, V.nact, V.active, tr_lrc, disp_out);
        } else {
            const unsigned gx = (unsigned)((V.H + kLrcRows - 1) / kLrcRows);
            hipLaunchKernelGGL(k_lrc<kLrcPx>, dim3(gx, V.active), dim3(kTL), 0, st, disp_lf, disp_rt, V.W, V.H,
                               V.nact, V.active, tr_lrc, disp_out, disp_pitch);
        }
    }
    if (hipGetLastError() != hipSuccess) return LD_E_HIP;
    return ldi_frame_set_last(f, hip_stream);
}
