// Harmonic summing and peak candidates on the f-fdot power plane (Sec. 3:
// a pulsed signal spreads its power over harmonics, whose powers are added
// to the fundamental's before the search for peaks, and the power is
// compared with a precomputed threshold to find candidates).
//
// A constant-fdot signal at (r, z) has its h-th harmonic at (h r, h z).  On
// a plane P[K][N] with rows z_k = (k - c) dz, c = (K - 1)/2, the H-fold sum
// at the fundamental (k, r) is S_H[k][r] = sum_{h=1}^{H} P[c + h (k - c)][h r]
// over the fundamentals whose harmonics all lie on the plane: r < ceil(N/H),
// |k - c| <= floor(c/H).  Harmonics of grid points are grid points, so the
// sums are exact gathers; they are formed in FP32 in the order h = 1..H, so
// a fold built on top of the previous one (H/2 terms already summed) equals
// the fold built from scratch bit for bit.
//
// Memory: the plane is read with stride h along a row for harmonic h, so
// each harmonic touches whole rows of the plane; folding up to 2^f reads
// about half a plane per fold on top of the previous fold's sums.  The
// kernels are gathers bound by the lines they fetch; a lane owns a few
// fundamental columns and walks their harmonics with independent loads.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/fdas.h"
#include "fdas_internal.h"

namespace fdas {

namespace {

constexpr int kHarmThreads = 256;
constexpr int kHScanThreads = 256;

// ---- chains of folds on one plane ------------------------------------------------
//
// S_H[k][r] continues S_{H/2}[k][r] at the same (k, r), so one wave carries its
// columns through all the folds whose domain holds them: the sums stay in
// registers between folds, and each fold's new harmonics are loaded at once
// (kFoldPerLane columns x kFoldGroup harmonics in flight per lane).
//
// Order of the work: harmonic 2h of the fundamental (k, r) is harmonic h of
// (2k, 2r), so columns one octave apart share their plane lines.  The chunks
// of kFoldCols columns are taken in an order in which chunk c and chunk 2c are
// neighbours in time (fold_chunk), with all the rows of a chunk together, so
// the shared lines are found in the caches: the plane lines of the even
// harmonics then come from memory once per octave chain instead of once per
// harmonic.
//
// Measured, folds 2..32 of a plane of 85 x 2^20: 119 us in one launch, 179 us
// as one launch per fold that reads the fold below back; 165 us with the same
// chains without the deal to the XCDs, and 122 / 136 us with runs of 16 / 8
// places instead of 32 (64 and 128 the same as 32).
constexpr int kFoldThreads = 64;      // one wave: its row is uniform
constexpr int kFoldPerLane = 4;       // lane t takes columns t + 64 j
constexpr int kFoldCols = kFoldThreads * kFoldPerLane;
constexpr int kFoldGroup = 8;         // harmonics loaded before they are added
constexpr int kMaxFolds = 7;          // H = 1, 2, .., 64
constexpr int64_t kMaxFoldGridX = int64_t(1) << 22, kMaxFoldGridY = 1 << 15;

struct FoldOut {
    float* p[kMaxFolds];              // S_H at log2 H, or NULL
};

// The p-th chunk of the octave order on [0, P): an odd part q and a power of two
// 2^a with p + 1 = (2q + 1) 2^a give the q-th chunk of the a-th octave from the
// top, (P / 2^(a+1), P / 2^a] counted from 1.  There are as many odd multiples of
// 2^a up to P as chunks in that octave, so each chunk is taken once; the q-th of
// an octave is half the 2q-th of the octave above and sits beside it.
__device__ __forceinline__ int fold_chunk(int p, int P)
{
    const int a = __builtin_ctz((unsigned)(p + 1));
    return (int)((uint32_t)P >> (a + 1)) + ((p + 1) >> (a + 1));
}

// Work item l of [0, P rows): a chunk (place p in the octave order) and a row.
// Consecutive workgroups go to the 8 XCDs in turn, each with an L2 of its own, so
// the items are dealt out in runs of kFoldRun places x all rows per XCD: the
// waves that share lines share an L2.  (The host emulation of the tests builds with a
// short run, to reach several rounds.)
#ifndef FDAS_FOLD_RUN
#define FDAS_FOLD_RUN 32
#endif
constexpr int kFoldRun = FDAS_FOLD_RUN, kXcds = 8;

__device__ __forceinline__ void fold_item(int64_t l, int P, int rows, int& p, int& row)
{
    const int run = P >= kXcds * kFoldRun ? kFoldRun : P / kXcds;
    const int dealt = run > 0 ? P / (kXcds * run) * (kXcds * run) : 0;   // places in full rounds
    if (l >= (int64_t)dealt * rows) {
        const uint32_t i = (uint32_t)(l - (int64_t)dealt * rows);    // < 2^20
        const uint32_t q = i / (uint32_t)rows;
        p = dealt + (int)q;
        row = (int)(i - q * (uint32_t)rows);
        return;
    }
    const uint32_t span = (uint32_t)(kXcds * run) * (uint32_t)rows;   // < 2^20
    const int64_t round = l >> 32 ? l / span : (int64_t)((uint32_t)l / span);
    const uint32_t j = (uint32_t)(l - round * span);
    const uint32_t x = j % kXcds, i = j / kXcds;
    const uint32_t q = i / (uint32_t)rows;
    p = (int)((round * kXcds + x) * run + q);
    row = (int)(i - q * (uint32_t)rows);
}

// Adds harmonics H/2 + 1 .. H of columns r0 + t + 64 j to s, in that order (FULL:
// all of them lie below NH).  Harmonic h is at h (dk N + r) from the centre row.
//
// The last chunk of a row, from 32 harmonics on: columns past NH read the last one's
// values (their sums are not stored), so that no load waits for a test of its own,
// and addresses are a scalar base and a 32-bit offset per lane.  Tested and addressed
// one by one these loads took more registers than there are (166 spilled) and ran
// one after another: the 64-harmonic fold of a 21 x 5000 plane 14.8 us, now 3.9,
// folds 2..64 of 201 x 300000 121 us, now 97; up to 16 harmonics the same either way.
template <int H, bool FULL>
__device__ __forceinline__ void fold_add(const float* __restrict__ centre, int64_t N, int64_t dk,
                                         int64_t r0, int t, int64_t NH, float (&s)[kFoldPerLane])
{
    constexpr int FIRST = H == 1 ? 1 : H / 2 + 1;
    constexpr int COUNT = H == 1 ? 1 : H / 2;
    constexpr int GROUP = COUNT < kFoldGroup ? COUNT : kFoldGroup;
    constexpr bool LAST_VALUES = !FULL && H >= 32;
    const int64_t r = r0 + t;
    uint32_t at[kFoldPerLane];            // column offsets of LAST_VALUES, in bytes
    if constexpr (LAST_VALUES) {
#pragma unroll
        for (int j = 0; j < kFoldPerLane; ++j)
            at[j] = 4u * min((uint32_t)(t + j * kFoldThreads), (uint32_t)(NH - 1 - r0));
    }
#pragma unroll
    for (int g = 0; g < COUNT; g += GROUP) {
        float v[GROUP][kFoldPerLane];
#pragma unroll
        for (int i = 0; i < GROUP; ++i) {
            const int h = FIRST + g + i;
            const float* row = centre + h * (dk * N + (LAST_VALUES ? r0 : r));
#pragma unroll
            for (int j = 0; j < kFoldPerLane; ++j) {
                if constexpr (LAST_VALUES)
                    v[i][j] = *reinterpret_cast<const float*>(
                        reinterpret_cast<const char*>(row) + (uint32_t)h * at[j]);
                else
                    v[i][j] = FULL || r + j * kFoldThreads < NH ? row[h * j * kFoldThreads] : 0.f;
            }
        }
#pragma unroll
        for (int i = 0; i < GROUP; ++i)
#pragma unroll
            for (int j = 0; j < kFoldPerLane; ++j)
                s[j] += v[i][j];
    }
}

__device__ __forceinline__ void fold_put(float* __restrict__ o, int64_t r, int64_t NH,
                                         const float (&s)[kFoldPerLane])
{
#pragma unroll
    for (int j = 0; j < kFoldPerLane; ++j)
        if (r + j * kFoldThreads < NH)
            o[j * kFoldThreads] = s[j];
}

// One stage of a wave's chain: if (dk, r) lies in fold H's domain, add its new
// harmonics and store the sums where the fold is wanted; false ends the chain.
template <int LOG>
__device__ __forceinline__ bool fold_stage(const float* __restrict__ centre, int64_t N, int c,
                                           int64_t dk, int64_t r0, int t, const FoldOut& out,
                                           float (&s)[kFoldPerLane])
{
    constexpr int H = 1 << LOG;
    const int kc = c / H;
    const int64_t NH = (N + H - 1) / H;
    if (dk > kc || -dk > kc || r0 >= NH)
        return false;                 // uniform in the wave
    if (r0 + kFoldCols <= NH)
        fold_add<H, true>(centre, N, dk, r0, t, NH, s);
    else
        fold_add<H, false>(centre, N, dk, r0, t, NH, s);
    if (out.p[LOG] != nullptr)
        fold_put(out.p[LOG] + (dk + kc) * NH + r0 + t, r0 + t, NH, s);
    return true;
}

// The chain of one wave at row offset dk and columns r0 + t + 64 j: folds 2^log_first
// .. 2^log_last, from prev (the fold below the first) or, without it, from the
// plane itself.
__device__ __forceinline__ void fold_chain(const float* __restrict__ plane, int64_t N, int c,
                                           int64_t dk, int64_t r0, int t,
                                           const float* __restrict__ prev, int log_first,
                                           int log_last, const FoldOut& out)
{
    const float* centre = plane + (int64_t)c * N;
    const int64_t r = r0 + t;
    float s[kFoldPerLane];
#pragma unroll
    for (int j = 0; j < kFoldPerLane; ++j)
        s[j] = 0.f;
    int log = 0;
    if (prev != nullptr) {
        const int Hp = 1 << (log_first - 1);
        const int64_t NHp = (N + Hp - 1) / Hp;
        const float* p = prev + (dk + c / Hp) * NHp + r;
#pragma unroll
        for (int j = 0; j < kFoldPerLane; ++j)
            if (r + j * kFoldThreads < NHp)
                s[j] = p[j * kFoldThreads];
        log = log_first;
    }
    if (log <= 0 && !fold_stage<0>(centre, N, c, dk, r0, t, out, s)) return;
    if (log <= 1 && (log_last < 1 || !fold_stage<1>(centre, N, c, dk, r0, t, out, s))) return;
    if (log <= 2 && (log_last < 2 || !fold_stage<2>(centre, N, c, dk, r0, t, out, s))) return;
    if (log <= 3 && (log_last < 3 || !fold_stage<3>(centre, N, c, dk, r0, t, out, s))) return;
    if (log <= 4 && (log_last < 4 || !fold_stage<4>(centre, N, c, dk, r0, t, out, s))) return;
    if (log <= 5 && (log_last < 5 || !fold_stage<5>(centre, N, c, dk, r0, t, out, s))) return;
    if (log <= 6 && log_last >= 6)
        fold_stage<6>(centre, N, c, dk, r0, t, out, s);
}

// One wave per (chunk, row of the first fold): workgroup b takes row b mod KH
// of the (b / KH)-th chunk of the octave order.
__global__ __launch_bounds__(kFoldThreads, 8) void fold_chain_kernel(
    const float* __restrict__ plane, int64_t N, int K, const float* __restrict__ prev,
    int log_first, int log_last, FoldOut out, int P, int KH)
{
    const int64_t b = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (b >= (int64_t)P * KH)
        return;
    int p, row;
    fold_item(b, P, KH, p, row);
    const int64_t dk = row - (KH - 1) / 2;
    fold_chain(plane, N, (K - 1) / 2, dk, (int64_t)fold_chunk(P - 1 - p, P) * kFoldCols,
               threadIdx.x, prev, log_first, log_last, out);
}

// ---- one fold -----------------------------------------------------------------
//
// One row of the H-fold sum per blockIdx.y, kHarmCols columns per
// blockIdx.x: lane t takes columns t + kHarmThreads j, j < kHarmCols /
// kHarmThreads, so each load instruction is coalesced and every lane keeps
// several independent gathers in flight.  With prev (the H/2-fold, KHp x
// NHp), the sum starts from it and adds harmonics H/2 + 1 .. H; without, it
// adds 1 .. H from zero.
constexpr int kHarmPerLane = 4;
constexpr int kHarmCols = kHarmThreads * kHarmPerLane;

__global__ __launch_bounds__(kHarmThreads) void harmonic_sum_kernel(
    const float* __restrict__ plane, int64_t N, int K, int H, const float* __restrict__ prev,
    int64_t NHp, int KHp, float* __restrict__ out, int64_t NH, int KH)
{
    const int64_t r0 = (int64_t)blockIdx.x * kHarmCols + threadIdx.x;
    const int c = (K - 1) / 2;
    const int krow = blockIdx.y;                       // row of the fold
    const int dk = krow - (KH - 1) / 2;                // k - c of the fundamental
    float s[kHarmPerLane];
    bool in[kHarmPerLane];
#pragma unroll
    for (int j = 0; j < kHarmPerLane; ++j) {
        in[j] = r0 + (int64_t)j * kHarmThreads < NH;
        s[j] = 0.f;
    }
    int h0 = 1;
    if (prev != nullptr) {
        const float* p = prev + (int64_t)(dk + (KHp - 1) / 2) * NHp + r0;
#pragma unroll
        for (int j = 0; j < kHarmPerLane; ++j)
            if (in[j])
                s[j] = p[(int64_t)j * kHarmThreads];
        h0 = H / 2 + 1;
    }
    for (int h = h0; h <= H; ++h) {
        const float* row = plane + (int64_t)(c + h * dk) * N + (int64_t)h * r0;
#pragma unroll
        for (int j = 0; j < kHarmPerLane; ++j)
            if (in[j])
                s[j] += row[(int64_t)h * j * kHarmThreads];
    }
    float* o = out + (int64_t)krow * NH + r0;
#pragma unroll
    for (int j = 0; j < kHarmPerLane; ++j)
        if (in[j])
            o[(int64_t)j * kHarmThreads] = s[j];
}

// One fold goes to this kernel or, with one stage, to fold_chain_kernel, whose lanes
// keep more loads in flight but whose order of the chunks is made for chains.
// Measured, this kernel -> the chain's (us):
//   H = 1: 85 x 20000 4.5 -> 5.3, 121 x 35391 8.6 -> 8.9, 201 x 44772 15.3 -> 14.4, 85 x
//   2^20 170 -> 141;
//   H = 2: 61 x 17537 3.7 -> 3.6, 61 x 83834 4.7 -> 5.3, 121 x 73983 9.0 -> 7.1, 85 x 2^20
//   75 -> 57; one row of 2065151 columns 5.7 -> 6.6;
//   H = 4 to 16 on top of the fold below: 85 x 2^22 134 -> 156, 106 -> 112, 79 -> 82,
//   85 x 2^20 29.5 -> 30.4, 24.4 -> 24.9, 19.8 -> 21; where this kernel's workgroups are
//   fewer than the CUs, 41 x 131073 (H = 8, 16) 4.7 -> 3.7, 6.7 -> 3.8; 4-fold of short
//   rows, 201 x 29908 4.0 -> 4.2 but 1025 x 30000 14.5 -> 12.6;
//   H = 4, 8 from the plane: 85 x 2^20 39 -> 32, 34 -> 30; 85 x 2^22 153 -> 161, 124 ->
//   130; 16: 29 -> 26, 103 -> 99;
//   H = 32 and 64 of small folds, H = 64 of large ones and 32 from the plane: 1025 x 30000
//   24 -> 9, 25 -> 12.5, 85 x 2^22 49 -> 17 (64), 122 -> 116 (32 from the plane);
//   H = 32 on top of the fold below, from 2^17 points of the fold on: at most one workgroup
//   of this kernel per CU, 41 x 6291456 37 -> 44, 401 x 496989 45 -> 49, 85 x 2097153 40.5 ->
//   42.8 (85 x 2^21 39.8 -> 38.4); the second only on some, 85 x 3000001 74 -> 62, 401 x
//   640000 71 -> 63, but one row of 265625 columns 55 -> 60; two on most, 85 x 5000000 103 ->
//   107, 401 x 2^20 96 -> 100; more, 85 x 5600000 129 -> 116, 85 x 2^23 175 -> 172.
bool one_fold_by_chain(int64_t N, int K, int H, int64_t NH, int KH, bool prev)
{
    const int64_t points = N * K, blocks = (NH + kHarmCols - 1) / kHarmCols * KH;
    if (H == 1)
        return points >= 1 << 23;
    if (H == 2)
        return points < 1 << 21 || (points >= 1 << 23 && KH > 1);
    if (H == 32 && prev && NH * KH >= 1 << 17)
        return blocks > 512 || (blocks > 256 && blocks <= 384 && KH > 1);
    if (H >= 32)
        return true;
    if (!prev)
        return H == 16 || points < (int64_t)1 << 28;
    return blocks < 256 || (H == 4 && NH < 1 << 14 && points >= 1 << 24);
}

__global__ void zero_count_kernel(unsigned* __restrict__ count)
{
    if (threadIdx.x == 0)
        *count = 0u;
}

// Whether v = S[k][r] is >= each of its neighbours inside the fold.  All eight are read
// at once; one outside the fold is replaced by the nearest point inside, another
// neighbour or v itself.
__device__ __forceinline__ bool is_peak(const float* __restrict__ S, int64_t NH, int KH, int k,
                                        int64_t r, float v)
{
    const float* row = S + (int64_t)k * NH;
    const float* up = k > 0 ? row - NH : row;
    const float* down = k + 1 < KH ? row + NH : row;
    const int64_t left = r > 0 ? r - 1 : r, right = r + 1 < NH ? r + 1 : r;
    const float near[8] = {up[left],   up[r],      up[right], row[left],
                           row[right], down[left], down[r],   down[right]};
    bool peak = true;
#pragma unroll
    for (int i = 0; i < 8; ++i)
        peak = peak && v >= near[i];
    return peak;
}

__device__ __forceinline__ void put_candidate(fdas_candidate* __restrict__ out, int capacity,
                                              unsigned* __restrict__ count, int64_t r, int row,
                                              float power)
{
    const unsigned slot = atomicAdd(count, 1u);
    if (slot < (unsigned)capacity) {
        fdas_candidate cand;
        cand.r = r;
        cand.row = row;
        cand.power = power;
        out[slot] = cand;
    }
}

// Peaks of one fold: S > threshold and S >= each neighbour inside the fold.
// Bound by reading the fold once; a lane keeps PER loads in flight (lane t takes
// columns t + kHarmThreads j), which is what the rate hangs on: 57 us for 85 x 2^20
// with 8 (6.3 TB/s), 107 us with one.  Where points pass the threshold a lane looks at
// its columns one after the other, and the last waves' looks are the tail of the
// call: with the neighbours read one by one 82 -> 87 us for 10^4 peaks in 201 x 300000
// (8 columns per lane against one), all at once 81 us.
constexpr int kCandPerLane = 8;
constexpr int kCandCols = kHarmThreads * kCandPerLane;

// Columns c0 .. c0 + kHarmThreads PER of row k of one fold; a candidate's r is reported
// from column r_at on.
template <int PER>
__device__ __forceinline__ void find_peaks(const float* __restrict__ S, int64_t NH, int KH, int k,
                                           int64_t c0, float threshold, int row0, int64_t r_at,
                                           fdas_candidate* __restrict__ out, int capacity,
                                           unsigned* __restrict__ count)
{
    const int64_t r = c0 + threadIdx.x;
    const float* row = S + (int64_t)k * NH + r;
    float v[PER];
    if (c0 + kHarmThreads * PER <= NH) {
#pragma unroll
        for (int j = 0; j < PER; ++j)
            v[j] = row[j * kHarmThreads];
    } else {
        // a column outside the fold gets the threshold itself: no candidate
#pragma unroll
        for (int j = 0; j < PER; ++j)
            v[j] = r + j * kHarmThreads < NH ? row[j * kHarmThreads] : threshold;
    }
    bool any = false;
#pragma unroll
    for (int j = 0; j < PER; ++j)
        any = any || v[j] > threshold;
    if (!any)
        return;
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (v[j] > threshold && is_peak(S, NH, KH, k, r + j * kHarmThreads, v[j]))
            put_candidate(out, capacity, count, r_at + r + j * kHarmThreads, row0 + k, v[j]);
}

template <int PER>
__global__ __launch_bounds__(kHarmThreads) void candidates_kernel(
    const float* __restrict__ S, int64_t NH, int KH, float threshold, int row0,
    fdas_candidate* __restrict__ out, int capacity, unsigned* __restrict__ count)
{
    find_peaks<PER>(S, NH, KH, blockIdx.y, (int64_t)blockIdx.x * (kHarmThreads * PER), threshold,
                    row0, 0, out, capacity, count);
}

// ---- batched: the planes of fdas_correlate_batched (plane b at K offsets[b],
// [K][N_b]), every fold in one launch --------------------------------------------

// fold column prefix sums over the spectra: colpre[b] = sum_{b' < b}
// ceil(N_b' / H), and the same for H/2 in prevpre (one workgroup).

__global__ __launch_bounds__(kHScanThreads) void harmonic_scan_kernel(
    const int64_t* __restrict__ offsets, int nspec, int H, int64_t* __restrict__ colpre,
    int64_t* __restrict__ prevpre)
{
    __shared__ int64_t part[2][kHScanThreads];
    __shared__ int64_t carry[2];
    const int t = threadIdx.x;
    const int Hp = H > 1 ? H / 2 : 1;
    if (t == 0) {
        carry[0] = carry[1] = 0;
        colpre[0] = prevpre[0] = 0;
    }
    __syncthreads();
    for (int base = 0; base < nspec; base += kHScanThreads) {
        const int b = base + t;
        int64_t a = 0, p = 0;
        if (b < nspec) {
            const int64_t n = offsets[b + 1] - offsets[b];
            a = n > 0 ? (n + H - 1) / H : 0;
            p = n > 0 ? (n + Hp - 1) / Hp : 0;
        }
        part[0][t] = a;
        part[1][t] = p;
        __syncthreads();
        for (int d = 1; d < kHScanThreads; d <<= 1) {
            const int64_t x = t >= d ? part[0][t - d] : 0;
            const int64_t y = t >= d ? part[1][t - d] : 0;
            __syncthreads();
            part[0][t] += x;
            part[1][t] += y;
            __syncthreads();
        }
        if (b < nspec) {
            colpre[b + 1] = carry[0] + part[0][t];
            prevpre[b + 1] = carry[1] + part[1][t];
        }
        __syncthreads();
        if (t == kHScanThreads - 1) {
            carry[0] += part[0][t];
            carry[1] += part[1][t];
        }
        __syncthreads();
    }
}

// Spectrum of fold column g: the b with colpre[b] <= g < colpre[b + 1]
// (binary search; empty spectra have equal bounds and are skipped).
__device__ __forceinline__ int column_spectrum(const int64_t* __restrict__ colpre, int nspec,
                                               int64_t g)
{
    int lo = 0, hi = nspec - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (colpre[mid] <= g)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// Batched chains.  Work item = (spectrum, chunk of the octave order, row of
// fold 2), numbered in that order.
__host__ __device__ inline int fold2_rows(int K) { return 2 * ((K - 1) / 2 / 2) + 1; }

__device__ __forceinline__ int64_t fold_columns(int64_t N, int log)
{
    return (N + (1 << log) - 1) >> log;
}

// Prefix sums over the spectra, one workgroup each: row 0 of pre[.][nspec + 1]
// counts the work items (fold 2^log in chunks of `cols` columns, times `rows`),
// row i <= folds the columns of fold 2^(log + i - 1).  A workgroup
// beyond those writes the row behind them, the prefix of the spectra's lengths, and the
// next, their starts.  Offsets are clamped to [0, cap].  `zero` (or NULL) is set to 0.
// A chain of dependent steps: 1024 lanes take a third of the steps that 256 took (folds 2 of 3000 spectra of 200 bins, 7 rows: 28.9 -> 20.8 us).
constexpr int kFoldScanThreads = 1024;

__global__ __launch_bounds__(kFoldScanThreads) void fold_scan_kernel(
    const int64_t* __restrict__ offsets, int nspec, int64_t cap, int log, int folds, int cols,
    int rows, int64_t* __restrict__ pre, unsigned* __restrict__ zero)
{
    __shared__ int64_t part[2][kFoldScanThreads];
    __shared__ int64_t carry;
    const int t = threadIdx.x;
    const int i = blockIdx.x;
    int64_t* const out = pre + (int64_t)i * (nspec + 1);
    if (t == 0) {
        carry = 0;
        out[0] = 0;
        if (i == 0 && zero != nullptr)
            *zero = 0u;
    }
    __syncthreads();
    for (int base = 0; base < nspec; base += kFoldScanThreads) {
        const int b = base + t;
        int64_t v = 0;
        if (b < nspec) {
            int64_t off, n;
            spec_range(offsets, b, cap, off, n);
            if (i > folds) {
                v = n;
                out[nspec + 1 + b] = off;
            } else if (n > 0) {
                v = i == 0 ? (fold_columns(n, log) + cols - 1) / cols * rows
                           : fold_columns(n, log + i - 1);
            }
        }
        // the steps the batch needs, from one buffer into the other
        const int count = min(nspec - base, kFoldScanThreads);
        int from = 0;
        part[0][t] = v;
        __syncthreads();
        for (int d = 1; d < count; d <<= 1) {
            v += t >= d ? part[from][t - d] : 0;
            part[from ^= 1][t] = v;
            __syncthreads();
        }
        if (b < nspec)
            out[b + 1] = carry + v;
        __syncthreads();
        if (t == count - 1)
            carry += v;
        __syncthreads();
    }
}

// One wave per work item (more waves than the host's bound on them stride on),
// so the waves of the moment work on neighbouring chunks of one spectrum.  Fold
// 2^i of spectrum b lies at out.p[i] + KH pre[i][b].  The spectra are those of the
// offsets clamped to the bins the planes hold, from the scan's last two rows
// (clamped here, wave by wave, the same took fold 2 of 85 x 2^20 from 64.1 to 72.5
// us); overlapping ones whose lengths add up to more than cap, and so their folds
// to more than cap / 2^i + nspec columns, are left out.  Measured, 8 spectra of
// 131073 bins, 41 rows, folds 2..16: 51 us; 64 us as one launch per fold, and
// 83 us with persistent waves, which paid for a new spectrum nearly every item.
__global__ __launch_bounds__(kFoldThreads, 8) void fold_chain_batched_kernel(
    const float* __restrict__ planes, int nspec, int64_t cap, int K, int log_last, FoldOut out,
    const int64_t* __restrict__ pre)
{
    const int64_t* const length = pre + (int64_t)(log_last + 1) * (nspec + 1);
    const int64_t* const start = length + nspec + 1;
    const int c = (K - 1) / 2, kc = c / 2;
    const int rows = fold2_rows(K);
    const int64_t total = pre[nspec];
    for (int64_t g = (int64_t)blockIdx.y * gridDim.x + blockIdx.x; g < total;
         g += (int64_t)gridDim.x * gridDim.y) {
        const int b = column_spectrum(pre, nspec, g);
        const int64_t off = start[b], N = length[b + 1] - length[b];
        FoldOut o = {};
#pragma unroll
        for (int i = 1; i < kMaxFolds; ++i)
            if (i <= log_last)
                o.p[i] = out.p[i] + (int64_t)(2 * (c >> i) + 1) * pre[(int64_t)i * (nspec + 1) + b];
        if (length[b + 1] > cap)
            return;
        const int P = (int)((fold_columns(N, 1) + kFoldCols - 1) / kFoldCols);
        int p, row;
        fold_item(g - pre[b], P, rows, p, row);
        fold_chain(planes + (int64_t)K * off, N, c, row - kc,
                   (int64_t)fold_chunk(P - 1 - p, P) * kFoldCols, threadIdx.x, nullptr, 1,
                   log_last, o);
    }
}

// Persistent grid: each lane takes fold columns g (stride gridDim.x x
// threads) over all spectra and walks the fold's KH rows for it, so a row's
// loads stay coalesced across the lanes.  Fold b lives at sums + KH
// colpre[b] as [KH][NH_b]; the previous fold (H/2) at prev + KHp prevpre[b].  This is
// one fold on top of the fold below; all folds at once come from the chains above, in
// half the time or less (8 spectra of 131073 bins, 41 rows, folds 2..32: 54 us against
// 105 one by one).
__global__ __launch_bounds__(kHarmThreads) void harmonic_batched_kernel(
    const float* __restrict__ planes, const int64_t* __restrict__ offsets, int nspec, int K, int H,
    const float* __restrict__ prev, int KHp, const int64_t* __restrict__ colpre,
    const int64_t* __restrict__ prevpre, float* __restrict__ sums, int KH)
{
    const int64_t total = colpre[nspec];
    const int c = (K - 1) / 2;
    const int h0 = prev != nullptr ? H / 2 + 1 : 1;
    for (int64_t g = (int64_t)blockIdx.x * kHarmThreads + threadIdx.x; g < total;
         g += (int64_t)gridDim.x * kHarmThreads) {
        const int b = column_spectrum(colpre, nspec, g);
        const int64_t Nb = offsets[b + 1] - offsets[b];
        const int64_t NH = (Nb + H - 1) / H;
        const int64_t r = g - colpre[b];
        const float* plane = planes + (int64_t)K * offsets[b];
        float* out = sums + (int64_t)KH * colpre[b] + r;
        const float* pv = nullptr;
        int64_t NHp = 0;
        if (prev != nullptr) {
            NHp = (Nb + H / 2 - 1) / (H / 2);
            pv = prev + (int64_t)KHp * prevpre[b] + r;
        }
        for (int krow = 0; krow < KH; ++krow) {
            const int dk = krow - (KH - 1) / 2;
            float s = 0.f;
            if (pv != nullptr)
                s = pv[(int64_t)(dk + (KHp - 1) / 2) * NHp];
            for (int h = h0; h <= H; ++h)
                s += plane[(int64_t)(c + h * dk) * Nb + (int64_t)h * r];
            out[(int64_t)krow * NH] = s;
        }
    }
}

// Peaks of every spectrum's fold H = 2^log; the record's r is the packed bin
// index offsets[b] + r, which names the spectrum too.  Workgroup row y takes fold
// row y, its workgroups stride over the chunks of kCandCols columns that pre row 0
// counts (a spectrum found per chunk; one found per column and lane took 67 us for
// 8 x 41 x 131073, this 28 us).  Chunks that hold under an eighth of their columns, and
// more of them than workgroups, each pay the search for next to nothing: there every
// lane takes one column of one spectrum and walks its rows (3000 spectra of 200 bins, 7
// rows, 420 peaks: 49 -> 21 us, all 467000 peaks 901 -> 759; 300 of 128 columns, a
// chunk for every workgroup, 8.8 us by chunks and 10.5 by lanes).
__global__ __launch_bounds__(kHarmThreads) void candidates_batched_kernel(
    const float* __restrict__ sums, const int64_t* __restrict__ offsets, int nspec, int log,
    const int64_t* __restrict__ pre, int KH, float threshold, int row0,
    fdas_candidate* __restrict__ out, int capacity, unsigned* __restrict__ count)
{
    const int64_t total = pre[nspec];
    const int64_t* const column = pre + nspec + 1;
    if (total > gridDim.x && column[nspec] < total * kHarmThreads) {
        const int64_t lanes = (int64_t)gridDim.x * gridDim.y * kHarmThreads;
        for (int64_t g = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * kHarmThreads + threadIdx.x;
             g < column[nspec]; g += lanes) {
            const int b = column_spectrum(column, nspec, g);
            const int64_t off = offsets[b], NH = fold_columns(offsets[b + 1] - off, log);
            const int64_t r = g - column[b];
            const float* S = sums + (int64_t)KH * column[b];
            for (int k = 0; k < KH; ++k) {
                const float v = S[(int64_t)k * NH + r];
                if (v > threshold && is_peak(S, NH, KH, k, r, v))
                    put_candidate(out, capacity, count, off + r, row0 + k, v);
            }
        }
        return;
    }
    for (int64_t g = blockIdx.x; g < total; g += gridDim.x) {
        const int b = column_spectrum(pre, nspec, g);
        const int64_t off = offsets[b], NH = fold_columns(offsets[b + 1] - off, log);
        find_peaks<kCandPerLane>(sums + (int64_t)KH * column[b], NH, KH, blockIdx.y,
                                 (g - pre[b]) * kCandCols, threshold, row0, off, out, capacity,
                                 count);
    }
}

// Persistent workgroups of the batched kernels (grid-stride loops, so any
// count is correct; the host emulation of the tests builds with a small one).
#ifndef FDAS_HARM_BATCHED_GRID
#define FDAS_HARM_BATCHED_GRID 2048
#endif
constexpr int kHarmBatchedGrid = FDAS_HARM_BATCHED_GRID;
constexpr int kCandBatchedGrid = FDAS_HARM_BATCHED_GRID < 512 ? FDAS_HARM_BATCHED_GRID : 512;

}  // namespace

void harmonic_shape(int64_t N, int K, int H, int* KH, int64_t* NH)
{
    const int c = (K - 1) / 2;
    *KH = 2 * (c / H) + 1;
    *NH = (N + H - 1) / H;
}

// Folds 2^log_first .. 2^log_last (those with an output pointer), on top of prev
// if given.
hipError_t launch_fold_chain(const float* plane, int64_t N, int K, const float* prev,
                             int log_first, int log_last, float* const* sums, hipStream_t s)
{
    int KH = 0;
    int64_t NH = 0;
    harmonic_shape(N, K, 1 << log_first, &KH, &NH);
    if (NH == 0)
        return hipSuccess;
    const int64_t P = (NH + kFoldCols - 1) / kFoldCols;
    FoldOut out = {};
    for (int i = log_first; i <= log_last; ++i)
        out.p[i] = sums[i - log_first];
    const int64_t waves = P * KH, gx = waves < kMaxFoldGridX ? waves : kMaxFoldGridX;
    hipLaunchKernelGGL(fold_chain_kernel,
                       dim3((unsigned)gx, (unsigned)((waves + gx - 1) / gx)), dim3(kFoldThreads),
                       0, s, plane, N, K, prev, log_first, log_last, out, (int)P, KH);
    return hipGetLastError();
}

hipError_t launch_harmonic_sum(const float* plane, int64_t N, int K, int H, const float* prev,
                               float* out, hipStream_t s)
{
    int KH = 0, KHp = 0;
    int64_t NH = 0, NHp = 0;
    harmonic_shape(N, K, H, &KH, &NH);
    if (prev != nullptr)
        harmonic_shape(N, K, H / 2, &KHp, &NHp);
    if (NH == 0)
        return hipSuccess;
    if (one_fold_by_chain(N, K, H, NH, KH, prev != nullptr)) {
        int log = 0;
        while ((1 << log) < H)
            ++log;
        return launch_fold_chain(plane, N, K, prev, log, log, &out, s);
    }
    const dim3 grid((unsigned)((NH + kHarmCols - 1) / kHarmCols), (unsigned)KH);
    hipLaunchKernelGGL(harmonic_sum_kernel, grid, dim3(kHarmThreads), 0, s, plane, N, K, H, prev,
                       NHp, KHp, out, NH, KH);
    return hipGetLastError();
}

hipError_t launch_candidates(const float* S, int64_t N, int K, int H, float threshold,
                             fdas_candidate* out, int capacity, unsigned* count, hipStream_t s)
{
    int KH = 0;
    int64_t NH = 0;
    harmonic_shape(N, K, H, &KH, &NH);
    hipLaunchKernelGGL(zero_count_kernel, dim3(1), dim3(64), 0, s, count);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || NH == 0)
        return e;
    const int row0 = (K - 1) / 2 - (KH - 1) / 2;
    // One column per lane while that gives no more workgroups than run at once (8 per
    // CU): there is nothing to wait for but the looks themselves.  Every local maximum of
    // 1 x 5000 4.9 us against 8.5, of the 32-fold of 41 x 131073 4.7 against 9.1.
    const int64_t blocks = (NH + kHarmThreads - 1) / kHarmThreads;
    if (blocks * KH <= 2048)
        hipLaunchKernelGGL((candidates_kernel<1>), dim3((unsigned)blocks, (unsigned)KH),
                           dim3(kHarmThreads), 0, s, S, NH, KH, threshold, row0, out, capacity,
                           count);
    else
        hipLaunchKernelGGL((candidates_kernel<kCandPerLane>),
                           dim3((unsigned)((NH + kCandCols - 1) / kCandCols), (unsigned)KH),
                           dim3(kHarmThreads), 0, s, S, NH, KH, threshold, row0, out, capacity,
                           count);
    return hipGetLastError();
}

hipError_t launch_harmonic_batched(const float* planes, const int64_t* offsets, int nspec, int K,
                                   int H, const float* prev, float* sums, int64_t* colpre,
                                   int64_t* prevpre, hipStream_t s)
{
    int KH = 0, KHp = 0;
    int64_t NH = 0, NHp = 0;
    harmonic_shape(1, K, H, &KH, &NH);
    if (prev != nullptr)
        harmonic_shape(1, K, H / 2, &KHp, &NHp);
    hipLaunchKernelGGL(harmonic_scan_kernel, dim3(1), dim3(kHScanThreads), 0, s, offsets, nspec, H,
                       colpre, prevpre);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(harmonic_batched_kernel, dim3(kHarmBatchedGrid), dim3(kHarmThreads), 0, s,
                       planes, offsets, nspec, K, H, prev, KHp, colpre, prevpre, sums, KH);
    return hipGetLastError();
}

hipError_t launch_fold_chain_batched(const float* planes, const int64_t* offsets, int nspec,
                                     int64_t capacity, int K, int log_last, float* const* sums,
                                     int64_t* pre, hipStream_t s)
{
    hipLaunchKernelGGL(fold_scan_kernel, dim3((unsigned)(log_last + 2)), dim3(kFoldScanThreads), 0, s,
                       offsets, nspec, capacity, 1, log_last, kFoldCols, fold2_rows(K), pre,
                       (unsigned*)nullptr);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    FoldOut out = {};
    for (int i = 1; i <= log_last; ++i)
        out.p[i] = sums[i - 1];
    // sum_b chunks(N_b) <= capacity / (2 kFoldCols) + 2 nspec
    const int64_t waves = (capacity / (2 * kFoldCols) + 2 * (int64_t)nspec) * fold2_rows(K);
    const int64_t gx = waves < kMaxFoldGridX ? waves : kMaxFoldGridX;
    const int64_t gy = (waves + gx - 1) / gx;
    hipLaunchKernelGGL(fold_chain_batched_kernel,
                       dim3((unsigned)gx, (unsigned)(gy < kMaxFoldGridY ? gy : kMaxFoldGridY)),
                       dim3(kFoldThreads), 0, s, planes, nspec, capacity, K, log_last, out, pre);
    return hipGetLastError();
}

hipError_t launch_candidates_batched(const float* sums, const int64_t* offsets, int nspec, int K,
                                     int H, float threshold, fdas_candidate* out, int capacity,
                                     unsigned* count, int64_t* pre, hipStream_t s)
{
    int KH = 0;
    int64_t NH = 0;
    harmonic_shape(1, K, H, &KH, &NH);
    int log = 0;
    while ((1 << log) < H)
        ++log;
    hipLaunchKernelGGL(fold_scan_kernel, dim3(2), dim3(kFoldScanThreads), 0, s, offsets, nspec,
                       INT64_MAX, log, 1, kCandCols, 1, pre, count);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    const int row0 = (K - 1) / 2 - (KH - 1) / 2;
    hipLaunchKernelGGL(candidates_batched_kernel, dim3(kCandBatchedGrid, (unsigned)KH),
                       dim3(kHarmThreads), 0, s, sums, offsets, nspec, log, pre, KH, threshold,
                       row0, out, capacity, count);
    return hipGetLastError();
}

}  // namespace fdas
