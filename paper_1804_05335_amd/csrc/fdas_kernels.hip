// HIP kernels for gfx950: template-bank preparation, the fused forward
// overlap-save correlation (Sec. 3, Fig. 1; Sec. 4.2), its batched ragged
// form, and the adjoint.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <type_traits>

#include "fdas_fft.hpp"
#include "fdas_internal.h"
#include "fdas_response.hpp"

namespace fdas {

typedef float f32x2 __attribute__((ext_vector_type(2)));


// ---- range-checked segment access ---------------------------------------------
//
// A segment's window positions q in [0, L) map to output u = q - M/2; only
// q in [M/2, M/2 + nvalid) are valid outputs (nvalid = min(B, N - out0)).
// Per-element branches are replaced by buffer instructions whose resource
// starts at position q = 0 of the row and ends after the last valid output:
// the hardware drops stores past the end and returns 0 for loads past it,
// and positions q < M/2 are given byte offset 2^31, which is past it as
// well.  Offsets are built from non-negative terms only, so no wrap-around
// is involved however the compiler splits them into register and immediate
// parts.
constexpr int kRsrcWord3 = 0x00020000;   // gfx9 raw buffer: 32-bit data format, no swizzle
constexpr int kNonTemporal = 2;          // cache policy: non-temporal

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t seg_rsrc(const void* row_q0, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(row_q0), (short)0, bytes,
                                             kRsrcWord3);
}

template <int BYTES>
__device__ __forceinline__ int seg_off(int q, int half_m)
{
    return q >= half_m ? q * BYTES : (int)0x80000000u;
}

// ---- templates and bank preparation -------------------------------------------
//
// Templates of the grid (Sec. 2, text before eq. 23), one lane per tap:
// taps[k][j] = R(j - M/2, z_k), z_k = (k - (K-1)/2) dz, or with HALF the
// half-bin taps of the two-bin interpolation, taps[k][j] = R(1/2 - (j -
// Mt/2), z_k) for j >= 2 and 0 below.  Mt is the row length.  Bound by one
// lane's FP64 chain (up to ~40 steps of a continued fraction or a series per
// end of the integral), so the lanes are spread over as many one-wave
// workgroups as there are: 10 us at K = 85, M = 256, where the host took 8 ms
// of one core and a blocking copy.
constexpr int kTemplateThreads = 64;

template <bool HALF>
__global__ __launch_bounds__(kTemplateThreads) void templates_kernel(double dz, int K, int Mt,
                                                                     float2* __restrict__ taps)
{
    const int i = blockIdx.x * kTemplateThreads + threadIdx.x;
    if (i >= K * Mt)
        return;
    const int k = i / Mt, j = i - k * Mt;
    const double z = ((double)k - 0.5 * (double)(K - 1)) * dz;
    cplx64 r = {0.0, 0.0};
    if (!HALF || j >= 2)
        r = response64(HALF ? 0.5 - (double)(j - Mt / 2) : (double)(j - Mt / 2), z);
    taps[i] = make_float2((float)r.re, (float)r.im);
}

hipError_t launch_templates(double dz, int K, int Mt, bool half, float2* taps, hipStream_t s)
{
    const dim3 grid((unsigned)(((int64_t)K * Mt + kTemplateThreads - 1) / kTemplateThreads));
    if (half)
        hipLaunchKernelGGL((templates_kernel<true>), grid, dim3(kTemplateThreads), 0, s, dz, K, Mt,
                           taps);
    else
        hipLaunchKernelGGL((templates_kernel<false>), grid, dim3(kTemplateThreads), 0, s, dz, K,
                           Mt, taps);
    return hipGetLastError();
}

// H_z[k] = (1/L) sum_j conj(T[z][j]) W_L^{((M/2 - j) mod L) k}: tap j of the
// template placed so that the filter is centred on bin 0, its two halves at
// the ends of the L-array (Sec. 3, Fig. 1); accumulated in FP64.
//
// With v = W_L^{-k} the sum is W_L^{(M/2) k} sum_j c_j v^j, c = conj T.  A
// lane takes the eight rows k = k0 + m L/8: v^8 is the same for all of them,
// so it evaluates S_b = sum_a c_{8a+b} (v^8)^a, b < 8, once, by Horner's rule
// (eight independent chains of four FP64 FMAs per tap), and combines them
// with one eight-point transform of S_b W_L^{-b k0}.  Few lanes and short
// chains: the row's taps come from LDS (scalar loads in the loop waited for
// memory once per group of taps: 17 us), and one sine and cosine pair serves
// all the powers W_L^{-b k0} (a pair for each took 16 of them per lane).
// Measured: 8-10 us at K = 85, M = 256, L = 2048 and 43 us at K = 201, M =
// 512, L = 8192; one lane per (z, k) with a sine and cosine per tap took 151
// and 2031 us with its launch for the twiddles.
// The row z = K holds the twiddles exp(-2 pi i n / L).
constexpr int kBankThreads = 64;

// Row lengths the LDS copy is sized for: the ordinary banks, whose small copy
// leaves room for many workgroups per CU, and the longest (L/2 at L = 8192).
constexpr int kBankTaps = 512, kBankMaxTaps = 4096;

__device__ __forceinline__ cplx64 bank_root(int64_t p, int L)   // W_L^p
{
    double s, c;
    sincospi(-2.0 * (double)(p & (L - 1)) / (double)L, &s, &c);
    return {c, s};
}

__device__ __forceinline__ void bank_bfly(cplx64& a, cplx64& b)
{
    const cplx64 d = a - b;
    a = a + b;
    b = d;
}

template <int MAXM>
__global__ __launch_bounds__(kBankThreads) void bank_rows_kernel(const float2* __restrict__ taps,
                                                                 int K, int M, int L,
                                                                 float2* __restrict__ bank)
{
    __shared__ float2 tz[MAXM];
    const int k0 = blockIdx.x * kBankThreads + threadIdx.x;
    const int z = blockIdx.y;
    const int P = L / 8;
    float2* row = bank + (int64_t)z * L + k0;
    if (z == K) {
#pragma unroll
        for (int m = 0; m < 8; ++m)
            if (k0 < P) {
                const cplx64 w = bank_root(k0 + m * P, L);
                row[m * P] = make_float2((float)w.re, (float)w.im);
            }
        return;
    }
    for (int j = threadIdx.x; j < M; j += kBankThreads)
        tz[j] = taps[(int64_t)z * M + j];
    const cplx64 v8 = bank_root(-8 * (int64_t)k0, L);
    const cplx64 v1 = bank_root(-(int64_t)k0, L);
    const cplx64 centre = bank_root((int64_t)(M / 2) * k0, L);
    __syncthreads();
    cplx64 S[8];
#pragma unroll
    for (int b = 0; b < 8; ++b)
        S[b] = {0.0, 0.0};
    auto step = [&](int b, float2 t) {           // S <- S v^8 + conj(t)
        const double re = fma(S[b].re, v8.re, (double)t.x);
        const double im = fma(S[b].re, v8.im, -(double)t.y);
        S[b] = {fma(-S[b].im, v8.im, re), fma(S[b].im, v8.re, im)};
    };
    int a = M / 8 * 8;
    if (a < M) {                                 // the last, shorter group of taps
#pragma unroll
        for (int b = 0; b < 8; ++b)
            if (a + b < M)
                step(b, tz[a + b]);
    }
#pragma unroll 2
    for (a -= 8; a >= 0; a -= 8) {
#pragma unroll
        for (int b = 0; b < 8; ++b)
            step(b, tz[a + b]);
    }
    // S_b <- S_b v^b
    const cplx64 v2 = v1 * v1, v4 = v2 * v2, v3 = v2 * v1;
    S[1] = S[1] * v1;
    S[2] = S[2] * v2;
    S[3] = S[3] * v3;
    S[4] = S[4] * v4;
    S[5] = S[5] * (v4 * v1);
    S[6] = S[6] * (v4 * v2);
    S[7] = S[7] * (v4 * v3);
    // X[m] = sum_b S[b] e^{+2 pi i b m / 8}
    const double h = 0.70710678118654752440084436210485;
#pragma unroll
    for (int b = 0; b < 4; ++b)
        bank_bfly(S[b], S[b + 4]);
    S[5] = cplx64{S[5].re - S[5].im, S[5].re + S[5].im} * h;
    S[6] = {-S[6].im, S[6].re};
    S[7] = cplx64{-(S[7].re + S[7].im), S[7].re - S[7].im} * h;
#pragma unroll
    for (int g = 0; g < 8; g += 4) {
        bank_bfly(S[g], S[g + 2]);
        bank_bfly(S[g + 1], S[g + 3]);
        S[g + 3] = {-S[g + 3].im, S[g + 3].re};
        bank_bfly(S[g], S[g + 1]);
        bank_bfly(S[g + 2], S[g + 3]);
    }
    if (k0 >= P)
        return;
    // times W_L^{(M/2)(k0 + m L/8)} / L = W_L^{(M/2) k0} W_8^{(M/2) m} / L
    const double inv = 1.0 / (double)L;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        // the decimation leaves X[m] at the bit-reversed place
        cplx64 r = S[((m & 1) << 2) | (m & 2) | (m >> 2)] * centre;
        const int e = (M / 2 * m) & 7;           // uniform: eighth turns
        if (e & 1)
            r = cplx64{r.re + r.im, r.im - r.re} * h;
        if (e & 2)
            r = {r.im, -r.re};
        if (e & 4)
            r = {-r.re, -r.im};
        row[m * P] = make_float2((float)(r.re * inv), (float)(r.im * inv));
    }
}

hipError_t launch_prepare_bank(const float2* taps, int K, int M, int L, float2* bank,
                               hipStream_t s)
{
    const dim3 grid((L / 8 + kBankThreads - 1) / kBankThreads, K + 1);
    if (M <= kBankTaps)
        hipLaunchKernelGGL((bank_rows_kernel<kBankTaps>), grid, dim3(kBankThreads), 0, s, taps, K,
                           M, L, bank);
    else
        hipLaunchKernelGGL((bank_rows_kernel<kBankMaxTaps>), grid, dim3(kBankThreads), 0, s, taps,
                           K, M, L, bank);
    return hipGetLastError();
}

// ---- fused forward correlation ---------------------------------------------

// The waves of a SIMD share its issue ports by age, so with equal work the
// oldest workgroup of a CU runs ahead and the youngest finishes alone, with
// nothing to fill its waits: measured on the half-bin plane of 10^6 bins (K = 85,
// M = 256, L = 2048), the four workgroups of a CU ended at 58, 74, 87 and 100 %
// of its time.  Every workgroup therefore starts its n-th template at priority 3 -
// n mod 4: the one ahead gives way until the others have caught up, and they end
// within 5 % of one another.  Measured: that plane 232 -> 217 us, the two-bin
// plane of 300007 bins (K = 41, M = 128, L = 1024) 37.8 -> 37.1 us; the plane of
// 2^21 bins at L = 2048, where the four workgroups differ less, unchanged.  Not
// below L = 1024, whose one-wave workgroups pay more for the branch than they
// gain (300001 bins, K = 85, M = 64, L = 512: 39.1 -> 41.5 us), nor at L = 8192,
// where one workgroup fills the CU and the two-bin kernel has no register to
// spare for the count (709 -> 1020 us).
//
// Where a workgroup has one or two templates there is little to catch up with, and
// the branches, or the registers they take, cost 1 to 4 %.  At L = 2048 and 4096 the
// kernels that lose are built without turns too, for the calls below so many eighths
// of a template per workgroup (turn_eighths).  Time without turns / with them, on
// planes of K = 85 (the largest and smallest of three tap counts):
//   templates per workgroup        1          1.5         2          3          4
//   half-bin,  L = 2048       0.99 0.99   0.98 0.99   1.00 1.02  1.00 1.04  1.02 1.05
//              L = 4096       0.99 1.00   0.99 0.99   1.02 1.08  1.07 1.10  1.07 1.08
//   symmetric, L = 2048       0.98 0.99   0.96 0.98   0.99 1.00  0.99 1.00  0.99 1.00
//              L = 4096       0.99 1.01   0.99 1.00   1.00 1.02  1.02 1.03  1.02 1.03
//   two-bin,   L = 2048       0.99 1.00   1.00 1.00   1.00 1.01  1.01 1.03  1.01 1.03
//              L = 4096       0.98 0.99   1.00 1.01   0.99 0.99  1.03 1.03  1.02 1.07
//   batched,   L = 2048       0.99 1.00   0.98 1.00   0.99 1.01  1.00 1.00  1.00 1.01
//              L = 4096       0.99 0.99   0.99 1.00   1.00 1.01  1.00 1.01  1.02 1.02
// The plain kernel (13.8 -> 13.4 us at L = 4096) and the two-bin kernel with no dead
// slots at L = 4096 (20.5 -> 18.1: fewer spilled registers) gain at every size.
// Kernels of other streams on the same CU run at priority 0 and yield to the waves
// above it.  Measured beside the plane of 2^21 bins without turns -> with: a copy of 64 MB
// 33.7 -> 34.7 us a call, a candidate search of 85 x 2^18 71.5 -> 58.3, an addition of 4096
// values 4.4 -> 4.7; beside the half-bin plane 40.2 -> 41.9, 63.5 -> 57.3, 4.5 -> 4.6.
template <int L, bool IB, bool SYM, bool DUAL, int DEAD, bool BATCH>
constexpr int turn_eighths()
{
    if (L != 2048 && L != 4096)
        return 0;
    if (BATCH)
        return L == 2048 ? 24 : 14;
    if (SYM)
        return L == 2048 ? 32 : 0;
    if (DUAL)
        return L == 2048 ? 16 : (DEAD > 0 ? 12 : 0);
    return IB ? 13 : 0;
}

__device__ __forceinline__ void give_way(int n)
{
#ifdef __HIP_DEVICE_COMPILE__   // the host pass and the CPU emulation have no priorities
    switch (n & 3) {
    case 0: __builtin_amdgcn_s_setprio(3); break;
    case 1: __builtin_amdgcn_s_setprio(2); break;
    case 2: __builtin_amdgcn_s_setprio(1); break;
    default: __builtin_amdgcn_s_setprio(0); break;
    }
#endif
}

// DPP lane patterns (gfx9 wave-wide forms): lane i reads lane i + 1
// (lane 63 reads nothing), or lane (i + 1) mod 64.
constexpr int kDppWaveShl1 = 0x130;
constexpr int kDppWaveRol1 = 0x134;
constexpr float kQuarterPi2 = 0.61685027506808491368f;   // (pi/4)^2, interbinning

//
// Segment s produces the B = L - M outputs [s B, s B + B) from the window of
// input bins [s B - M/2, s B - M/2 + L) (zero outside [0, N)):
//   1. coalesced window load (lane t: positions t + T m);
//   2. forward FFT of the window (kept in registers for all its templates);
//   3. per template z: multiply by H_z (natural order, fused into the first
//      inverse pass), inverse FFT, |.|^2, non-temporal stores of the B valid
//      outputs to plane[z][s B + u].
// Nothing but the valid plane values reaches HBM (Sec. 4.2 first paragraph).
// A workgroup's consecutive work needs no extra barrier: the LDS buffers la/lb keep
// alternating from one transform to the next, the plan split over waves writes each of
// its regions behind a barrier that follows all reads of it, and the plan with one
// buffer ends its reads in a wave fence.
template <int L, int EV = Geometry<L>::E, class PLAN = SwapPlan<L, EV>>
struct Fwd {
    static constexpr bool kTurns = L >= 1024 && L <= 4096;    // see give_way
    static constexpr int E = EV;
    using F = FFT<L, E, typename PLAN::R>;
    static constexpr int T = F::T;
    static constexpr int NTW = F::NTW;
    // interbinned epilogue: waves per workgroup, and the `edge` slots
    // ([wave][E + 1]) of several waves below L = 8192 (at 8192 LDS is full:
    // the slots borrow the free exchange buffer)
    static constexpr int IB_NW = T / 64;
    static constexpr bool IB_OWN_EDGE = IB_NW > 1 && L < 8192;
    static constexpr int kEdgeAlloc = IB_OWN_EDGE ? IB_NW * (E + 1) : 1;

    __device__ static void load_row(float2 (&H)[E], const float2* __restrict__ bank, int row,
                                    int t)
    {
        const float2* h = bank + (int64_t)row * L + t;
#pragma unroll
        for (int m = 0; m < E; ++m)
            H[m] = h[T * m];
    }

    // Symmetric bank (only the rows z >= 0, template index c = (K-1)/2 on):
    // the row of template zi < c is the mirror of row c - zi, since
    // T_{-z} = conj T_z gives H_{-z}[p] = conj H_z[(L - p) mod L].  For lane
    // t and p = t + T m, (L - p) mod L = (b + T (E-1-m)) mod L with
    // b = T - t, so the mirrored row is read like a plain one from the lane
    // base b, in "load order" H[m'] = H_row[(b + T m') mod L] (only lane 0's
    // last slot wraps, to index 0), and its consumer takes
    // H_zi[t + T m] = conj(H[E-1-m]): a register renaming and a conjugate
    // that the multiply absorbs.  Rows zi >= c (row zi - c) load in natural
    // order.  The choice is uniform, so the load has no branch.
    __device__ static void load_row_sym(float2 (&H)[E], const float2* __restrict__ bank, int zi,
                                        int c, int t)
    {
        const bool mir = zi < c;
        const float2* h = bank + (int64_t)(mir ? c - zi : zi - c) * L;
        const int b = mir ? T - t : t;
#pragma unroll
        for (int m = 0; m < E - 1; ++m)
            H[m] = h[b + T * m];
        H[E - 1] = h[(b + T * (E - 1)) & (L - 1)];
    }

    template <bool SYM>
    __device__ static void load_bank_row(float2 (&H)[E], const float2* __restrict__ bank, int zi,
                                         int K, int t)
    {
        if constexpr (SYM)
            load_row_sym(H, bank, zi, (K - 1) / 2, t);
        else
            load_row(H, bank, zi, t);
    }

    __device__ static void load_window(float2 (&X)[E], const float2* __restrict__ spec,
                                       int64_t N, int64_t in0, int t)
    {
#pragma unroll
        for (int m = 0; m < E; ++m) {
            const int64_t idx = in0 + t + T * m;
            X[m] = (idx >= 0 && idx < N) ? spec[idx] : make_float2(0.f, 0.f);
        }
    }

    // Templates [z0, z1) of segment s, the workgroup's templates turn, turn + 1, ..
    // (see give_way).  H holds bank row z0 on entry; each template's successor
    // row (row 0 after the last template, ready for the next segment) is loaded
    // into H as soon as the first inverse pass has consumed it, so the load
    // overlaps the rest of the transform without a second register buffer.
    //
    // IB (interbinning, Sec. 3 eq. f-interp): the plane has 2N columns per
    // row; column 2r holds |y_r|^2 and column 2r+1 |(pi/4)(y_r - y_{r+1})|^2.
    // Each lane gets its right-hand neighbour's y by a DPP lane shift; the
    // segment's spare valid output supplies y_{r+1} for its last output.
    //
    // DUAL (two-bin Fourier interpolation): bank2 holds the half-bin
    // filters on the same segment geometry; per template both inverse
    // transforms run on the window's X (the half-bin row is loaded as soon
    // as the first has consumed the integer row) and the [K][2N] plane gets
    // the pair (|y_r|^2, |y_half_r|^2) in one 8-byte store.
    // DEAD: output slots m < DEAD and m >= E - DEAD hold no valid output in
    // any lane (positions below M/2 or from L - M/2 on, which needs
    // M/2 >= DEAD T); their power and stores are skipped, so the compiler
    // also drops the last butterfly operations that feed only them.
    template <bool IB, bool SYM = false, bool DUAL = false, int DEAD = 0, bool TURNS = kTurns>
    __device__ static void item(const float2* __restrict__ spec, int64_t N,
                                const float2* __restrict__ bank, int K, int M, int64_t s, int z0,
                                int z1, float* __restrict__ plane, const typename F::TW& tw,
                                float2*& la, float2*& lb, int t, float2 (&H)[E],
                                int& turn, const float2* __restrict__ bank2 = nullptr,
                                float2* __restrict__ edge = nullptr)
    {
        const int B = L - M;
        const int64_t out0 = s * B;
        const int nvalid = (int)min<int64_t>(B, N - out0);   // >= 1: segment s < nseg
        float2 X[E];
        load_window(X, spec, N, out0 - M / 2, t);
        F::template run<false>(X, la, lb, tw, t);

        static_assert(!(SYM && (IB || DUAL)), "the symmetric bank is for the plain plane");
        // One template; MIR: H holds a mirrored row in load order (symmetric
        // bank, z < c), consumed reversed and conjugated.
        auto one = [&](int z, auto mir_tag) {
            constexpr bool MIR = decltype(mir_tag)::value;
            if constexpr (TURNS)
                give_way(turn++);
            float2 v[E];
            const int znext = z + 1 == K ? 0 : z + 1;
            auto next = [&]() { load_bank_row<SYM>(H, bank, znext, K, t); };
            if constexpr (DUAL) {
                auto half = [&]() { load_row(H, bank2, z, t); };
                F::template run_mul_hook<true, kMul>(X, H, v, la, lb, tw, t, half);
                float p1[E];
#pragma unroll
                for (int m = DEAD; m < E - DEAD; ++m)
                    p1[m] = fmaf(v[m].x, v[m].x, v[m].y * v[m].y);
                F::template run_mul_hook<true, kMul>(X, H, v, la, lb, tw, t, next);
                const float* row_q0 = plane + 2 * ((int64_t)z * N + out0 - M / 2);
                const auto rs = seg_rsrc(row_q0, (M / 2 + nvalid) * 8);
#pragma unroll
                for (int m = DEAD; m < E - DEAD; ++m) {
                    const float p2 = fmaf(v[m].x, v[m].x, v[m].y * v[m].y);
                    const u32x2 pp = {__float_as_uint(p1[m]), __float_as_uint(p2)};
                    __builtin_amdgcn_raw_buffer_store_b64(pp, rs, seg_off<8>(t + T * m, M / 2), 0,
                                                          kNonTemporal);
                }
                return;
            }
            if constexpr (MIR) {
                float2 Hr[E];
#pragma unroll
                for (int m = 0; m < E; ++m)
                    Hr[m] = H[E - 1 - m];
                F::template run_mul_hook<true, kMulConj>(X, Hr, v, la, lb, tw, t, next);
            } else if constexpr (!IB) {
                F::template run_mul_hook<true, kMul>(X, H, v, la, lb, tw, t, next);
            } else {
                // the interbinned epilogue holds more values; the next row is
                // loaded once y has gone to LDS, which keeps H out of the
                // transform's register peak
                NoHook none;
                F::template run_mul_hook<true, kMul>(X, H, v, la, lb, tw, t, none);
            }
            if constexpr (!IB) {
                const float* row_q0 = plane + ((int64_t)z * N + out0 - M / 2);
                const auto rs = seg_rsrc(row_q0, (M / 2 + nvalid) * 4);
#pragma unroll
                for (int m = DEAD; m < E - DEAD; ++m) {
                    const float p = fmaf(v[m].x, v[m].x, v[m].y * v[m].y);
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(p), rs,
                                                          seg_off<4>(t + T * m, M / 2), 0,
                                                          kNonTemporal);
                }
            } else if constexpr (IB_NW == 1) {
                // one wave: y at q + 1 = (t + 1) + 64 m is lane t + 1's
                // v[m], and for lane 63 lane 0's v[m + 1]; lane 0 offers
                // v[m + 1] instead of v[m] and a rotation by one lane hands
                // every lane its neighbour (slot E, position L, is never a
                // valid output)
                next();
                const int lane = t & 63;
                const float* row_q0 = plane + 2 * ((int64_t)z * N + out0 - M / 2);
                const auto rs = seg_rsrc(row_q0, (M / 2 + nvalid) * 8);
#pragma unroll
                for (int m = DEAD; m < E - DEAD; ++m) {
                    const float2 nx = m + 1 < E ? v[m + 1] : v[m];
                    const float sx = lane == 0 ? nx.x : v[m].x;
                    const float sy = lane == 0 ? nx.y : v[m].y;
                    const float dx = __int_as_float(__builtin_amdgcn_mov_dpp(
                                         __float_as_int(sx), kDppWaveRol1, 0xf, 0xf, true)) -
                                     v[m].x;
                    const float dy = __int_as_float(__builtin_amdgcn_mov_dpp(
                                         __float_as_int(sy), kDppWaveRol1, 0xf, 0xf, true)) -
                                     v[m].y;
                    const float p = fmaf(v[m].x, v[m].x, v[m].y * v[m].y);
                    const float h = kQuarterPi2 * fmaf(dx, dx, dy * dy);
                    const u32x2 ph = {__float_as_uint(p), __float_as_uint(h)};
                    __builtin_amdgcn_raw_buffer_store_b64(ph, rs, seg_off<8>(t + T * m, M / 2), 0,
                                                          kNonTemporal);
                }
            } else {
                // several waves: lanes 0..62 take lane t + 1's v[m] by a lane
                // shift; lane 63 takes the next wave's lane 0 at the same m,
                // or in the last wave wave 0's lane 0 at m + 1, from slots
                // each wave's lane 0 fills behind a barrier of their own (an
                // array of their own below L = 8192, so the exchange buffers
                // keep their parity across templates and their addresses stay
                // loop-invariant; at 8192 the free exchange buffer, which
                // then swaps parity once more per template; slot E is read
                // only for position L, never a valid output).  For valid
                // outputs q + 1 <= M/2 + B = L - M/2 stays inside the
                // segment.  Deferring lane 63's pairs to the next transform's
                // first barrier instead leaves 8-byte holes in the plane's
                // lines that a second, partial write fills: measured 1.4-1.8x
                // slower.
                constexpr int NW = IB_NW;
                const int lane = t & 63, wave = t >> 6;
                float2* const ex = IB_OWN_EDGE ? edge : la;
                if (lane == 0) {
                    // slots DEAD .. E - DEAD: the live ones and, one past
                    // them, the spare output at L - M/2
#pragma unroll
                    for (int m = DEAD; m < E - DEAD + (DEAD > 0 ? 1 : 0); ++m)
                        ex[wave * (E + 1) + m] = v[m];
                }
                next();
                __syncthreads();
                const int ew = wave + 1 < NW ? wave + 1 : 0;
                const int em = wave + 1 < NW ? 0 : 1;
                const float* row_q0 = plane + 2 * ((int64_t)z * N + out0 - M / 2);
                const auto rs = seg_rsrc(row_q0, (M / 2 + nvalid) * 8);
#pragma unroll
                for (int m = DEAD; m < E - DEAD; ++m) {
                    const float2 e = ex[ew * (E + 1) + em + m];     // broadcast read
                    // lane t + 1's v[m]; lane 63 keeps e
                    const float bx = __int_as_float(__builtin_amdgcn_update_dpp(
                        __float_as_int(e.x), __float_as_int(v[m].x), kDppWaveShl1, 0xf, 0xf, false));
                    const float by = __int_as_float(__builtin_amdgcn_update_dpp(
                        __float_as_int(e.y), __float_as_int(v[m].y), kDppWaveShl1, 0xf, 0xf, false));
                    const float p = fmaf(v[m].x, v[m].x, v[m].y * v[m].y);
                    const float dx = v[m].x - bx, dy = v[m].y - by;
                    const float h = kQuarterPi2 * fmaf(dx, dx, dy * dy);
                    const u32x2 ph = {__float_as_uint(p), __float_as_uint(h)};
                    __builtin_amdgcn_raw_buffer_store_b64(ph, rs, seg_off<8>(t + T * m, M / 2), 0,
                                                          kNonTemporal);
                }
                if constexpr (!IB_OWN_EDGE) {
                    float2* tmp = la;
                    la = lb;
                    lb = tmp;
                }
            }
        };
        if constexpr (SYM) {
            // the mirrored templates first, then the stored rows: each loop
            // has one multiply form and no per-template branch
            const int zm = min(max((K - 1) / 2, z0), z1);
            for (int z = z0; z < zm; ++z)
                one(z, std::true_type{});
            for (int z = zm; z < z1; ++z)
                one(z, std::false_type{});
        } else {
            for (int z = z0; z < z1; ++z)
                one(z, std::false_type{});
        }
    }
};

// Work partition of the persistent kernels: the flattened (segment,
// template) items [0, total) are split into P contiguous ranges, one per
// workgroup, so every workgroup gets the same number of templates (+-1)
// and recomputes a window FFT only where its range enters a segment.
__device__ __forceinline__ void item_range(int64_t total, int64_t P, int64_t& i0, int64_t& i1)
{
    const int64_t w = blockIdx.x;
    i0 = total * w / P;
    i1 = total * (w + 1) / P;
}

// One spectrum of N bins in nseg segments; persistent grid.  IB selects the
// interbinned plane ([K][2N]) instead of the plain one ([K][N]); SYM a bank
// that stores only the z >= 0 rows; DUAL adds the half-bin bank bank2 and
// writes interleaved [K][2N] pairs.
template <int L, bool IB, bool SYM, bool DUAL, int DEAD, bool TURNS>
__global__ __launch_bounds__(Fwd<L>::T, 2) void forward_kernel(
    const float2* __restrict__ spec, int64_t N, const float2* __restrict__ bank, int K, int M,
    int64_t nseg, float* __restrict__ plane, const float2* __restrict__ bank2)
{
    // the interbinned kernel's neighbouring outputs must sit in neighbouring lanes
    constexpr int E = Geometry<L>::E;
    using W = Fwd<L, E, std::conditional_t<IB && L == 8192, Plan<L, E>, SwapPlan<L, E>>>;
    __shared__ __align__(16) float2 lds[W::F::kLds];
    __shared__ float2 twl[W::F::kLdsTwAlloc];
    __shared__ __align__(16) float2 edge[IB ? W::kEdgeAlloc : 1];   // interbinning
    int64_t i, i1;
    item_range(nseg * K, gridDim.x, i, i1);
    if (i >= i1)
        return;     // uniform across the workgroup, before any barrier
    const int t = W::F::place(threadIdx.x);
    typename W::F::TW tw;
    const int rows = SYM ? (K + 1) / 2 : K;      // bank rows before the twiddle row
    W::F::twiddles(tw, bank + (int64_t)rows * L, twl, t);
    __syncthreads();
    float2* la = lds;
    float2* lb = lds + W::F::kLdsSplit;
    float2 H[W::E];
    W::template load_bank_row<SYM>(H, bank, (int)(i % K), K, t);
    int turn = 0;
    while (i < i1) {
        const int64_t s = i / K;
        const int zs = (int)(i - s * K);
        const int ze = (int)min<int64_t>(K, zs + (i1 - i));
        W::template item<IB, SYM, DUAL, DEAD, TURNS>(spec, N, bank, K, M, s, zs, ze, plane, tw, la, lb,
                                               t, H, turn, bank2, edge);
        i += ze - zs;
    }
}

// ---- batched ragged correlation --------------------------------------------
//
// Spectra b = 0..nspec-1 are packed back to back: spectrum b is
// specs[offsets[b] .. offsets[b+1]) and its plane starts at
// planes + K * offsets[b] ([K][N_b] row-major).  A single-workgroup scan
// turns the lengths into segment counts and their prefix sums segpre[0..nspec]
// (segpre[nspec] = total segments); the persistent kernel then splits the
// flattened (segment, template) items of all spectra into contiguous ranges,
// so one launch of a fixed grid covers any batch and every workgroup reaches
// the end of its range.  The offsets are read on the device, so every use
// clamps them to the caller's capacity (the bins specs holds; planes holds K
// times as many floats): an offset past it, or a negative length, makes the
// spectrum shorter or empty, never an access outside the buffers.

constexpr int kScanThreads = 1024;

// segpre[b + 1] = sum over b' <= b of ceil(N_b' / B) (segments of length B,
// or the adjoint's windows, which have the same count).
__global__ __launch_bounds__(kScanThreads) void segment_scan_kernel(
    const int64_t* __restrict__ offsets, int nspec, int64_t cap, int B, int64_t* __restrict__ segpre)
{
    __shared__ int64_t part[kScanThreads];
    __shared__ int64_t carry;
    const int t = threadIdx.x;
    if (t == 0) {
        carry = 0;
        segpre[0] = 0;
    }
    __syncthreads();
    for (int base = 0; base < nspec; base += kScanThreads) {
        const int b = base + t;
        int64_t segs = 0;
        if (b < nspec) {
            int64_t off, n;
            spec_range(offsets, b, cap, off, n);
            segs = (n + B - 1) / B;
        }
        part[t] = segs;
        __syncthreads();
        // Hillis-Steele inclusive scan over the chunk
        for (int d = 1; d < kScanThreads; d <<= 1) {
            const int64_t add = t >= d ? part[t - d] : 0;
            __syncthreads();
            part[t] += add;
            __syncthreads();
        }
        if (b < nspec)
            segpre[b + 1] = carry + part[t];
        __syncthreads();
        if (t == kScanThreads - 1)
            carry += part[t];
        __syncthreads();
    }
}

// The spectrum that owns flattened segment `tile`: the last b with
// segpre[b] <= tile (segpre is non-decreasing, segpre[0] = 0 <= tile).
__device__ __forceinline__ int owner(const int64_t* __restrict__ segpre, int nspec, int64_t tile)
{
    int lo = 0, hi = nspec - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (segpre[mid] <= tile) lo = mid; else hi = mid - 1;
    }
    return lo;
}

template <int L, int E, int DEAD, bool TURNS>
__global__ __launch_bounds__((Fwd<L, E>::T), 2) void batched_kernel(
    const float2* __restrict__ specs, const int64_t* __restrict__ offsets,
    const int64_t* __restrict__ segpre, int nspec, int64_t cap, const float2* __restrict__ bank,
    int K, int M, float* __restrict__ planes)
{
    using W = Fwd<L, E>;
    __shared__ __align__(16) float2 lds[W::F::kLds];
    __shared__ float2 twl[W::F::kLdsTwAlloc];
    int64_t i, i1;
    // Fewer items than workgroups, which only the device knows: the first ones take one
    // each.  Spread over the whole grid they shared CUs while others idled: 168 items,
    // E = 8, L = 4096, grid 512: 17.1 us, so 12.7; L = 2048, 1024: 15.9 and 10.1; E = 16, L =
    // 2048, 512: 14.6 and 10.9.
    const int64_t items = segpre[nspec] * K, P = min<int64_t>(gridDim.x, items);
    if (blockIdx.x >= P)
        return;
    item_range(items, P, i, i1);
    if (i >= i1)
        return;
    const int t = W::F::place(threadIdx.x);
    typename W::F::TW tw;
    W::F::twiddles(tw, bank + (int64_t)K * L, twl, t);
    __syncthreads();
    float2* la = lds;
    float2* lb = lds + W::F::kLdsSplit;
    float2 H[W::E];
    W::load_row(H, bank, (int)(i % K), t);
    int turn = 0;
    while (i < i1) {
        const int64_t tile = i / K;
        const int zs = (int)(i - tile * K);
        const int ze = (int)min<int64_t>(K, zs + (i1 - i));
        const int b = owner(segpre, nspec, tile);
        int64_t off, Nb;
        spec_range(offsets, b, cap, off, Nb);
        W::template item<false, false, false, DEAD, TURNS>(specs + off, Nb, bank, K, M,
                                                    tile - segpre[b], zs, ze,
                                                    planes + (int64_t)K * off, tw, la, lb, t, H,
                                                    turn);
        i += ze - zs;
    }
}

// ---- adjoint (backward) ------------------------------------------------------
//
// Loss Lw = sum_{z,r} w[z][r] P[z][r] with w = dLw/dP given.  In PyTorch's
// complex convention (grad = dLw/dRe + i dLw/dIm), with g = 2 w Y:
//   grad_A[k]    = sum_z sum_j T[z][j] g[z][k - e_j]
//   grad_T[z][j] = sum_r conj(g[z][r]) A[r + e_j].
// Per forward window s (input bins [w0, w0 + L), w0 = s B - M/2; owned outputs
// t in [M/2, M/2 + B)), the correlation is y = IFFT(X H_z) with X = FFT(a_w);
// its adjoint is IFFT(conj(H_z) FFT(g_w)), and the window's part of grad_T is
// the circular cross-correlation IFFT(conj(G) X)/L at lags e_j.  Because g_w
// is supported on the owned outputs only, neither wraps, and summing the
// windows' contributions gives the exact gradients.  Y is recomputed, never
// stored.  Window contributions go to per-(chunk, window) partial buffers and
// are summed in FP64, in a fixed order, by the two reduction kernels.
template <int L, class PLAN = SwapPlan<L, BwdGeometry<L>::E>>
struct Bwd {
    using W = Fwd<L, BwdGeometry<L>::E, PLAN>;
    using F = typename W::F;
    static constexpr int E = W::E;
    static constexpr int T = W::T;
    static constexpr int NTW = W::NTW;

    // Templates [z0, z1) of window s.  Hc holds bank row z0 on entry.  Per
    // template the weights w_z are loaded before the inverse transform and
    // the next bank row is loaded once the first pass of FFT(g) has started,
    // so neither load's latency sits on the critical path; row z stays live
    // for the accumulate step.  WANT_T is a compile-time switch: without the
    // taps gradient's transform the kernel needs ~80 fewer VGPRs, which buys
    // a third wave per SIMD.
    // EDGE (M/2 = T exactly): slot 0 holds the positions below M/2 and slot
    // E-1 those from L - M/2 on in every lane.  No window owns them, so g is
    // zero there (w is not read), and they are exactly the taps gradient's
    // lags, which are then stored without a per-lane test; the compiler
    // drops the transform outputs nothing reads.
    template <bool WANT_T, bool EDGE = false>
    __device__ static void item(const float2* __restrict__ spec, int64_t N,
                                const float2* __restrict__ bank, int M, int64_t s, int z0,
                                int z1, const float* __restrict__ dLdP, bool want_A,
                                float2* __restrict__ partA,
                                float2* __restrict__ partT, const typename F::TW& tw,
                                float2*& la, float2*& lb, int t, float2 (&Hc)[E])
    {
        const int B = L - M;
        const int64_t out0 = s * B;
        const int nvalid = (int)min<int64_t>(B, N - out0);   // >= 1: window s < nwin
        float2 X[E];
        W::load_window(X, spec, N, out0 - M / 2, t);
        F::template run<false>(X, la, lb, tw, t);

        float2 acc[E];
#pragma unroll
        for (int m = 0; m < E; ++m)
            acc[m] = make_float2(0.f, 0.f);

        for (int z = z0; z < z1; ++z) {
            // 2 w on the owned outputs, zero elsewhere (w is read exactly once;
            // out-of-range buffer loads return 0)
            const auto rw = seg_rsrc(dLdP + ((int64_t)z * N + out0 - M / 2), (M / 2 + nvalid) * 4);
            float wv[E];
#pragma unroll
            for (int m = 0; m < E; ++m)
                wv[m] = (EDGE && (m == 0 || m == E - 1))
                            ? 0.f
                            : 2.f * __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                                        rw, seg_off<4>(t + T * m, M / 2), 0, kNonTemporal));
            float2 v[E];
            F::template run_mul<true, kMul>(X, Hc, v, la, lb, tw, t);     // y = IFFT(X H_z)
#pragma unroll
            for (int m = 0; m < E; ++m)                                   // g = 2 w y
                v[m] = (EDGE && (m == 0 || m == E - 1))
                           ? make_float2(0.f, 0.f)
                           : make_float2(wv[m] * v[m].x, wv[m] * v[m].y);
            float2 Hn[E];
            const int zn = z + 1 < z1 ? z + 1 : z0;
            auto next = [&]() { W::load_row(Hn, bank, zn, t); };
            F::template run_hook<false>(v, la, lb, tw, t, next);          // G = FFT(g)
            if (want_A) {
#pragma unroll
                for (int m = 0; m < E; ++m) {                             // acc += conj(H) G
                    acc[m].x = fmaf(v[m].x, Hc[m].x, fmaf(v[m].y, Hc[m].y, acc[m].x));
                    acc[m].y = fmaf(v[m].y, Hc[m].x, fmaf(-v[m].x, Hc[m].y, acc[m].y));
                }
            }
            if constexpr (WANT_T) {
                F::template run_mul<true, kMulConj>(X, v, v, la, lb, tw, t);  // IFFT(X conj(G))
                float2* pz = partT + (int64_t)z * M;
                if constexpr (EDGE) {
                    pz[t + M / 2] = v[0];                                 // p = t < M/2
                    pz[t] = v[E - 1];                                     // p - L + M/2 = t
                } else {
#pragma unroll
                    for (int m = 0; m < E; ++m) {
                        const int p = t + T * m;
                        if (p < M / 2)
                            pz[p + M / 2] = v[m];
                        else if (p >= L - M / 2)
                            pz[p - L + M / 2] = v[m];
                    }
                }
            }
#pragma unroll
            for (int m = 0; m < E; ++m)
                Hc[m] = Hn[m];
        }
        if (want_A) {
            F::template run<true>(acc, la, lb, tw, t);
#pragma unroll
            for (int m = 0; m < E; ++m)
                partA[t + T * m] = acc[m];
        }
    }

    // One window of a group: its spectrum, bin count, window index in that
    // spectrum, weights and partial-gradient row.  n = 0 marks an absent
    // window (the group's tail past the last window).
    struct Win {
        const float2* spec;
        int64_t N;
        int64_t s;
        const float* dLdP;
        float2* partA;
    };

    // Both gradients for NW windows at once.  The taps gradient of template
    // z is sum_s IFFT(X_s conj(G_{z,s})) at the lags; the inverse transform
    // is linear, so the group accumulates P_z = sum_s X_s conj(G_{z,s}) in
    // the frequency domain and runs one inverse transform per template for
    // all its windows: 2 + 1/NW transforms per (window, template) instead
    // of 3, and partT holds one [K][M] row per group instead of per window.
    // The spectrum gradient is computed exactly as by item(), window by
    // window (bitwise the same partials).
    template <bool EDGE, int NW>
    __device__ static void item_group(const Win (&win)[NW], const float2* __restrict__ bank,
                                      int M, int z0, int z1, bool want_A,
                                      float2* __restrict__ partT, const typename F::TW& tw,
                                      float2*& la, float2*& lb, int t, float2 (&Hc)[E])
    {
        const int B = L - M;
        float2 X[NW][E];
        float2 acc[NW][E];
        int nvalid[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const int64_t out0 = win[w].s * B;
            nvalid[w] = win[w].spec ? (int)min<int64_t>(B, win[w].N - out0) : 0;
            if (win[w].spec) {
                W::load_window(X[w], win[w].spec, win[w].N, out0 - M / 2, t);
                F::template run<false>(X[w], la, lb, tw, t);
            }
#pragma unroll
            for (int m = 0; m < E; ++m)
                acc[w][m] = make_float2(0.f, 0.f);
        }

        for (int z = z0; z < z1; ++z) {
            float2 P[E];
#pragma unroll
            for (int m = 0; m < E; ++m)
                P[m] = make_float2(0.f, 0.f);
            float2 Hn[E];
            const int zn = z + 1 < z1 ? z + 1 : z0;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                if (!win[w].spec)           // uniform: the group's tail
                    continue;
                const int64_t out0 = win[w].s * B;
                const auto rw = seg_rsrc(win[w].dLdP + ((int64_t)z * win[w].N + out0 - M / 2),
                                         (M / 2 + nvalid[w]) * 4);
                float wv[E];
#pragma unroll
                for (int m = 0; m < E; ++m)
                    wv[m] = (EDGE && (m == 0 || m == E - 1))
                                ? 0.f
                                : 2.f * __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                                            rw, seg_off<4>(t + T * m, M / 2), 0, kNonTemporal));
                float2 v[E];
                F::template run_mul<true, kMul>(X[w], Hc, v, la, lb, tw, t);   // y
#pragma unroll
                for (int m = 0; m < E; ++m)                                   // g = 2 w y
                    v[m] = (EDGE && (m == 0 || m == E - 1))
                               ? make_float2(0.f, 0.f)
                               : make_float2(wv[m] * v[m].x, wv[m] * v[m].y);
                if (w == NW - 1 || !win[w + 1 < NW ? w + 1 : w].spec) {
                    auto next = [&]() { W::load_row(Hn, bank, zn, t); };
                    F::template run_hook<false>(v, la, lb, tw, t, next);      // G = FFT(g)
                } else {
                    F::template run<false>(v, la, lb, tw, t);
                }
                if (want_A) {
#pragma unroll
                    for (int m = 0; m < E; ++m) {                             // acc += conj(H) G
                        acc[w][m].x = fmaf(v[m].x, Hc[m].x, fmaf(v[m].y, Hc[m].y, acc[w][m].x));
                        acc[w][m].y = fmaf(v[m].y, Hc[m].x, fmaf(-v[m].x, Hc[m].y, acc[w][m].y));
                    }
                }
#pragma unroll
                for (int m = 0; m < E; ++m) {                                 // P += X conj(G)
                    P[m].x = fmaf(X[w][m].x, v[m].x, fmaf(X[w][m].y, v[m].y, P[m].x));
                    P[m].y = fmaf(X[w][m].y, v[m].x, fmaf(-X[w][m].x, v[m].y, P[m].y));
                }
            }
            F::template run<true>(P, la, lb, tw, t);                          // lags
            float2* pz = partT + (int64_t)z * M;
            if constexpr (EDGE) {
                pz[t + M / 2] = P[0];
                pz[t] = P[E - 1];
            } else {
#pragma unroll
                for (int m = 0; m < E; ++m) {
                    const int p = t + T * m;
                    if (p < M / 2)
                        pz[p + M / 2] = P[m];
                    else if (p >= L - M / 2)
                        pz[p - L + M / 2] = P[m];
                }
            }
#pragma unroll
            for (int m = 0; m < E; ++m)
                Hc[m] = Hn[m];
        }
        if (want_A) {
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                if (!win[w].spec)
                    continue;
                F::template run<true>(acc[w], la, lb, tw, t);
#pragma unroll
                for (int m = 0; m < E; ++m)
                    win[w].partA[t + T * m] = acc[w][m];
            }
        }
    }
};

template <int L, bool WANT_T, bool EDGE, class PLAN = SwapPlan<L, BwdGeometry<L>::E>>
__global__ __launch_bounds__(Bwd<L>::T, WANT_T ? BwdGeometry<L>::kMinWaves
                                               : BwdGeometry<L>::kMinWavesSpec) void backward_kernel(
    const float2* __restrict__ spec, int64_t N, const float2* __restrict__ bank, int K, int M,
    int zchunk, int64_t nwin, const float* __restrict__ dLdP, int want_A,
    float2* __restrict__ partA, float2* __restrict__ partT)
{
    using Bk = Bwd<L, PLAN>;
    __shared__ __align__(16) float2 lds[Bk::F::kLds];
    __shared__ float2 twl[Bk::F::kLdsTwAlloc];
    const int t = Bk::F::place(threadIdx.x);
    typename Bk::F::TW tw;
    Bk::F::twiddles(tw, bank + (int64_t)K * L, twl, t);
    __syncthreads();
    float2* la = lds;
    float2* lb = lds + Bk::F::kLdsSplit;
    const int64_t s = blockIdx.x;
    const int c = blockIdx.y;
    const int z0 = c * zchunk;
    const int z1 = min(K, z0 + zchunk);
    float2 H[Bk::E];
    Bk::W::load_row(H, bank, z0, t);
    constexpr int NW = WANT_T && EDGE ? BwdGeometry<L>::kWinGroupEdge : 1;
    if constexpr (NW == 1) {
        Bk::template item<WANT_T, EDGE>(spec, N, bank, M, s, z0, z1, dLdP, want_A != 0,
                                        partA + ((int64_t)c * nwin + s) * L,
                                        partT + s * (int64_t)K * M, tw, la, lb, t, H);
    } else {
        // workgroup x takes windows x NW .. x NW + NW - 1 (those below nwin)
        typename Bk::Win win[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const int64_t sw = s * NW + w;
            const bool ok = sw < nwin;
            win[w] = {ok ? spec : nullptr, N, sw, dLdP,
                      partA + ((int64_t)c * nwin + (ok ? sw : 0)) * L};
        }
        Bk::template item_group<EDGE, NW>(win, bank, M, z0, z1, want_A != 0,
                                          partT + s * (int64_t)K * M, tw, la, lb, t, H);
    }
}

// grad_A[k] = sum over chunks c and windows s covering k of
// partA[c][s][k - (s B - M/2)], summed in FP64 in (c, s) order.
__global__ void reduce_grad_spec_kernel(const float2* __restrict__ partA, int64_t N, int L, int M,
                                        int64_t nwin, int nzc, float2* __restrict__ grad)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= N)
        return;
    const int B = L - M;
    int64_t s_hi = (k + M / 2) / B;            // windows with s B - M/2 <= k
    if (s_hi > nwin - 1)
        s_hi = nwin - 1;
    const int64_t lo_num = k + M / 2 - L;      // windows with s B - M/2 + L > k
    const int64_t s_lo = lo_num < 0 ? 0 : lo_num / B + 1;
    double sr = 0.0, si = 0.0;
    for (int c = 0; c < nzc; ++c)
        for (int64_t s = s_lo; s <= s_hi; ++s) {
            const int64_t p = k - (s * B - M / 2);
            const float2 v = partA[((int64_t)c * nwin + s) * L + p];
            sr += v.x;
            si += v.y;
        }
    grad[k] = make_float2((float)sr, (float)si);
}

// grad_T[z][j] = (1/L) sum_s partT[s][z][j] in FP64 (s: the rows of partT,
// one per window or per group of windows), in two fixed-order
// stages.  Stage 1: block (x, y) covers kTapsCols consecutive (z, j) entries
// and the windows s of chunk y; lane row q sums s = s0 + q, s0 + q +
// kTapsRows, ..., the rows are added in order q = 0, 1, ..., and the FP64
// sum goes to tpart[y][(z, j)].  Stage 2 adds the chunks in order y = 0,
// 1, ... and scales.  The chunking depends only on the geometry, so the
// result is deterministic.
constexpr int kTapsCols = 64, kTapsRows = 16;

__global__ __launch_bounds__(kTapsCols * kTapsRows) void reduce_grad_taps_kernel(
    const float2* __restrict__ partT, int64_t nwin, const int64_t* __restrict__ nwin_dev,
    int group, int64_t chunk, int KM, double2* __restrict__ tpart)
{
    __shared__ double part[kTapsRows][kTapsCols][2];
    const int c = threadIdx.x % kTapsCols, q = threadIdx.x / kTapsCols;
    const int i = blockIdx.x * kTapsCols + c;
    // rows present: nwin, or (batched) the groups of the windows actually
    // present (a device window count, rows of `group` windows, at most nwin)
    const int64_t nw = nwin_dev ? min(nwin, (*nwin_dev + group - 1) / group) : nwin;
    const int64_t s0 = (int64_t)blockIdx.y * chunk;
    const int64_t s1 = min(nw, s0 + chunk);
    double sr = 0.0, si = 0.0;
    if (i < KM)
        for (int64_t s = s0 + q; s < s1; s += kTapsRows) {
            const float2 v = partT[s * KM + i];
            sr += v.x;
            si += v.y;
        }
    part[q][c][0] = sr;
    part[q][c][1] = si;
    __syncthreads();
    if (q == 0 && i < KM) {
        double tr = 0.0, ti = 0.0;
        for (int r = 0; r < kTapsRows; ++r) {
            tr += part[r][c][0];
            ti += part[r][c][1];
        }
        tpart[(int64_t)blockIdx.y * KM + i] = make_double2(tr, ti);
    }
}

__global__ void reduce_grad_taps_final_kernel(const double2* __restrict__ tpart, int nsplit,
                                              int KM, int L, float2* __restrict__ grad)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= KM)
        return;
    double tr = 0.0, ti = 0.0;
    for (int y = 0; y < nsplit; ++y) {
        const double2 v = tpart[(int64_t)y * KM + i];
        tr += v.x;
        ti += v.y;
    }
    const double inv = 1.0 / (double)L;
    grad[i] = make_float2((float)(tr * inv), (float)(ti * inv));
}

// ---- batched adjoint -----------------------------------------------------------
//
// The adjoint over the spectra of a batched forward (packed as for
// batched_kernel, dL/dP packed like the planes).  A window of spectrum b is
// the same window as in the single-spectrum adjoint; windows of all spectra
// are numbered globally by the scan winpre (windows per spectrum =
// ceil(N_b / B), the segment count).  The grid is fixed by the host's bound
// maxwin on the window count (which only offsets that overlap could exceed)
// times the template chunks, so one launch covers any batch within the
// bound and a captured graph serves new batches.  Workgroups past the
// batch's actual window count exit at once, so no partial buffer is overrun.
// One window per workgroup (global window blockIdx.z * gridDim.x +
// blockIdx.x), as in the single-spectrum kernel, so the body allocates the
// same registers (a grid-stride loop over windows made the compiler keep
// more values live and spill).
template <int L, bool WANT_T, bool EDGE, class PLAN = SwapPlan<L, BwdGeometry<L>::E>>
__global__ __launch_bounds__(Bwd<L>::T, WANT_T ? BwdGeometry<L>::kMinWaves
                                               : BwdGeometry<L>::kMinWavesSpec) void
backward_batched_kernel(const float2* __restrict__ specs, const int64_t* __restrict__ offsets,
                        const int64_t* __restrict__ winpre, int nspec, int64_t cap,
                        const float2* __restrict__ bank, int K, int M, int zchunk, int64_t maxwin,
                        const float* __restrict__ dLdP, int want_A, float2* __restrict__ partA,
                        float2* __restrict__ partT)
{
    using Bk = Bwd<L, PLAN>;
    __shared__ __align__(16) float2 lds[Bk::F::kLds];
    __shared__ float2 twl[Bk::F::kLdsTwAlloc];
    const int64_t nw = min(winpre[nspec], maxwin);
    const int c = blockIdx.y;
    const int z0 = c * zchunk;
    const int z1 = min(K, z0 + zchunk);
    constexpr int NW = WANT_T && EDGE ? BwdGeometry<L>::kWinGroupEdge : 1;
    const int64_t g = (int64_t)blockIdx.z * gridDim.x + blockIdx.x;   // window, or group
    if (g * NW >= nw)
        return;     // uniform across the workgroup, before any barrier
    const int t = Bk::F::place(threadIdx.x);
    typename Bk::F::TW tw;
    Bk::F::twiddles(tw, bank + (int64_t)K * L, twl, t);
    __syncthreads();
    float2* la = lds;
    float2* lb = lds + Bk::F::kLdsSplit;
    float2 H[Bk::E];
    Bk::W::load_row(H, bank, z0, t);
    if constexpr (NW == 1) {
        const int b = owner(winpre, nspec, g);
        int64_t off, Nb;
        spec_range(offsets, b, cap, off, Nb);
        Bk::template item<WANT_T, EDGE>(specs + off, Nb, bank, M, g - winpre[b], z0, z1,
                                        dLdP + (int64_t)K * off, want_A != 0,
                                        partA + ((int64_t)c * maxwin + g) * L,
                                        partT + g * (int64_t)K * M, tw, la, lb, t, H);
    } else {
        // group g: global windows g NW .. g NW + NW - 1 (those below the
        // batch's count), each from its own spectrum
        typename Bk::Win win[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const int64_t gw = g * NW + w;
            if (gw < nw) {
                const int b = owner(winpre, nspec, gw);
                int64_t off, Nb;
                spec_range(offsets, b, cap, off, Nb);
                win[w] = {specs + off, Nb, gw - winpre[b], dLdP + (int64_t)K * off,
                          partA + ((int64_t)c * maxwin + gw) * L};
            } else {
                win[w] = {nullptr, 0, 0, nullptr, partA};
            }
        }
        Bk::template item_group<EDGE, NW>(win, bank, M, z0, z1, want_A != 0,
                                          partT + g * (int64_t)K * M, tw, la, lb, t, H);
    }
}

// grad[k] for every packed bin k < cap: the bins of spectrum b (the last b
// whose clamped range starts at or before k and contains it) sum their
// windows' partials as reduce_grad_spec_kernel does, in the same (chunk,
// window) order, so each spectrum's gradient is bitwise the single-spectrum
// one; bins outside every spectrum get 0.
__global__ void reduce_grad_spec_batched_kernel(const float2* __restrict__ partA,
                                                const int64_t* __restrict__ offsets,
                                                const int64_t* __restrict__ winpre, int nspec,
                                                int64_t cap, int L, int M, int64_t maxwin,
                                                int nzc, float2* __restrict__ grad)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= cap)
        return;
    if (nspec == 0) {
        grad[k] = make_float2(0.f, 0.f);
        return;
    }
    // the last spectrum whose (clamped) start is <= k
    int lo = 0, hi = nspec - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        int64_t o = offsets[mid];
        o = o < 0 ? 0 : (o > cap ? cap : o);
        if (o <= k) lo = mid; else hi = mid - 1;
    }
    int64_t off, n;
    spec_range(offsets, lo, cap, off, n);
    if (k < off || k >= off + n) {
        grad[k] = make_float2(0.f, 0.f);
        return;
    }
    const int64_t kl = k - off;
    const int B = L - M;
    const int64_t nwin = (n + B - 1) / B;
    int64_t s_hi = (kl + M / 2) / B;           // windows with s B - M/2 <= kl
    if (s_hi > nwin - 1)
        s_hi = nwin - 1;
    const int64_t lo_num = kl + M / 2 - L;     // windows with s B - M/2 + L > kl
    const int64_t s_lo = lo_num < 0 ? 0 : lo_num / B + 1;
    double sr = 0.0, si = 0.0;
    for (int c = 0; c < nzc; ++c)
        for (int64_t s = s_lo; s <= s_hi; ++s) {
            const int64_t g = winpre[lo] + s;
            if (g >= maxwin)
                continue;
            const int64_t p = kl - (s * B - M / 2);
            const float2 v = partA[((int64_t)c * maxwin + g) * L + p];
            sr += v.x;
            si += v.y;
        }
    grad[k] = make_float2((float)sr, (float)si);
}

// ---- launchers -------------------------------------------------------------------

// Resident workgroups of `kernel` on the current device (occupancy x CUs),
// queried once per (device, kernel) and cached so later calls -- e.g. under
// graph capture -- make no runtime queries.
template <class Kern>
static hipError_t resident_grid(Kern kernel, int threads, std::atomic<int>* cache, int* grid)
{
    constexpr int kMaxDev = 64;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return e;
    if (dev >= 0 && dev < kMaxDev) {
        const int c = cache[dev].load(std::memory_order_relaxed);
        if (c > 0) {
            *grid = c;
            return hipSuccess;
        }
    }
    int per_cu = 0, cus = 0;
    if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0)) !=
        hipSuccess)
        return e;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) !=
        hipSuccess)
        return e;
    *grid = (per_cu > 0 ? per_cu : 1) * (cus > 0 ? cus : 1);
    if (dev >= 0 && dev < kMaxDev)
        cache[dev].store(*grid, std::memory_order_relaxed);
    return hipSuccess;
}

template <int L, bool IB, bool SYM, bool DUAL, int DEAD, bool TURNS>
static hipError_t resident_forward(int* grid)
{
    static std::atomic<int> cache[64];
    return resident_grid(forward_kernel<L, IB, SYM, DUAL, DEAD, TURNS>, Fwd<L>::T, cache, grid);
}

template <int L, bool IB, bool SYM, bool DUAL, int DEAD>
static hipError_t launch_forward_LD(const float2* spec, int64_t N, const float2* bank, int K,
                                    int M, float* plane, int grid, const float2* bank2,
                                    hipStream_t s)
{
    constexpr bool TURNS = Fwd<L>::kTurns;
    constexpr int FEW = turn_eighths<L, IB, SYM, DUAL, DEAD, false>();
    const int64_t nseg = (N + (L - M) - 1) / (L - M);
    if (grid <= 0) {
        hipError_t e = resident_forward<L, IB, SYM, DUAL, DEAD, TURNS>(&grid);
        if (e != hipSuccess)
            return e;
    }
    if ((int64_t)grid > nseg * K)
        grid = (int)(nseg * K);
    if (8 * nseg * K < (int64_t)FEW * grid)
        hipLaunchKernelGGL((forward_kernel<L, IB, SYM, DUAL, DEAD, FEW == 0 && TURNS>), dim3(grid),
                           dim3(Fwd<L>::T), 0, s, spec, N, bank, K, M, nseg, plane, bank2);
    else
        hipLaunchKernelGGL((forward_kernel<L, IB, SYM, DUAL, DEAD, TURNS>), dim3(grid),
                           dim3(Fwd<L>::T), 0, s, spec, N, bank, K, M, nseg, plane, bank2);
    return hipGetLastError();
}

// Output slots with no valid output in any lane at each end (0..2): the
// first covers positions below T, the second below 2T, all inside M/2.
template <int L, int E = Geometry<L>::E>
static int dead_slots(int M)
{
    const int d = (M / 2) / Fwd<L, E>::T;
    return d < 2 ? d : 2;
}

template <int L, bool IB, bool SYM, bool DUAL>
static hipError_t launch_forward_L(const float2* spec, int64_t N, const float2* bank, int K,
                                   int M, float* plane, int grid, const float2* bank2,
                                   hipStream_t s)
{
    switch (dead_slots<L>(M)) {
    case 0: return launch_forward_LD<L, IB, SYM, DUAL, 0>(spec, N, bank, K, M, plane, grid, bank2, s);
    case 1: return launch_forward_LD<L, IB, SYM, DUAL, 1>(spec, N, bank, K, M, plane, grid, bank2, s);
    default: return launch_forward_LD<L, IB, SYM, DUAL, 2>(spec, N, bank, K, M, plane, grid, bank2, s);
    }
}

template <bool IB, bool SYM, bool DUAL>
static hipError_t launch_forward_ib(const float2* spec, int64_t N, const float2* bank, int K,
                                    int M, int L, float* plane, int grid, const float2* bank2,
                                    hipStream_t s)
{
    switch (L) {
    case 256:  return launch_forward_L<256, IB, SYM, DUAL>(spec, N, bank, K, M, plane, grid, bank2, s);
    case 512:  return launch_forward_L<512, IB, SYM, DUAL>(spec, N, bank, K, M, plane, grid, bank2, s);
    case 1024: return launch_forward_L<1024, IB, SYM, DUAL>(spec, N, bank, K, M, plane, grid, bank2, s);
    case 2048: return launch_forward_L<2048, IB, SYM, DUAL>(spec, N, bank, K, M, plane, grid, bank2, s);
    case 4096: return launch_forward_L<4096, IB, SYM, DUAL>(spec, N, bank, K, M, plane, grid, bank2, s);
    case 8192: return launch_forward_L<8192, IB, SYM, DUAL>(spec, N, bank, K, M, plane, grid, bank2, s);
    default:   return hipErrorInvalidValue;
    }
}

hipError_t launch_forward(const float2* spec, int64_t N, const float2* bank, int K, int M,
                          int L, float* plane, int grid, bool interbin, bool sym, hipStream_t s)
{
    if (sym)   // the symmetric bank serves the plain plane only
        return interbin ? hipErrorInvalidValue
                        : launch_forward_ib<false, true, false>(spec, N, bank, K, M, L, plane,
                                                                grid, nullptr, s);
    return interbin
               ? launch_forward_ib<true, false, false>(spec, N, bank, K, M, L, plane, grid,
                                                       nullptr, s)
               : launch_forward_ib<false, false, false>(spec, N, bank, K, M, L, plane, grid,
                                                        nullptr, s);
}

hipError_t launch_forward_dual(const float2* spec, int64_t N, const float2* bank,
                               const float2* bank_half, int K, int Mgeom, int L, float* plane2,
                               int grid, hipStream_t s)
{
    return launch_forward_ib<false, false, true>(spec, N, bank, K, Mgeom, L, plane2, grid,
                                                 bank_half, s);
}

template <int L, int E, int DEAD>
static hipError_t resident_batched_LD(int* grid)
{
    static std::atomic<int> cache[64];
    const hipError_t e = resident_grid(batched_kernel<L, E, DEAD, Fwd<L, E>::kTurns>,
                                       Fwd<L, E>::T, cache, grid);
    // Five of the eight workgroups that fit a CU: with all of them at work the 960 or 896
    // columns of each, in rows of any alignment, leave more half-written lines than
    // the caches hold until a neighbour completes them.  Spectra of odd length, K = 85,
    // M = 64: 2048 workgroups 97.8 us, 1280 83.7 (1536 of the plan before 87.3); of even
    // length 81.1 and 85.0 (88.9).
    if (L == 1024 && E == 8 && DEAD == 0)
        *grid = *grid * 5 / 8;
    return e;
}

template <int L, int E>
static hipError_t resident_batched_LE(int M, int* grid)
{
    switch (dead_slots<L, E>(M)) {
    case 0: return resident_batched_LD<L, E, 0>(grid);
    case 1: return resident_batched_LD<L, E, 1>(grid);
    default: return resident_batched_LD<L, E, 2>(grid);
    }
}

template <int L>
static hipError_t resident_batched_L(int E, int M, int* grid)
{
    constexpr int E0 = Geometry<L>::E;
    if (E == 0 || E == E0)
        return resident_batched_LE<L, E0>(M, grid);
    if constexpr (L >= 1024) {
        constexpr int E1 = E0 == 16 ? 8 : 16;
        if (E == E1)
            return resident_batched_LE<L, E1>(M, grid);
    }
    return hipErrorInvalidValue;
}

hipError_t batched_resident_grid(int L, int E, int M, int* grid)
{
    switch (L) {
    case 256:  return resident_batched_L<256>(E, M, grid);
    case 512:  return resident_batched_L<512>(E, M, grid);
    case 1024: return resident_batched_L<1024>(E, M, grid);
    case 2048: return resident_batched_L<2048>(E, M, grid);
    case 4096: return resident_batched_L<4096>(E, M, grid);
    case 8192: return resident_batched_L<8192>(E, M, grid);
    default:   return hipErrorInvalidValue;
    }
}

template <int L, int E, int DEAD>
static hipError_t launch_batched_LD(const float2* specs, const int64_t* offsets, int nspec,
                                    int64_t cap, const float2* bank, int K, int M, float* planes,
                                    int64_t* segpre, int grid, hipStream_t s)
{
    if (grid <= 0) {
        hipError_t e = resident_batched_LD<L, E, DEAD>(&grid);
        if (e != hipSuccess)
            return e;
    }
    // the templates of a full batch (E = 8 is faster with turns at every size)
    constexpr bool TURNS = Fwd<L, E>::kTurns;
    constexpr int FEW = E == Geometry<L>::E ? turn_eighths<L, false, false, false, DEAD, true>() : 0;
    if (8 * (cap / (L - M)) * K < (int64_t)FEW * grid)
        hipLaunchKernelGGL((batched_kernel<L, E, DEAD, FEW == 0 && TURNS>), dim3(grid),
                           dim3(Fwd<L, E>::T), 0, s, specs, offsets, segpre, nspec, cap, bank, K,
                           M, planes);
    else
        hipLaunchKernelGGL((batched_kernel<L, E, DEAD, TURNS>), dim3(grid), dim3(Fwd<L, E>::T), 0,
                           s, specs, offsets, segpre, nspec, cap, bank, K, M, planes);
    return hipGetLastError();
}

template <int L, int E>
static hipError_t launch_batched_LE(const float2* specs, const int64_t* offsets, int nspec,
                                    int64_t cap, const float2* bank, int K, int M, float* planes,
                                    int64_t* segpre, int grid, hipStream_t s)
{
    switch (dead_slots<L, E>(M)) {
    case 0: return launch_batched_LD<L, E, 0>(specs, offsets, nspec, cap, bank, K, M, planes, segpre, grid, s);
    case 1: return launch_batched_LD<L, E, 1>(specs, offsets, nspec, cap, bank, K, M, planes, segpre, grid, s);
    default: return launch_batched_LD<L, E, 2>(specs, offsets, nspec, cap, bank, K, M, planes, segpre, grid, s);
    }
}

template <int L>
static hipError_t launch_batched_L(const float2* specs, const int64_t* offsets, int nspec,
                                   int64_t cap, const float2* bank, int K, int M, int E,
                                   float* planes, int64_t* segpre, int grid, hipStream_t s)
{
    constexpr int E0 = Geometry<L>::E;
    if (E == 0 || E == E0)
        return launch_batched_LE<L, E0>(specs, offsets, nspec, cap, bank, K, M, planes, segpre, grid, s);
    if constexpr (L >= 1024) {
        constexpr int E1 = E0 == 16 ? 8 : 16;
        if (E == E1)
            return launch_batched_LE<L, E1>(specs, offsets, nspec, cap, bank, K, M, planes, segpre, grid, s);
    }
    return hipErrorInvalidValue;
}

bool batched_values_per_lane_ok(int L, int E)
{
    if (E == 0)
        return true;
    if (L <= 256)
        return E == 4;
    if (L == 512)
        return E == 8;
    return E == 8 || E == 16;
}

// ---- allocation-free batched correlation -------------------------------------
//
// fdas_correlate_batched_noalloc keeps the segment prefix segpre[nspec + 1]
// in this file-scope device array instead of a caller workspace.  Every GPU
// the library runs on holds its own copy until the process ends.  Host code
// never passes the array's name to a kernel (on the host it is only a
// stand-in symbol): the device address is looked up once per device with
// hipGetSymbolAddress and kept in g_noalloc_ptr.  The scan kernel writes
// every entry the correlation kernel reads (segpre[0] = 0 and segpre[1..nspec]),
// so nothing has to be cleared between calls; calls that overlap on one GPU
// share the array and race.
static __device__ __align__(256) int64_t scratch[FDAS_NOALLOC_MAX_SPECTRA + 1];

constexpr int kMaxDevices = 64;
static std::atomic<int64_t*> g_noalloc_ptr[kMaxDevices];

hipError_t noalloc_segpre(int64_t** out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return e;
    if (dev < 0 || dev >= kMaxDevices)
        return hipErrorInvalidDevice;
    int64_t* p = g_noalloc_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        void* addr = nullptr;
        e = hipGetSymbolAddress(&addr, HIP_SYMBOL(scratch));
        if (e != hipSuccess)
            return e;
        if (!addr)
            return hipErrorInvalidSymbol;
        p = static_cast<int64_t*>(addr);
        g_noalloc_ptr[dev].store(p, std::memory_order_release);
    }
    *out = p;
    return hipSuccess;
}

hipError_t launch_batched(const float2* specs, const int64_t* offsets, int nspec, int64_t cap,
                          const float2* bank, int K, int M, int L, int E, float* planes,
                          int64_t* segpre, int grid, hipStream_t s)
{
    if (!batched_values_per_lane_ok(L, E))
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(segment_scan_kernel, dim3(1), dim3(kScanThreads), 0, s, offsets, nspec,
                       cap, L - M, segpre);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    switch (L) {
    case 256:  return launch_batched_L<256>(specs, offsets, nspec, cap, bank, K, M, E, planes, segpre, grid, s);
    case 512:  return launch_batched_L<512>(specs, offsets, nspec, cap, bank, K, M, E, planes, segpre, grid, s);
    case 1024: return launch_batched_L<1024>(specs, offsets, nspec, cap, bank, K, M, E, planes, segpre, grid, s);
    case 2048: return launch_batched_L<2048>(specs, offsets, nspec, cap, bank, K, M, E, planes, segpre, grid, s);
    case 4096: return launch_batched_L<4096>(specs, offsets, nspec, cap, bank, K, M, E, planes, segpre, grid, s);
    case 8192: return launch_batched_L<8192>(specs, offsets, nspec, cap, bank, K, M, E, planes, segpre, grid, s);
    default:   return hipErrorInvalidValue;
    }
}

// Whether the adjoint at L = 4096 runs in passes over the workgroup
// (BwdGeometry::kSplitPoints); points: of the plane, or of all planes of a batch.
template <int L>
static bool by_passes(int64_t points, int want_T, bool edge)
{
    return want_T ? edge && points >= BwdGeometry<L>::kSplitPointsEdge
                  : points >= BwdGeometry<L>::kSplitPoints;
}

template <int L>
static hipError_t launch_backward_L(const float2* spec, int64_t N, const float2* bank, int K,
                                   int M, int zchunk, int64_t nwin, const float* dLdP,
                                   int want_A, int want_T, float2* partA, float2* partT,
                                   hipStream_t s)
{
    const int nzc = (K + zchunk - 1) / zchunk;
    const dim3 grid((unsigned)nwin, (unsigned)nzc);
    const int NW = backward_window_group(L, M);
    const dim3 grid_t((unsigned)((nwin + NW - 1) / NW), (unsigned)nzc);
    // The edge specialisation pays off with the taps transform (fewer
    // instructions and cycles); without it the compiler waits for the w
    // loads early in the transform and the kernel ran slower, so the
    // spectrum-only kernel keeps the general form.
    const bool edge = M / 2 == Bwd<L>::T;
    auto launch = [&](auto kernel, dim3 g) {
        hipLaunchKernelGGL(kernel, g, dim3(Bwd<L>::T), 0, s, spec, N, bank, K, M, zchunk, nwin,
                           dLdP, want_A, partA, partT);
    };
    if (L == 4096 && by_passes<L>((int64_t)K * N, want_T, edge)) {
        if constexpr (L == 4096) {
            if (want_T)
                launch(backward_kernel<L, true, true, PassesPlan>, grid_t);
            else
                launch(backward_kernel<L, false, false, PassesPlan>, grid);
        }
    } else if (want_T && edge) {
        launch(backward_kernel<L, true, true>, grid_t);
    } else if (want_T) {
        launch(backward_kernel<L, true, false>, grid_t);
    } else {
        launch(backward_kernel<L, false, false>, grid);
    }
    return hipGetLastError();
}

hipError_t launch_backward(const float2* spec, int64_t N, const float2* bank, int K, int M,
                          int L, const float* dLdP, float2* grad_spec, float2* grad_taps,
                          int zchunk, float2* partA, float2* partT, int tsplit, double2* tpart,
                          hipStream_t s)
{
    const int64_t nwin = (N + (L - M) - 1) / (L - M);
    const int want_A = grad_spec != nullptr, want_T = grad_taps != nullptr;
    hipError_t e = hipSuccess;
    if (nwin > 0) {
        switch (L) {
        case 256:  e = launch_backward_L<256>(spec, N, bank, K, M, zchunk, nwin, dLdP, want_A, want_T, partA, partT, s); break;
        case 512:  e = launch_backward_L<512>(spec, N, bank, K, M, zchunk, nwin, dLdP, want_A, want_T, partA, partT, s); break;
        case 1024: e = launch_backward_L<1024>(spec, N, bank, K, M, zchunk, nwin, dLdP, want_A, want_T, partA, partT, s); break;
        case 2048: e = launch_backward_L<2048>(spec, N, bank, K, M, zchunk, nwin, dLdP, want_A, want_T, partA, partT, s); break;
        case 4096: e = launch_backward_L<4096>(spec, N, bank, K, M, zchunk, nwin, dLdP, want_A, want_T, partA, partT, s); break;
        case 8192: e = launch_backward_L<8192>(spec, N, bank, K, M, zchunk, nwin, dLdP, want_A, want_T, partA, partT, s); break;
        default:   return hipErrorInvalidValue;
        }
    }
    if (e != hipSuccess)
        return e;
    const int bs = 256;
    if (want_A && N > 0) {
        const int nzc = (K + zchunk - 1) / zchunk;
        hipLaunchKernelGGL(reduce_grad_spec_kernel, dim3((unsigned)((N + bs - 1) / bs)), dim3(bs),
                           0, s, partA, N, L, M, nwin, nzc, grad_spec);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
    }
    if (want_T) {
        const int KM = K * M;
        const int NW = backward_window_group(L, M);
        const int64_t ngrp = (nwin + NW - 1) / NW;       // rows of partT
        const int64_t chunk = ngrp > 0 ? (ngrp + tsplit - 1) / tsplit : 1;
        hipLaunchKernelGGL(reduce_grad_taps_kernel,
                           dim3((KM + kTapsCols - 1) / kTapsCols, (unsigned)tsplit),
                           dim3(kTapsCols * kTapsRows), 0, s, partT, ngrp,
                           (const int64_t*)nullptr, 1, chunk, KM, tpart);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
        hipLaunchKernelGGL(reduce_grad_taps_final_kernel, dim3((KM + bs - 1) / bs), dim3(bs), 0,
                           s, tpart, tsplit, KM, L, grad_taps);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
    }
    return hipSuccess;
}

constexpr int64_t kMaxBwdGridX = int64_t(1) << 22;

template <int L>
static int window_group_L(int M)
{
    return M / 2 == Bwd<L>::T ? BwdGeometry<L>::kWinGroupEdge : 1;
}

int backward_window_group(int L, int M)
{
    switch (L) {
    case 256:  return window_group_L<256>(M);
    case 512:  return window_group_L<512>(M);
    case 1024: return window_group_L<1024>(M);
    case 2048: return window_group_L<2048>(M);
    case 4096: return window_group_L<4096>(M);
    default:   return window_group_L<8192>(M);
    }
}

template <int L>
static hipError_t launch_backward_batched_L(const float2* specs, const int64_t* offsets,
                                            const int64_t* winpre, int nspec, int64_t cap,
                                            const float2* bank, int K, int M, int zchunk,
                                            int64_t maxwin, const float* dLdP, int want_A,
                                            int want_T, float2* partA, float2* partT,
                                            hipStream_t s)
{
    const int nzc = (K + zchunk - 1) / zchunk;
    // one workgroup per (window, chunk), or per (group of windows, chunk)
    // with the taps gradient: items x + gridDim.x * z
    auto grid_for = [&](int64_t items) {
        const int64_t gx = items < kMaxBwdGridX ? items : kMaxBwdGridX;
        return dim3((unsigned)gx, (unsigned)nzc, (unsigned)((items + gx - 1) / (gx > 0 ? gx : 1)));
    };
    if (maxwin < 1)
        return hipSuccess;
    const dim3 grid = grid_for(maxwin);
    const int NW = backward_window_group(L, M);
    const dim3 grid_t = grid_for((maxwin + NW - 1) / NW);
    const bool edge = M / 2 == Bwd<L>::T;
    auto launch = [&](auto kernel, dim3 g) {
        hipLaunchKernelGGL(kernel, g, dim3(Bwd<L>::T), 0, s, specs, offsets, winpre, nspec, cap,
                           bank, K, M, zchunk, maxwin, dLdP, want_A, partA, partT);
    };
    if (L == 4096 && by_passes<L>((int64_t)K * cap, want_T, edge)) {
        if constexpr (L == 4096) {
            if (want_T)
                launch(backward_batched_kernel<L, true, true, PassesPlan>, grid_t);
            else
                launch(backward_batched_kernel<L, false, false, PassesPlan>, grid);
        }
    } else if (want_T && edge) {
        launch(backward_batched_kernel<L, true, true>, grid_t);
    } else if (want_T) {
        launch(backward_batched_kernel<L, true, false>, grid_t);
    } else {
        launch(backward_batched_kernel<L, false, false>, grid);
    }
    return hipGetLastError();
}

hipError_t launch_backward_batched(const float2* specs, const int64_t* offsets, int nspec,
                                   int64_t cap, const float2* bank, int K, int M, int L,
                                   const float* dLdP, float2* grad_specs, float2* grad_taps,
                                   int zchunk, int64_t maxwin, int64_t* winpre, float2* partA,
                                   float2* partT, int tsplit, double2* tpart, hipStream_t s)
{
    const int want_A = grad_specs != nullptr, want_T = grad_taps != nullptr;
    hipLaunchKernelGGL(segment_scan_kernel, dim3(1), dim3(kScanThreads), 0, s, offsets, nspec,
                       cap, L - M, winpre);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    switch (L) {
    case 256:  e = launch_backward_batched_L<256>(specs, offsets, winpre, nspec, cap, bank, K, M, zchunk, maxwin, dLdP, want_A, want_T, partA, partT, s); break;
    case 512:  e = launch_backward_batched_L<512>(specs, offsets, winpre, nspec, cap, bank, K, M, zchunk, maxwin, dLdP, want_A, want_T, partA, partT, s); break;
    case 1024: e = launch_backward_batched_L<1024>(specs, offsets, winpre, nspec, cap, bank, K, M, zchunk, maxwin, dLdP, want_A, want_T, partA, partT, s); break;
    case 2048: e = launch_backward_batched_L<2048>(specs, offsets, winpre, nspec, cap, bank, K, M, zchunk, maxwin, dLdP, want_A, want_T, partA, partT, s); break;
    case 4096: e = launch_backward_batched_L<4096>(specs, offsets, winpre, nspec, cap, bank, K, M, zchunk, maxwin, dLdP, want_A, want_T, partA, partT, s); break;
    case 8192: e = launch_backward_batched_L<8192>(specs, offsets, winpre, nspec, cap, bank, K, M, zchunk, maxwin, dLdP, want_A, want_T, partA, partT, s); break;
    default:   return hipErrorInvalidValue;
    }
    if (e != hipSuccess)
        return e;
    const int bs = 256;
    if (want_A && cap > 0) {
        const int nzc = (K + zchunk - 1) / zchunk;
        hipLaunchKernelGGL(reduce_grad_spec_batched_kernel, dim3((unsigned)((cap + bs - 1) / bs)),
                           dim3(bs), 0, s, partA, offsets, winpre, nspec, cap, L, M, maxwin, nzc,
                           grad_specs);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
    }
    if (want_T) {
        const int KM = K * M;
        const int NW = backward_window_group(L, M);
        const int64_t ngrp = (maxwin + NW - 1) / NW;     // rows of partT
        const int64_t chunk = ngrp > 0 ? (ngrp + tsplit - 1) / tsplit : 1;
        hipLaunchKernelGGL(reduce_grad_taps_kernel,
                           dim3((KM + kTapsCols - 1) / kTapsCols, (unsigned)tsplit),
                           dim3(kTapsCols * kTapsRows), 0, s, partT, ngrp,
                           (const int64_t*)(winpre + nspec), NW, chunk, KM, tpart);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
        hipLaunchKernelGGL(reduce_grad_taps_final_kernel, dim3((KM + bs - 1) / bs), dim3(bs), 0,
                           s, tpart, tsplit, KM, L, grad_taps);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
    }
    return hipSuccess;
}

}  // namespace fdas
