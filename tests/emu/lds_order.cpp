// Host build of the transforms alone that records every LDS access, to check that
// accesses of different lanes to one place are ordered by a barrier (test
// infrastructure only).  The device's plans run, lane swaps included: the swaps
// make the lanes of a wave meet but order no memory accesses, and that the
// hardware keeps one wave's accesses in order does not bind the compiler, so
// neither counts.
#include <algorithm>
#include <atomic>
#include <barrier>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <memory>
#include <thread>
#include <vector>

namespace order {
struct Event {
    int place, lane;
    bool write;
    unsigned syncs, wave_syncs;
};
inline const char* base;
inline size_t bytes;
void record(const void* p, bool write);
}  // namespace order

#define EMU_OWN_VECTORS
struct float2 {
    float x, y;
    float2() = default;
    float2(float a, float b) : x(a), y(b) {}
    float2(const float2& o) : x(o.x), y(o.y) { order::record(&o, false); }
    float2& operator=(const float2& o)
    {
        order::record(&o, false);
        order::record(this, true);
        x = o.x;
        y = o.y;
        return *this;
    }
};
inline float2 make_float2(float a, float b) { return float2(a, b); }
struct float4 {
    float x, y, z, w;
    float4& operator=(const float4& o)
    {
        order::record(this, true);
        order::record(&z, true);
        std::memcpy(&x, &o.x, sizeof(float4));
        return *this;
    }
};
inline float4 make_float4(float a, float b, float c, float d) { return float4{a, b, c, d}; }

static uint64_t load64(const uint64_t* p)
{
    order::record(p, false);
    return *p;
}
static void store64(uint64_t* p, uint64_t v)
{
    order::record(p, true);
    *p = v;
}
#define __atomic_load_n(p, o) load64(p)
#define __atomic_store_n(p, v, o) store64(p, v)

#define __HIP_DEVICE_COMPILE__ 1
#include <hip/hip_runtime.h>

#include "../../paper_1804_05335_amd/csrc/fdas_fft.hpp"

static std::vector<order::Event> events[1024];      // per lane

void order::record(const void* p, bool write)
{
    const size_t at = (size_t)(static_cast<const char*>(p) - base);
    if (static_cast<const char*>(p) >= base && at < bytes)
        events[threadIdx.x].push_back({(int)(at / 8), (int)threadIdx.x, write, emu_syncs,
                                       emu_wave_syncs});
}

// Two transforms of the same input one after the other, forward and inverse: the
// second does not depend on the first.
template <class F, int L, int E>
static long long run(const float2* in, const float2* table, float2* fwd, float2* inv)
{
    constexpr int T = L / E;
    alignas(16) static char mem[(F::kLds + F::kLdsTwAlloc) * sizeof(float2)];
    order::base = mem;
    order::bytes = sizeof(mem);
    for (auto& e : events)
        e.clear();
    auto kernel = [](const float2* in, const float2* table, float2* fwd, float2* inv) {
        float2* lds = reinterpret_cast<float2*>(mem);
        const int t = F::place(threadIdx.x);
        typename F::TW tw;
        F::twiddles(tw, table, lds + F::kLds, t);
        __syncthreads();
        float2 *la = lds, *lb = lds + F::kLdsSplit;
        float2 v[E], w[E];
        for (int m = 0; m < E; ++m)
            v[m] = w[m] = in[t + T * m];
        F::template run<false>(v, la, lb, tw, t);
        F::template run<true>(w, la, lb, tw, t);
        for (int m = 0; m < E; ++m) {
            fwd[t + T * m] = v[m];
            inv[t + T * m] = w[m];
        }
    };
    emu_launch(kernel, dim3(1), dim3(T), in, table, fwd, inv);
    std::vector<std::vector<order::Event>> at(sizeof(mem) / 8);
    for (const auto& lane : events)
        for (const auto& e : lane)
            at[e.place].push_back(e);
    long long unordered = 0;
    for (const auto& es : at)
        for (size_t i = 0; i < es.size(); ++i)
            for (size_t j = 0; j < i; ++j) {
                const auto &a = es[i], &b = es[j];
                unordered += (a.write || b.write) && a.lane != b.lane && a.syncs == b.syncs &&
                             !(a.lane / 64 == b.lane / 64 && a.wave_syncs != b.wave_syncs);
            }
    return unordered;
}

// Pairs of LDS accesses that nothing orders, or -1 for an unknown plan.  swap: the
// plan of the kernels; 0: the plan without lane swaps.
extern "C" long long emu_unordered(int L, int E, int swap, const float2* in, const float2* table,
                                   float2* fwd, float2* inv)
{
    using namespace fdas;
#define CASE(l, e)                                                                              \
    if (L == l && E == e)                                                                       \
        return swap ? run<FFT<l, e, typename SwapPlan<l, e>::R>, l, e>(in, table, fwd, inv)     \
                    : run<FFT<l, e, typename Plan<l, e>::R>, l, e>(in, table, fwd, inv);
    CASE(256, 4)
    CASE(512, 8)
    CASE(1024, 8)
    CASE(1024, 16)
    CASE(2048, 8)
    CASE(2048, 16)
    CASE(4096, 8)
    CASE(4096, 16)
    CASE(8192, 8)
    CASE(8192, 16)
#undef CASE
    return -1;
}
