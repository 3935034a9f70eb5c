// Host export of the transforms' LDS layouts (test infrastructure only), for
// the bank-conflict model checks.
#include <hip/hip_runtime.h>

#include "../../paper_1804_05335_amd/csrc/fdas_fft.hpp"

extern "C" int emu_lds_pad(int idx, int pair)
{
    return pair ? fdas::lds_pad<true>(idx) : fdas::lds_pad<false>(idx);
}
extern "C" int emu_pair_writes(int L)
{
    switch (L) {
    case 256:  return fdas::PairWrites<256>::value;
    case 512:  return fdas::PairWrites<512>::value;
    case 1024: return fdas::PairWrites<1024>::value;
    case 2048: return fdas::PairWrites<2048>::value;
    case 4096: return fdas::PairWrites<4096>::value;
    case 8192: return fdas::PairWrites<8192>::value;
    default:   return -1;
    }
}

// The transforms split over 2^b waves: the stride of bit k in the first exchange, and
// the values in a region of each exchange buffer.
template <int L>
static int split_stride(int k)
{
    return fdas::FFT<L, 8, fdas::WaveSplit>::stride_a(k);
}
template <int L>
static int split_region(int buffer)
{
    using F = fdas::FFT<L, 8, fdas::WaveSplit>;
    return buffer == 0 ? F::kRegionA : F::kRegionB;
}
extern "C" int emu_split_stride(int b, int k)
{
    return b == 1 ? split_stride<1024>(k) : (b == 2 ? split_stride<2048>(k) : split_stride<4096>(k));
}
extern "C" int emu_split_region(int b, int buffer)
{
    return b == 1 ? split_region<1024>(buffer)
                  : (b == 2 ? split_region<2048>(buffer) : split_region<4096>(buffer));
}
