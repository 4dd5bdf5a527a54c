// croft_bluestein.hip -- the compiled Bluestein kernels: one per convolution
// length, storage and line geometry, with its launch shape.
#include <hip/hip_runtime.h>

#include "croft_bluestein.h"
#include "croft_internal.h"

namespace croft {
using namespace dev;
namespace {

// Threads per line and lines per block (256 threads), whether the exchange goes
// in two halves, and whether the tables are copied into LDS.  What bounds these
// passes is VALU issue (about 85 instructions per point of the convolution)
// and the LDS trips between, with few waves resident where a line is long: so
// threads hold 8 to 16 elements (32 at 4096 and 8192), the exchange is halved
// where that brings another block onto the CU, and from 2048 points on, where
// a block has one or two lines, each table entry would be copied for one or
// two uses and take the room of other blocks.  One sweep of a 509 x 509 x 509
// complex64 grid (m = 1024): x 0.83, y 0.98, z 0.84 ms against 1.89, 2.00,
// 2.04 for one LDS trip per stage, chirp and product; 64 elements a thread
// (one trip per FFT) took 0.95 and 1.32 ms (one wave per SIMD).  33 million
// points (us, contiguous; strided with rows of n/2): m = 512 8 elements 171;
// 222, 16 halved 187; 204; 2048 16 halved, tables in global memory 267; 340,
// in LDS 303; 388; 4096 16 halved 269; 441, 32 halved 285; 375, tables in LDS
// 577; 725; 8192 285; 518, tables in LDS 708; 1206.
template <int M, int KIND, int CB>
struct BlueShape {
    static constexpr bool k64 = CB == 16;  // FP64 compute
    static constexpr bool kLines = KIND == kContiguous;
    static constexpr int T = M == 16     ? 1
                             : M == 32   ? 4
                             : M <= 128  ? 8
                             : M == 256  ? (k64 ? 16 : 32)
                             : M == 512  ? (kLines ? 64 : 32)
                             : M == 1024 ? 64
                             : M == 2048 ? 128
                             : M == 4096 ? (k64 || kLines ? 256 : 128)
                                         : 256;
    static constexpr int E = M / T;
    static constexpr int kSplit = (M == 256 && k64) || (M == 512 && !kLines) || (M >= 1024 && M < 8192);
    static constexpr bool kTab = M <= 1024;
    static constexpr int L = M <= 32 ? 64 : M == 64 ? (k64 ? 16 : 32) : M == 128 ? 16 : 256 / T;
};

template <class St, int KIND, int M>
BluesteinLaunch launch_of() {
    BluesteinLaunch b;
    constexpr int CB = (int)sizeof(cx<typename St::R>);
    // FP64 convolutions stop at 4096 points (lengths up to 2048)
    if constexpr (CB == 8 || M <= 4096) {
        using S = BlueShape<M, KIND, CB>;
        using Cfg = GCfg<M, KIND, S::L, S::E, CB, S::kSplit, 0, S::T>;
        static_assert(Cfg::kBlock <= 256 && BlueLds<Cfg, S::kTab>::kBytes <= 160 * 1024, "launch shape");
        b.func = reinterpret_cast<const void *>(&fft_bluestein<Cfg, St, KIND, S::kTab>);
        b.T = Cfg::T;
        b.L = Cfg::L;
        b.lds = BlueLds<Cfg, S::kTab>::kBytes;
    }
    return b;
}

template <class St, int KIND>
BluesteinLaunch for_length(int m) {
    switch (m) {
        case 16: return launch_of<St, KIND, 16>();
        case 32: return launch_of<St, KIND, 32>();
        case 64: return launch_of<St, KIND, 64>();
        case 128: return launch_of<St, KIND, 128>();
        case 256: return launch_of<St, KIND, 256>();
        case 512: return launch_of<St, KIND, 512>();
        case 1024: return launch_of<St, KIND, 1024>();
        case 2048: return launch_of<St, KIND, 2048>();
        case 4096: return launch_of<St, KIND, 4096>();
        case 8192: return launch_of<St, KIND, 8192>();
        default: return BluesteinLaunch{};
    }
}

template <int KIND>
BluesteinLaunch for_dtype(int dtype, int m) {
    switch (dtype) {
        case kC64: return for_length<StC64, KIND>(m);
        case kC128: return for_length<StC128, KIND>(m);
        case kC16F: return for_length<StHalf<false>, KIND>(m);
        default: return for_length<StHalf<true>, KIND>(m);
    }
}

}  // namespace

BluesteinLaunch bluestein_kernel(int kind, int dtype, int m) {
    return kind == kContiguous ? for_dtype<kContiguous>(dtype, m) : for_dtype<kStrided>(dtype, m);
}

}  // namespace croft
