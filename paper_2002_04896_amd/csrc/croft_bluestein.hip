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
// FEW: the shape for launches of few tiles (at most one a CU), where a tile's
// own time counts and LDS has room: more threads a line, fewer lines a block,
// the exchange whole.  (us, FEW against the ordinary shape and against one LDS
// trip per stage: complex64 64 x 1009 x 4 10.8, 14.7, 12.6, 1009 x 32 x 8 9.1, 13.8,
// 10.9, 64 x 2039 x 2 15.4, 23.2, 19.2; complex128 64 x 97 x 21 8.3, 12.1, 10.0;
// FP16 1021 x 32 x 16 (256 tiles) 10.8, 14.9, 14.3; beyond it complex64 64 x 1021 x
// 16 (512) 21.6, 20.2, 27.0, FP16 64 x 614 x 13 (416) 18.2, 17.3, 27.7)
template <int M, int KIND, int CB, bool FEW>
struct BlueShape {
    static constexpr bool k64 = CB == 16;  // FP64 compute
    static constexpr bool kLines = KIND == kContiguous;
    static constexpr bool kMore = FEW && (M == 2048 || M == 4096 || (M == 512 && !kLines) || (M == 256 && k64));
    static constexpr int T = kMore       ? (M / 8 < 256 ? M / 8 : 256)
                             : M == 16   ? 1
                             : M == 32   ? 4
                             : M <= 128  ? 8
                             : M == 256  ? (k64 ? 16 : 32)
                             : M == 512  ? (kLines ? 64 : 32)
                             : M == 1024 ? 64
                             : M == 2048 ? 128
                             : M == 4096 ? (k64 || kLines ? 256 : 128)
                                         : 256;
    static constexpr int E = M / T;
    static constexpr int kSplit = kMore ? 0 : (M == 256 && k64) || (M == 512 && !kLines) || (M >= 1024 && M < 8192);
    static constexpr bool kTab = M <= 1024;
    static constexpr int L = M <= 32 ? 64 : M == 64 ? (k64 ? 16 : 32) : M == 128 ? 16 : 256 / T;
};

template <class St, int KIND, int M, bool FEW>
BluesteinLaunch launch_of() {
    BluesteinLaunch b;
    constexpr int CB = (int)sizeof(cx<typename St::R>);
    // FP64 convolutions stop at 4096 points (lengths up to 2048)
    if constexpr (CB == 8 || M <= 4096) {
        using S = BlueShape<M, KIND, CB, FEW>;
        using Cfg = GCfg<M, KIND, S::L, S::E, CB, S::kSplit, 0, S::T>;
        static_assert(Cfg::kBlock <= 256 && BlueLds<Cfg, S::kTab>::kBytes <= 160 * 1024, "launch shape");
        b.func = reinterpret_cast<const void *>(&fft_bluestein<Cfg, St, KIND, S::kTab>);
        b.T = Cfg::T;
        b.L = Cfg::L;
        b.lds = BlueLds<Cfg, S::kTab>::kBytes;
    }
    return b;
}

template <class St, int KIND, bool FEW>
BluesteinLaunch for_length(int m) {
    switch (m) {
        case 16: return launch_of<St, KIND, 16, FEW>();
        case 32: return launch_of<St, KIND, 32, FEW>();
        case 64: return launch_of<St, KIND, 64, FEW>();
        case 128: return launch_of<St, KIND, 128, FEW>();
        case 256: return launch_of<St, KIND, 256, FEW>();
        case 512: return launch_of<St, KIND, 512, FEW>();
        case 1024: return launch_of<St, KIND, 1024, FEW>();
        case 2048: return launch_of<St, KIND, 2048, FEW>();
        case 4096: return launch_of<St, KIND, 4096, FEW>();
        case 8192: return launch_of<St, KIND, 8192, FEW>();
        default: return BluesteinLaunch{};
    }
}

template <int KIND, bool FEW>
BluesteinLaunch for_dtype(int dtype, int m) {
    switch (dtype) {
        case kC64: return for_length<StC64, KIND, FEW>(m);
        case kC128: return for_length<StC128, KIND, FEW>(m);
        case kC16F: return for_length<StHalf<false>, KIND, FEW>(m);
        default: return for_length<StHalf<true>, KIND, FEW>(m);
    }
}

}  // namespace

BluesteinLaunch bluestein_kernel(int kind, int dtype, int m, bool few_tiles) {
    if (few_tiles)
        return kind == kContiguous ? for_dtype<kContiguous, true>(dtype, m) : for_dtype<kStrided, true>(dtype, m);
    return kind == kContiguous ? for_dtype<kContiguous, false>(dtype, m) : for_dtype<kStrided, false>(dtype, m);
}

}  // namespace croft
