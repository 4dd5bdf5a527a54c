// croft_group_c64.hip -- complex64: the passes of croft_group.h (several stages
// per register group), and the short 2^a 3^b 5^c lengths on the stage-by-stage
// kernels.
#include "croft_group.h"

namespace croft {
namespace dev {

// strided above 240 and contiguous above 480; below, the stage-by-stage tiles
// are as fast or faster.  Contiguous lines shorter than 75 and strided ones
// shorter than 18 stay on the runtime-radix kernel.
#define STRIDED(N) make_group_entry<N, StC64, 8, kC64, kStrided>(0),
// beside the stage-by-stage tile (candidate 0): taken where rows are not whole 128-byte lines
#define PARTIAL(N) make_group_entry<N, StC64, 8, kC64, kStrided>(1),
#define SHORT(N) make_entry<N, kStrided, StC64, 8, kC64>(0),
#define LINES(N) make_entry<N, kContiguous, StC64, 8, kC64>(0),
#define GLINES(N) make_group_entry<N, StC64, 8, kC64, kContiguous>(0),
// contiguous 3: non-temporal, numbered as in croft_entries_c64.hip
#define NTLINES(N) make_group_entry<N, StC64, 8, kC64, kContiguous, 1>(3),

// strided 1: the stage-by-stage tile, taken where the launch has few tiles (kBuiltinSized in croft_tune.cpp);
// from 576 on, where a CU holds one, in the XCD-contiguous order (64 x 576 x 28 9.2 us against 12.6)
#define STAGED(N) make_entry<N, kStrided, StC64, 8, kC64>(1),
#define STAGEDX(N) make_entry<N, kStrided, StC64, 8, kC64, 0, 0, 0, 0, 0, 1>(1),

std::vector<Entry> group_entries_c64() {
    return {
        CROFT_GROUP_LONG(STRIDED)
        // 384: 8, beside the candidates of croft_entries_c64.hip (174/136 us against 182/148)
        make_group_entry<384, StC64, 8, kC64, kStrided>(8),
        STAGED(288) STAGED(320) STAGED(360) STAGED(400) STAGED(480) STAGEDX(576) STAGEDX(640) STAGEDX(720) STAGEDX(768)
        STAGEDX(960)
        CROFT_GROUP_SHORT(SHORT)
        CROFT_GROUP_PARTIAL(PARTIAL)
        // the same at 128 and 256: 6, beside the candidates of croft_entries_c64.hip
        make_group_entry<128, StC64, 8, kC64, kStrided>(6), make_group_entry<256, StC64, 8, kC64, kStrided>(6),
        LINES(75) LINES(81) LINES(90) LINES(108) LINES(125) LINES(135) LINES(144) LINES(150) LINES(162) LINES(180)
        LINES(216) LINES(225) LINES(243) LINES(250) LINES(270) LINES(300) LINES(324) LINES(375) LINES(405) LINES(432)
        LINES(450)
        // contiguous, 0.8 GB moved (us, plain; non-temporal): 576 150, 148 (188 stage by stage), 864 149
        // (178), 960 146, 143 (157).  640 stays stage by stage: 240 MB moved 45.5 against 47.5, beyond the
        // cache (0.6 GB, non-temporal) 124 against 133
        GLINES(486) GLINES(500) GLINES(540) GLINES(576) GLINES(600) GLINES(625) GLINES(648) GLINES(675)
        GLINES(720) GLINES(729) GLINES(750) GLINES(768) GLINES(800) GLINES(810) GLINES(864) GLINES(900) GLINES(960)
        GLINES(972) GLINES(1000)
        LINES(640) make_entry<640, kContiguous, StC64, 8, kC64, 0, 0, 0, 1, 1>(3),
        NTLINES(576) NTLINES(720) NTLINES(768) NTLINES(960)
    };
}

}  // namespace dev
}  // namespace croft
