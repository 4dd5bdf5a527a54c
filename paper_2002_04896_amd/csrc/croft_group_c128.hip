// croft_group_c128.hip -- complex128: the strided passes of croft_group.h, and
// the other 2^a 3^b 5^c lengths on the stage-by-stage kernels.
#include "croft_group.h"

namespace croft {
namespace dev {

// strided above 240; contiguous lines stay stage by stage at every length
// (0.8 GB moved: 400 149 us against 151, 864 148 against 144, 1000 142
// against 189)
#define STRIDED(N) make_group_entry<N, StC128, 16, kC128, kStrided>(0),
// beside the stage-by-stage tile (candidate 0): taken where rows are not whole 128-byte lines
#define PARTIAL(N) make_group_entry<N, StC128, 16, kC128, kStrided>(1),
#define SHORT(N) make_entry<N, kStrided, StC128, 16, kC128>(0),
#define LINES(N) make_entry<N, kContiguous, StC128, 16, kC128>(0),

// strided 1: the stage-by-stage tile, in the XCD-contiguous order but at 384, taken where the launch has few
// tiles and at some sizes of 384, 400 and 480 (kBuiltinSized in croft_tune.cpp)
#define STAGED(N) make_entry<N, kStrided, StC128, 16, kC128, 0, 0, 0, 1, 0, 1>(1),

std::vector<Entry> group_entries_c128() {
    return {
        CROFT_GROUP_LONG(STRIDED)
        make_group_entry<384, StC128, 16, kC128, kStrided>(0),
        STAGED(320) STAGED(360) STAGED(400) STAGED(480) STAGED(576) STAGED(640) STAGED(768) STAGED(960)
        make_entry<384, kStrided, StC128, 16, kC128>(1),
        CROFT_GROUP_SHORT(SHORT)
        CROFT_GROUP_PARTIAL(PARTIAL)
        // the same at 128 and 256: 6, beside the candidates of croft_entries_c128.hip
        make_group_entry<128, StC128, 16, kC128, kStrided>(6), make_group_entry<256, StC128, 16, kC128, kStrided>(6),
        LINES(75) LINES(81) LINES(90) LINES(108) LINES(125) LINES(135) LINES(144) LINES(150) LINES(162) LINES(180)
        LINES(216) LINES(225) LINES(243) LINES(250) LINES(270) LINES(300) LINES(324) LINES(375) LINES(405) LINES(432)
        LINES(450) LINES(486) LINES(500) LINES(540) LINES(600) LINES(625) LINES(648) LINES(675) LINES(729) LINES(750)
        LINES(800) LINES(810) LINES(864) LINES(900) LINES(972) LINES(1000)
    };
}

}  // namespace dev
}  // namespace croft
