// croft_group_c16b.hip -- BF16 storage: the strided passes of croft_group.h.
#include "croft_group.h"

namespace croft {
namespace dev {

#define STRIDED(N) make_group_entry<N, StHalf<true>, 4, kC16B, kStrided>(0),

// strided 1: the stage-by-stage tile, taken where the launch has few tiles (kBuiltinSized in croft_tune.cpp);
// at 400 and 576 to 768 in the XCD-contiguous order (64 x 640 x 12 9.0 us against 10.8)
#define STAGED(N) make_entry<N, kStrided, StHalf<true>, 4, kC16B>(1),
#define STAGEDX(N) make_entry<N, kStrided, StHalf<true>, 4, kC16B, 0, 0, 0, 0, 0, 1>(1),

std::vector<Entry> group_entries_c16b() {
    return {
        CROFT_GROUP_LONG(STRIDED)
        CROFT_GROUP_SHORT(STRIDED)
        STRIDED(32) STRIDED(48) STRIDED(60) STRIDED(64) STRIDED(72) STRIDED(80) STRIDED(96) STRIDED(100) STRIDED(120)
        STRIDED(160) STRIDED(192) STRIDED(200) STRIDED(240) STRIDED(384)
        STAGED(32) STAGED(60) STAGED(64) STAGED(80) STAGED(96) STAGED(100) STAGED(120) STAGED(160) STAGED(192) STAGED(200)
        STAGED(288) STAGED(320) STAGED(360) STAGED(384) STAGEDX(400) STAGED(480) STAGEDX(576) STAGEDX(640) STAGEDX(720)
        STAGEDX(768) STAGED(900) STAGED(960) STAGED(972)
        // 128 and 256: 6, beside the candidates of croft_entries_c16b.hip
        make_group_entry<128, StHalf<true>, 4, kC16B, kStrided>(6), make_group_entry<256, StHalf<true>, 4, kC16B, kStrided>(6),
    };
}

}  // namespace dev
}  // namespace croft
