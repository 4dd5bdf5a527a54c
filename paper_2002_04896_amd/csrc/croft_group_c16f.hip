// croft_group_c16f.hip -- FP16 storage: the strided passes of croft_group.h.
#include "croft_group.h"

namespace croft {
namespace dev {

#define STRIDED(N) make_group_entry<N, StHalf<false>, 4, kC16F, kStrided>(0),

std::vector<Entry> group_entries_c16f() {
    return {
        CROFT_GROUP_LONG(STRIDED)
        CROFT_GROUP_SHORT(STRIDED)
        STRIDED(32) STRIDED(48) STRIDED(60) STRIDED(64) STRIDED(72) STRIDED(80) STRIDED(96) STRIDED(100) STRIDED(120)
        STRIDED(160) STRIDED(192) STRIDED(200) STRIDED(240) STRIDED(384)
        // 128 and 256: 6, beside the candidates of croft_entries_c16f.hip
        make_group_entry<128, StHalf<false>, 4, kC16F, kStrided>(6), make_group_entry<256, StHalf<false>, 4, kC16F, kStrided>(6),
    };
}

}  // namespace dev
}  // namespace croft
