// croft_group_c16f_x.hip -- FP16 storage: the contiguous passes of croft_group.h.
#include "croft_group.h"

namespace croft {
namespace dev {

// 0.8 GB moved (us; the stage-by-stage tile before): 81 198 (267), 108 181
// (270), 144 158 (239), 180 161 (283), 400 182 (237), 648 175 (289), 864 178
// (283), 960 198 (240).  1000 (three trips) stays stage by stage: 251 against 290
#define LINES(N) make_group_entry<N, StHalf<false>, 4, kC16F, kContiguous>(0),

// contiguous 1: the stage-by-stage tile, taken on small grids (kBuiltinSized in croft_tune.cpp)
#define STAGED(N) make_entry<N, kContiguous, StHalf<false>, 4, kC16F>(1),

std::vector<Entry> group_entries_c16f_x() {
    return {
        STAGED(96) STAGED(100) STAGED(160) STAGED(192) STAGED(200) STAGED(288) STAGED(320) STAGED(360) STAGED(384)
        STAGED(480) STAGED(640) STAGED(768) STAGED(960)
        LINES(72) LINES(80) LINES(96) LINES(100) LINES(120) LINES(160) LINES(192) LINES(200) LINES(240) LINES(384)
        LINES(75) LINES(81) LINES(90) LINES(108) LINES(125) LINES(135) LINES(144) LINES(150) LINES(162) LINES(180)
        LINES(216) LINES(225)
        LINES(243) LINES(250) LINES(270) LINES(288) LINES(300) LINES(320) LINES(324) LINES(360) LINES(375) LINES(400)
        LINES(405) LINES(432) LINES(450) LINES(480) LINES(486) LINES(500) LINES(540) LINES(576) LINES(600) LINES(625)
        LINES(640) LINES(648) LINES(675) LINES(720) LINES(729) LINES(750) LINES(768) LINES(800) LINES(810) LINES(864)
        LINES(900) LINES(960) LINES(972) make_entry<1000, kContiguous, StHalf<false>, 4, kC16F>(0),
    };
}

}  // namespace dev
}  // namespace croft
