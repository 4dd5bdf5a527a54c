// croft_group_conv.hip -- the fused multiply passes on grouped stages
// (complex64 and complex128).  Which candidate a plan takes: conv_choice in
// croft_tune.cpp.
#include "croft_group.h"

namespace croft {
namespace dev {

// complex64: 16-line tiles (128-byte rows) up to 512, above 256 also 8-line
// tiles with fewer registers (candidate 1), 8-line tiles alone above 512;
// complex128: 8-line tiles (128-byte rows)
#define SHORT(N) make_group_conv_entry<N, StC64, 8, kC64, 16, short_elements(N)>(0),
#define BOTH(N) make_group_conv_entry<N, StC64, 8, kC64, 16, 32>(0), make_group_conv_entry<N, StC64, 8, kC64, 8, 16>(1),
#define NARROW(N) make_group_conv_entry<N, StC64, 8, kC64, 8, 16>(0),
#define DSHORT(N) make_group_conv_entry<N, StC128, 16, kC128, 8, short_elements(N)>(0),
#define DLONG(N) make_group_conv_entry<N, StC128, 16, kC128, 8, 16>(0),
#define SHORT_LENGTHS(X)                                                                                            \
    X(72) X(75) X(80) X(81) X(90) X(96) X(100) X(108) X(120) X(125) X(135) X(144) X(150) X(160) X(162) X(180) X(192) \
    X(200) X(216) X(225) X(240) X(243) X(250)

std::vector<Entry> group_conv_entries_c64() {
    return {
        SHORT_LENGTHS(SHORT)
        BOTH(270) BOTH(288) BOTH(300) BOTH(320) BOTH(324) BOTH(360) BOTH(375) BOTH(400) BOTH(405) BOTH(432) BOTH(450)
        BOTH(480) BOTH(486) BOTH(500)
        NARROW(540) NARROW(576) NARROW(600) NARROW(625) NARROW(640) NARROW(648) NARROW(675) NARROW(720) NARROW(729)
        NARROW(750) NARROW(768) NARROW(800) NARROW(810) NARROW(864) NARROW(900) NARROW(960) NARROW(972) NARROW(1000)
        // beside the candidates of croft_entries_c64.hip
        make_group_conv_entry<128, StC64, 8, kC64, 16, 16>(2), make_group_conv_entry<256, StC64, 8, kC64, 16, 10>(2),
        make_group_conv_entry<384, StC64, 8, kC64, 16, 32>(2), make_group_conv_entry<384, StC64, 8, kC64, 8, 16>(3),
        make_group_conv_entry<512, StC64, 8, kC64, 16, 32>(2), make_group_conv_entry<512, StC64, 8, kC64, 8, 16>(3),
        make_group_conv_entry<1024, StC64, 8, kC64, 8, 16>(2),
    };
}

std::vector<Entry> group_conv_entries_c128() {
    return {
        SHORT_LENGTHS(DSHORT)
        DLONG(270) DLONG(288) DLONG(300) DLONG(320) DLONG(324) DLONG(360) DLONG(375) DLONG(384) DLONG(400) DLONG(405)
        DLONG(432) DLONG(450) DLONG(480) DLONG(486) DLONG(500) DLONG(540) DLONG(576) DLONG(600) DLONG(625) DLONG(640)
        DLONG(648) DLONG(675) DLONG(720) DLONG(729) DLONG(750) DLONG(768) DLONG(800) DLONG(810) DLONG(864) DLONG(900)
        DLONG(960) DLONG(972) DLONG(1000)
        // beside the candidates of croft_entries_c128.hip
        make_group_conv_entry<128, StC128, 16, kC128, 8, 16>(2), make_group_conv_entry<256, StC128, 16, kC128, 8, 10>(2),
        make_group_conv_entry<512, StC128, 16, kC128, 8, 16>(2),
        make_group_conv_entry<1024, StC128, 16, kC128, 8, 16>(2),
    };
}

}  // namespace dev
}  // namespace croft
