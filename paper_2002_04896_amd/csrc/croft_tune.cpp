// croft_tune.cpp -- wisdom: remembered kernel choices per (length, pass kind,
// dtype), the FFTW-style cache of the autotuner's results.
//
// The choice is a compiled candidate configuration and the persistent grid
// size (in resident-block waves; 0 = one block per tile).  Choices measured in
// this process are kept in memory; when the environment variable CROFT_WISDOM
// names a file, plans also read it and CROFT_MEASURE plans append to it.
// File format, one choice per line:  n kind dtype candidate waves [axis]
// (and "slabs nx ny nz dtype K" for the slab count of a grid, below)
// A choice that CROFT_MEASURE made holds for the class of passes it was timed
// on (measure_class: size to a factor of two, alignment of the rows, place in
// the plan), as the best configuration changes between them; its line has
// dtype + 4 class in the place of dtype.  A line with a plain dtype serves
// every class.
// A strided pass also has a choice of its own per grid axis (1 = y, 2 = z:
// their strides differ, and so can their best tiles); a line without an axis
// serves every axis.  Lookup order: the CROFT_WISDOM file, choices measured
// in this process, for forward plans the forward-only built-in choices, the
// per-axis built-in choices, the built-in table below (measured on an MI355X
// with CROFT_MEASURE on cubic grids, and before it the choices that hold for
// some sizes only; kinds 2 and 3, the real x pass and the
// fused multiply pass, on real and convolution plans of cubic grids), then
// candidate 0 on the grid size the caller starts from.  At each step an entry for the pass's
// axis comes before one for any axis, and one for its class before one for any.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>
#include <tuple>

#include "croft_internal.h"

namespace croft {
namespace {
struct Builtin {
    int n, kind, dtype, cand, waves;
};
// n kind dtype candidate waves
const Builtin kBuiltin[] = {
    // complex64 (384: from a sweep of the 384^3 grid, too large for the
    // Infinity Cache: the non-temporal contiguous tile, x 186 -> 163 us;
    // strided, the grouped stages, 174/136 us against 182/148 for the 32-line
    // wide tile (0.8 GB moved, rows of 360 and of 36000 elements))
    {32, 0, 0, 0, 1}, {32, 1, 0, 0, 1}, {48, 0, 0, 0, 0}, {48, 1, 0, 0, 2}, {60, 0, 0, 0, 4}, {60, 1, 0, 0, 0},
    {64, 0, 0, 0, 4}, {64, 1, 0, 0, 4}, {72, 0, 0, 0, 1}, {72, 1, 0, 0, 0}, {80, 0, 0, 0, 0}, {80, 1, 0, 0, 4},
    {96, 0, 0, 0, 1}, {96, 1, 0, 0, 1}, {100, 0, 0, 0, 2}, {100, 1, 0, 0, 4}, {128, 0, 0, 1, 2},
    {128, 1, 0, 5, 1}, {256, 0, 0, 1, 0}, {256, 1, 0, 1, 0}, {384, 0, 0, 3, 0}, {384, 1, 0, 8, 0},
    // (the real x pass of the 512^3 real grid, length 256 above: the non-temporal
    // candidate, forward 0.613 -> 0.587 ms, backward 0.675 -> 0.640, convolution
    // 1.207 -> 1.194)
    // complex64 at the larger compiled 2^a 3^b 5^c lengths: the streaming
    // contiguous tile for x (strided: the grouped stages, their only candidate);
    // 160 to 240 strided: the grouped stages too (200 x 400 x 800 z 666 -> 641
    // us, 384 x 768 x 192 z 556 -> 545, 240^3 y 120.2 -> 118.4)
    {160, 1, 0, 1, 0}, {192, 1, 0, 1, 0}, {200, 1, 0, 1, 0}, {240, 1, 0, 1, 0},
    {480, 0, 0, 3, 0}, {576, 0, 0, 3, 0}, {640, 0, 0, 3, 0}, {720, 0, 0, 3, 0}, {768, 0, 0, 3, 0},
    {960, 0, 0, 3, 0},
    {512, 0, 0, 3, 0}, {512, 1, 0, 4, 4}, {1024, 0, 0, 3, 0}, {1024, 1, 0, 7, 1}, {32, 2, 0, 0, 0},
    {64, 2, 0, 0, 2}, {64, 3, 0, 0, 2}, {128, 2, 0, 0, 1}, {256, 2, 0, 1, 0},
    // complex64 batched tile shapes (kinds 4 and 5: the batched kernel's
    // contiguous and strided passes; candidate = shape), the majority of six
    // CROFT_MEASURE runs (both directions) on the 64-grid PME batch; the
    // lengths not listed keep shape 0
    {60, 4, 0, 1, 0}, {60, 5, 0, 1, 0}, {64, 4, 0, 1, 0}, {64, 5, 0, 1, 0}, {72, 4, 0, 1, 0}, {72, 5, 0, 1, 0},
    {80, 4, 0, 1, 0}, {80, 5, 0, 1, 0}, {96, 4, 0, 1, 0}, {96, 5, 0, 1, 0}, {100, 5, 0, 1, 0},
    // complex128 (128 x: the padded tile, 128 x 256 x 256 153 -> 138 us against
    // the non-temporal one)
    {32, 0, 1, 0, 4}, {32, 1, 1, 0, 0}, {48, 0, 1, 0, 2}, {48, 1, 1, 0, 4}, {60, 0, 1, 0, 2}, {60, 1, 1, 0, 2},
    {64, 0, 1, 0, 0}, {64, 1, 1, 0, 4}, {72, 0, 1, 0, 1}, {72, 1, 1, 0, 0}, {80, 0, 1, 0, 1}, {80, 1, 1, 0, 0},
    {96, 0, 1, 0, 2}, {96, 1, 1, 0, 1}, {100, 0, 1, 0, 4}, {100, 1, 1, 0, 1}, {128, 0, 1, 1, 0},
    {128, 1, 1, 5, 4}, {256, 0, 1, 3, 0}, {256, 1, 1, 5, 0}, {384, 0, 1, 0, 0},
    // complex128 at the larger compiled lengths (one forward sweep of n^3): the
    // streaming x tile; 720 keeps the default, which it did not beat
    {480, 0, 1, 3, 0}, {576, 0, 1, 3, 0}, {640, 0, 1, 3, 0}, {768, 0, 1, 3, 0},
    {512, 0, 1, 3, 0}, {512, 1, 1, 4, 2}, {1024, 0, 1, 2, 0}, {1024, 1, 1, 5, 0}, {32, 2, 1, 0, 2},
    {64, 2, 1, 0, 1}, {64, 3, 1, 0, 0}, {128, 2, 1, 0, 1}, {256, 2, 1, 0, 2},
    // FP16 storage (strided 128 and 256: the grouped stages; 512 x: the
    // non-temporal contiguous tile on four waves of resident blocks, 0.217 ->
    // 0.195 ms in both directions; the same for BF16)
    {32, 0, 2, 0, 2}, {48, 0, 2, 0, 0}, {60, 0, 2, 0, 1}, {64, 0, 2, 0, 0}, {128, 0, 2, 1, 1}, {128, 1, 2, 6, 0},
    {256, 0, 2, 1, 0}, {256, 1, 2, 6, 0}, {512, 0, 2, 3, 4}, {512, 1, 2, 6, 1}, {1024, 0, 2, 3, 4},
    {1024, 1, 2, 7, 1},
    // BF16 storage
    {32, 0, 3, 0, 0}, {48, 0, 3, 0, 2}, {60, 0, 3, 0, 4}, {64, 0, 3, 0, 2}, {128, 0, 3, 1, 2}, {128, 1, 3, 6, 0},
    {256, 0, 3, 1, 0}, {256, 1, 3, 6, 0}, {512, 0, 3, 3, 4}, {512, 1, 3, 6, 1}, {1024, 0, 3, 3, 4},
    {1024, 1, 3, 7, 1},
};

// Forward-only choices, looked up before the table above by forward plans:
// where the best configuration for both directions together is not the best
// forward one (512 strided complex64 passes with no per-axis choice, such as
// the convolution plan's: the 1024-thread wide tile is the fastest forward
// but spills in its inverse).
const Builtin kBuiltinForward[] = {
    {512, 1, 0, 2, 1},
};

// Per-axis choices (n kind dtype axis candidate waves), looked up before
// the two tables above, all one line per lane; at 512 in 256-thread blocks
// (two share a CU), one block per tile, unless noted: the y pass (4 KiB
// stride for complex64) with non-temporal loads, complex64 with the tiles
// in reverse order (0.377 -> 0.350 ms), 16-bit storage in the
// XCD-contiguous order (0.230 -> 0.213 ms); a real grid's half-spectrum y
// pass, whose rows are not whole 128-byte lines, takes the plain twin (the
// XCD-ordered plain kernel, 0.20 ms); the complex64 z pass (2 MiB stride)
// with non-temporal loads and stores.
struct BuiltinAxis {
    int n, kind, dtype, axis, cand, waves;
};
const BuiltinAxis kBuiltinAxis[] = {
    // 128 and 256, from sweeps of the whole transform over cubes and flat and
    // long grids (both directions; us, the choice for any axis before).  The
    // non-temporal hint pays in the pass along z, which nothing follows, and
    // costs in the passes before it, whose output the next one reads: complex64
    // 256^3 z 133 -> 125, 512 x 512 x 256 z 613 -> 541, 512 x 256 x 512 y 570
    // -> 559, 256 x 128 x 256 y 75.3 -> 69.3; complex128 128^3 y 39.5 -> 35.3,
    // 256^3 y 296 -> 259 (512 x 256 x 512 1130 -> 1147, 256 x 256 x 1024 1282
    // -> 1237)
    {128, 1, 0, 1, 1, 1},
    {128, 1, 0, 2, 5, 0},
    {256, 1, 0, 1, 2, 0},
    {256, 1, 0, 2, 5, 0},
    {128, 1, 1, 1, 2, 1},
    {128, 1, 1, 2, 5, 0},
    {256, 1, 1, 1, 4, 0},
    // complex64 at 1024, 512-thread blocks, one block per tile: y in the
    // XCD-contiguous order (3.40 -> 3.29 ms), z non-temporal (4.16 -> 3.97)
    {1024, 1, 0, 1, 8, 0},
    {1024, 1, 0, 2, 7, 0},
    // 16-bit storage at 1024: y in dispatch order, plain (2.29 -> 2.23 ms
    // FP16, 2.25 -> 2.16 BF16); z in XCD-contiguous order, non-temporal, one
    // block per tile (2.91 -> 2.86)
    {1024, 1, 2, 1, 6, 1},
    {1024, 1, 2, 2, 9, 0},
    {1024, 1, 3, 1, 6, 1},
    {1024, 1, 3, 2, 9, 0},
    {512, 1, 0, 1, 15, 0},
    // complex64 z at 512: the same 256-thread blocks, non-temporal, the
    // candidate that copies half a tile into LDS, one block per tile (so each
    // block copies the first half of its own tile): 0.400 -> 0.382 ms on two
    // waves of resident blocks, then 0.382 -> 0.371 ms with one block per
    // tile (both directions, two GPUs; real plans 0.618 -> 0.615 ms forward,
    // 0.684 -> 0.677 ms backward)
    {512, 1, 0, 2, 18, 0},
    {512, 1, 2, 1, 14, 0},
    {512, 1, 3, 1, 14, 0},
    // complex128 y at 512: the wide tile with fewer threads, one block per
    // tile.  The 16-line tile in the XCD-contiguous order (candidate 6) runs
    // the y pass itself faster (0.79-0.80 against 0.80-0.81 ms), but the z
    // pass after it takes 0.91 against 0.86 ms: the transform is faster with
    // this one (2.404-2.423 against 2.440-2.461 ms, both directions)
    {512, 1, 1, 1, 4, 0},
    // 16-bit storage z at 512: 64-line tiles loading the next tile into
    // registers during the current one (BF16 0.272-0.277 -> 0.264-0.268 ms,
    // FP16 the same within the spread, both directions, two GPUs); FP16 with
    // the non-temporal hint on those loads (0.242-0.243 -> 0.238-0.239 ms,
    // transform 0.675-0.679 -> 0.665-0.666 ms; on BF16 the hint gains nothing)
    {512, 1, 2, 2, 23, 1},
    {512, 1, 3, 2, 20, 1},
};

// Choices for some sizes only, looked up before the tables above: the first
// entry whose limits hold.  axis -1: any; rows: any, whole 128-byte lines, not,
// or whole in a number of planes that is no power of two; segments: at most so many 128-byte row segments (0: no
// limit); MiB the pass reads: more than `above`, at most `upto` (0: no limit).
// dtype kHalves: either 16-bit storage.
struct BuiltinSized {
    int n, kind, dtype, axis, rows, segments, above, upto, cand, waves;
};
constexpr int kAny = 0, kWhole = 1, kPartial = 2, kWholeUneven = 3;
constexpr int kHalves = -1;
const BuiltinSized kBuiltinSized[] = {
    // 256: the wide tiles of the choices by axis leave most CUs without one on
    // small grids (us, wide against 16 or 8 lines: complex64 y 64 x 256 x 16
    // 8.1, 6.4, 64 x 256 x 64 (256 segments, the whole transform) 20.1, 19.8, z
    // 64 x 16 x 256 8.4, 6.8; complex128 y 64 x 256 x 8 7.8, 6.4, 64 x 256 x 32
    // 9.3, 8.2, 64 x 256 x 64 (512, whole) 35.1, 33.1)
    {256, 1, 0, 1, kWhole, 128, 0, 0, 1, 0},
    {256, 1, 0, 2, kWhole, 128, 0, 0, 1, 0},
    {256, 1, 1, 1, kWhole, 512, 0, 0, 0, 1},
    // and beyond the cache complex128 y keeps the non-temporal one where the planes
    // are no power of two (512 x 256 x 300 736, 746, 512 x 256 x 400 963, 979, 360 x 256
    // x 300 506, 520; 512 x 256 x 256 563, 545, 256 x 256 x 1024 1282, 1237, but 512 x
    // 256 x 512 1130, 1147)
    {256, 1, 1, 1, kWholeUneven, 0, 256, 0, 5, 0},
    // and the non-temporal z stores stay off grids that the eight 4 MiB L2s hold
    // between calls (whole transforms, us, non-temporal against plain: complex64
    // 128 x 72 x 256 (18 MiB) 31.5, 27.7, 128 x 96 x 256 35.4, 28.4, 128 x 120 x 256 40.0,
    // 34.2, but 128 x 64 x 256 (16 MiB) 25.5, 32.2, 256 x 64 x 256 (32 MiB) 34.5, 36.5;
    // complex128 128 x 88 x 128 (22 MiB) 49.1, 45.7, 256 x 56 x 128 50.2, 45.3, 128 x 52 x
    // 256 48.9, 44.1, real 192 x 64 x 256 39.4, 33.8, but 20 and 30 MiB level)
    {256, 1, 0, 2, kWhole, 0, 16, 31, 1, 0},
    {128, 1, 1, 2, kWhole, 0, 20, 29, 2, 0},
    {256, 1, 1, 2, kWhole, 0, 20, 29, 6, 0},
    // complex64 384 beyond the cache: the 32-line wide tile on one wave (whole
    // transforms, us, against the grouped stages: 384^3 496, 516, 384 x 384 x 256
    // 357, 363; in the cache 384 x 384 x 96 124, 123, 64 x 384 x 160 47, 44)
    {384, 1, 0, -1, kWhole, 0, 256, 0, 2, 1},
    // complex128 y at 512 around the cache's size: two waves (whole transforms,
    // us, one block per tile against it: 512 x 512 x 48 (192 MiB) 208, 202, 512 x
    // 512 x 64 287, 276, 512 x 512 x 96 414, 405; 128 MiB 146.3, 146.3, 512 MiB
    // 571, 570)
    {512, 1, 1, 1, kWhole, 0, 160, 400, 4, 2},
    // Strided launches of few tiles: the stage-by-stage tiles, whose lines have
    // more threads, against the grouped stages, whose threads hold up to 64
    // elements and take longest over a tile (a pass, us, stage by stage against
    // grouped, at about a quarter of the limit | at the limit | beyond it:
    // complex64 320 7.0, 8.6 | 8.2, 9.8 | 14.6, 13.2; 960 8.7, 13.7 | 10.2, 14.9 |
    // 17.0, 15.6; complex128 320 0.88 | 0.91 | 1.12 of the time, 768 0.77 | 0.91 |
    // 1.04; FP16 100 6.4, 7.0 | 0.95 | 1.07, 256 8.5, 9.4 | 11.5,
    // 13.3 | 26.2, 18.7, 320 0.67 | 0.84 |
    // 1.00, 900 0.60 | 0.78 | 1.01)
    {288, 1, 0, -1, kAny, 256, 0, 0, 1, 0}, {320, 1, 0, -1, kAny, 256, 0, 0, 1, 0},
    {360, 1, 0, -1, kAny, 256, 0, 0, 1, 0}, {400, 1, 0, -1, kAny, 256, 0, 0, 1, 0},
    {480, 1, 0, -1, kAny, 256, 0, 0, 1, 0}, {576, 1, 0, -1, kAny, 128, 0, 0, 1, 0},
    {640, 1, 0, -1, kAny, 128, 0, 0, 1, 0}, {720, 1, 0, -1, kAny, 128, 0, 0, 1, 0},
    {768, 1, 0, -1, kAny, 128, 0, 0, 1, 0}, {960, 1, 0, -1, kAny, 128, 0, 0, 1, 0},
    {320, 1, 1, -1, kAny, 256, 0, 0, 1, 0}, {360, 1, 1, -1, kAny, 256, 0, 0, 1, 0},
    {384, 1, 1, -1, kPartial, 256, 0, 0, 1, 0}, {400, 1, 1, -1, kAny, 256, 0, 0, 1, 0},
    {480, 1, 1, -1, kAny, 256, 0, 0, 1, 0}, {576, 1, 1, -1, kAny, 128, 0, 0, 1, 0},
    {640, 1, 1, -1, kAny, 128, 0, 0, 1, 0}, {768, 1, 1, -1, kAny, 512, 0, 0, 1, 0},
    {960, 1, 1, -1, kAny, 128, 0, 0, 1, 0},
    {32, 1, kHalves, -1, kWhole, 2048, 0, 0, 1, 0}, {60, 1, kHalves, -1, kWhole, 1024, 0, 0, 1, 0},
    {60, 1, kHalves, -1, kPartial, 256, 0, 0, 1, 0}, {64, 1, kHalves, -1, kWhole, 4096, 0, 0, 1, 0},
    {64, 1, kHalves, -1, kPartial, 256, 0, 0, 1, 0}, {80, 1, kHalves, -1, kWhole, 512, 0, 0, 1, 0},
    {80, 1, kHalves, -1, kPartial, 128, 0, 0, 1, 0}, {96, 1, kHalves, -1, kWhole, 512, 0, 0, 1, 0},
    {96, 1, kHalves, -1, kPartial, 128, 0, 0, 1, 0}, {100, 1, kHalves, -1, kWhole, 256, 0, 0, 1, 0},
    {100, 1, kHalves, -1, kPartial, 128, 0, 0, 1, 0}, {120, 1, kHalves, -1, kWhole, 512, 0, 0, 1, 0},
    {120, 1, kHalves, -1, kPartial, 128, 0, 0, 1, 0},
    {256, 1, kHalves, -1, kWhole, 512, 0, 0, 0, 0}, {160, 1, kHalves, -1, kPartial, 128, 0, 0, 1, 0}, {192, 1, kHalves, -1, kWhole, 512, 0, 0, 1, 0},
    {192, 1, kHalves, -1, kPartial, 128, 0, 0, 1, 0}, {200, 1, kHalves, -1, kAny, 128, 0, 0, 1, 0},
    {288, 1, kHalves, -1, kAny, 128, 0, 0, 1, 0}, {320, 1, kHalves, -1, kAny, 256, 0, 0, 1, 0},
    {360, 1, kHalves, -1, kAny, 128, 0, 0, 1, 0}, {384, 1, kHalves, -1, kAny, 128, 0, 0, 1, 0},
    {400, 1, kHalves, -1, kAny, 128, 0, 0, 1, 0}, {480, 1, kHalves, -1, kAny, 128, 0, 0, 1, 0},
    {576, 1, kHalves, -1, kAny, 64, 0, 0, 1, 0}, {640, 1, kHalves, -1, kAny, 64, 0, 0, 1, 0},
    {720, 1, kHalves, -1, kAny, 32, 0, 0, 1, 0}, {768, 1, kHalves, -1, kAny, 64, 0, 0, 1, 0},
    {900, 1, kHalves, -1, kAny, 64, 0, 0, 1, 0}, {960, 1, kHalves, -1, kAny, 64, 0, 0, 1, 0},
    {972, 1, kHalves, -1, kAny, 32, 0, 0, 1, 0},
    // 16-bit 128 in whole rows, whole transforms: along z at every size (512 x 512 x
    // 128 179, 187, 256 x 512 x 128 92, 97, 250 x 1024 x 128 192, 190), along y up to
    // 64 MiB (128 x 128 x 128 21.1, 23.2, 128 x 128 x 1024 88, 91)
    {128, 1, kHalves, 2, kWhole, 0, 0, 0, 1, 4}, {128, 1, kHalves, 1, kWhole, 0, 0, 64, 1, 1},
    // and at every size of whole rows at 16-bit 160 (one wave: 64 x 160 x 768 19.5,
    // 22.6; 250 x 768 x 160 57.4, 59.0) and complex128 384 (one wave: 384 x 384 x
    // 48 38.9, 45.5, 64 x 768 x 384 120, 128); at complex128 480 up to 64 MiB (64 x
    // 480 x 64 15.7, 17.2; 120 MiB 42.5, 41.9) and along y beyond the cache, as at
    // 400, in the XCD-contiguous order (64 x 480 x 640 110, 127, 384 x 480 x 96 107,
    // 117, 64 x 400 x 768 119, 129)
    {160, 1, kHalves, -1, kWhole, 0, 0, 0, 1, 1},
    {384, 1, 1, -1, kWhole, 0, 0, 0, 1, 1},
    {480, 1, 1, -1, kWhole, 0, 0, 64, 1, 0},
    {480, 1, 1, 1, kWhole, 0, 256, 0, 1, 0},
    {400, 1, 1, 1, kWhole, 0, 256, 0, 1, 0},
    // 16-bit contiguous lines of small grids, likewise (7 MiB: 100 11.4, 12.4,
    // 160 11.0, 12.7, 288 10.1, 13.1, 480 10.3, 12.4, 960 (2 MiB) 7.8, 8.7; 28 MiB:
    // 96 16.1, 18.4, 192 18.3, 21.4, 360 22.2, 23.6, 480 23.0, 24.7; 72 to 120 MiB:
    // 288 48.9, 47.4, 360 54.9, 48.6, 480 69.4, 61.3), at 640 at every size
    // (160 MiB 84, 90)
    {96, 0, kHalves, -1, kAny, 0, 0, 64, 1, 0}, {100, 0, kHalves, -1, kAny, 0, 0, 64, 1, 0},
    {160, 0, kHalves, -1, kAny, 0, 0, 64, 1, 0}, {192, 0, kHalves, -1, kAny, 0, 0, 64, 1, 0},
    {200, 0, kHalves, -1, kAny, 0, 0, 64, 1, 0}, {288, 0, kHalves, -1, kAny, 0, 0, 64, 1, 0},
    {320, 0, kHalves, -1, kAny, 0, 0, 64, 1, 0}, {360, 0, kHalves, -1, kAny, 0, 0, 32, 1, 0},
    {384, 0, kHalves, -1, kAny, 0, 0, 64, 1, 0}, {480, 0, kHalves, -1, kAny, 0, 0, 32, 1, 0},
    {640, 0, kHalves, -1, kAny, 0, 0, 0, 1, 1}, {768, 0, kHalves, -1, kAny, 0, 0, 16, 1, 0},
    {960, 0, kHalves, -1, kAny, 0, 0, 4, 1, 0},
};

std::mutex g_mu;
std::map<std::tuple<int, int, int, int, int>, std::pair<int, int>> g_mem;  // (n, kind, dtype, class, axis or -1)

// The last matching line for this axis (axis >= 0) or for any axis (axis -1),
// and for this class or (0) for any.
bool read_file(const char *path, int n, int kind, int dtype, int cls, int axis, int *cand, int *waves) {
    FILE *f = std::fopen(path, "r");
    if (!f) return false;
    bool found = false;
    int a, b, c, d, e, x;
    char line[256];
    while (std::fgets(line, sizeof line, f)) {
        const int got = std::sscanf(line, "%d %d %d %d %d %d", &a, &b, &c, &d, &e, &x);
        if (got < 5 || a != n || b != kind || c != dtype + 4 * cls) continue;
        if ((axis < 0 && got == 5) || (axis >= 0 && got == 6 && x == axis)) {
            *cand = d;
            *waves = e;
            found = true;
        }
    }
    std::fclose(f);
    return found;
}
}  // namespace

bool wisdom_measured(int n, int kind, int dtype, int axis, int cls, int *cand, int *waves) {
    std::lock_guard<std::mutex> lk(g_mu);
    const int axes[2] = {axis, -1}, classes[2] = {cls, 0};
    const char *path = std::getenv("CROFT_WISDOM");
    if (path && *path)
        for (int i = axis >= 0 ? 0 : 1; i < 2; ++i)
            for (int j = cls > 0 ? 0 : 1; j < 2; ++j)
                if (read_file(path, n, kind, dtype, classes[j], axes[i], cand, waves)) return true;
    for (int i = axis >= 0 ? 0 : 1; i < 2; ++i) {
        auto it = g_mem.find({n, kind, dtype, cls, axes[i]});
        if (it != g_mem.end()) {
            *cand = it->second.first;
            *waves = it->second.second;
            return true;
        }
    }
    return false;
}

bool wisdom_lookup(int n, int kind, int dtype, int dir, int axis, int cls, int *cand, int *waves) {
    return wisdom_measured(n, kind, dtype, axis, cls, cand, waves) ||
           builtin_choice(n, kind, dtype, dir, axis, cand, waves);
}

bool sized_choice(int n, int kind, int dtype, int axis, const PassSize &size, int *cand, int *waves) {
    for (const BuiltinSized &b : kBuiltinSized) {
        if (b.n != n || b.kind != kind || (b.dtype == kHalves ? dtype < kC16F : b.dtype != dtype) || (b.axis >= 0 && b.axis != axis)) continue;
        if (b.rows != kAny && (b.rows == kPartial) != size.partial_lines) continue;
        if (b.rows == kWholeUneven && (size.planes & (size.planes - 1)) == 0) continue;
        if (b.segments && size.segments > b.segments) continue;
        if (size.bytes <= ((long long)b.above << 20) || (b.upto && size.bytes > ((long long)b.upto << 20))) continue;
        *cand = b.cand;
        *waves = b.waves;
        return true;
    }
    return false;
}

bool builtin_choice(int n, int kind, int dtype, int dir, int axis, int *cand, int *waves) {
    if (axis >= 0) {
        for (const BuiltinAxis &b : kBuiltinAxis) {
            if (b.n == n && b.kind == kind && b.dtype == dtype && b.axis == axis) {
                *cand = b.cand;
                *waves = b.waves;
                return true;
            }
        }
    }
    if (dir == -1) {
        for (const Builtin &b : kBuiltinForward) {
            if (b.n == n && b.kind == kind && b.dtype == dtype) {
                *cand = b.cand;
                *waves = b.waves;
                return true;
            }
        }
    }
    for (const Builtin &b : kBuiltin) {
        if (b.n == n && b.kind == kind && b.dtype == dtype) {
            *cand = b.cand;
            *waves = b.waves;
            return true;
        }
    }
    return false;
}

void wisdom_record(int n, int kind, int dtype, int axis, int cls, int cand, int waves, bool persist) {
    std::lock_guard<std::mutex> lk(g_mu);
    g_mem[{n, kind, dtype, cls, axis}] = {cand, waves};
    const char *path = std::getenv("CROFT_WISDOM");
    if (!persist || !path || !*path) return;
    if (FILE *f = std::fopen(path, "a")) {
        const int key = dtype + 4 * cls;
        if (axis >= 0) std::fprintf(f, "%d %d %d %d %d %d\n", n, kind, key, cand, waves, axis);
        else std::fprintf(f, "%d %d %d %d %d\n", n, kind, key, cand, waves);
        std::fclose(f);
    }
}

// The fused multiply pass: the grouped stages at every length that has them
// (us on a half spectrum of 129 x 256 and of 257 x 512 lines; stage by stage
// before: complex64 75 14.6, 40 (15.5, 42), 150 25, 88 (30, 101), 200 34, 126
// (38, 138), 256 39, 142 (42, 147), 360 67, 228 (87, 317), 512 95, 299 (118,
// 373); complex128 108 32, 126 (38, 142), 180 50, 207 (74, 303), 256 97, 270
// (93, 303), 512 209, 548 (244, 704)), but complex128 128 on whole-line rows beyond
// 64 MiB: the wide stage-by-stage tile (whole convolutions 512 x 400 x 128 454, 470,
// 256 x 400 x 128 228, 235, 512 x 128 x 128 140, 143; 128^3 (17 MB) 63.8, 61.1; on
// partial ones, 512 x 300 x 128, 333, 320).  Above 256 complex64 has 16- and 8-line
// tiles: the narrow ones (half a line of memory each, so in XCD order, but
// more blocks on a CU) where rows share lines anyway and the spectrum stays in
// the last-level cache (97 x 180 lines: 360 29 against 39, 512 35 against 46;
// of 211 MB and above they lose, 360 309 against 262; the line is drawn at
// 64 MiB), and alone above 512 (625 488 against 594).
void conv_choice(int n, int dtype, long long spectrum_bytes, bool partial_lines, int *cand, int *waves) {
    const bool narrow = partial_lines && spectrum_bytes <= (64LL << 20);
    *cand = 0;
    *waves = 1;  // the stage-by-stage tiles: one wave of resident blocks
    if (n == 128 && dtype == kC128 && !partial_lines && spectrum_bytes > (64LL << 20)) *cand = 1;
    else if (n == 128 || n == 256 || n == 1024 || (n == 512 && dtype == kC128)) *cand = 2;
    else if (dtype == kC64 && (n == 384 || n == 512)) *cand = narrow ? 3 : 2;
    else if (dtype == kC64 && n > 256 && n < 512) *cand = narrow ? 1 : 0;
}

// ---- slab count K of the pipelined schedule ----
// File lines "slabs nx ny nz dtype K"; the same lookup order as the pass
// choices (file, this process, built-in).  No built-in grid takes K > 1: on
// an MI355X the measured gain of the slab schedule at 512^3 and 1024^3 is
// within the spread of repeated runs.
namespace {
std::map<std::tuple<int, int, int, int>, int> g_slabs;  // (nx, ny, nz, dtype) -> K

bool read_slabs(const char *path, int nx, int ny, int nz, int dtype, int *k) {
    FILE *f = std::fopen(path, "r");
    if (!f) return false;
    bool found = false;
    int a, b, c, d, e;
    char line[256];
    while (std::fgets(line, sizeof line, f)) {
        if (std::sscanf(line, "slabs %d %d %d %d %d", &a, &b, &c, &d, &e) != 5) continue;
        if (a == nx && b == ny && c == nz && d == dtype && e >= 1 && nz % e == 0) {
            *k = e;
            found = true;
        }
    }
    std::fclose(f);
    return found;
}
}  // namespace

bool slab_wisdom_lookup(int nx, int ny, int nz, int dtype, int *k) {
    std::lock_guard<std::mutex> lk(g_mu);
    const char *path = std::getenv("CROFT_WISDOM");
    if (path && *path && read_slabs(path, nx, ny, nz, dtype, k)) return true;
    auto it = g_slabs.find({nx, ny, nz, dtype});
    if (it != g_slabs.end()) {
        *k = it->second;
        return true;
    }
    return false;
}

void slab_wisdom_record(int nx, int ny, int nz, int dtype, int k, bool persist) {
    std::lock_guard<std::mutex> lk(g_mu);
    g_slabs[{nx, ny, nz, dtype}] = k;
    const char *path = std::getenv("CROFT_WISDOM");
    if (!persist || !path || !*path) return;
    if (FILE *f = std::fopen(path, "a")) {
        std::fprintf(f, "slabs %d %d %d %d %d\n", nx, ny, nz, dtype, k);
        std::fclose(f);
    }
}

}  // namespace croft
