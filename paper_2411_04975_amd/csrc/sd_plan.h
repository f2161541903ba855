// How many waves a workgroup of k_speculate gets, and how much LDS.  Host code without any HIP
// call, so that it can be held to its promises without a GPU.
#pragma once
#include <stddef.h>

// A compute unit hands LDS out in pieces of this many bytes (gfx950: 160 KiB in 128 pieces).
constexpr size_t SD_LDS_PIECE = 1280;
constexpr int SD_PLAN_OCC = 6;       // waves per SIMD that one or two resident workgroups may fill
constexpr size_t SD_PLAN_SMALL_TREES = 4096;  // LDS of a wave with trees of up to 53 nodes
constexpr int SD_PLAN_RESIDENT = 4;  // workgroups per compute unit that a large batch is sized for

struct sd_plan {
    int waves;     // of a workgroup; 0: not even one wave's share fits
    int resident;  // workgroups that are on a compute unit together with this much LDS, if there are so many
    size_t lds;    // dynamic LDS of a workgroup
};

// requests: of the launch, one workgroup each; lds_cu: LDS of a compute unit; lds_dyn_max: the most dynamic LDS
// that a launch may ask for; lds_static: what the kernel holds besides; lds_wave: a wave's frontier, trees and
// staging; lds_least: what the occurrence sort needs whatever the waves do; lds_most: what it can use, of LDS that would
// lie idle (where all workgroups of a compute unit are resident).
//
// One workgroup per compute unit takes the 16 waves a workgroup can have; two share SD_PLAN_OCC waves per
// SIMD between them (12 each: the kernel's registers leave room for 6 per SIMD); three and four get 8
// and 6.  More requests are throughput work: 5 waves up to eight per compute unit, 4 from there on (five
// of the larger workgroups resident, and less idle time at their barriers).  Where it is known how many waves the
// registers of a compute unit have room for (wave_room; 0: not), five to eight get 4 as well if that makes as many
// resident waves or more, which six workgroups of four do and four of five don't; but trees of more than some 50 nodes keep 5 at five
// requests, as many as are resident then but for one.
// sd_speculate, us, 5 and 4 waves, by nodes:  1100 requests  64: 34.3 34.7     1280  32: 31.1 25.6  48: 33.7 30.0  64: 37.4 37.4
//    1536  32: 33.2 27.8  48: 36.7 32.7  64: 40.1 38.2     2048  32: 43.3 36.4  48: 46.3 42.1  64: 50.8 46.2
//
// Up to four workgroups of a compute unit are counted on to be resident together, and the waves are cut
// down until they are: a workgroup that does not fit runs behind the others, which costs more than the
// waves are worth.  Only where that leaves less than two waves, or (up to eight requests per compute
// unit) less than eight in all, two to a SIMD, it is one workgroup less.
// sd_speculate, us, geometric means over five kinds of contexts and corpora, by waves x resident:
//    64 nodes  1000 requests   6 x 3  33.1    5 x 4  25.2
//   128 nodes   300            8 x 1  29.7    7 x 2  22.8      700   5 x 2  35.6    4 x 3  27.1
//              1000            4 x 3  37.8    3 x 4  31.0     4096   4 x 3  99.2    3 x 4  85.3
//   180 nodes  1000            3 x 3  41.9    2 x 4  36.9     4096   3 x 3   111    2 x 4  99.1
//   256 nodes   700            2 x 3  57.5    4 x 2  48.0     4096   2 x 3   152    4 x 2   167
inline sd_plan sd_plan_waves(int requests, int n_cu, size_t lds_cu, size_t lds_dyn_max, size_t lds_static,
                             size_t lds_wave, size_t lds_least, size_t lds_most = 0, int wave_room = 0) {
    const int per_cu = (requests + n_cu - 1) / n_cu;
    int most = per_cu <= 2 ? 4 * SD_PLAN_OCC / per_cu : per_cu == 3 ? 8 : per_cu == 4 ? 6 : per_cu <= 8 ? 5 : 4;
    if (most > 16) most = 16;
    if (wave_room > 0 && per_cu > 4 && per_cu <= 8 && (per_cu > 5 || lds_wave <= SD_PLAN_SMALL_TREES)) {
        auto resident = [&](int waves) {  // waves of a compute unit
            const size_t whole = (lds_static + waves * lds_wave + SD_LDS_PIECE - 1) / SD_LDS_PIECE * SD_LDS_PIECE;
            int n = (int)(lds_cu / whole);
            if (n > wave_room / waves) n = wave_room / waves;
            return (n < per_cu ? n : per_cu) * waves;
        };
        if (resident(4) >= resident(5)) most = 4;
    }
    int r = per_cu < SD_PLAN_RESIDENT ? per_cu : SD_PLAN_RESIDENT, fit = 0;
    size_t dyn = 0;
    for (;; r--) {  // the waves of a workgroup if r of them are to be resident
        const size_t share = lds_cu / (size_t)r / SD_LDS_PIECE * SD_LDS_PIECE;
        dyn = share > lds_static ? share - lds_static : 0;
        if (dyn > lds_dyn_max) dyn = lds_dyn_max;
        fit = dyn >= lds_least ? (int)(dyn / lds_wave) : 0;
        if (r == 1 || (fit >= 2 && (per_cu > 8 || fit * r >= 8))) break;
    }
    sd_plan p;
    p.waves = fit < most ? fit : most;
    p.resident = r;
    p.lds = (size_t)p.waves * lds_wave;
    if (p.lds < lds_least) p.lds = lds_least;
    if (r == per_cu && p.lds < lds_most) p.lds = lds_most < dyn ? lds_most : dyn;
    return p;
}
