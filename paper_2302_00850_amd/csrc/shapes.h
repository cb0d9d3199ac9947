// The launch shapes of the hops: which ones a launch accepts, the default of each kind of
// launch, and the candidates of the tuner.  Host code without device or runtime calls.
#pragma once

#include <cstdlib>
#include <string>
#include <vector>

#include "../../include/cola.h"
#include "common.h"

namespace cola {

constexpr int kMaxGrid = kRedMaxBlocks;

struct TuneEntry {
    int rpt = 1;
    int sites_per_block = 64;
    int grid = 0;    // 0: one block per sites_per_block site columns; -1: the blocks
                     // resident at once (grid-stride loop, no tail of late blocks)
    int tchunk = 1;  // timeslices walked by one lane
    int tile_y = 0;  // spatial tile (all x-rows x tile_y x tile_z); 0 = lexicographic
    int tile_z = 0;
    int stage = 0;   // 1: links staged in LDS by the lanes of a site (see stage_ok); 2: a
                     // wavefront per direction (see dirs_ok)
    double ms = 0;
};

// A spatial tile must divide the y and z extents (tile_y = 0: no tiling).
inline bool tile_ok(const Geom &g, int ty, int tz) {
    if (ty == 0 && tz == 0) return true;
    return ty > 0 && tz > 0 && g.L[1] % ty == 0 && g.L[2] % tz == 0;
}

// Link staging: one or two rhs per lane, at least three lanes per site to share the
// eight links, whole sites of at most kStageSites per block, a 12-real FP16 or FP32 field
// and a packed field addressable with 32-bit byte offsets.
inline bool stage_ok(const Geom &g, int prec, int nrhs, const TuneEntry &t) {
    if (prec != COLA_FP16 && prec != COLA_FP32) return false;
    const double bytes = 8.0 * 3 * g.S * (prec == COLA_FP16 ? 8 : 16);
    return (t.rpt == 1 || t.rpt == 2) && nrhs / t.rpt >= 3 && t.sites_per_block <= kStageSites &&
           bytes < 2147483648.0;
}

// The hop with a wavefront per direction (stage = 2): FP64 and FP32, one rhs per lane, whole
// sites of at most kDirsSites lanes per block, one block per sites_per_block sites.
inline bool dirs_ok(const Geom &g, int prec, int nrhs, const TuneEntry &e) {
    return prec != COLA_FP16 && e.rpt == 1 && e.grid == 0 && e.tchunk == 1 && e.tile_y == 0 &&
           e.tile_z == 0 && e.sites_per_block >= 1 && e.sites_per_block * nrhs <= kDirsSites &&
           2.0 * ((double)g.Vh / e.sites_per_block + 1) <= kMaxGrid;
}

// A launch shape the hop kernels accept for this lattice, precision and rhs count.
inline bool shape_valid(const Geom &g, int prec, int nrhs, const TuneEntry &e) {
    if (e.stage == 2) return dirs_ok(g, prec, nrhs, e);
    const bool f64 = prec == COLA_FP64 || prec == COLA_FP64_12;
    return (e.rpt >= 1 && e.rpt <= 4) && nrhs % e.rpt == 0 && (e.rpt == 1 || !f64) &&
           e.sites_per_block >= 1 && (e.sites_per_block & (e.sites_per_block - 1)) == 0 &&
           e.sites_per_block * (nrhs / e.rpt) <= 256 && e.grid >= -1 && e.tchunk >= 1 &&
           g.L[3] % e.tchunk == 0 && tile_ok(g, e.tile_y, e.tile_z);
}

// The largest spatial tile (ty x tz columns of all x, dividing the lattice, tz >= 2) whose
// timeslice holds at most `most` checkerboard sites; the squarer one of equals.  0 x 0 when
// there is none.
inline void best_tile(const Geom &g, int most, int *ty, int *tz) {
    *ty = *tz = 0;
    // per divisor y the largest z that fits: a smaller z of the same y is a smaller tile
    for (int y = 2; y <= g.L[1]; ++y) {
        if (g.L[1] % y) continue;
        int z = most / (g.Lxh * y);
        if (z > g.L[2]) z = g.L[2];
        while (z >= 2 && g.L[2] % z) --z;
        if (z < 2) continue;
        const int now = y * z, had = *ty * *tz;
        if (now > had || (now == had && abs(y - z) < abs(*ty - *tz))) {
            *ty = y;
            *tz = z;
        }
    }
}

// The tile of at most `most` sites.  None where the whole timeslice is one, or but a quarter
// more (several rhs): the order is that of one tile, the index cheaper, and cutting it in two
// costs more than it keeps.  20 x 18 x 14 x 30 (2520 sites) against 9x14 tiles, D_eo D_oe: FP32 12
// rhs 162 -> 148 us, 10 rhs 152 -> 134, 3 rhs 54 -> 50; FP16 12 rhs 102 -> 92.
inline void set_tile(const Geom &g, int most, bool several, TuneEntry &t) {
    const double slice = g.s3;
    t.tile_y = t.tile_z = 0;
    if (slice > (several ? 1.25 : 1.0) * most) best_tile(g, most, &t.tile_y, &t.tile_z);
}

// A launch of few blocks takes smaller ones, down to a wavefront, so that more of the chip's
// compute units have one: FLIC FP32 8^4 D_eo D_oe, 3 rhs 24.4 -> 21.5 us, 7 rhs 26.1 -> 22.0.
inline void fill_chip(TuneEntry &t, double sites, int nrhs) {
    while (t.sites_per_block > 1 && t.sites_per_block * nrhs > 64 &&
           sites / t.tchunk / t.sites_per_block < 200.0)
        t.sites_per_block /= 2;
}

// Launch shapes.  Tiles are walked through t, so that the timeslices in flight of a tile and
// their links stay in one XCD's L2; the tile sizes below are where the times measured over
// all divisors of 24^3 x 48, 32^3 x 64 and 48^3 x 96 are flat or lowest.
inline TuneEntry plain_entry(const Geom &g, int prec, int nrhs, bool both, bool clover) {
    TuneEntry t;
    t.rpt = 1;
    const int G = nrhs;
    int T = 1;
    while (T * 2 * G <= 256) T *= 2;
    t.sites_per_block = T;
    t.grid = 0;
    const double sites = (double)g.Vh * (both ? 2 : 1);
    if (nrhs == 1) {
        // 8192 sites, or 4096 where both parities run side by side.  M^dag M (both): FP64
        // 48^3 x 96 7.12 ms with 16x16 tiles of 64-site blocks, 5.06 with 24x6 (256); 32^3 x
        // 64 1.14 and 1.04 ms with 16x16 (256); 24^3 x 48 410 us untiled, 353 with 24x12;
        // FP32 48^3 x 96 3.05 ms untiled, 2.36; FP16 1.60 ms with 16x8, 1.35.  S^dag S (one
        // parity): FP64 48^3 x 96 7.30 -> 6.81 ms, 32^3 x 64 1.27 -> 1.23; FP32 2.94 -> 2.78
        // ms and 528 -> 515 us.  Blocks of 256 sites where that leaves each CU several of
        // them, else 64.
        set_tile(g, both ? 4096 : 8192, false, t);
        t.sites_per_block = sites >= 524288.0 ? 256 : 64;
        return t;
    }
    if (prec == COLA_FP64 || prec == COLA_FP64_12) {
        // FP64 (2304 bytes a site with 12 rhs).  12 rhs, S^dag S: 24^3 x 48 2.76 ms with
        // 12x6, 2.82 with 8x8; 32^3 x 64 9.2 ms with 8x4 and 8x8; clover S 48^3 x 96 29.4
        // ms with 8x4, 28.7 with 6x6; with 2 to 8 rhs 12x6 or 12x12 are the fastest on 24^3
        // x 48.  M^dag M (both): 24^3 x 48 2.86 ms with 8x8, 2.73 with 6x4; 32^3 x 64 9.74
        // ms with 8x8, 8.95 with 4x4; up to 8 rhs 12x6 as for one parity.  Two rhs, and three
        // with one parity, up to 2048 sites: 32^3 x 64 2 rhs D_eo D_oe 1076 us untiled, 1275 with
        // 8x4, 948 with 16x8; 48 x 24 x 24 x 32 430 with 6x6, 415 with 12x6; 3 rhs 569 and 547.
        const bool wide = nrhs == 2 || (nrhs == 3 && !both);
        set_tile(g, wide ? 2048 : both && nrhs > 8 ? 288 : 900, true, t);
        return t;
    }
    // FP32 and FP16: the site's links staged in LDS.  Four rhs without a clover block, in
    // blocks of kStageSites sites walking time in chunks of 4 (one parity: where 4 rounds of
    // resident blocks remain, else 2), if that leaves a block for each SIMD.  M and D_eo D_oe,
    // unstaged and so: FP32 16^3 x 32 45.2 -> 41.1 and 53.7 -> 45.9 us, 24^3 x 48 254 -> 225
    // and 249 -> 229, 32^3 x 64 798 -> 663 and 869 -> 716; FP16 31.9 -> 30.9 and 35.4 -> 35.6,
    // 142 -> 128 and 157 -> 141, 468 -> 402 and 497 -> 434.  With clover blocks to stage as
    // well M takes 315 and 323 us in FP32 at 24^3 x 48, and in FP16 191 and 240.
    if (nrhs == 4 && !clover) {
        TuneEntry s = t;
        s.sites_per_block = kStageSites;
        const double blocks = sites / kStageSites;
        if (blocks / 2 >= 1024.0 && stage_ok(g, prec, nrhs, s)) {
            s.stage = 1;
            s.tchunk = blocks / 4 >= (both ? 1 : 4) * 1024.0 ? 4 : 2;
            while (g.L[3] % s.tchunk) s.tchunk /= 2;
            set_tile(g, 2048, true, s);
            return s;
        }
    }
    // From five rhs on always.  M, clover FP32, 5 rhs, unstaged and staged: 20 x 18 x 14 x 30
    // 105 and 89 us, 24^3 x 48 452 and 411; FP16 74 and 69, 274 and 297.
    t.stage = nrhs >= 5 && stage_ok(g, prec, nrhs, t) ? 1 : 0;
    if (t.stage) {
        // With staged links the lanes can walk time with the neighbours of their index in
        // registers: chunks of 8 timeslices where at least 12 rounds of resident blocks
        // remain, of 4 where 4 rounds do, else no walk.  S^dag S with 12 rhs: FP32 24^3 x 48
        // 1.29 ms with 8x8 in chunks of 8, 1.19 with 12x12 in 4; 32^3 x 64 3.99 and 3.78
        // with 16x8 in 4; clover S 48^3 x 96 11.24 and 11.09 with 12x6 in 8; FP16 24^3 x 48
        // 790 and 712 us.  5 to 8 rhs on 24^3 x 48 (2 to 3 rounds): 0 to 7% faster without
        // the walk.  Both parities (M^dag M): FP32 24^3 x 48 1.21 ms with 12x6.
        set_tile(g, both ? 1024 : 2048, true, t);
        fill_chip(t, sites, nrhs);
        const double blocks = sites / t.sites_per_block;
        t.tchunk = blocks / 8 >= 12 * 1024.0 ? 8 : blocks / 4 >= 4 * 1024.0 ? 4 : 1;
        while (g.L[3] % t.tchunk) t.tchunk /= 2;
        return t;
    }
    // two to four rhs per site (M, 24^3 x 48 FP16: 92 us untiled in 256-lane blocks, 78
    // with 12x12 tiles of 64-site blocks)
    if (T > 64) t.sites_per_block = 64;
    set_tile(g, 2048, true, t);
    fill_chip(t, sites, nrhs);
    return t;
}

// Launches of few lanes (sites of one parity x rhs) take the hop with a wavefront per
// direction.  The lines, from times of plain_entry's shape over times of this one (m: both
// parities, s: D_eo D_oe; c: with clover; 12 = FP64_12):
//   one rhs   FP32 s 28^3 x 48 1.29, c 1.20, 32^3 x 64 0.88; m 24^3 x 48 1.06; m c 16^3 x 32
//             1.02, 18^3 x 30 0.98, 20^3 x 32 0.97
//             FP64 s 24^3 x 32 1.12 (12: 1.18), 24^3 x 48 0.92 (1.03), 28^3 x 48 0.95 (0.98); m
//             28^3 x 48 1.11 (1.09), 32^3 x 64 0.83 (0.85); s c 20^3 x 32 1.04 (1.02), 24^3 x 32
//             0.98 (1.05); m c 16^3 x 32 1.19 (1.11), 20 x 18 x 14 x 30 (1.10), 20^3 x 24 1.05
//             (0.95), 20^3 x 32 1.07 (0.95), 24^3 x 32 0.98 (0.95)
//   more      (2 to 16 rhs, 4 thousand to 131 thousand lanes) FP32 at least 0.98 up to 65536;
//             m c 1.05 up to 41 thousand, then 0.83 to 0.94 from six rhs on
//             FP64 at least 0.97; m c 0.95 up to 41 thousand, then 0.91 to 0.94 with 11 and 12
//             rhs, 0.85 to 0.98 from 76 on, but with 7 and 8 rhs 1.03 to 1.09 up to 110 and with
//             16 1.08 at 110; s c at least 1.01, but with three and four rhs 0.91 from 98 on
inline bool few_lanes(const Geom &g, int prec, int nrhs, bool both, bool clover) {
    const double lanes = (double)g.Vh * nrhs;
    if (prec == COLA_FP32) {
        if (nrhs == 1) return lanes <= (clover && both ? 65536 : 600000);
        return lanes <= (clover && both && nrhs > 5 ? 43008 : 65536);
    }
    if (!clover) return lanes <= (nrhs > 1 ? 131072 : both ? 600000 : 262144);
    if (nrhs == 1) return lanes <= (both && prec == COLA_FP64_12 ? 81920 : 131072);
    if (both && nrhs < 16) return lanes <= (nrhs > 8 ? 43008 : nrhs > 6 ? 114688 : 73728);
    return lanes <= (nrhs == 3 || nrhs == 4 ? 90112 : 131072);
}

// The shape of the hop with a wavefront per direction: as many whole sites as a block takes.
inline TuneEntry dirs_entry(int nrhs) {
    TuneEntry t;
    t.stage = 2;
    t.sites_per_block = kDirsSites / nrhs;
    return t;
}

inline TuneEntry default_entry(const Geom &g, int prec, int nrhs, bool both, bool clover) {
    const TuneEntry t = dirs_entry(nrhs);
    if (few_lanes(g, prec, nrhs, both, clover) && dirs_ok(g, prec, nrhs, t)) return t;
    return plain_entry(g, prec, nrhs, both, clover);
}

// The FLIC hops load both links per lane, one rhs per lane, and neither stage links nor walk
// time.  Blocks: one wavefront where the rhs fill it (2, 4, 8, 16); else in FP64 up to one
// wavefront, with both parities up to 256 lanes; FP32 and three rhs as plain_entry.  Tiles of
// 1024 sites, in FP64 with both parities 512 up to 8 rhs, with both parities 256 beyond; FP32
// counts that do not fill a wavefront keep the tile and chunk of plain_entry (12 rhs: within 2%
// of the best of 80 shapes), three rhs in FP64 with one parity 2048.  FP64 takes chunks of 4
// timeslices from five rhs on where 4 rounds of resident blocks remain, with three where one
// does.  Against plain_entry, D_eo D_oe and M at 32^3 x 64: FP64 12 rhs 8.47 -> 7.76 and 6.95 ->
// 6.50 ms, 8 rhs 4.89 -> 4.26 and 4.39 -> 3.88, 4 rhs 2.58 -> 2.34 and 2.25 -> 2.00, 3 rhs 2.32 ->
// 2.13 and 1.95 -> 1.74, one rhs 1.20 -> 1.11 and 0.89 -> 0.74; FP32 (with the bases of its
// arrays formed singly) 16 rhs 4.10 -> 3.82 and 4.25 -> 4.01, 4 rhs 1.18 -> 1.01 and 1.07 -> 0.94.
inline TuneEntry flic_entry(const Geom &g, int prec, int nrhs, bool both) {
    TuneEntry t = plain_entry(g, prec, nrhs, both, false);
    t.stage = 0;
    const bool f64 = prec == COLA_FP64 || prec == COLA_FP64_12;
    const double sites = (double)g.Vh * (both ? 2 : 1);
    const auto chunk = [&](int rounds) {
        t.tchunk = sites / t.sites_per_block / 4 >= rounds * 1024.0 ? 4 : 1;
        while (g.L[3] % t.tchunk) t.tchunk /= 2;
    };
    if (nrhs == 1) {
        if (f64 && t.sites_per_block == 256) {
            t.sites_per_block = 128;
            set_tile(g, both ? 2048 : 4096, false, t);
        }
        return t;
    }
    int T = 64;
    while (T * nrhs > 64) T /= 2;
    const bool fills = T * nrhs == 64;
    if (f64 && nrhs == 3) {
        if (!both) set_tile(g, 2048, true, t);
        chunk(1);
    } else if (fills || f64) {
        if (fills || !both) t.sites_per_block = T;
        const int most = !both || nrhs == 2 ? 1024 : nrhs > 8 ? 256 : f64 ? 512 : 1024;
        set_tile(g, most, true, t);
        t.tchunk = 1;
        if (f64 && nrhs >= 5) chunk(4);
    }
    fill_chip(t, sites, nrhs);
    return t;
}

// A shape that the FLIC hops take.
inline bool flic_ok(const Geom &g, int prec, int nrhs, const TuneEntry &t) {
    return t.rpt == 1 && t.stage == 0 && shape_valid(g, prec, nrhs, t);
}

// The shapes that the tuner times: the defaults first, so that a tuned shape is never a slower
// one; blocks by rhs per lane in plain order and chunks, with power-of-two tiles and, one rhs
// per lane, the tiles that the defaults are made of; each also staged where that applies.
inline std::vector<TuneEntry> tune_candidates(const Geom &g, int prec, int nrhs, bool both,
                                              bool clover) {
    std::vector<TuneEntry> cand;
    const auto add = [&](const TuneEntry &t) {
        for (const TuneEntry &c : cand)
            if (c.rpt == t.rpt && c.sites_per_block == t.sites_per_block && c.grid == t.grid &&
                c.tchunk == t.tchunk && c.tile_y == t.tile_y && c.tile_z == t.tile_z &&
                c.stage == t.stage)
                return;
        cand.push_back(t);
    };
    add(default_entry(g, prec, nrhs, both, clover));
    add(plain_entry(g, prec, nrhs, both, clover));
    if (dirs_ok(g, prec, nrhs, dirs_entry(nrhs))) add(dirs_entry(nrhs));
    std::vector<TuneEntry> base;
    for (int rpt : {1, 2, 3, 4}) {
        if (nrhs % rpt) continue;
        if (rpt > 1 && (prec == COLA_FP64 || prec == COLA_FP64_12)) continue;
        const int G = nrhs / rpt;
        // blocks of whole wavefronts when some block size allows it
        bool whole = false;
        for (int T : {4, 8, 16, 32, 64, 128, 256}) whole |= T * G <= 256 && (T * G) % 64 == 0;
        for (int T : {4, 8, 16, 32, 64, 128, 256}) {
            if (T * G > 256 || T * G < 64) continue;
            if (whole && (T * G) % 64 != 0) continue;
            TuneEntry t;
            t.rpt = rpt;
            t.sites_per_block = T;
            for (int tc : {1, 2, 4, 8, 16}) {
                if (g.L[3] % tc) continue;
                t.tchunk = tc;
                for (int grid : {0, -1}) {
                    t.grid = grid;
                    base.push_back(t);
                }
            }
            t.tchunk = 1;
            t.grid = 0;
            const int tiles[][2] = {{4, 4}, {8, 4}, {4, 8}, {8, 8}, {16, 8}, {8, 16}, {16, 16}};
            for (const auto &tl : tiles) {
                t.tile_y = tl[0];
                t.tile_z = tl[1];
                if (tile_ok(g, tl[0], tl[1])) base.push_back(t);
            }
            if (rpt > 1) continue;
            for (int most : {288, 900, 1024, 2048, 4096, 8192}) {
                best_tile(g, most, &t.tile_y, &t.tile_z);
                base.push_back(t);
            }
        }
    }
    for (const TuneEntry &b : base) add(b);
    for (const TuneEntry &b : base) {
        if (!stage_ok(g, prec, nrhs, b)) continue;
        TuneEntry t = b;
        t.stage = 1;
        add(t);
        // the time walk of staged FP32 / FP16 hops: tiles in chunks of 4 and 8 timeslices
        if ((prec == COLA_FP32 || prec == COLA_FP16) && t.rpt == 1 && t.tile_y > 0) {
            for (int tc : {4, 8}) {
                if (g.L[3] % tc) continue;
                t.tchunk = tc;
                add(t);
            }
        }
    }
    return cand;
}

// The key of the table of tuned shapes: device and version, launch.  Entries of another
// version, timed against other kernels and other defaults, stay in the file and are not used;
// the number goes up whenever a kernel, a kind of shape or a default changes.
constexpr const char *kShapeVersion = ":v2 ";

inline std::string table_key(const std::string &arch, int num_cu, const std::string &key) {
    return arch + ":" + std::to_string(num_cu) + kShapeVersion + key;
}

}  // namespace cola
