// How the cluster solver (cluster.hpp) lays an instance out over workgroups:
// host arithmetic on sizes alone.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <vector>

#include "plan.hpp"

namespace hms {

constexpr int kXcds = 8;              // XCDs of the GPU, each with its own L2
constexpr int kXcdCus = 32;           // CUs per XCD: the most workgroups a cluster can have
constexpr int kClusterThreads = 1024;
constexpr int kClusterWaves = kClusterThreads / 64;
constexpr int kClusterMaxPos = 32768; // LDS slots a 15-bit literal field can name
constexpr int kClusterMaxWide = 65536; // positions a 16-bit literal field can name (wide form)
constexpr int kOneSlots = 4096;       // LDS slots up to which t is exchanged as {t, step} words
constexpr uint32_t kAltByte = 0x20000;  // second copy of t in LDS (a bit past every record offset)
constexpr size_t kClusterSharedBytes = 320;  // the workgroup variables after the arrays

// How a cluster's wavefronts hold their tiles: several each (state in LDS), or
// at most one (state in registers), the latter exchanging t behind flags or,
// for few variables, as words that carry their step.  Wide: several each, with
// only the roundings of all variables in LDS (more variables than t fits for).
enum ClusterMode : int32_t { kClusterMany = 0, kClusterOne = 1, kClusterOneWords = 2, kClusterWide = 3 };

// What the shape depends on.
struct ClusterSize {
    int32_t v_tiles = 0;   // variable tiles
    int32_t NO = 0;        // other literals per occurrence record (2, 3 or 4)
};

// Shape of a cluster solve of an instance.
struct ClusterShape {
    int32_t mode = kClusterMany;
    int32_t C = 0;         // workgroups per restart (a power of two)
    int32_t NO = 0;
    int32_t slice = 0;     // variables per workgroup, padded to whole tiles
    size_t lds = 0;        // dynamic LDS per workgroup
    int32_t per_launch = 0;  // restarts one launch holds
};

constexpr size_t cluster_up16(size_t b) { return (b + 15) & ~size_t(15); }
// LDS of a workgroup: t of all variables and two constants, own x, m, v, own
// rounded bits (current and best).
constexpr size_t cluster_t_bytes(int32_t C, int32_t slice) { return cluster_up16(((size_t)C * slice + 2) * 4); }
constexpr size_t cluster_many_lds(int32_t C, int32_t slice) {
    return cluster_up16(cluster_t_bytes(C, slice) + (size_t)slice * 12 + (size_t)(slice / 64) * 16) + kClusterSharedBytes;
}
// The same in the wide form: a bit per variable and for the two constants, own
// t, x, m, v, own rounded bits.
constexpr size_t cluster_bits_bytes(int32_t C, int32_t slice) {
    return cluster_up16(((size_t)C * slice / 64 + 1) * 8);
}
constexpr size_t cluster_wide_lds(int32_t C, int32_t slice) {
    return cluster_up16(cluster_bits_bytes(C, slice) + (size_t)slice * 16 + (size_t)(slice / 64) * 16) +
           kClusterSharedBytes;
}
// One tile per wavefront: t of all variables, twice where it goes in words.
constexpr size_t cluster_one_lds(int32_t C, int32_t slice, bool words) {
    return (words ? kAltByte : 0) + cluster_t_bytes(C, slice) + kClusterSharedBytes;
}

// Which shapes are looked at: any (a single instance), or those of the two forms
// for several tiles per wavefront.
enum ClusterForm : int32_t { kFormAny = 0, kFormMany = 1, kFormWide = 2 };

// Shape for R restarts together; false when there is none.
inline bool cluster_shape_of(const ClusterSize& Z, int32_t R, size_t lds_cap, ClusterShape& sh,
                             ClusterForm form = kFormAny) {
    sh.NO = Z.NO;
    // as many workgroups per restart as leave every restart its own at once
    int32_t C = kXcdCus;
    while (C > 2 && (int64_t)kXcds * (kXcdCus / C) < R) C /= 2;
    while (C > 2 && C > Z.v_tiles) C /= 2;
    // at most one tile per wavefront: the fewest workgroups that leave each of
    // their four SIMDs one tile, half as many tiles where t goes in words (n =
    // 4000, 3-CNF, one restart: 2.33 us a step at one, 2.31 at two, 2.39 at
    // four, 2.94 at sixteen tiles)
    if (form == kFormAny && Z.v_tiles <= kClusterWaves * C) {
        const int per = Z.v_tiles * kTile <= kOneSlots ? 2 : 4;  // tiles per workgroup
        int32_t c1 = 2;
        while (c1 < C && Z.v_tiles > per * c1) c1 *= 2;
        const int32_t slice = (Z.v_tiles + c1 - 1) / c1 * kTile;
        const bool words = c1 * slice <= kOneSlots && slice / kTile <= kClusterWaves / 2;
        const size_t lds = cluster_one_lds(c1, slice, words);
        if (lds <= lds_cap && c1 * slice + 2 <= kClusterMaxPos) {
            sh.C = c1;
            sh.slice = slice;
            sh.lds = lds;
            sh.mode = words ? kClusterOneWords : kClusterOne;
            sh.per_launch = kXcds * (kXcdCus / c1);
            return true;
        }
    }
    auto slice_at = [&](int32_t c) { return (Z.v_tiles + c - 1) / c * kTile; };
    auto fits = [&](int32_t c, bool wide) {
        const int64_t P = (int64_t)c * slice_at(c);
        if (wide) return P + 64 <= kClusterMaxWide && cluster_wide_lds(c, slice_at(c)) <= lds_cap;
        return P + 2 <= kClusterMaxPos && cluster_many_lds(c, slice_at(c)) <= lds_cap;
    };
    // wide where t fits LDS neither with so many workgroups nor with more.  481 to
    // 496 tiles fit with 16 only and so change form past eight restarts (n = 31000,
    // us a step with 16 in that form and wide with 32: 3-CNF 6.6 and 6.9, counted
    // every step 17.1 and 12.7; nine restarts, both with 16, 6.6 and 10.0)
    const int32_t C0 = C;
    bool wide = form == kFormWide;
    while (C <= kXcdCus && !fits(C, wide)) C *= 2;
    if (C > kXcdCus && form == kFormAny) {
        wide = true;
        for (C = C0; C <= kXcdCus && !fits(C, wide);) C *= 2;
    }
    if (C > kXcdCus) return false;
    sh.mode = wide ? kClusterWide : kClusterMany;
    sh.slice = slice_at(C);
    sh.lds = wide ? cluster_wide_lds(C, sh.slice) : cluster_many_lds(C, sh.slice);
    sh.C = C;
    sh.per_launch = kXcds * (kXcdCus / C);
    return true;
}

// Shapes of instances whose solves run together, largest first, R[i] restarts
// of instance i: as many workgroups per restart as leave every restart its own
// at once.  One launch runs one kernel.  `wide`: which form each instance has by
// itself (the form may change with the number of restarts, so it is fixed here
// for all of them); those that are not wide take the form for several tiles per
// wavefront unless all fit the same other one.  What CUs are left in that form go
// to the largest instances (twelve 3-CNF instances of 15000 to 26000 variables: 16
// workgroups each, 32 for the four largest).  False when an instance does not fit
// the form or their kernels differ.
inline bool cluster_group(const std::vector<ClusterSize>& Z, const std::vector<int32_t>& R, bool wide, size_t lds_cap,
                          std::vector<ClusterShape>& sh) {
    const size_t count = Z.size();
    sh.assign(count, ClusterShape());
    int32_t units = 0;
    for (int32_t r : R) units += r;
    for (size_t i = 0; i < count; ++i)
        if (Z[i].NO != Z[0].NO) return false;
    bool one = !wide;  // all at most one tile per wavefront, with one exchange
    for (size_t i = 0; i < count && one; ++i)
        one = cluster_shape_of(Z[i], units, lds_cap, sh[i]) && sh[i].mode == sh[0].mode &&
              (sh[i].mode == kClusterOne || sh[i].mode == kClusterOneWords);
    if (one) return true;
    const ClusterForm form = wide ? kFormWide : kFormMany;
    int32_t left = kXcds * kXcdCus;
    for (size_t i = 0; i < count; ++i) {
        if (!cluster_shape_of(Z[i], units, lds_cap, sh[i], form)) return false;
        left -= R[i] * sh[i].C;
    }
    for (size_t i = 0; i < count; ++i) {
        ClusterShape more;
        const int32_t C = sh[i].C;
        if (C == kXcdCus || R[i] * C > left) break;
        if (!cluster_shape_of(Z[i], kXcds * (kXcdCus / (2 * C)), lds_cap, more, form) || more.C != 2 * C) break;
        sh[i] = more;
        left -= R[i] * C;
    }
    return true;
}

}  // namespace hms
