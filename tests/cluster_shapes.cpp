// Checks cluster_shape.hpp over all sizes (run by test_cluster_shapes.py):
// prints the number of shapes and groups looked at, or the first one that is wrong.
#include <cstdio>
#include <cstdlib>

#include "cluster_shape.hpp"

using namespace hms;

namespace {

constexpr size_t kCap = 160 * 1024;
constexpr int kMaxTiles = 1023;

[[noreturn]] void wrong(const char* what, int tiles, int NO, int R) {
    std::printf("wrong: %s (tiles %d, NO %d, restarts %d)\n", what, tiles, NO, R);
    std::exit(1);
}

void check_shape(const ClusterShape& s, int tiles, int NO, int R) {
    const int64_t P = (int64_t)s.C * s.slice;
    const bool one = s.mode == kClusterOne || s.mode == kClusterOneWords;
    if (s.C < 2 || s.C > kXcdCus || (s.C & (s.C - 1)) || s.per_launch != kXcds * (kXcdCus / s.C)) wrong("workgroups", tiles, NO, R);
    if (s.slice % 64 || P < (int64_t)tiles * 64 || (int64_t)(tiles - 1) / s.C * 64 >= s.slice) wrong("slice", tiles, NO, R);
    if (s.lds > kCap) wrong("LDS over the limit", tiles, NO, R);
    if (one && s.slice > kClusterWaves * 64) wrong("more than a tile per wavefront", tiles, NO, R);
    if (s.mode == kClusterOneWords && (P > kOneSlots || s.slice > kClusterWaves * 32)) wrong("words", tiles, NO, R);
    if (s.mode == kClusterWide ? P + 64 > kClusterMaxWide : P + 2 > kClusterMaxPos) wrong("literal field", tiles, NO, R);
    const size_t need = s.mode == kClusterWide ? cluster_wide_lds(s.C, s.slice)
                        : one ? cluster_one_lds(s.C, s.slice, s.mode == kClusterOneWords) : cluster_many_lds(s.C, s.slice);
    if (s.lds != need || s.NO != NO) wrong("LDS of another form", tiles, NO, R);
}

bool is_wide(int tiles, int NO, int R) {
    ClusterShape s;
    return cluster_shape_of(ClusterSize{tiles, NO}, R, kCap, s) && s.mode == kClusterWide;
}

// One launch: one kernel, every shape a valid one.
bool check_group(const std::vector<ClusterSize>& Z, const std::vector<int32_t>& R, bool wide) {
    std::vector<ClusterShape> sh;
    int units = 0;
    for (int32_t r : R) units += r;
    if (!cluster_group(Z, R, wide, kCap, sh)) return false;
    for (size_t i = 0; i < Z.size(); ++i) {
        check_shape(sh[i], Z[i].v_tiles, Z[i].NO, units);
        if (sh[i].mode != sh[0].mode || sh[i].NO != sh[0].NO) wrong("two kernels in one launch", Z[i].v_tiles, Z[i].NO, units);
        if ((sh[i].mode == kClusterWide) != wide) wrong("not the group's form", Z[i].v_tiles, Z[i].NO, units);
    }
    return true;
}

}  // namespace

int main() {
    long shapes = 0, groups = 0;
    std::vector<int> least(kMaxTiles + 1, 0);  // fewest restarts it runs with
    for (int NO = 2; NO <= 4; ++NO)
        for (int tiles = 2; tiles <= kMaxTiles; ++tiles) {
            least[tiles] = 0;
            for (int R = 1; R <= 300; ++R) {
                ClusterShape s;
                if (!cluster_shape_of(ClusterSize{tiles, NO}, R, kCap, s)) {
                    if (tiles <= 992) wrong("refused", tiles, NO, R);
                    if (least[tiles]) wrong("refused with more restarts only", tiles, NO, R);
                    continue;
                }
                if (!least[tiles]) least[tiles] = R;
                check_shape(s, tiles, NO, R);
                ++shapes;
            }
        }
    // equal instances, one or several restarts each
    for (int NO = 2; NO <= 4; ++NO)
        for (int tiles = 2; tiles <= kMaxTiles; ++tiles)
            for (int count = 2; count <= 64; ++count)
                for (int r : {1, 2, 5, 9}) {
                    if (!least[tiles] || least[tiles] > r) continue;
                    if (!check_group(std::vector<ClusterSize>(count, ClusterSize{tiles, NO}), std::vector<int32_t>(count, r),
                                     is_wide(tiles, NO, r)))
                        wrong("equal instances refused", tiles, NO, r);
                    ++groups;
                }
    // instances of one form as a batch brings them: largest first, restarts of their own
    unsigned z = 12345;
    auto rnd = [&](int n) { return (int)((z = z * 1664525u + 1013904223u) >> 8) % n; };
    for (int it = 0; it < 400000; ++it) {
        const int count = 2 + rnd(it % 4 == 0 ? 63 : 15), w = rnd(2), NO = 2 + rnd(3);
        const int lo = it % 3 == 0 ? 470 : 2, hi = it % 3 == 0 ? 510 : kMaxTiles;
        std::vector<ClusterSize> Z;
        std::vector<int32_t> R;
        while ((int)Z.size() < count) {
            const int tiles = lo + rnd(hi - lo + 1), r = 1 + rnd(rnd(2) ? 3 : 20);
            if (!least[tiles] || least[tiles] > r || is_wide(tiles, NO, r) != (w != 0)) continue;
            Z.push_back(ClusterSize{tiles, NO});
            R.push_back(r);
        }
        std::stable_sort(Z.begin(), Z.end(), [](const ClusterSize& a, const ClusterSize& b) { return a.v_tiles > b.v_tiles; });
        if (!check_group(Z, R, w != 0)) wrong("instances of one form refused", Z[0].v_tiles, NO, count);
        ++groups;
    }
    // sizes in no order, with either form asked for: one kernel, or none
    for (int a = 2; a <= kMaxTiles; ++a)
        for (int b = 470; b <= 520; ++b)
            for (int r : {1, 2, 9})
                for (bool w : {false, true}) {
                    check_group({ClusterSize{std::max(a, b), 2}, ClusterSize{std::min(a, b), 2}}, {r, r}, w);
                    ++groups;
                }
    if (check_group({ClusterSize{100, 2}, ClusterSize{100, 3}}, {1, 1}, false)) wrong("two record sizes in one launch", 100, 2, 1);
    std::printf("ok %ld shapes %ld groups\n", shapes, groups);
    return 0;
}
