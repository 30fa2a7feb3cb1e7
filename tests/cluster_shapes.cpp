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

// One launch: one kernel, shapes in order, every restart its own workgroups or less room than that.
bool check_group(const std::vector<ClusterSize>& Z, const std::vector<int32_t>& R) {
    std::vector<ClusterShape> sh;
    int units = 0;
    for (int32_t r : R) units += r;
    if (!cluster_group(Z, R, kCap, sh)) return false;
    for (size_t i = 0; i < Z.size(); ++i) {
        check_shape(sh[i], Z[i].v_tiles, Z[i].NO, units);
        if (sh[i].mode != sh[0].mode || sh[i].NO != sh[0].NO) wrong("two kernels in one launch", Z[i].v_tiles, Z[i].NO, units);
    }
    return true;
}

}  // namespace

int main() {
    long shapes = 0, groups = 0;
    std::vector<int> wide(kMaxTiles + 1, -1);  // whether an instance's roundings alone are in LDS
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
                const int w = s.mode == kClusterWide;
                if (wide[tiles] < 0) wide[tiles] = w;
                if (wide[tiles] != w) wrong("the form depends on the restarts", tiles, NO, R);
            }
        }
    // equal instances, one or several restarts each
    for (int NO = 2; NO <= 4; ++NO)
        for (int tiles = 2; tiles <= kMaxTiles; ++tiles)
            for (int count = 2; count <= 64; ++count)
                for (int r : {1, 2, 5, 9}) {
                    if (!least[tiles] || least[tiles] > r) continue;
                    if (!check_group(std::vector<ClusterSize>(count, ClusterSize{tiles, NO}), std::vector<int32_t>(count, r)))
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
            if (wide[tiles] != w || least[tiles] > r) continue;
            Z.push_back(ClusterSize{tiles, NO});
            R.push_back(r);
        }
        std::stable_sort(Z.begin(), Z.end(), [](const ClusterSize& a, const ClusterSize& b) { return a.v_tiles > b.v_tiles; });
        if (!check_group(Z, R)) wrong("instances of one form refused", Z[0].v_tiles, NO, count);
        ++groups;
    }
    // of two forms: never one launch
    for (int a = 2; a <= kMaxTiles; ++a)
        for (int b = 470; b <= 520; ++b)
            for (int r : {1, 2, 9}) {
                if (wide[a] < 0 || wide[b] < 0 || least[a] > r || least[b] > r) continue;
                const bool ok = check_group({ClusterSize{std::max(a, b), 2}, ClusterSize{std::min(a, b), 2}}, {r, r});
                if (ok != (wide[a] == wide[b])) wrong("two forms in one launch", a, b, r);
                ++groups;
            }
    std::printf("ok %ld shapes %ld groups\n", shapes, groups);
    return 0;
}
