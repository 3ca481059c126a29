// Host check of the 3-D pass planner (csrc/smap_steps.hpp): over boxes and
// generations, the pieces of an H pass cover every column of the 3-simplex
// once, plane by plane, their numbers fit the fields the kernel reads them
// from, and up to n = 3000 the cut is the one whose rounds over the chip take the
// fewest planes (beyond, whole columns may be taken instead).
#include <cstdio>
#include <cstdlib>
#include <map>

#include "../../paper_2208_11617_amd/csrc/smap_plan.hpp"
#include "../../paper_2208_11617_amd/csrc/smap_steps.hpp"

using namespace smap;

static long bad = 0;
static void fail(const char *what, int64_t n, int gens, int64_t a, int64_t b)
{
    if (++bad < 20) std::printf("%s: n=%lld gens=%d: %lld %lld\n", what, (long long)n, gens, (long long)a, (long long)b);
}

static int64_t planes(int64_t n, int gens, const Steps3Plan &S, int64_t rz)
{
    const int64_t pieces = steps3_pieces(n, S.rho, rz);
    return (pieces + S.slots - 1) / S.slots * (rz + 2 * gens);
}

int main()
{
    const int64_t sizes[] = {0, 1, 14, 15, 31, 32, 47, 48, 63, 64, 100, 200, 301, 383, 384, 385, 512, 700, 1024,
                             1250, 1700, 2500, 3000, 3500, 3750, 4200, 5000, 5240, 6000, 8000};
    for (const int64_t n : sizes) {
        for (int gens = 1; gens <= kCa3kMaxGens; ++gens) {
            Steps3Plan S = steps3_plan(n, gens);
            for (int64_t rz = 1; n <= 3000 && rz <= n + 1; rz += 1 + rz / 16) {
                if (steps3_pieces(n, S.rho, rz) > 8 * S.slots) continue;
                if (planes(n, gens, S, rz) < planes(n, gens, S, S.rz))
                    fail("better cut", n, gens, S.rz, rz);
            }
            Plan P;
            if (make_plan(2, n, 2, S.rho, false, &P, nullptr) != kOk) { fail("plan", n, gens, 0, 0); continue; }
            steps3_units(P, S);
            if ((int64_t)S.units.size() != steps3_pieces(n, S.rho, S.rz)) fail("count", n, gens, S.units.size(), S.rz);
            std::map<std::pair<uint32_t, uint32_t>, std::vector<int>> seen;
            for (const uint32_t u : S.units) {
                auto &v = seen[{u & 1023u, u >> 10 & 1023u}];
                const size_t k = u >> 20;
                if (v.size() <= k) v.resize(k + 1);
                ++v[k];
            }
            int64_t columns = 0;
            for (int64_t x = 0; x <= n / S.rho; ++x) {
                for (int64_t y = 0; (x + y) * S.rho <= n; ++y, ++columns) {
                    // the kernel's cut of a column: pieces of `each` planes from 0 to its height
                    const int64_t height = n - (x + y) * S.rho + 1, cnt = (height + S.rz - 1) / S.rz,
                                  each = (height + cnt - 1) / cnt;
                    const auto it = seen.find({(uint32_t)x, (uint32_t)y});
                    if (it == seen.end()) { fail("column", n, gens, x, y); continue; }
                    const int64_t k = (int64_t)it->second.size();
                    if (k * each < height || (k - 1) * each >= height || each > S.rz) fail("cover", n, gens, k, each);
                    for (const int c : it->second)
                        if (c != 1) fail("twice", n, gens, x, y);
                }
            }
            if (columns != (int64_t)seen.size()) fail("columns", n, gens, columns, seen.size());
        }
    }
    std::printf("bad=%ld\n", bad);
    return bad != 0;
}
