"""The division of the head's products into work items (csrc/lm_plan.hpp), taken by the host compiler alone: over
sizes, whole and cut contractions and numbers of CUs, every 128 rows x 256 columns of the result get every K step
exactly once, no item leaves the matrix, no two parts share a block of partial results, a launch of fewer
workgroups than CUs has one for every place, and the lanes of a wavefront agree with the host on the number of parts."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_07291_amd", "csrc")

HARNESS = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <type_traits>
#include <vector>
#include "lm_plan.hpp"
// two kernels derive one plan: in whole numbers, whatever a compiler makes of the expression in each
static_assert(std::is_integral<decltype(lm_split_cost(1, 1, 1, 1, 1, 1, 256))>::value, "whole numbers");
// the choice of a wavefront: a lane to a candidate, exchanges with lane ^ 1, ^ 2, ... ^ 32
static int wavefront_choice(int lane, int over, int thin, int kt, int blocks, int cu)
{
    long long c[64], d[64];
    int s[64], t[64];
    for (int l = 0; l < 64; ++l) c[l] = lm_split_candidate(s[l] = l + 1, over, thin, kt, blocks, cu);
    for (int o = 1; o < 64; o <<= 1) {
        for (int l = 0; l < 64; ++l) {
            const bool other = lm_split_better(c[l ^ o], s[l ^ o], c[l], s[l]);
            d[l] = other ? c[l ^ o] : c[l];
            t[l] = other ? s[l ^ o] : s[l];
        }
        std::copy(d, d + 64, c);
        std::copy(t, t + 64, s);
    }
    return s[lane];
}
static int fail(const char *what, int M, int tn, int kt, int split, int cu)
{
    printf("%s: M %d tiles_n %d k_tiles %d split %d cu %d\n", what, M, tn, kt, split, cu);
    return 1;
}
int main()
{
    long plans = 0;
    srand(7);
    // 320 live rows of 511, two columns of tiles: four halves and two thin tiles
    if (lm_items_per_xcd(lm_plan(320, 2, 16, false, 0, 256)) > lm_workgroups_per_xcd(511, 2, false, 256))
        return fail("two places for one of few workgroups", 320, 2, 16, 0, 256);
    for (int cu : {64, 256, 304})
        for (int split = 0; split < 2; ++split)
            for (int it = 0; it < 5000; ++it) {
                const int M = it < 700 ? it + 1 : 1 + rand() % 9000, tn = 1 + rand() % (rand() % 2 ? 40 : 600);
                const int kt = 1 + rand() % (rand() % 2 ? 30 : 2400), blocks_max = rand() % 4 ? 20000 : rand() % 400;
                const LmPlan pl = lm_plan(M, tn, kt, split, blocks_max, cu);
                if (const int over = pl.rows_w * tn % cu; split && over + pl.thin > 0) {
                    for (int lane : {0, 17, 63})
                        if (wavefront_choice(lane, over, pl.thin, kt, blocks_max, cu) != pl.s2)
                            return fail("a lane chooses otherwise", M, tn, kt, split, cu);
                }
                std::vector<int> cov((size_t)((M + 127) / 128) * tn, 0), blocks;
                const int most = M + rand() % 600;  // what the host knows about the rows
                const int per_xcd = lm_workgroups_per_xcd(most, tn, split, cu), items = lm_items_per_xcd(pl);
                if (per_xcd < 1 || per_xcd > cu / 8) return fail("workgroups", M, tn, kt, split, cu);
                if (per_xcd < cu / 8 && items > per_xcd) return fail("two places for one of few workgroups", M, tn, kt, split, cu);
                for (int b = 0; b < per_xcd * 8; ++b)
                    for (int idx = b / 8; idx < items; idx += per_xcd) {
                        LmItem i;
                        if (!lm_map_item(b % 8, idx, tn, pl, i)) continue;
                        for (int two = i.pair; two >= 0; --two, ++i.tn) {
                        if (i.tn < 0 || i.tn >= tn || i.row0 < 0 || i.row0 >= M || i.row0 % 128)
                            return fail("outside", M, tn, kt, split, cu);
                        const int k0 = (int)((unsigned)kt * (unsigned)i.part / (unsigned)i.parts);
                        const int k1 = (int)((unsigned)kt * (unsigned)(i.part + 1) / (unsigned)i.parts);
                        if (i.parts > 1 && k1 - k0 < 2) return fail("short part", M, tn, kt, split, cu);
                        for (int r = i.row0; r < std::min(M, i.row0 + i.height); r += 128) cov[(size_t)(r / 128) * tn + i.tn] += k1 - k0;
                        if (i.parts > 1) blocks.push_back(i.block);
                        }
                    }
                for (int c : cov)
                    if (c != kt) return fail("coverage", M, tn, kt, split, cu);
                std::sort(blocks.begin(), blocks.end());
                for (size_t q = 1; q < blocks.size(); ++q)
                    if (blocks[q] == blocks[q - 1]) return fail("shared block", M, tn, kt, split, cu);
                if (!blocks.empty() && (blocks[0] < 0 || blocks.back() >= blocks_max))
                    return fail("block outside", M, tn, kt, split, cu);
                ++plans;
            }
    printf("plans %ld\n", plans);
    return 0;
}
"""


def test_items_cover_every_product_once(tmp_path):
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(HARNESS)
    cc = subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, "-o", str(exe), str(src)],
                        capture_output=True, text=True)
    assert cc.returncode == 0, cc.stderr[-2000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0 and run.stdout == "plans 30000\n", run.stdout
