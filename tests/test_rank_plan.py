"""The plan of the ordered fetch (csrc/rank_plan.h), checked on the host with g++: at
the largest tables a plan from the test's hit words can lose them to an allocation on
the way, and the plan without them may need more workspace or not fit at all.  The
workspace that is handed out always holds the plan that is then carried out."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "rank_plan.h"
#include <cstdio>
#include <initializer_list>
using namespace gss;
static char mem[1];
int main() {
    uint64_t lost = 0, kept_ws = 0;
    const uint32_t widths[] = {8, 9, 16, 31, 64};
    for (uint32_t W : widths) {
        uint32_t RWc = 1;
        while (RWc < W) RWc <<= 1;
        const uint64_t edge = (1ull << 31) / RWc;  // ids whose hit words are 2^31 cells
        const uint64_t ids[] = {1000, 40000, edge / 8, edge - 64, edge - 1, edge, edge + 1, 2 * edge};
        for (uint64_t hits_ids : ids)
            for (uint64_t more : {0ull, 1ull, 100000ull})  // ids issued since the test
                for (uint64_t kept : {1ull, 20000ull, 1ull << 22, 1ull << 28})
                    for (int staged = 0; staged < 3; ++staged)      // none, as planned, much more
                        for (int gone = 0; gone < 4; ++gone) {      // hit words given up: never, by the stage, by the allocation, no room
                            bool has = rank_uses_hits((hits_ids * RWc / 8 + 63) / 64 * 64);
                            auto plan = [&] { return RankPlan(hits_ids + more, W, RWc, kept, has, hits_ids); };
                            uint64_t have = 0;
                            if (staged) have = plan().fits ? plan().bytes() + (staged == 2 ? 1 << 20 : 0) : 0;
                            if (gone == 1) has = false;
                            uint64_t got = 0, released = 0;
                            auto alloc = [&](uint64_t b) -> char * {
                                if (gone >= 2) has = false;
                                if (gone == 3) return nullptr;
                                got = b;
                                return mem;
                            };
                            const RankSpace s = rank_space(plan, have ? mem : nullptr, have, alloc, [&](char *) { ++released; });
                            const RankPlan p = plan();
                            const bool bad = s.ranked ? !p.small && (!p.fits || p.cells > (1ull << 31) || !s.ws || p.bytes() > s.bytes ||
                                                                     (s.own && s.bytes != got))
                                                      : s.ws != nullptr;
                            if (bad || (!s.own && got && !released)) {
                                std::printf("W %u ids %llu + %llu kept %llu staged %d gone %d: %llu bytes for %llu\n", W,
                                            (unsigned long long)hits_ids, (unsigned long long)more, (unsigned long long)kept, staged,
                                            gone, (unsigned long long)s.bytes, (unsigned long long)p.bytes());
                                return 1;
                            }
                            if (!s.ranked && gone) ++lost;
                            if (s.ranked && s.ws) ++kept_ws;
                        }
    }
    std::printf("ok %d %d\n", lost > 0, kept_ws > 0);
    return 0;
}
"""


def test_workspace_holds_the_plan(tmp_path):
    src = tmp_path / "rank_plan_check.cpp"
    exe = tmp_path / "rank_plan_check"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2012_03119_amd", "csrc"), str(src),
                    "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "ok 1 1", out.stdout
