"""Plans and requests of the row kernels, on the host: how the waves of a workgroup share the groups of K, that every request, those past
a wave's last group included, names bytes of the layer, and which shape serves layers that another would slow down."""
import os
import subprocess

from test_gpu_rows import SLICES, TILE

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "bf16_rows_plan.hpp"
#include "rows_plan.hpp"
#include "wave_share.hpp"
using namespace dmr;

// The waves of all splits cover the groups once and in order; each asks for `ahead` items beyond its own.
static int check(int groups, int gps, int splits, int held, int ahead) {
    int next = 0;
    for (int split = 0; split < splits; ++split)
        for (int wave = 0; wave < kSharingWaves; ++wave) {
            const WaveShare s = wave_share(groups, gps, split, wave);
            if (s.g0 != next || s.n < 0 || s.n > held) return 1;
            next += s.n;
            for (int i = 0; i < s.n + ahead; ++i) {
                const int g = requested_group(s, i, groups);
                if (g < 0 || g >= groups || (i < s.n && g != s.g0 + i)) return 2;
            }
        }
    return next == groups ? 0 : 3;
}

int main() {
    for (int K = 128; K <= 20480; K += 128)
        for (int N : {16, 272, 1024, 4096, 6160, 8208, 28672})
            for (int M : {2, 8, 9, 16, 17, 32, 33, 48, 49, 64, 100, 129, 145, 193, 250, 289, 385, 512}) {
                const int groups = K / kGroup;
                for (int max_splits : {1, 2, 4, 8}) {
                    int bad = 0;
                    const Bf16RowsPlan b = plan_bf16_rows(M, K, N, max_splits);
                    if (b.ok) bad = check(groups, b.gps, b.SK, b.GPW, b.GPW - 1);        // items of a tile: GPW, whatever the wave holds
                    if (!bad && M >= 17) {
                        const RowsPlan r = plan_rows(M, K, N, max_splits);
                        if (r.slices) bad = check(groups, r.gps, r.SK, groups, 1);
                        if (r.half && (r.slices || r.MT < 3)) bad = 4;              // not instantiated
                    }
                    if (bad) {
                        std::printf("K=%d N=%d M=%d splits<=%d: %d\n", K, N, M, max_splits, bad);
                        return 1;
                    }
                }
            }
    return 0;
}
"""


PLANS = r"""
#include <cstdio>
#include "row_splits.hpp"
using namespace dmr;

int main() {
    int bad = 0;
    auto want = [&](int M, int K, int N, bool slices, int MT, int WM, int R, int SK) {
        const RowsPlan p = rows_call(M, K, N);
        if (p.slices == slices && p.MT == MT && p.WM == WM && p.R == R && p.SK == SK) return;
        std::printf("%d x %d -> %d: slices %d MT %d WM %d R %d SK %d\n", M, K, N, p.slices, p.MT, p.WM, p.R, p.SK);
        bad = 1;
    };
    // a few more than 256 workgroups take what 512 do: not 288 or 320 of two tiles (23.9, 16.7 and 6.5 us) but K in three on the tile
    // kernel (18.3, 14.4) or 144 of four tiles (5.5)
    want(32, 8192, 9216, false, 2, 1, 0, 3);
    want(17, 6144, 10240, false, 2, 1, 0, 3);
    want(32, 1024, 9216, true, 2, 1, 4, 1);
    want(32, 4096, 8192, true, 2, 1, 2, 1);            // 256 of two
    // two and four blocks of 48 rows where one or two of 96 leave half of the chip idle (12.6 / 8.9 us, 15.7 / 10.5)
    want(96, 1024, 16384, false, 3, 1, 0, 1);
    want(192, 1536, 8192, false, 3, 1, 0, 1);
    want(128, 4096, 28672, false, 4, 2, 0, 1);         // more than a round of them: 128 rows
    // 256 workgroups of four tiles: K stays whole (27.6 / 24.9 us)
    want(17, 11008, 16384, true, 2, 1, 4, 1);
    return bad;
}
"""


def run(tmp_path, program):
    src, exe = tmp_path / "share.hip", tmp_path / "share"
    src.write_text(program)
    inc = os.path.join(ROOT, "paper_2602_02711_amd", "csrc")
    built = subprocess.run(["hipcc", "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-I", inc, str(src), "-o", str(exe)],
                           capture_output=True, text=True)
    assert built.returncode == 0, built.stderr[-2000:]
    ran = subprocess.run([str(exe)], capture_output=True, text=True)
    assert ran.returncode == 0, ran.stdout
    return ran.stdout


def test_every_request_names_a_group_of_the_layer(tmp_path):
    run(tmp_path, PROGRAM)


def test_shapes_of_the_row_kernels(tmp_path):
    run(tmp_path, PLANS)


def test_the_gpu_cases_cover_every_shape(tmp_path):
    cases = ", ".join("{%d, %d, %d}" % c for c in SLICES + TILE)
    out = run(tmp_path, r"""
#include <cstdio>
#include "row_splits.hpp"
struct Case {
    int M, K, N;
};
int main() {
    for (const auto &c : {%s}) {
        const dmr::RowsPlan p = dmr::rows_call(c.M, c.K, c.N);
        std::printf("%%d %%d %%d %%d %%d %%d\n", p.slices, p.MT, p.WM, p.R, p.half, p.SK > 1);
    }
    return 0;
}
""" % cases.replace("{", "Case{"))
    got = [tuple(map(int, line.split())) for line in out.splitlines()]
    assert all(p[0] == 1 for p in got[:len(SLICES)]) and all(p[0] == 0 for p in got[len(SLICES):])
    want = {(1, mt, 1, r, 0, split) for mt in (2, 3, 4) for r in (1, 2, 4) for split in (0, 1)}
    want |= {(0, mt, wm, 0, 0, split) for mt, wm in ((2, 1), (3, 1), (4, 1), (3, 2), (4, 2)) for split in (0, 1)}
    want |= {(0, mt, wm, 0, 1, 0) for mt, wm in ((3, 1), (4, 1), (3, 2), (4, 2))}
    assert want == set(got), (want - set(got), set(got) - want)
