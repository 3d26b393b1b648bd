"""Which wave takes which query rows in the bf16 forward and dQ kernels, over random shapes and row windows, on the CPU: the map that the
kernels use is compiled for the host.  Every row of every head has one wave, and all waves of a workgroup walk equally far."""
import os
import subprocess

import paper_2506_11498_amd as lrsa

SOURCE = r"""
#include "mfma_tiles.h"
#include <cstdio>
#include <random>
#include <vector>
using namespace lrsa;
static int fail(const char* what, const Dims& D, int waves) {
    printf("%s: B %d Hkv %d G %d n %d L %d S %d rows [%d, %d) waves %d\n", what, D.B, D.Hkv, D.G, D.n, D.L, D.S, D.row_begin, D.row_end, waves);
    return 1;
}
int main() {
    std::mt19937 r(17);
    auto pick = [&](std::vector<int> v) { return v[r() % v.size()]; };
    for (int it = 0; it < 3000; ++it) {
        Dims D{};
        D.B = pick({1, 1, 2, 3}); D.Hkv = pick({1, 2, 3, 8}); D.G = pick({1, 2, 3, 4, 5, 6, 7, 8, 12, 16, 20, 64}); D.Hq = D.Hkv * D.G;
        D.n = 1 + r() % pick({40, 400, 3000}); D.L = 2 + r() % pick({8, 40, 300, 2000}); D.S = r() % pick({1, 8, 70, 500}); D.K = 1 + r() % D.L;
        D.lp = 1; D.d = 128; D.dtype = 1;
        const int rest = D.n > D.S ? D.n - D.S : 0;
        D.nq = (rest + D.L - 1) / D.L; D.Ns = D.nq > 2 ? D.nq - 2 : 0;
        D.fq0 = 0; D.fq1 = D.nq; D.row_begin = 0; D.row_end = D.n;
        if (D.nq > 1 && r() % 3 == 0) {     // a filling step
            D.fq0 = r() % D.nq; D.fq1 = D.fq0 + 1 + r() % (D.nq - D.fq0);
            D.row_begin = D.fq0 == 0 ? 0 : D.S + D.fq0 * D.L; D.row_end = D.fq1 == D.nq ? D.n : D.S + D.fq1 * D.L;
        }
        for (int waves : {4, 8}) {
            const QTileMap M = make_qtile_map(D, waves);
            const int tiles = D.B * D.Hkv * M.per_unit;
            if (M.per_unit != tiles_per_unit(D, waves)) return fail("tiles_per_unit", D, waves);
            std::vector<unsigned char> seen(size_t(D.B) * D.Hq * D.n, 0);
            int used = 0;
            for (int i = 0; i < M.wgs; ++i) {
                int b, h, tix, last = -2;
                if (!decode_qtile(M, D, i, b, h, tix)) continue;
                ++used;
                if (b < 0 || b >= D.B || h < 0 || h >= D.Hkv || tix < M.tix_lo || tix >= M.tix_hi) return fail("tile out of range", D, waves);
                bool any = false;
                for (int w = 0; w < waves; ++w) {
                    int qc, seg_end, tw, head, t_last;
                    const bool there = qtile_rows(M, D, tix, waves, w, qc, seg_end, tw, head, t_last);
                    if (w && (there != any || (there && t_last != last))) return fail("waves disagree", D, waves);
                    any = there; last = t_last;
                    if (!there) continue;
                    if (head < 0 || head >= D.G || tw < 0) return fail("piece out of range", D, waves);
                    for (int t = tw; t < tw + 32 && t < seg_end; ++t) {
                        if (t > t_last) return fail("row behind the walk", D, waves);
                        if (t < D.S ? qc != -1 : (t - D.S) / D.L != qc) return fail("row of another chunk", D, waves);
                        ++seen[(size_t(b) * D.Hq + h * D.G + head) * D.n + t];
                    }
                }
            }
            if (used != tiles) return fail("tiles left out", D, waves);
            for (int bh = 0; bh < D.B * D.Hq; ++bh)
                for (int t = 0; t < D.n; ++t)
                    if (seen[size_t(bh) * D.n + t] != (t >= D.row_begin && t < D.row_end)) return fail("a row without one wave", D, waves);
        }
    }
    puts("ok");
}
"""


def test_every_row_has_one_wave(tmp_path):
    src = tmp_path / "map.hip"
    src.write_text(SOURCE)
    csrc = os.path.join(os.path.dirname(lrsa.__file__), "csrc")
    exe = str(tmp_path / "map")
    subprocess.run(["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "--offload-host-only", "-O2", "-std=c++17", "-w", f"-I{csrc}", str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr
