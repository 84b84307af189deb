"""Positions of query rows at the ends of their range: the host arithmetic the score kernels rely on, compiled on its own
with signed overflow trapped (no GPU needed)."""
import importlib.util
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "common.h"
using namespace lvlm;
int main() {
    const int top = 0x7fffffff, n_max = 1 << 22;
    for (int N : {1, 31, 64, 5219, n_max})
        for (int p : {0, 1, N - 1, N, N + 1, n_max + 1, top - 65535, top - 128, top - 1, top})
            for (int i : {0, 1, 127, 65534}) {
                lvlm_score_desc d{};
                d.N = N;
                d.q_pos0 = p;
                const int got = first_row_position(d) + i;                 // traps if it overflows
                const long long want = (long long)p + i;
                if ((got < N - 1 ? got : N - 1) != (want < N - 1 ? want : N - 1)) return 1;      // the keys this row sees
                for (int jb = 0; jb < N; jb += 64 * 37)
                    for (int je : {jb + 1, jb + 63, jb + 64, jb + 65, N}) {
                        if (je > N || je <= jb) continue;
                        long long steps = 0;
                        while (jb + 64 * (steps + 1) <= je && jb + 64 * (steps + 1) - 1 <= want && steps < 200) ++steps;
                        const int s = steps_seen(jb, je, got, 64);
                        if (s > (je - jb) / 64 || (steps < 200 && s != steps)) return 2;
                    }
            }
    // whatever the position is, the steps stay inside the keys
    for (int pos : {-top - 1, -1, 0, top - 1, top})
        for (int jb : {0, 64, n_max - 64}) {
            const int s = steps_seen(jb, n_max, pos, 64);
            if (s < 0 || s > (n_max - jb) / 64 || (pos < 0 && s != 0)) return 3;
        }
    return 0;
}
"""


def test_positions_of_rows_never_overflow_and_steps_stay_in_range(tmp_path):
    spec = importlib.util.spec_from_file_location("lvlm_build", os.path.join(ROOT, "paper_2509_00419_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    src, exe = tmp_path / "positions.hip", tmp_path / "positions"
    src.write_text(PROGRAM)
    subprocess.run([build.HIPCC, "--offload-host-only", "--offload-arch=gfx950", "-std=c++17", "-O1", "-Xarch_host",
                    "-fsanitize=signed-integer-overflow", "-Xarch_host", "-fsanitize-trap=signed-integer-overflow",
                    "-I" + build.CSRC, str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)]).returncode == 0
