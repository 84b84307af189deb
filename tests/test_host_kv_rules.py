"""Rules of the cache compression's launches: the library's own host arithmetic, compiled on its own (no GPU needed)."""
import importlib.util
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(tmp_path, body, header="common.h"):
    """Compiles `body` (the statements of main) against one of the library's headers, host side only, and runs it."""
    spec = importlib.util.spec_from_file_location("lvlm_build", os.path.join(ROOT, "paper_2509_00419_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    src, exe = str(tmp_path / "rules.hip"), str(tmp_path / "rules")
    with open(src, "w") as f:
        f.write(f'#include "{header}"\n#include <algorithm>\n#include <vector>\nusing namespace lvlm;\nint main() {{\n' + body +
                "\n    return 0;\n}\n")
    subprocess.run([build.HIPCC, "--offload-host-only", "--offload-arch=gfx950", "-std=c++17", "-O1", "-I" + build.CSRC, "-Xarch_host",
                    "-fsanitize=undefined", "-Xarch_host", "-fsanitize-trap=undefined", src, "-o", exe], check=True)
    code = subprocess.run([exe]).returncode
    assert code == 0, code


def test_fill_workgroups_with_work_are_spread_over_the_chip(tmp_path):
    """Workgroups go round 8 XCDs of 4 shader engines in launch order, and a head's first ones have its moves: whatever the
    heads and bounds, every engine gets its share of those."""
    _run(tmp_path, r"""
    for (long long heads : {256, 400, 500, 640, 800, 1000, 1024, 1536, 2048, 4096})
        for (int max_moves : {65, 250, 512, 1000, 1024, 2048, 8256}) {
            const int wgs = kv_fill_workgroups(heads, max_moves), most = (max_moves + kFillRows - 1) / kFillRows;
            for (int eighths = 1; eighths <= 8; ++eighths) {               // batches a head really has
                const int batches = std::max(1, most * eighths / 8);
                long long load[32] = {}, total = 0, top = 0;
                for (long long h = 0; h < heads; ++h)
                    for (int x = 0; x < wgs && x < batches; ++x) {
                        const long long at = h * wgs + x, n = (batches - x + wgs - 1) / wgs;
                        load[at % 8 * 4 + at / 8 % 4] += n;
                        total += n;
                    }
                for (long long l : load) top = std::max(top, l);
                if (32 * top > total + total / 4 + 64 * most) return 1;
            }
        }""")


def test_fill_workgroups_by_heads_and_batches(tmp_path):
    """One workgroup for every batch there can be while those are not too many; reserved caches start no more than 16384."""
    _run(tmp_path, r"""
    if (kv_fill_workgroups(112, 16512 / 2) != 147) return 1;                                   // 258 batches a head
    if (kv_fill_workgroups(8, 2000) != 63 || kv_fill_workgroups(64, 1000) != 33 || kv_fill_workgroups(800, 1000) != 33) return 2;
    if (kv_fill_workgroups(1536, 944) != 23 || kv_fill_workgroups(64, 8256) != 257 || kv_fill_workgroups(800, 100) != 5) return 3;
    if (kv_fill_workgroups(1, 1 << 30) != 16385 || kv_fill_workgroups(1 << 20, 100) != 1 || kv_fill_workgroups(1, 65) != 3) return 4;""")


def test_rows_go_past_the_caches_by_what_the_heads_hold(tmp_path):
    """The rule's line at 256 MiB of live rows, and no overflow at the largest calls."""
    _run(tmp_path, r"""
    if (fill_past_caches(112, 2115, 256) || !fill_past_caches(1536, 1888, 256)) return 1;
    if (fill_past_caches(256, 2048, 256) || !fill_past_caches(256, 2049, 256) || !fill_past_caches(1, (256ll << 20) / 1024 + 1, 512)) return 2;
    if (fill_past_caches(65535, 0, 512) || !fill_past_caches(1ll << 20, 1 << 30, 512)) return 3;""")


def test_select_form_of_few_heads(tmp_path):
    """Where every head has a compute unit of its own, long heads take 1024 threads; every form holds the heads it is taken for."""
    _run(tmp_path, r"""
    for (long long heads : {1, 8, 64, 256, 257, 300, 512, 513, 768, 769, 1280, 1281, 1536, 1537, 5000, 1 << 20})
        for (int bound : {1, 70, 1024, 1025, 1280, 1281, 2048, 2049, 2560, 2561, 4096, 4097, 8192, 8193, 17408, 17409, 1 << 30}) {
            const SelectForm f = kv_select_form(bound, heads);
            if (f.keys ? f.keys * f.threads < bound : bound <= 17408) return 1;
            if (f.waves * 4 * 64 < f.threads) return 2;
            const bool wide = (bound > 1024 && bound <= 2048) || bound > 2560;
            if (heads <= 256 && wide && f.threads != 1024) return 3;
            if (heads > 256 && bound <= 8192 && f.threads == 1024) return 4;
        }""")


def test_select_form_spills_only_where_it_saves_a_turn(tmp_path):
    """Eight keys per thread at six waves per SIMD put registers into scratch memory: taken only where the heads then need fewer
    turns of the chip (five heads of 256 threads, or two of 512, fit a compute unit without)."""
    _run(tmp_path, r"""
    for (long long heads = 257; heads < 9000; ++heads)
        for (int bound : {1500, 2048, 3000, 4096}) {
            const SelectForm f = kv_select_form(bound, heads);
            if (f.keys != 8) continue;
            const long long without = 256 * (f.threads == 256 ? 5 : 2), with = 256 * (f.threads == 256 ? 6 : 3);
            const bool saves = (heads + with - 1) / with < (heads + without - 1) / without;
            if ((f.waves == 6) != saves) return 1;
        }
    if (kv_select_form(2048, 1536).waves != 6 || kv_select_form(2048, 1000).waves != 5) return 2;
    if (kv_select_form(4096, 640).waves != 6 || kv_select_form(4096, 512).waves != 4) return 3;""")
