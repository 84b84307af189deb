"""What the compiler gives the kernels whose form, or whose launch rule, counts on it (no GPU needed): waves per SIMD, and no
registers in scratch memory.  Launch bounds that ask for it change the code (two waves per SIMD asked of prefill_attn_d64_kernel, its
registers are halved into two kinds: 2 x 4000 tokens, 32 heads 176 -> 180 us), so it is checked here instead."""
import importlib.util
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _reports(*sources):
    spec = importlib.util.spec_from_file_location("lvlm_build", os.path.join(ROOT, "paper_2509_00419_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    procs = [subprocess.Popen([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                               os.path.join(build.CSRC, s), "-o", os.devnull], stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                              text=True) for s in sources]
    out = {}
    for p in procs:
        text, _ = p.communicate()
        assert p.returncode == 0, text[-2000:]
        for part in text.split("Function Name: ")[1:]:
            got = {k: int(v) for k, v in re.findall(r"(Scratch|Occupancy)\w* \[[^\]]*\]: (\d+)", part)}
            out[part.split()[0]] = (got["Occupancy"], got["Scratch"])
    return out


def test_waves_per_simd_that_forms_and_rules_count_on():
    reports = _reports("prefill.hip", "merge.hip")
    for name, waves, n in (("prefill_attn_d64_kernel", 2, 1), ("prefill_attn_bf16_kernel", 1, 1), ("prefill_attn_safe_kernel", 1, 2),
                           ("11rank_kernelINS0_7ByScore", 8, 1),        # two workgroups of 16 waves, beside which norms are taken
                           ("rank_search_kernelINS0_7ByScoreELi2E", 8, 1), ("rank_search_kernelINS0_7ByScoreELi4E", 8, 1),
                           ("rank_search_kernelINS0_7ByOwnerELi2E", 8, 1), ("rank_search_kernelINS0_7ByOwnerELi4E", 8, 1)):
        found = {k: v for k, v in reports.items() if name in k}
        assert len(found) == n, (name, sorted(reports))
        for kernel, (occupancy, scratch) in found.items():
            assert occupancy >= waves and scratch == 0, (kernel, occupancy, scratch)
