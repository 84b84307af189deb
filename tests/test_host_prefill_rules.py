"""Rules of the fp32 prefill attention's launches: the library's own host arithmetic, compiled on its own (no GPU needed)."""
from test_host_kv_rules import _run

HEADER = "prefill_rules.h"


def test_dealt_blocks_are_all_done_once(tmp_path):
    """Every block of every head has one workgroup, however heads are cut for the XCDs and turns end, and the workgroups of an XCD
    have equally many of a level."""
    _run(tmp_path, r"""
    for (int heads : {1, 2, 3, 4, 5, 7, 8, 12, 25, 64, 250, 320})
        for (int blocks : {2, 3, 7, 8, 9, 31, 33, 44, 65, 130, 257}) {
            lvlm_prefill_desc d{};
            d.causal = 1; d.B = 1; d.Hq = heads;
            BlockDeal deal;
            const unsigned wgs = deal_blocks(d, blocks, deal);
            if ((wgs != 0) != (heads * blocks > 256)) return 1;
            std::vector<int> seen(heads * blocks);
            for (unsigned wg = 0; wg < wgs; ++wg) {
                int head, qb;
                if (!dealt_block(deal, blocks, wg, head, qb)) continue;
                if (head < 0 || head >= heads || qb >= blocks || seen[head * blocks + qb]++) return 2;
            }
            for (int s : seen)
                if (wgs && s != 1) return 3;
        }""", HEADER)


def test_launches_of_any_size_fit_their_grid(tmp_path):
    """A grid dimension holds less than 2^32 threads, 256 to a workgroup: calls of more workgroups take the grid of three."""
    _run(tmp_path, r"""
    int dealt = 0, plain = 0;
    for (int hd : {64, 128})
        for (int causal : {0, 1})
            for (int B : {1, 64, 4096, 16384, 32768, 65535})
                for (int Hq : {1, 8, 40, 128, 512, 1024})
                    for (int N : {1, 17, 33, 48, 129, 700, 4096, 1 << 22}) {
                        lvlm_prefill_desc d{};
                        d.dtype = LVLM_F32; d.hd = hd; d.causal = causal; d.B = B; d.N = N; d.Hq = Hq; d.Hkv = 1;
                        if ((long long)B * Hq * ((N + 127) / 128) >= 1ll << 28 || (long long)B * Hq * N >= 1ll << 33) continue;
                        const F32Form f = prefill_f32_form(d);
                        if (f.dealt) {
                            ++dealt;
                            if ((unsigned long long)f.dealt * 256 >= 1ull << 32) return 1;
                            if (f.dealt < f.blocks * B * Hq || !causal) return 2;
                            int head, qb;       // (the last workgroup: no product on the way overflows)
                            if (dealt_block(f.deal, (int)f.blocks, f.dealt - 1, head, qb) && (head < 0 || head >= B * Hq)) return 3;
                        } else {
                            ++plain;
                            if (f.blocks * 256 >= 1ll << 32) return 4;
                        }
                    }
    if (!dealt || !plain) return 5;
    lvlm_prefill_desc d{};
    d.dtype = LVLM_F32; d.hd = 64; d.causal = 1; d.B = 65535; d.N = 33; d.Hq = 136; d.Hkv = 1;
    if (prefill_f32_form(d).dealt) return 6;                    // 2^24 workgroups and more
    d.B = 30000;
    if (!prefill_f32_form(d).dealt) return 7;""", HEADER)


def test_gpu_tests_take_the_launches_they_name(tmp_path):
    """The fp32 cases of the GPU tests name the kernel they are for: a rule that moves takes no kernel out of the tests unseen."""
    from test_gpu_prefill_attn import F32_DEALT, F32_ROW_BLOCKS, F32_WHOLE_TURNS
    cases = F32_ROW_BLOCKS + F32_WHOLE_TURNS + F32_DEALT
    assert {(d, form) for _, _, _, _, d, _, form in cases} == {
        (d, form + dealt) for d in (64, 128) for form in ("one", "two", "shared") for dealt in ("", " dealt")}
    rows = ", ".join("{%d, %d, %d, %d, %d, %d, %d, %d}" % (*c[:6], ["one", "two", "shared"].index(c[6].split()[0]), "dealt" in c[6])
                     for c in cases)
    _run(tmp_path, r"""
    const int cases[][8] = {%s};
    int i = 0;
    for (const auto &c : cases) {
        lvlm_prefill_desc d{};
        d.dtype = LVLM_F32; d.B = c[0]; d.N = c[1]; d.Hq = c[2]; d.Hkv = c[3]; d.hd = c[4]; d.causal = c[5];
        const F32Form f = prefill_f32_form(d);
        ++i;
        if ((f.shared ? 2 : f.two ? 1 : 0) != c[6] || (f.dealt != 0) != (c[7] != 0)) return i;
    }""" % rows, HEADER)
