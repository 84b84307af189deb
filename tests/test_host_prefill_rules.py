"""Rules of the fp32 prefill attention's launches: the library's own host arithmetic, compiled on its own (no GPU needed)."""
from test_host_kv_rules import _run

HEADER = "prefill_rules.h"


def test_dealt_blocks_are_all_done_once(tmp_path):
    """Every block of every head has one workgroup, however heads are cut for the XCDs, taken in groups, and turns end."""
    _run(tmp_path, r"""
    int dealt = 0, grouped = 0, cut = 0;
    for (int heads : {1, 2, 3, 4, 5, 7, 8, 12, 25, 64, 123, 245, 250, 320, 401})
        for (int G : {1, 5})
            for (int rows : {16, 32, 128})
                for (int N : {113, 138, 140, 231, 500, 700, 1025, 2049, 4097}) {
                    lvlm_prefill_desc d{};
                    d.dtype = LVLM_F32; d.hd = 64; d.causal = 1; d.B = 1; d.N = N; d.Hq = heads; d.Hkv = heads % G ? heads : heads / G;
                    const int blocks = (N + rows - 1) / rows;
                    BlockDeal deal;
                    const unsigned wgs = deal_blocks(d, rows, deal);
                    if ((wgs != 0) != (blocks > 1 && heads * blocks > 256)) return 1;
                    if (!wgs) continue;
                    ++dealt;
                    const bool groups = deal.group < deal.xcd_parts;
                    grouped += groups;
                    cut += deal.parts_log2 > 0;
                    std::vector<int> seen(heads * blocks);
                    for (unsigned wg = 0; wg < wgs; ++wg) {
                        int head, qb;
                        if (!(groups ? dealt_block<true>(deal, blocks, wg, head, qb) : dealt_block<false>(deal, blocks, wg, head, qb))) continue;
                        if (head < 0 || head >= heads || qb >= blocks || seen[head * blocks + qb]++) return 2;
                    }
                    for (int s : seen)
                        if (s != 1) return 3;
                }
    if (!dealt || !grouped || !cut) return 4;""", HEADER)


def test_dealt_blocks_leave_few_workgroups_idle(tmp_path):
    """Parts of heads whose blocks do not fill them, and shares that heads do not, are idle workgroups in places of the chip."""
    _run(tmp_path, r"""
    for (int heads = 33; heads <= 1024; ++heads)
        for (int blocks : {2, 3, 4, 5, 8, 9, 15, 17, 33, 44, 71}) {
            lvlm_prefill_desc d{};
            d.dtype = LVLM_F32; d.hd = 128; d.causal = 1; d.B = 1; d.N = blocks < 6 ? 128 * blocks : 16 * blocks; d.Hq = d.Hkv = heads;
            BlockDeal deal;
            const long long wgs = deal_blocks(d, blocks < 6 ? 128 : 16, deal);
            if (4 * wgs > 5 * heads * blocks) return 1 + blocks;
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
                            const unsigned wg = f.dealt - 1;
                            if ((f.grouped ? dealt_block<true>(f.deal, (int)f.blocks, wg, head, qb) : dealt_block<false>(f.deal, (int)f.blocks, wg, head, qb)) &&
                                (head < 0 || head >= B * Hq)) return 3;
                        } else {
                            ++plain;
                            if (f.blocks * 256 >= 1ll << 32) return 4;
                        }
                    }
    if (!dealt || !plain) return 5;
    lvlm_prefill_desc d{};
    d.dtype = LVLM_F32; d.hd = 64; d.causal = 1; d.B = 65535; d.N = 130; d.Hq = 136; d.Hkv = 1;
    if (prefill_f32_form(d).dealt) return 6;                    // 2^24 workgroups and more
    d.B = 20000;
    if (!prefill_f32_form(d).dealt) return 7;""", HEADER)


def test_gpu_tests_take_the_launches_they_name(tmp_path):
    """The fp32 cases of the GPU tests name the kernel they are for: a rule that moves takes no kernel out of the tests unseen."""
    from test_gpu_prefill_attn import F32_DEALT, F32_ROW_BLOCKS, F32_WHOLE_TURNS
    cases = F32_ROW_BLOCKS + F32_WHOLE_TURNS + F32_DEALT
    assert {(d, form) for _, _, _, _, d, _, form in cases} == {
        (d, form + dealt) for d in (64, 128) for form in ("one", "two", "shared") for dealt in ("", " dealt", " grouped")
        if form + dealt != "shared grouped"}
    rows = ", ".join("{%d, %d, %d, %d, %d, %d, %d, %d}" % (*c[:6], ["one", "two", "shared"].index(c[6].split()[0]),
                                                            ["", "dealt", "grouped"].index((c[6] + " ").split(" ")[1])) for c in cases)
    _run(tmp_path, r"""
    const int cases[][8] = {%s};
    int i = 0;
    for (const auto &c : cases) {
        lvlm_prefill_desc d{};
        d.dtype = LVLM_F32; d.B = c[0]; d.N = c[1]; d.Hq = c[2]; d.Hkv = c[3]; d.hd = c[4]; d.causal = c[5];
        const F32Form f = prefill_f32_form(d);
        ++i;
        if ((f.shared ? 2 : f.two ? 1 : 0) != c[6] || (f.grouped ? 2 : f.dealt ? 1 : 0) != c[7]) return i;
    }""" % rows, HEADER)
