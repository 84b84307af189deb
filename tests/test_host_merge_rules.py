"""Rules of the rank merge's launches: the library's own host arithmetic, compiled on its own (no GPU needed)."""
from test_host_kv_rules import _run


def test_searches_stage_no_more_than_their_batch_needs(tmp_path):
    """A workgroup that searches for few tokens stages as much as one that searches for many: fewer than four times 64 only while
    every workgroup has one of the 256 compute units to itself.  The longest sequences share out all their rounds of eight blocks."""
    _run(tmp_path, r"""
    for (int B : {1, 2, 3, 5, 8, 9, 16, 64, 65536})
        for (int n : {4096, 4800, 5441, 8192, 8193, 12000, 16384, 16385, 32768, 32769, 100000, 1 << 22}) {
            const SearchForm f = rank_search_form(n, B);
            const long long wgs = (long long)B * ((n + 64 * f.groups - 1) / (64 * f.groups));
            if (f.groups != 1 && f.groups != 2 && f.groups != 4) return 1;
            if (f.groups < 4 && wgs > 256) return 2;
            if (f.groups > 1 && (long long)B * ((n + 32 * f.groups - 1) / (32 * f.groups)) <= 256) return 3;
            if (f.parts != (n > 32768 ? (n + 8191) / 8192 : 1)) return 4;
            if (f.parts > 1 && f.groups != 4) return 5;
        }""")
