"""The entries that a set's members' lists hold, as the service counts them from lengths of two bytes:
lists just below, at and above what those hold, past 2^32 entries in all, and repeated members."""
import host_unit


@host_unit.needs_hipcc
def test_list_entries():
    out = host_unit.run(r"""
#include <algorithm>
#include <cstdio>
#include <vector>
#include "skis_query.h"
int main()
{
    const int64_t lens[] = {0, 1, 7, 65534, 65535, 65536, 65537, 1 << 20, INT32_MAX, 3};
    std::vector<int64_t> ptr{0};
    std::vector<uint16_t> two;
    for (int64_t l : lens) {
        ptr.push_back(ptr.back() + l);
        two.push_back((uint16_t)std::min<int64_t>(l, skis::LONG_LIST));
    }
    const std::vector<std::vector<int32_t>> sets = {{}, {0}, {3}, {4}, {5}, {6}, {0, 1, 2, 9}, {4, 4, 3}, {8, 8, 8, 1},
                                                    {9, 8, 7, 6, 5, 4, 3, 2, 1, 0}};
    for (const auto &s : sets) {
        uint64_t want = 0;
        for (int32_t v : s) want += (uint64_t)lens[v];
        if (skis::list_entries(two.data(), ptr.data(), s.data(), (int32_t)s.size()) != want) std::printf("%zu\n", s.size());
    }
    std::puts("done");
}
""")
    assert out == "done\n"
