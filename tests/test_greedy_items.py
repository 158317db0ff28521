"""The queue records of the greedy's cover: a sample's first entry and its length come back as they
went in, also past 2^33 entries (a sketch of that size does not fit a test), and at the longest
sample there can be."""
import host_unit


@host_unit.needs_hipcc
def test_cover_items():
    out = host_unit.run(r"""
#include <cstdio>
#include "skis_query.h"
int main()
{
    const int64_t firsts[] = {0, 1, 2, (1ll << 31) - 1, 1ll << 32, (1ll << 33) - 1, 1ll << 33, (1ll << 33) + 1,
                              (1ll << 34) + 5, (1ll << 40) + 12345};
    const int32_t lens[] = {0, 1, 2, 45, 1 << 20, INT32_MAX - 1, INT32_MAX};
    for (int64_t a : firsts)
        for (int32_t len : lens) {
            skis::CoverItem x;
            x.set(a, a + len);
            if (x.first() != a || x.len() != len) std::printf("%lld %d\n", (long long)a, len);
        }
    std::puts("done");
}
""")
    assert out == "done\n"
