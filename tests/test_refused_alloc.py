"""A device buffer whose allocation is refused is empty afterwards: scratch that is kept between calls
is judged by its size, so a size without memory behind it would be written through a null pointer by
the next call."""
import host_unit


@host_unit.needs_hipcc
def test_refused_buffer_is_empty():
    out = host_unit.run(r"""
#include <cstdio>
#include <cstdlib>
#include "skis_query.h"
namespace skis { // an arena of host memory that gives out blocks of up to 1000 bytes
void *Arena::alloc(size_t bytes)
{
    if (bytes > 1000) throw Error{SKIS_ENOMEM, "no"};
    used += bytes;
    return std::malloc(bytes);
}
void Arena::release(void *p, size_t bytes)
{
    used -= bytes;
    std::free(p);
}
void Arena::trim(bool) {}
Arena::~Arena() {}
}
int main()
{
    skis::Arena a;
    skis::DevBuf<uint32_t> b;
    b.alloc(a, 250);
    if (!b.ptr || b.count != 250 || a.used != 1000) std::puts("alloc");
    for (int i = 0; i < 2; ++i) {
        try {
            b.alloc(a, 251);
            std::puts("not refused");
        } catch (const skis::Error &) {
        }
        if (b.ptr || b.count != 0 || b.bytes() != 0 || a.used != 0) std::puts("left over");
    }
    b.alloc(a, 0);
    if (!b.ptr || b.count != 0) std::puts("none");
    std::puts("done");
}
""")
    assert out == "done\n"
