// The numbers of launches that share a place in the memory they meet in, for tests/test_slot_numbers.py.  Host code only.
#include <stdio.h>

#include "slot_map.h"

int main()
{
    // Numbers of eight bits.  Every launch reports itself at once; a place has 255 of them, and each number once.
    addrms_host::SlotMap<3, uint8_t> map;
    uint32_t done[3] = {};
    int launches[3] = {}, last[3] = {};
    for (int i = 0; i < 3 * 255; ++i) {
        const int u = map.take(1, done);
        if (u < 0 || static_cast<int>(map.number(u)) != last[u] + 1) return printf("launch %d: place %d\n", i, u), 1;
        last[u] = static_cast<int>(map.number(u));
        ++launches[u];
        done[u] = map.number(u);
    }
    for (int u = 0; u < 3; ++u)
        if (launches[u] != 255) return printf("place %d: %d launches\n", u, launches[u]), 1;
    if (map.take(1, done) != -1 || map.take(2, done) != -1) return printf("a number twice\n"), 1;

    // A place whose last launch, of two units, is in flight: the unit behind it is that launch's.
    addrms_host::SlotMap<3, uint8_t> wide;
    uint32_t ends[3] = {};
    for (int i = 0; i < 255; ++i) {
        const int u = wide.take(2, ends);
        if (u != 0) return printf("wide launch %d: %d\n", i, u), 1;
        if (i < 254) ends[0] = wide.number(0);
    }
    if (wide.take(1, ends) != 2 || wide.take(1, ends) != -1) return printf("units of a launch in flight\n"), 1;
    ends[0] = wide.number(0);
    if (wide.take(1, ends) != 1) return printf("the unit behind a place that is used up\n"), 1;
    printf("ok\n");
    return 0;
}
