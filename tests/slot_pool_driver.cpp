// Which launches may use the same piece of the memory that workgroups meet in (slot_pool.h), on a HIP of a few lines
// (fake_hip), for tests/test_slot_pool.py.  Argument: the test; prints "ok".
#include <stdio.h>
#include <string.h>

#include "slot_pool.h"

using namespace addrms_host;

#define EXPECT(c) do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)

static hipStream_t stream(size_t handle, int device)
{
    const hipStream_t s = reinterpret_cast<hipStream_t>(handle);
    fake_hip::device[s] = device;
    return s;
}

// A launch that is queued and does not end: the slot it has.
static int launch(SlotPool& pool, hipStream_t s)
{
    SlotPool::Lease lease;
    if (!pool.take(s, &lease)) return -1;
    lease.launched();
    return static_cast<int>(lease.slot());
}

// Launches on streams of one GPU, in flight together, with another GPU current at some of the calls.
static int devices()
{
    static SlotPool pool;
    const hipStream_t a = stream(0x1000, 1), b = stream(0x2000, 1);
    fake_hip::current = 0;
    const int first = launch(pool, a);
    EXPECT(first >= 0);
    fake_hip::current = 1;
    const int second = launch(pool, b);
    EXPECT(second >= 0 && second != first);
    const int third = launch(pool, nullptr);                 // GPU 1's null stream
    EXPECT(third >= 0 && third != first && third != second);
    fake_hip::current = 0;
    EXPECT(launch(pool, nullptr) >= 0);                      // GPU 0's
    return 0;
}

int main(int, char** argv)
{
    const int bad = !strcmp(argv[1], "devices") ? devices() : 1;
    if (!bad) printf("ok\n");
    return bad;
}
