// Which launches may use the same piece of the memory that workgroups meet in (slot_pool.h), on a HIP of a few lines
// (fake_hip), for tests/test_slot_pool.py.  Argument: the test; prints "ok".
#include <stdio.h>
#include <string.h>

#include "slot_pool.h"

using namespace addrms_host;

#define EXPECT(c) do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)

using Pool = SlotPool<8>;

static hipStream_t stream(size_t handle, int device)
{
    const hipStream_t s = reinterpret_cast<hipStream_t>(handle);
    fake_hip::device[s] = device;
    return s;
}

// A launch that is queued and does not end: the unit it has.
static int launch(Pool& pool, hipStream_t s)
{
    Pool::Lease lease;
    if (pool.take(s, 1, &lease) != Units::taken) return -1;
    lease.launched();
    return static_cast<int>(lease.unit());
}

// Launches on streams of one GPU, in flight together, with another GPU current at some of the calls.
static int devices()
{
    static Pool pool;
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

// A stream that is destroyed with its launch in flight, and another one that is created and gets the same handle.
static int handles()
{
    static Pool pool;
    const int first = launch(pool, stream(0x1000, 0));
    fake_hip::device.clear();
    const int second = launch(pool, stream(0x1000, 0));
    EXPECT(first >= 0 && second >= 0 && first != second);
    return 0;
}

// All units in flight: a call waits for one, for a bounded time, and after that nobody does until one has been free again.
static int waiting()
{
    static Pool pool;
    using clock = std::chrono::steady_clock;
    const auto ms = [](clock::time_point since) { return std::chrono::duration<double, std::milli>(clock::now() - since).count(); };
    const hipStream_t s = stream(0x1000, 0);
    Pool::Lease all;
    EXPECT(pool.take(s, 8, &all) == Units::taken);
    all.launched();
    clock::time_point t = clock::now();
    EXPECT(launch(pool, s) == -1 && ms(t) > 4.0);
    t = clock::now();
    for (int i = 0; i < 20; ++i) EXPECT(launch(pool, s) == -1);
    EXPECT(ms(t) < 60.0);                                    // 20 waits would be 80
    *all.done() = all.number();
    int got = -1;
    for (int trial = 0; trial < 50 && got < 0; ++trial) {    // a machine that is busy may end the launch too late
        Pool::Lease one;
        EXPECT(pool.take(s, 8, &one) == Units::taken);
        one.launched();
        std::thread ends([&] {
            std::this_thread::sleep_for(std::chrono::milliseconds(1));
            __atomic_store_n(one.done(), one.number(), __ATOMIC_SEQ_CST);
        });
        got = launch(pool, s);
        ends.join();
    }
    EXPECT(got >= 0);
    return 0;
}

// The null stream cannot be asked while another stream captures: no units, and no error is left, nor one of the caller's taken.
static int errors()
{
    static Pool pool;
    fake_hip::capturing.insert(stream(0x1000, 0));
    Pool::Lease lease;
    EXPECT(pool.take(nullptr, 1, &lease) == Units::none && hipPeekAtLastError() == hipSuccess);
    fake_hip::is(hipErrorInvalidHandle);
    EXPECT(pool.take(nullptr, 1, &lease) == Units::none && hipPeekAtLastError() != hipSuccess);
    fake_hip::capturing.clear();
    fake_hip::last = hipErrorInvalidHandle;
    EXPECT(pool.take(nullptr, 1, &lease) == Units::taken && hipPeekAtLastError() == hipErrorInvalidHandle);
    return 0;
}

// Units go back where nothing was launched, and once a launch has reported itself; a capturing stream has none.
static int leases()
{
    static Pool pool;
    const hipStream_t s = stream(0x1000, 0), capturing = stream(0x2000, 0);
    for (int i = 0; i < 100; ++i) {
        Pool::Lease lease;
        EXPECT(pool.take(s, 3, &lease) == Units::taken);
    }
    for (int i = 0; i < 100; ++i) {
        Pool::Lease lease;
        EXPECT(pool.take(hipStreamPerThread, 3, &lease) == Units::taken);
        lease.launched();
        *lease.done() = lease.number();
    }
    fake_hip::capturing.insert(capturing);
    Pool::Lease lease;
    EXPECT(pool.take(capturing, 1, &lease) == Units::capturing && pool.take(s, 8, &lease) == Units::taken);
    fake_hip::capturing.clear();
    return 0;
}

int main(int, char** argv)
{
    const struct { const char* name; int (*run)(); } tests[] = {{"devices", devices}, {"handles", handles}, {"leases", leases},
                                                                {"waiting", waiting}, {"errors", errors}};
    int bad = 1;
    for (const auto& t : tests)
        if (!strcmp(argv[1], t.name)) bad = t.run();
    if (!bad) printf("ok\n");
    return bad;
}
