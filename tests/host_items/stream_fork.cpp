// Host check of StreamFork (stream_fork.hpp) against a stand-in for the HIP stream
// calls that records them and fails where told to.  Prints one line per case: name,
// streams had, whether an error was left behind, join's code, waits of the caller's
// stream, synchronisations.
#include <cstdio>
#include <cstring>

typedef struct ihipStream_t *hipStream_t;
typedef struct ihipEvent_t *hipEvent_t;
enum hipError_t { hipSuccess = 0, hipErrorUnknown = 999 };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone, hipStreamCaptureStatusActive };
enum hipStreamCaptureMode { hipStreamCaptureModeGlobal, hipStreamCaptureModeRelaxed = 2 };
constexpr unsigned hipEventDisableTiming = 2, hipStreamNonBlocking = 1;

static hipError_t last;
static hipStream_t const caller = (hipStream_t)0x10;
static int made, side_waits, caller_waits, syncs, fail_side_wait, fail_record, fail_create;
static bool capturing;
static hipError_t set(bool bad)
{
    if (bad) last = hipErrorUnknown;
    return bad ? hipErrorUnknown : hipSuccess;
}
static hipError_t hipGetLastError() { hipError_t e = last; last = hipSuccess; return e; }
static hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    *e = (hipEvent_t)(size_t)(0x1000 + ++made);
    return set(fail_create && made >= fail_create);
}
static hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    *s = (hipStream_t)(size_t)(0x1000 + ++made);
    return set(fail_create && made >= fail_create);
}
static hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }
static hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *c)
{
    *c = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
static hipError_t hipEventRecord(hipEvent_t, hipStream_t s)
{
    return set(s != caller && fail_record);
}
static hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t, unsigned)
{
    if (s == caller) return ++caller_waits, hipSuccess;
    return set(++side_waits == fail_side_wait);
}
static hipError_t hipStreamSynchronize(hipStream_t) { return ++syncs, hipSuccess; }

#include "stream_fork.hpp"

using namespace ptf;

static SideSets sets[8];

static void run(const char *name, SideSets *x, int want)
{
    side_waits = caller_waits = syncs = 0;
    last = hipSuccess;
    int n, rc;
    {
        StreamFork f(x, caller, want);
        n = f.count();
        for (int k = 1; k < n; ++k)
            if (f.stream(k) == caller || f.stream(k) == f.stream(k - 1)) n = -1;
        const bool left = last != hipSuccess;
        last = hipSuccess;
        rc = f.join();
        printf("%s %d %d %d %d %d\n", name, n, (int)left, rc, caller_waits, syncs);
    }
}

int main()
{
    run("all", &sets[0], 4);
    run("again", &sets[0], 9);
    run("two", &sets[0], 2);
    run("one", nullptr, 1);
    capturing = true;
    run("capture", &sets[0], 4);
    capturing = false;
    fail_side_wait = 2;
    run("second_wait", &sets[0], 4);
    fail_side_wait = 1;
    run("first_wait", &sets[0], 4);
    fail_side_wait = 0;
    fail_record = 1;
    run("join", &sets[0], 4);
    fail_record = 0;
    fail_create = made + 3;
    run("create", &sets[1], 4);
    run("create_again", &sets[1], 4);
    fail_create = 0;
    run("after", &sets[0], 4);
    return 0;
}
