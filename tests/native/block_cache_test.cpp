// The cache of free device blocks over a model of the HIP runtime: two devices,
// streams whose work ends when the test says so, events bound to the device
// they were created on.  block_cache_test NAME runs one case.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>

#include "../../paper_2507_23700_amd/csrc/block_cache.hpp"

struct ihipStream_t {
    int dev;
    long queued = 0, done = 0;
    std::vector<hipEvent_t> waits;
};
struct ihipEvent_t {
    int dev;
    hipStream_t on = nullptr;
    long at = 0;
};

namespace {
thread_local int t_dev = 0;
thread_local hipStreamCaptureMode t_mode = hipStreamCaptureModeGlobal;
bool g_other_captures = false;  // another thread captures a graph, in global mode
int g_synced = 0, g_destroyed = 0;
size_t g_total = 1000 << 20;
struct Freed {
    void *p;
    int dev;  // of the stream
};
std::vector<Freed> g_freed;
bool forbidden() { return g_other_captures && t_mode != hipStreamCaptureModeRelaxed; }
}  // namespace

extern "C" {
hipError_t hipGetDevice(int *d) { *d = t_dev; return hipSuccess; }
hipError_t hipSetDevice(int d) { t_dev = d; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *m) { std::swap(*m, t_mode); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = new ihipStream_t{t_dev}; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { ++g_synced; s->done = s->queued; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) { s->waits.push_back(e); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = new ihipEvent_t{t_dev}; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { ++g_destroyed; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    if (e->dev != s->dev)
        return hipErrorInvalidHandle;
    e->on = s;
    e->at = ++s->queued;
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e)
{
    if (forbidden())
        return hipErrorStreamCaptureUnsupported;
    return !e->on || e->on->done >= e->at ? hipSuccess : hipErrorNotReady;
}
hipError_t hipEventSynchronize(hipEvent_t e)
{
    if (e->on && e->on->done < e->at)
        e->on->done = e->at;
    return hipSuccess;
}
hipError_t hipFreeAsync(void *p, hipStream_t s) { g_freed.push_back({p, s ? s->dev : -1}); return hipSuccess; }
hipError_t hipMemGetInfo(size_t *avail, size_t *total)
{
    if (forbidden())
        return hipErrorStreamCaptureUnsupported;
    *avail = *total = g_total >> t_dev;  // the second device has half the memory
    return hipSuccess;
}
hipError_t hipDeviceGetDefaultMemPool(hipMemPool_t *, int) { return hipErrorNotSupported; }
hipError_t hipMemPoolTrimTo(hipMemPool_t, size_t) { return hipSuccess; }
}

using namespace ax;

namespace {
int g_failed = 0;
#define CHECK(x)                                                      \
    do {                                                              \
        if (!(x)) {                                                   \
            std::printf("%s:%d: %s\n", __FILE__, __LINE__, #x);      \
            ++g_failed;                                               \
        }                                                             \
    } while (0)

hipStream_t stream_on(int dev)
{
    hipStream_t s = nullptr;
    const int before = t_dev;
    t_dev = dev;
    (void)hipStreamCreateWithFlags(&s, 0);
    t_dev = before;
    return s;
}
void *block(size_t bytes, int dev)
{
    void *p = std::malloc(1);
    cache_note(p, bytes, dev);
    return p;
}

// Two devices in turn: an event of one is never recorded on the other, which
// fails, and the release would then wait for its stream.
void events_by_device()
{
    hipStream_t s[2] = {stream_on(0), stream_on(1)};
    for (int round = 0; round < 6; ++round) {
        void *p[2];
        for (int d = 0; d < 2; ++d) {
            t_dev = d;
            p[d] = cache_take(d, 4096, s[d]);
            if (!p[d])
                p[d] = block(4096, d);
        }
        for (int d = 0; d < 2; ++d) {
            t_dev = d;
            cache_release({p[d]}, s[d], nullptr);
            s[d]->done = s[d]->queued;
        }
    }
    CHECK(g_synced == 0);
    CHECK(g_freed.empty());
}

// A block whose last use is still to come on another stream makes no one wait
// while there is a finished one, or other memory.
void unfinished_elsewhere()
{
    hipStream_t a = stream_on(0), b = stream_on(0);
    void *p = block(8192, 0);
    cache_release({p}, b, nullptr);  // taken for a, read last by work on b that goes on
    CHECK(cache_take(0, 8192, a) == nullptr);
    CHECK(a->waits.empty());
    void *q = block(8192, 0);
    cache_release({q}, b, nullptr);
    b->done = b->queued - 1;  // p's use has ended, q's has not
    CHECK(cache_take(0, 8192, a) == p);
    CHECK(cache_take(0, 8192, a) == nullptr);
    CHECK(cache_take(0, 8192, b) == q);  // b's own work is in order
    CHECK(a->waits.empty());
    CHECK(b->waits.size() == 1);
    CHECK(g_synced == 0 && g_freed.empty());
}

// Blocks of a device that is not the current one when they are freed keep that
// device's bound, and go back on a stream of theirs.
void other_device_is_trimmed()
{
    hipStream_t s = stream_on(0);
    t_dev = 0;
    const size_t bytes = (size_t)25 << 20;  // device 1 has 500 MiB: 125 may stay
    for (int i = 0; i < 8; ++i)
        cache_release({block(bytes, 1)}, s, nullptr);
    CHECK(t_dev == 0);
    CHECK(g_free_bytes[1] <= (size_t)126 << 20 && g_free_bytes[1] >= (size_t)100 << 20);
    CHECK(g_freed.size() >= 3);
    for (const Freed &f : g_freed)
        CHECK(f.dev == 1);
}
}  // namespace

int main(int argc, char **argv)
{
    const std::string name = argc > 1 ? argv[1] : "";
    if (name == "events_by_device")
        events_by_device();
    else if (name == "unfinished_elsewhere")
        unfinished_elsewhere();
    else if (name == "other_device_is_trimmed")
        other_device_is_trimmed();
    else
        return 2;
    return g_failed ? 1 : 0;
}
