// Free device blocks kept for later calls (capi.cpp's default allocator).
// Calls of the HIP runtime and the standard library only.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <stdint.h>

#include <map>
#include <mutex>
#include <unordered_map>
#include <vector>

namespace ax {
namespace {

// Stream of the calling device on which destroyed structures release their
// memory, after waiting for the build and every recorded use.
hipStream_t release_stream()
{
    static std::mutex mu;
    static hipStream_t streams[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)
        return nullptr;
    std::lock_guard<std::mutex> lock(mu);
    if (!streams[dev] && hipStreamCreateWithFlags(&streams[dev], hipStreamNonBlocking) != hipSuccess) {
        (void)hipGetLastError();
        streams[dev] = nullptr;
    }
    return streams[dev];
}

// Blocks of the default allocator that are free, kept for later calls.  A
// build and a query take and give back some thirty blocks, up to gigabytes;
// left to hipMallocAsync and hipFreeAsync, whose memory went back to the
// device and was mapped again, a build and CSR query at 10^7 points took
// 84 ms for 7 ms of kernels, and 10^6 box overlaps 5.3 ms for 0.8 ms.
//
// A block is freed with an event on the stream that had its last use (one
// event for all the blocks of a call).  It goes to a later allocation for that
// stream, which waits for the event on the device, or for any stream once the
// event has completed; never to work that could overlap its last use, and
// nothing waits for another stream's work where memory is left.  What is kept is bounded by a quarter of the device's memory, the
// longest unused given back first, and all of it is given back when an
// allocation fails or the caller installs an allocator or names the default.  While a stream is
// being captured its allocations and releases pass the cache by.
struct FreeGroup {
    hipEvent_t done = nullptr;  // NULL: complete
    int dev = 0;                // the event's device
    hipStream_t on = nullptr;   // the stream that recorded it
    int blocks = 0;             // free blocks that refer to the group
};
struct CachedBlock {
    void *p = nullptr;
    size_t bytes = 0;
    int dev = 0;
    FreeGroup *group = nullptr;
    uint64_t age = 0;
};
std::mutex g_cache_mu;
std::unordered_map<void *, CachedBlock> g_live_blocks;
std::multimap<size_t, CachedBlock> g_free_blocks[64];
size_t g_free_bytes[64] = {};
size_t g_cache_limit[64] = {};
uint64_t g_cache_age = 0;
std::vector<hipEvent_t> g_event_pool[64];  // by the device an event was created on, the only one that records it

bool is_capturing(hipStream_t s)
{
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    return hipStreamIsCapturing(s, &cs) == hipSuccess && cs != hipStreamCaptureStatusNone;
}

// Lets this thread query events while another thread captures a graph.
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

bool group_complete(FreeGroup *g)
{
    if (!g->done)
        return true;
    RelaxedCapture relaxed;
    if (hipEventQuery(g->done) != hipSuccess) {
        (void)hipGetLastError();  // "not ready" must not surface as a later call's error
        return false;
    }
    g_event_pool[g->dev].push_back(g->done);
    g->done = nullptr;
    return true;
}

void group_leave(FreeGroup *g)
{
    if (--g->blocks == 0) {
        if (g->done)  // an event may be recorded again while waits on its earlier record are queued
            g_event_pool[g->dev].push_back(g->done);
        delete g;
    }
}

// Give a cached block back to the device, after its last use.
void give_back(CachedBlock &b, bool wait)
{
    hipStream_t rs = release_stream();
    if (b.group->done) {
        if (wait || !rs)
            (void)hipEventSynchronize(b.group->done);
        else
            (void)hipStreamWaitEvent(rs, b.group->done, 0);
    }
    (void)hipFreeAsync(b.p, rs);
    group_leave(b.group);
}

// Give back the longest unused blocks of a device until at most `keep` bytes
// stay (g_cache_mu held, dev the current device).
void trim_cache(int dev, size_t keep, bool wait)
{
    auto &blocks = g_free_blocks[dev];
    while (g_free_bytes[dev] > keep && !blocks.empty()) {
        auto oldest = blocks.begin();
        for (auto it = blocks.begin(); it != blocks.end(); ++it)
            if (it->second.age < oldest->second.age)
                oldest = it;
        g_free_bytes[dev] -= oldest->second.bytes;
        give_back(oldest->second, wait);
        blocks.erase(oldest);
    }
    if (wait) {
        hipStream_t rs = release_stream();
        (void)hipStreamSynchronize(rs);
        hipMemPool_t pool;
        if (hipDeviceGetDefaultMemPool(&pool, dev) == hipSuccess)
            (void)hipMemPoolTrimTo(pool, 0);
        (void)hipGetLastError();
    }
}

// A free block of at least `bytes` (and not much more) for work on s, or NULL.
void *cache_take(int dev, size_t bytes, hipStream_t s)
{
    std::lock_guard<std::mutex> lock(g_cache_mu);
    auto &blocks = g_free_blocks[dev];
    const size_t most = bytes + bytes / 4 + 4096;
    auto found = blocks.end();
    for (int pass = 0; pass < 2 && found == blocks.end(); ++pass)
        for (auto it = blocks.lower_bound(bytes); it != blocks.end() && it->first <= most; ++it) {
            FreeGroup *g = it->second.group;
            if (pass == 0 ? g->on == s : group_complete(g)) {
                found = it;
                break;
            }
        }
    if (found == blocks.end())
        return nullptr;
    CachedBlock b = found->second;
    // on the stream that recorded it this costs nothing; it is never left out,
    // because a stream's handle may be given to a new stream
    if (b.group->done && hipStreamWaitEvent(s, b.group->done, 0) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    blocks.erase(found);
    g_free_bytes[dev] -= b.bytes;
    group_leave(b.group);
    b.group = nullptr;
    g_live_blocks[b.p] = b;
    return b.p;
}

// What may be kept on the current device.
size_t cache_limit(int dev)
{
    if (!g_cache_limit[dev]) {
        RelaxedCapture relaxed;
        size_t avail = 0, total = 0;
        if (hipMemGetInfo(&avail, &total) != hipSuccess) {
            (void)hipGetLastError();
            total = (size_t)4 << 30;
        }
        g_cache_limit[dev] = total / 4 + 1;
    }
    return g_cache_limit[dev];
}

void flush_cache()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess)
        return;
    std::lock_guard<std::mutex> lock(g_cache_mu);
    for (int d = 0; d < 64; ++d)
        if (!g_free_blocks[d].empty() && hipSetDevice(d) == hipSuccess)
            trim_cache(d, 0, true);
    (void)hipSetDevice(dev);
}

// Remember a block of the device.
void cache_note(void *p, size_t bytes, int dev)
{
    std::lock_guard<std::mutex> lock(g_cache_mu);
    CachedBlock b;
    b.p = p;
    b.bytes = bytes;
    b.dev = dev;
    g_live_blocks[p] = b;
}

// Keep blocks that are free after the work queued on s so far, or after `done`
// (owned by this call; then no call is made on s, which may be gone).
void cache_release(const std::vector<void *> &ptrs, hipStream_t s, hipEvent_t done)
{
    std::vector<CachedBlock> mine;
    const bool capturing = !ptrs.empty() && !done && is_capturing(s);
    std::lock_guard<std::mutex> lock(g_cache_mu);
    for (void *p : ptrs) {
        CachedBlock b;
        auto it = g_live_blocks.find(p);
        if (it != g_live_blocks.end()) {
            b = it->second;
            g_live_blocks.erase(it);
        }
        if (!b.p || capturing)
            (void)hipFreeAsync(p, s);
        else
            mine.push_back(b);
    }
    if (mine.empty()) {
        if (done)
            (void)hipEventDestroy(done);
        return;
    }
    int cur = -1;
    if (hipGetDevice(&cur) != hipSuccess || cur < 0 || cur >= 64)
        cur = 0;
    FreeGroup *g = new FreeGroup();
    g->dev = done ? mine[0].dev : cur;
    g->on = s;
    hipEvent_t e = done;
    if (!e && !g_event_pool[cur].empty()) {
        e = g_event_pool[cur].back();
        g_event_pool[cur].pop_back();
    } else if (!e && hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
        (void)hipGetLastError();
        e = nullptr;
    }
    if (e && (done || hipEventRecord(e, s) == hipSuccess)) {
        g->done = e;
    } else {
        (void)hipGetLastError();
        if (e)
            (void)hipEventDestroy(e);  // not to be met by the next release
        (void)hipStreamSynchronize(s);
    }
    bool touched[64] = {};
    for (CachedBlock &b : mine) {
        b.group = g;
        b.age = ++g_cache_age;
        ++g->blocks;
        g_free_bytes[b.dev] += b.bytes;
        g_free_blocks[b.dev].emplace(b.bytes, b);
        touched[b.dev] = true;
    }
    for (int d = 0; d < 64; ++d)  // blocks may be of another device than the current one
        if (touched[d] && (d == cur || hipSetDevice(d) == hipSuccess)) {
            trim_cache(d, cache_limit(d), false);
            if (d != cur)
                (void)hipSetDevice(cur);
        }
}

}  // namespace
}  // namespace ax
