// A HIP runtime that runs on the CPU, for the library's host code alone.  Streams are queues; a queue that is
// `held` runs only as far as a wait makes it, every other one at once, so that whatever the calls do not order
// happens in the worst order.  A launch compares the pointer table that it was given with the one that the
// caller meant.  Copies, launches, events and waits are queue entries; memory is malloc's, so that a table freed
// under a queued launch is for the address sanitizer to find.
#ifndef FAKE_HIP_H
#define FAKE_HIP_H

#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <memory>
#include <utility>
#include <vector>

#include "kt_internal.h"

namespace fake {

struct Event;
struct Op {
    enum Kind { COPY, LAUNCH, RECORD, WAIT, WORK } kind;
    void *dst;
    const void *src;
    size_t n;                        // bytes of a copy
    std::vector<uint64_t> want;      // table that a launch should find at `src`
    Event *ev;
    uint64_t version;
};
struct Stream {
    std::deque<Op> q;
    uint64_t id = 0;
    bool held = false, capturing = false, invalidated = false;
};
struct Event {
    uint64_t asked = 0, done = 0;    // records issued, records passed
    Stream *on = nullptr;
};
struct Handle { Stream *cur = nullptr; };

inline std::vector<std::unique_ptr<Stream>> all;
inline std::vector<std::unique_ptr<Event>> events;
inline std::vector<std::unique_ptr<Handle>> handles;
inline std::vector<Handle *> free_handles;
inline std::vector<uint64_t> want;               // table that the next launch is meant to read
inline std::vector<Op> recorded;                 // launches under capture
inline int wrong = 0, launched = 0, device_syncs = 0, stream_syncs = 0, work_done = 0;
inline bool destroy_drains = true;

inline Stream *new_stream()
{
    static uint64_t next = 1;
    all.emplace_back(new Stream);
    all.back()->id = next++;
    return all.back().get();
}
inline Stream *null_stream()
{
    static Stream *s = new_stream();
    return s;
}
inline Stream *of(hipStream_t h)
{
    if (!h) return null_stream();
    if (h == hipStreamPerThread) {
        static thread_local Stream *mine = new_stream();
        return mine;
    }
    return reinterpret_cast<Handle *>(h)->cur;
}

inline void run(Stream &s, bool force, const Event *until = nullptr, uint64_t version = 0)
{
    while (!s.q.empty() && !(until && until->done >= version)) {
        Op &op = s.q.front();
        if (op.kind == Op::WAIT && op.ev->done < op.version) {
            if (!force) return;
            run(*op.ev->on, true, op.ev, op.version);
        }
        switch (op.kind) {
        case Op::COPY: memcpy(op.dst, op.src, op.n); break;
        case Op::LAUNCH:
            if (memcmp(op.src, op.want.data(), op.want.size() * 8) != 0) ++wrong;
            break;
        case Op::RECORD: op.ev->done = op.version; break;
        case Op::WORK: ++work_done; break;
        case Op::WAIT: break;
        }
        s.q.pop_front();
    }
}
inline void pump()
{
    for (auto &s : all)
        if (!s->held) run(*s, false);
}
inline void push(Stream *s, Op op)
{
    s->q.push_back(std::move(op));
    pump();
}
inline void finish()
{
    for (auto &s : all) s->held = false;
    for (auto it = all.rbegin(); it != all.rend(); ++it) run(**it, true);
}
// Waiting for anything of a stream under capture, or for the device, ends the capture; so do waits for other streams
// (but the null stream) and allocations, unless the thread has exchanged its mode for the relaxed one.
inline thread_local hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
inline bool breaks_capture(Stream *s)
{
    bool broken = false;
    for (auto &x : all)
        if (x->capturing && (!s || x.get() == s || (mode != hipStreamCaptureModeRelaxed && s != null_stream())))
            x->invalidated = broken = true;
    return broken;
}
inline hipError_t last = hipSuccess;             // what a launch reports
inline bool refused()
{
    bool any = false;
    if (mode != hipStreamCaptureModeRelaxed)
        for (auto &x : all)
            if (x->capturing) x->invalidated = any = true;
    return any;
}
inline void begin_capture(hipStream_t s) { of(s)->capturing = true; }
inline bool end_capture(hipStream_t s)
{
    of(s)->capturing = false;
    return !of(s)->invalidated;
}

inline hipStream_t create()
{
    Handle *h;
    if (!free_handles.empty()) {
        h = free_handles.back();          // the handle of the stream destroyed last
        free_handles.pop_back();
    } else {
        handles.emplace_back(new Handle);
        h = handles.back().get();
    }
    h->cur = new_stream();
    return reinterpret_cast<hipStream_t>(h);
}
inline void destroy(hipStream_t st)
{
    Handle *h = reinterpret_cast<Handle *>(st);
    if (destroy_drains) run(*h->cur, true);
    h->cur = nullptr;                     // otherwise what is queued runs later
    free_handles.push_back(h);
}
inline void work(hipStream_t st) { push(of(st), Op{Op::WORK, nullptr, nullptr, 0, {}, nullptr, 0}); }

}  // namespace fake

extern "C" {
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 100000; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError(void) { return std::exchange(fake::last, hipSuccess); }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *m) { std::swap(*m, fake::mode); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = fake::create(); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { fake::destroy(s); return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n)
{
    *p = nullptr;
    if (fake::refused()) return hipErrorStreamCaptureUnsupported;
    *p = calloc(1, n);
    return hipSuccess;
}
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st)
{
    fake::push(fake::of(st), fake::Op{fake::Op::COPY, d, s, n, {}, nullptr, 0});
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    fake::events.emplace_back(new fake::Event);
    *e = reinterpret_cast<hipEvent_t>(fake::events.back().get());
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t st)
{
    fake::Event *ev = reinterpret_cast<fake::Event *>(e);
    ev->on = fake::of(st);
    fake::push(ev->on, fake::Op{fake::Op::RECORD, nullptr, nullptr, 0, {}, ev, ++ev->asked});
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e)
{
    fake::Event *ev = reinterpret_cast<fake::Event *>(e);
    if (!ev->on) return hipSuccess;
    if (fake::breaks_capture(ev->on)) return hipErrorCapturedEvent;
    fake::run(*ev->on, true, ev, ev->asked);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t st, hipEvent_t e, unsigned)
{
    fake::Event *ev = reinterpret_cast<fake::Event *>(e);
    fake::push(fake::of(st), fake::Op{fake::Op::WAIT, nullptr, nullptr, 0, {}, ev, ev->asked});
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t st)
{
    ++fake::stream_syncs;
    fake::Stream *s = fake::of(st);
    if (!s) return hipSuccess;           // a destroyed stream: no error, no wait
    if (fake::breaks_capture(s)) return hipErrorStreamCaptureUnsupported;
    fake::run(*s, true);
    return hipSuccess;
}
#ifdef FAKE_STREAM_IDS                   // newer runtimes have it
hipError_t hipStreamGetId(hipStream_t st, unsigned long long *id)
{
    fake::Stream *s = fake::of(st);
    if (!s) return hipErrorInvalidHandle;
    *id = s->id;
    return hipSuccess;
}
#endif
hipError_t hipDeviceSynchronize(void)
{
    ++fake::device_syncs;
    if (fake::breaks_capture(nullptr)) return hipErrorStreamCaptureUnsupported;
    for (auto &s : fake::all) fake::run(*s, true);
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t st, hipStreamCaptureStatus *c)
{
    fake::Stream *s = fake::of(st);
    if (!st)                                      // the streams here are ones that the null stream waits for
        for (auto &x : fake::all)
            if (x->capturing) return fake::last = hipErrorStreamCaptureImplicit;
    *c = s && s->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
}

int kt_launch_pack(const KtDeviceTables &, kt_dtype, int64_t, int64_t, const void *const *table, void *const *, void *stream)
{
    ++fake::launched;
    fake::Stream *s = fake::of(static_cast<hipStream_t>(stream));
    fake::Op op{fake::Op::LAUNCH, nullptr, table, 0, fake::want, nullptr, 0};
    if (s->capturing) fake::recorded.push_back(op); else fake::push(s, op);
    return (int)hipGetLastError();
}
int kt_launch_unpack(const KtDeviceTables &, kt_dtype, int64_t, int64_t, const void *const *, float, void *const *, void *) { return 0; }
int kt_launch_reduce(const KtDeviceTables &, kt_dtype, int64_t, int64_t, const void *const *, int, const KtWeights &, void *const *, void *) { return 0; }
int kt_launch_fused(const KtDeviceTables &, kt_dtype, int64_t, int64_t, const void *const *, const void *const *, int, const KtWeights &, float, void *const *, void *) { return 0; }
int kt_launch_unpack_sgd(const KtDeviceTables &, kt_dtype, int64_t, int64_t, const void *const *, void *const *, void *const *, void *const *, const KtSgd &, void *) { return 0; }
int kt_launch_fused_sgd(const KtDeviceTables &, kt_dtype, int64_t, int64_t, const void *const *, const void *const *, int, const KtWeights &, void *const *, void *const *, void *const *, const KtSgd &, void *) { return 0; }

#endif
