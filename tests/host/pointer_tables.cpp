// The library's pointer tables on streams, threads and destroyed streams (fake_hip.h).  usage: pointer_tables CASE
#include <thread>

#include "fake_hip.h"

static const int KEPT = 8;          // tables that a plan keeps
static const int T = 3;

#define CHECK(x)                                                        \
    do {                                                                \
        if (!(x)) { printf("line %d: %s\n", __LINE__, #x); exit(1); }   \
    } while (0)

struct Plan {
    kt_plan *p = nullptr;
    Plan()
    {
        const int64_t numel[T] = {40, 7, 100};
        CHECK(kt_plan_create(numel, T, KT_F32, 0, 16, &p) == KT_OK);
    }
    ~Plan() { CHECK(kt_plan_destroy(p) == KT_OK); }
    // one call with the pointers of set `set`
    kt_status pack(int set, hipStream_t s)
    {
        const void *t[T];
        void *b = reinterpret_cast<void *>(0x900000000ull + (uint64_t)set * 4096);
        fake::want.assign(T + 1, reinterpret_cast<uintptr_t>(b));
        for (int i = 0; i < T; ++i) {
            t[i] = reinterpret_cast<const void *>(0x100000000ull + (uint64_t)set * 4096 + (uint64_t)i * 512);
            fake::want[(size_t)i] = reinterpret_cast<uintptr_t>(t[i]);
        }
        return kt_bucket_pack(p, KT_ALL_BUCKETS, t, &b, s);
    }
    void call(int set, hipStream_t s) { CHECK(pack(set, s) == KT_OK); }
};
template <typename F> static void in_thread(F f) { std::thread(f).join(); }
static void end(int launches)
{
    fake::finish();
    CHECK(fake::launched == launches);
    CHECK(fake::wrong == 0);
}

// hipStreamPerThread names another stream in every thread: a table that one thread's stream is still uploading is
// not read by another's
static void per_thread_hit()
{
    Plan p;
    fake::of(hipStreamPerThread)->held = true;
    p.call(0, hipStreamPerThread);
    in_thread([&] { p.call(0, hipStreamPerThread); });
    end(2);
}
static void per_thread_eviction()
{
    Plan p;
    fake::of(hipStreamPerThread)->held = true;
    for (int r = 0; r < KEPT; ++r) p.call(r, hipStreamPerThread);
    in_thread([&] { for (int r = 0; r < 2 * KEPT; ++r) p.call(100 + r, hipStreamPerThread); });
    for (int r = 0; r < KEPT; ++r) p.call(r, hipStreamPerThread);
    end(4 * KEPT);
}
// one thread on its per-thread stream is one stream: new pointers on every call wait for no device
static void per_thread_new_pointers()
{
    Plan p;
    fake::of(hipStreamPerThread)->held = true;
    for (int r = 0; r < 8 * KEPT; ++r) p.call(r, hipStreamPerThread);
    CHECK(fake::device_syncs == 0 && fake::stream_syncs == 0);
    end(8 * KEPT);
}

// A stream destroyed with its launches queued, and a new one at the same handle: the new one's uploads are not
// ordered behind those launches, nor its launches behind the old one's uploads.  Without stream ids the runtime
// drains a stream that it destroys.
static void destroyed_stream(bool drains)
{
    fake::destroy_drains = drains;
    Plan p;
    hipStream_t a = fake::create();
    fake::of(a)->held = true;
    for (int r = 0; r < KEPT; ++r) p.call(r, a);
    fake::destroy(a);
    hipStream_t b = fake::create();
    CHECK(a == b);
    for (int r = 0; r < 2 * KEPT; ++r) p.call(r < 3 ? r + 1 : 100 + r, b);      // some of the old pointers, then new ones
    end(3 * KEPT);
}
static void destroyed_stream_undrained() { destroyed_stream(false); }
static void destroyed_stream_drained() { destroyed_stream(true); }
// the stream behind a later table's upload is not the one of the launch that is waited for
static void destroyed_stream_later_upload()
{
    fake::destroy_drains = false;
    Plan p;
    hipStream_t a = fake::create(), c = fake::create();
    fake::of(a)->held = true;
    for (int r = 0; r < KEPT - 1; ++r) p.call(r, a);
    fake::destroy(a);
    hipStream_t b = fake::create();
    CHECK(a == b);
    p.call(50, b);
    for (int r = 0; r < 2 * KEPT; ++r) p.call(100 + r, c);
    end(3 * KEPT);
}

// Two streams with new pointers: from the second round on, what one stream's program has queued behind its launches
// is not waited for when the other takes its tables.
static void other_streams_queue()
{
    Plan p;
    hipStream_t a = fake::create(), b = fake::create();
    fake::of(a)->held = true;
    int calls = 0;
    for (int round = 0; round < 3; ++round) {
        for (int r = 0; r < 8; ++r, ++calls) p.call(r % 4, a);      // every table again after the last upload
        for (int r = 0; r < 4; ++r, ++calls) p.call(3, a);
        fake::work(a);
        for (int r = 0; r < KEPT - 1; ++r, ++calls) p.call(100 * (round + 1) + r, b);      // all but a's last
        CHECK(round == 0 || fake::work_done <= round);
    }
    CHECK(fake::device_syncs == 0);
    end(calls);
}
// one stream alone: no event but the uploads'
static void one_stream_marks_nothing()
{
    Plan p;
    hipStream_t a = fake::create();
    for (int r = 0; r < 4 * KEPT; ++r) p.call(r, a);
    const size_t n = fake::events.size();
    for (int r = 0; r < 4 * KEPT; ++r) p.call(r % 3, a);
    CHECK(n == (size_t)KEPT && fake::events.size() == n);
    CHECK(fake::device_syncs == 0 && fake::stream_syncs == 0);
    end(8 * KEPT);
}

// A call recorded after the same call was made on the stream that is captured, on another one, on the null
// stream; the recorded launch runs before anything else that is queued.
static void recorded_after(int where)
{
    Plan p;
    hipStream_t a = fake::create(), b = fake::create();
    hipStream_t eager = where == 0 ? a : where == 1 ? b : nullptr;
    fake::of(eager)->held = true;
    for (int r = 0; r < 3; ++r) p.call(r, eager);
    fake::begin_capture(a);
    for (int r = 0; r < 3; ++r) p.call(r, a);
    CHECK(fake::end_capture(a));
    CHECK(fake::recorded.size() == 3);
    for (const fake::Op &op : fake::recorded) fake::push(fake::of(fake::create()), op);
    for (int r = 0; r < 2 * KEPT; ++r) p.call(100 + r, b);
    end(6 + 2 * KEPT);
}
static void recorded_after_captured_stream() { recorded_after(0); }
static void recorded_after_other_stream() { recorded_after(1); }
static void recorded_after_null_stream() { recorded_after(2); }

// New pointers on one stream while another, which used some of the tables last, is being captured
static void new_pointers_beside_a_capture()
{
    Plan p;
    hipStream_t a = fake::create(), b = fake::create();
    fake::of(a)->held = true;
    for (int r = 0; r < 2 * KEPT - 3; ++r) p.call(r, r < KEPT ? b : a);      // 5 tables of a, 3 of b
    fake::begin_capture(a);
    p.call(2 * KEPT - 4, a);
    for (int r = 0; r < 3 * KEPT; ++r) p.call(100 + r, b);
    CHECK(fake::end_capture(a));
    for (int r = 0; r < KEPT; ++r) p.call(200 + r, a);
    fake::begin_capture(a);
    CHECK(p.pack(300, b) == KT_EUNSUPPORTED);
    CHECK(fake::end_capture(a));
    p.call(300, b);
    end(2 * KEPT - 3 + 1 + 3 * KEPT + KEPT + 1);
}

int main(int argc, char **argv)
{
    const struct { const char *name; void (*run)(); } cases[] = {
        {"per_thread_hit", per_thread_hit},
        {"per_thread_eviction", per_thread_eviction},
        {"per_thread_new_pointers", per_thread_new_pointers},
        {"other_streams_queue", other_streams_queue},
        {"one_stream_marks_nothing", one_stream_marks_nothing},
        {"recorded_after_captured_stream", recorded_after_captured_stream},
        {"recorded_after_other_stream", recorded_after_other_stream},
        {"recorded_after_null_stream", recorded_after_null_stream},
        {"new_pointers_beside_a_capture", new_pointers_beside_a_capture},
        {"destroyed_stream_undrained", destroyed_stream_undrained},
        {"destroyed_stream_drained", destroyed_stream_drained},
        {"destroyed_stream_later_upload", destroyed_stream_later_upload},
    };
    for (const auto &c : cases)
        if (argc > 1 && strcmp(argv[1], c.name) == 0) {
            c.run();
            printf("ok\n");
            return 0;
        }
    printf("no such case\n");
    return 2;
}
