// Test program (CPU only): the batched accept of host matchers beside a fill that is still running, with the HIP runtime and the
// kernels replaced by what a device with a queue of fills would do as far as the host can see.  Exits with 0 and "ok" if every check of
// the mode holds; built by tests/test_host_accept_beside.py with sanitizers.
//   accept_beside_main MODE
#include "../../paper_2601_04426_amd/csrc/api.cpp"

#include <cstdio>
#include <cstdlib>
#include <new>

#define CHECK(x) do { if (!(x)) { std::printf("%s:%d: %s (%s)\n", __FILE__, __LINE__, #x, xg2_last_error()); std::fflush(stdout); std::_Exit(1); } } while (0)

// ---- allocations: the next but `countdown` of this thread fails; `on_new` is called once, at the next one ------------
static thread_local long countdown = -1;
static thread_local void (*on_new)() = nullptr;
void* operator new(size_t n) {
    if (auto* f = on_new) { on_new = nullptr; f(); }
    if (countdown >= 0 && countdown-- == 0) throw std::bad_alloc();
    if (void* p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

// ---- the device: fills are numbered as they are enqueued and end when somebody waits for one ----------------------------
struct ihipEvent_t { std::atomic<long> fill{0}; };
static std::atomic<long> enqueued{0}, ended{0};
static std::atomic<bool> leave_undecided{false};              // of the fills to come
static void (*after_query)() = nullptr;

extern "C" {
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 1; return hipSuccess; }
hipError_t hipDeviceSynchronize() { ended = enqueued.load(); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = new ihipEvent_t; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t e) {
    if (auto* f = after_query) { after_query = nullptr; on_new = f; }
    return e->fill > ended ? hipErrorNotReady : hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { e->fill = enqueued.load(); return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { for (long n = ended; n < e->fill && !ended.compare_exchange_weak(n, e->fill);) {} return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { *p = std::calloc(n, 1); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void* d, int v, size_t n) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* st) { *st = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
}

namespace xg2 {
uint32_t wave_slots() { return 8192; }
hipError_t noalloc_scratch(void** p) { static void* const mem = std::calloc(kNoAllocScratchBytes, 1); *p = mem; return hipSuccess; }
void launch_copy_masked(const CopyJob*, uint32_t, uint32_t, hipStream_t) {}
void launch_copy_structure(const CopyJob*, uint32_t, uint32_t, hipStream_t) {}
void launch_copy_first_byte(const FirstByteCopyJob*, uint32_t, const uint8_t*, uint32_t, hipStream_t) {}
void launch_expand_chunks(const uint4*, const uint4*, const uint32_t*, uint32_t, uint4*, hipStream_t) {}
void launch_stage(void*, const void*, size_t, const StageZero&, const uint4*, const uint4*, const uint32_t*, uint32_t, uint4*, hipStream_t) {}
void launch_build(const DevTables&, const DevVocab&, BuildPlan, const SlowScratch&, hipStream_t) {}
void launch_build_slow(const DevTables&, const DevVocab&, const BuildPlan&, const SlowScratch&, hipStream_t) {}
void launch_finish_planes(uint32_t* const*, const FinishJob*, uint32_t, const uint8_t*, uint32_t, uint32_t*, hipStream_t) {}
void launch_plane_summary(uint32_t* const*, uint32_t, uint32_t, uint32_t*, hipStream_t) {}
void launch_recheck_slow(const FillBatch&, const DevVocab&, int32_t*, int64_t, const SlowScratch&, hipStream_t) {}
void launch_token_records(const DevVocab&, TokenRecord*, hipStream_t) {}
void launch_accept(const BatchDev&, const DevVocab&, uint32_t, const int32_t*, int32_t*, hipStream_t) {}
void launch_batch_assign(const BatchDev&, const int32_t*, uint32_t, uint32_t, hipStream_t) {}
void launch_upload(void* d, const void* s, size_t n, hipStream_t, uint64_t*, hipEvent_t) { std::memcpy(d, s, n); }
void launch_clear(uint32_t*, uint32_t, hipStream_t) {}
void launch_apply(void*, int32_t, int32_t, int32_t, int64_t, const int32_t*, int64_t, hipStream_t) {}
void launch_fill(const FillBatch&, const DevVocab&, int32_t*, int64_t, const SlowScratch& S, hipStream_t, hipEvent_t done) {
    const long n = ++enqueued;
    if (done) done->fill = n;
    if (leave_undecided) { S.unresolved[0] = 1; S.unresolved[2] = 0; S.unresolved[3] = 1; }
}
}  // namespace xg2

// ---- what the checks work with ------------------------------------------------------------------------------------------
static const char* const TOKENS[] = {"", "(", ")", ",", "a", "b", "aab,", "x"};
enum { END, OPEN, CLOSE, COMMA, A, B, LONG, BAD };
static xg2_vocab* vocab;
static xg2_mask_cache* cache;
static std::vector<int32_t> mask(64);

static std::vector<xg2_matcher*> some_matchers(int n) {       // each behind "("
    std::vector<xg2_matcher*> ms((size_t)n);
    for (xg2_matcher*& m : ms) {
        CHECK(xg2_matcher_create(cache, &m) == XG2_OK);
        CHECK(xg2_matcher_accept_token(m, OPEN) == XG2_OK);
    }
    return ms;
}
static void fill(const std::vector<xg2_matcher*>& ms) { CHECK(xg2_fill_next_token_bitmask(ms.data(), (int32_t)ms.size(), mask.data(), 1, nullptr) == XG2_OK); }
static size_t length(const xg2_matcher* m) { return m->p->chart.length(); }
static bool undecided_error(int32_t rc) { return rc == XG2_EOVERFLOW && std::strstr(xg2_last_error(), "undecided"); }

static void setup() {
    std::string bytes;
    std::vector<uint64_t> offs{0};
    for (const char* t : TOKENS) { bytes += t; offs.push_back(bytes.size()); }
    const int32_t special[] = {END};
    CHECK(xg2_vocab_create((const uint8_t*)bytes.data(), offs.data(), (int32_t)offs.size() - 1, END, special, 1, &vocab) == XG2_OK);
    const std::string ebnf = "root ::= \"(\" list \")\"\nlist ::= item (\",\" item)*\nitem ::= \"a\"+ \"b\"* | \"(\" list \")\"\n";
    CHECK(xg2_compile_grammar(vocab, ebnf.data(), ebnf.size(), "root", nullptr, nullptr, nullptr, &cache, nullptr) == XG2_OK);
}

// Every allocation of the call fails once: no exception leaves it, nothing the fill left undecided goes unreported, and a call that
// reports it moves no matcher.
static void allocations() {
    for (bool undecided : {false, true})
        for (long n = 0;; ++n) {
            CHECK(n < 1000);
            auto ms = some_matchers(3);
            leave_undecided = undecided;
            fill(ms);
            leave_undecided = false;
            const int32_t ids[3] = {LONG, BAD, A};
            int32_t status[3];
            const size_t before = length(ms[0]);
            bool threw = false;
            int32_t rc = XG2_OK;
            countdown = n;
            try { rc = xg2_matcher_accept_tokens(ms.data(), ids, 3, status); } catch (...) { threw = true; }
            const bool reached = countdown < 0;
            countdown = -1;
            CHECK(!threw);
            if (undecided) {
                if (!undecided_error(rc)) { CHECK(rc != XG2_OK); CHECK(undecided_error(xg2_matcher_accept_tokens(ms.data(), ids, 3, status))); }
                if (!reached) for (const xg2_matcher* m : ms) CHECK(length(m) == before);
            } else if (!reached) CHECK(rc == XG2_OK && status[0] == XG2_OK && status[1] == XG2_EREJECTED && status[2] == XG2_OK);
            for (xg2_matcher* m : ms) xg2_matcher_destroy(m);
            if (!reached) break;
        }
    // the same of a single token
    for (long n = 0;; ++n) {
        CHECK(n < 1000);
        auto ms = some_matchers(1);
        leave_undecided = true;
        fill(ms);
        leave_undecided = false;
        const size_t before = length(ms[0]);
        bool threw = false;
        int32_t rc = XG2_OK;
        countdown = n;
        try { rc = xg2_matcher_accept_token(ms[0], A); } catch (...) { threw = true; }
        const bool reached = countdown < 0;
        countdown = -1;
        CHECK(!threw);
        if (!undecided_error(rc)) { CHECK(rc != XG2_OK); CHECK(undecided_error(xg2_matcher_accept_token(ms[0], A))); }
        CHECK(length(ms[0]) == before);
        for (xg2_matcher* m : ms) xg2_matcher_destroy(m);
        if (!reached) break;
    }
}

// Where the call ends early, the statuses of the rows it has not come to are left as the caller had them, and so for a fill that has ended.
static void statuses() {
    int ended_early = 0;
    for (bool running : {false, true})
        for (long n = 0;; ++n) {
            CHECK(n < 1000);
            auto ms = some_matchers(3);
            fill(ms);
            if (!running) ended = enqueued.load();
            const int32_t ids[3] = {LONG, LONG, LONG};
            int32_t status[3] = {77, 78, 79};
            const size_t before = length(ms[0]);
            countdown = n;
            const int32_t rc = xg2_matcher_accept_tokens(ms.data(), ids, 3, status);
            const bool reached = countdown < 0;
            countdown = -1;
            if (rc != XG2_OK) {
                ++ended_early;
                for (int b = 0; b < 3; ++b) {
                    if (length(ms[(size_t)b]) == before) CHECK(status[b] == 77 + b || status[b] == XG2_EOVERFLOW);
                    else CHECK(status[b] == XG2_OK || status[b] == XG2_EOVERFLOW);
                }
            }
            for (xg2_matcher* m : ms) xg2_matcher_destroy(m);
            if (!reached) break;
        }
    CHECK(ended_early > 6);
}

// Another thread's calls while this one parses: the fill that was under way is this call's to report, and no other fill is.
static xg2_matcher* other;
static std::thread other_thread;
static std::atomic<int> other_fills{0};
static int32_t other_rc;
static void threads() {
    auto ms = some_matchers(2), theirs = some_matchers(1);
    other = theirs[0];
    const int32_t ids[2] = {LONG, A};
    int32_t status[2];
    const size_t before = length(ms[0]);

    // a call that would have taken the report
    leave_undecided = true;
    fill(ms);
    leave_undecided = false;
    after_query = [] { std::thread([] { other_rc = xg2_matcher_accept_token(other, A); }).join(); };
    CHECK(undecided_error(xg2_matcher_accept_tokens(ms.data(), ids, 2, status)));
    CHECK(after_query == nullptr && other_rc == XG2_OK && length(other) == before + 1);
    CHECK(length(ms[0]) == before && length(ms[1]) == before);

    // a fill of its own, with undecided pairs: reported to the call after
    fill(ms);
    after_query = [] { std::thread([] { leave_undecided = true; fill({other}); leave_undecided = false; }).join(); };
    CHECK(xg2_matcher_accept_tokens(ms.data(), ids, 2, status) == XG2_OK && status[0] == XG2_OK && status[1] == XG2_OK);
    CHECK(after_query == nullptr && length(ms[0]) == before + 4 && length(ms[1]) == before + 1);
    CHECK(undecided_error(xg2_matcher_accept_token(other, A)) && xg2_matcher_accept_token(other, A) == XG2_OK);

    // more fills than there are staging slots: the one whose outcome this call has yet to read is not handed out again
    leave_undecided = true;
    fill(ms);
    leave_undecided = false;
    after_query = [] {
        other_thread = std::thread([] { for (int k = 0; k < 9; ++k) { fill({other}); ++other_fills; } });
        while (other_fills < 3) std::this_thread::yield();
    };
    CHECK(undecided_error(xg2_matcher_accept_tokens(ms.data(), ids, 2, status)));
    CHECK(after_query == nullptr && length(ms[0]) == before + 4);
    other_thread.join();
    CHECK(other_fills == 9 && xg2_matcher_accept_tokens(ms.data(), ids, 2, status) == XG2_OK);
}

int main(int argc, char** argv) {
    setup();
    const std::string mode = argc > 1 ? argv[1] : "";
    if (mode == "allocations") allocations();
    else if (mode == "statuses") statuses();
    else if (mode == "threads") threads();
    else return 2;
    std::printf("ok\n");
    std::fflush(stdout);
    std::_Exit(0);                                                // (the library's threads live until the process ends)
}
