// The device allocations that destroyed batches leave for later ones, on a runtime of this program's own: relserve_api.hip is linked with
// it, the kernel launchers and every HIP call the batches make are defined below, and time passes when the driver says so.
// A stream is a count of what was submitted to it and a count of what is done; an event is a place in the default stream.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include "relserve_internal.h"

namespace {
std::mutex g_m;
std::map<void*, size_t> g_live;          // device allocations
std::map<void*, long> g_last_use;        // of a live allocation: the default stream's place of the last work on it
long g_submitted = 0, g_done = 0;        // default stream
std::set<void*> g_other_busy;            // allocations with work outstanding on another stream
int g_mallocs = 0, g_frees = 0, g_waits = 0, g_misuse = 0;
bool g_capturing = false, g_capture_broken = false, g_no_new = false;
thread_local hipStreamCaptureMode t_mode = hipStreamCaptureModeGlobal;
void* g_batch_blob = nullptr;            // the allocation the running call works on
struct Event { long place = 0; };

void submit(hipStream_t s, void* blob) {
    std::lock_guard<std::mutex> lock(g_m);
    if (s) {
        // work on another stream may begin at once: nothing of the default stream may still use the allocation
        if (g_last_use[blob] > g_done) ++g_misuse;
        g_other_busy.insert(blob);
    } else {
        if (g_other_busy.count(blob)) ++g_misuse;
        g_last_use[blob] = ++g_submitted;
    }
}
void pass_time() {
    std::lock_guard<std::mutex> lock(g_m);
    g_done = g_submitted;
    g_other_busy.clear();
}
bool unsafe_call() {   // what a capture in global mode does not allow
    if (!g_capturing || t_mode == hipStreamCaptureModeRelaxed) return false;
    g_capture_broken = true;
    return true;
}
}  // namespace

void* operator new(std::size_t n) {
    if (g_no_new) throw std::bad_alloc();
    if (void* p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void* operator new(std::size_t n, const std::nothrow_t&) noexcept { return g_no_new ? nullptr : std::malloc(n ? n : 1); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

extern "C" {
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) { std::memset(p, 0, sizeof *p); std::strcpy(p->gcnArchName, "gfx950"); return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) {
    std::lock_guard<std::mutex> lock(g_m);
    if (unsafe_call()) return hipErrorStreamCaptureUnsupported;
    *p = std::malloc(n);
    g_live[*p] = n;
    ++g_mallocs;
    return hipSuccess;
}
hipError_t hipFree(void* p) {   // waits for the whole device
    std::lock_guard<std::mutex> lock(g_m);
    if (unsafe_call()) return hipErrorStreamCaptureUnsupported;
    g_done = g_submitted;
    g_other_busy.clear();
    ++g_waits;
    ++g_frees;
    g_live.erase(p);
    g_last_use.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t s) {
    submit(s, dst);
    g_batch_blob = dst;
    std::memcpy(dst, src, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
    std::lock_guard<std::mutex> lock(g_m);
    if (s) g_other_busy.clear(); else g_done = g_submitted;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = reinterpret_cast<hipEvent_t>(std::malloc(sizeof(Event)));
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) { std::free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    std::lock_guard<std::mutex> lock(g_m);
    if (s) ++g_misuse;
    reinterpret_cast<Event*>(e)->place = g_submitted;
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
    std::lock_guard<std::mutex> lock(g_m);
    return reinterpret_cast<Event*>(e)->place <= g_done ? hipSuccess : hipErrorNotReady;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) { std::swap(*m, t_mode); return hipSuccess; }
}

namespace relserve {
hipError_t launch_rope_table(const int32_t*, const float*, int32_t, int32_t, float2*, hipStream_t) { return hipSuccess; }
hipError_t launch_rmsnorm(const void*, bool, const void*, float, int32_t, int32_t, void*, hipStream_t, const int32_t*, float) { return hipSuccess; }
hipError_t launch_quantise_bf16(const void*, int64_t, float, void*, hipStream_t) { return hipSuccess; }
hipError_t launch_embedding(const int32_t*, const void*, int32_t, int32_t, int32_t, void*, hipStream_t) { return hipSuccess; }
hipError_t launch_greedy_sample(const float*, int32_t, int32_t, int32_t*, hipStream_t) { return hipSuccess; }
// the work on a batch that the driver submits: relserve_kv_append
hipError_t launch_kv_append(const BatchDev& b, const void*, const void*, void*, void*, int32_t, hipStream_t s) {
    submit(s, const_cast<int32_t*>(b.tok_req));   // the first table of the allocation
    return hipSuccess;
}
hipError_t launch_rope_append(const BatchDev&, const relserve_layer&, void*, void*, void*, hipStream_t) { return hipSuccess; }
int64_t gemm_scratch_floats(int64_t T, int64_t n_max) { return T * n_max; }
void gemm_force_plan(int, int) {}
hipError_t launch_linear(const void*, const void*, int32_t, int32_t, int32_t, int32_t, const void*, void*, hipStream_t, float*, bool, const CodeScales*) { return hipSuccess; }
hipError_t launch_pack_weight(const void*, int32_t, int32_t, void*, hipStream_t) { return hipSuccess; }
hipError_t launch_qkv_rope_append(const BatchDev&, const relserve_layer&, const void*, const void*, void*, void*, void*, hipStream_t, float*, bool, KvFormat, const CodeScales*) { return hipSuccess; }
hipError_t launch_attention(const BatchDev&, const relserve_layer&, const void*, int32_t, const void*, const void*, void*, float*, float*, hipStream_t, relserve_layer*, KvFormat) { return hipSuccess; }
hipError_t launch_peak_mfma(float*, int32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_peak_stream(const void*, int64_t, uint32_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_peak_stream_pattern(const void*, int64_t, int32_t, uint32_t*, hipStream_t) { return hipSuccess; }
}  // namespace relserve

#define EXPECT(cond) do { if (!(cond)) { std::printf("FAILED %s, line %d: %s\n", __func__, __LINE__, #cond); std::exit(1); } } while (0)

namespace {
const relserve_layer_config cfg{256, 8, 2, 64, 688, 16, 1e-5f, 10000.0f};
void* const kOther = reinterpret_cast<void*>(0x5000);   // a stream that is not the default one

relserve_layer* layer() {
    relserve_layer* L = nullptr;
    EXPECT(relserve_layer_create(&cfg, &L) == RELSERVE_OK);
    return L;
}
relserve_batch* prepare(relserve_layer* L, int tokens, void* stream = nullptr) {
    std::vector<int32_t> bt((tokens + 15) / 16);
    for (size_t i = 0; i < bt.size(); ++i) bt[i] = (int32_t)i;
    const int32_t q[2] = {0, tokens}, ctx[1] = {tokens};
    relserve_batch_desc d{};
    d.num_reqs = 1;
    d.max_blocks = d.num_pages = (int32_t)bt.size();
    d.q_start = q;
    d.ctx_len = ctx;
    d.block_table = bt.data();
    relserve_batch* b = nullptr;
    EXPECT(relserve_batch_prepare(L, &d, stream, &b) == RELSERVE_OK);
    return b;
}
void work(relserve_layer* L, relserve_batch* b, void* stream) {
    static char pool[64];
    relserve_kv_cache c{};
    c.k_pages = c.v_pages = pool;
    c.num_pages = 1 << 20;
    EXPECT(relserve_kv_append(L, b, pool, pool, c, stream) == RELSERVE_OK);
}
void end(relserve_layer* L) {
    EXPECT(relserve_layer_destroy(L) == RELSERVE_OK);
    EXPECT(g_live.empty() && g_misuse == 0);
    g_mallocs = g_frees = g_waits = 0;
}

void reuse() {
    relserve_layer* L = layer();
    for (int i = 0; i < 20; ++i) {
        relserve_batch* b = prepare(L, 40 + i);
        work(L, b, nullptr);
        EXPECT(relserve_batch_destroy(b) == RELSERVE_OK);
        pass_time();
    }
    EXPECT(g_mallocs == 1 && g_frees == 0 && g_waits == 0);
    end(L);
}
// work of the default stream is outstanding as its batch goes and another stream prepares the next one
void other_stream_behind_default() {
    relserve_layer* L = layer();
    relserve_batch* b = prepare(L, 40);
    work(L, b, nullptr);
    EXPECT(relserve_batch_destroy(b) == RELSERVE_OK);
    relserve_batch* c = prepare(L, 40, kOther);   // (submit counts a misuse if this is the first one's allocation)
    EXPECT(g_misuse == 0 && g_mallocs == 2);
    pass_time();
    relserve_batch* d = prepare(L, 40, kOther);
    EXPECT(g_misuse == 0 && g_mallocs == 2);
    EXPECT(relserve_batch_destroy(c) == RELSERVE_OK && relserve_batch_destroy(d) == RELSERVE_OK);
    end(L);
}
void default_behind_other_stream() {
    relserve_layer* L = layer();
    for (int prepared_there = 0; prepared_there < 2; ++prepared_there) {
        relserve_batch* b = prepare(L, 40, prepared_there ? kOther : nullptr);
        if (!prepared_there) work(L, b, kOther);
        const int frees = g_frees;
        EXPECT(relserve_batch_destroy(b) == RELSERVE_OK && g_frees == frees + 1);   // hipFree waits
        b = prepare(L, 40);
        EXPECT(g_misuse == 0);
        EXPECT(relserve_batch_destroy(b) == RELSERVE_OK);
        pass_time();
        EXPECT(relserve_layer_destroy(L) == RELSERVE_OK);
        L = layer();
    }
    end(L);
}
void bounded() {
    relserve_layer* L = layer();
    std::vector<relserve_batch*> all;
    for (int i = 0; i < 30; ++i) all.push_back(prepare(L, 40));
    for (relserve_batch* b : all) EXPECT(relserve_batch_destroy(b) == RELSERVE_OK);
    EXPECT(g_live.size() == 8);
    relserve_batch* big = prepare(L, 40000);   // 10 MB of tables
    const size_t live = g_live.size();
    EXPECT(relserve_batch_destroy(big) == RELSERVE_OK && g_live.size() == live - 1);
    end(L);
}
void batch_outlives_the_layers() {
    relserve_layer *L = layer(), *M = layer();
    relserve_batch *b = prepare(L, 40), *c = prepare(L, 40);
    EXPECT(relserve_batch_destroy(c) == RELSERVE_OK);
    EXPECT(relserve_layer_destroy(L) == RELSERVE_OK && g_live.size() == 2);   // the other handle keeps the list
    EXPECT(relserve_layer_destroy(M) == RELSERVE_OK && g_live.size() == 1);
    EXPECT(relserve_batch_destroy(b) == RELSERVE_OK);
    EXPECT(g_live.empty());
    end(layer());
}
void destroy_allocates_nothing() {
    relserve_layer* L = layer();
    std::vector<relserve_batch*> all;
    for (int i = 0; i < 12; ++i) all.push_back(prepare(L, 40));
    g_no_new = true;   // the host is out of memory
    for (relserve_batch* b : all) {
        bool ok = false;
        try { ok = relserve_batch_destroy(b) == RELSERVE_OK; } catch (...) {}
        if (!ok) g_no_new = false;
        EXPECT(ok);
    }
    g_no_new = false;
    end(L);
}
void inside_a_capture() {
    relserve_layer* L = layer();
    relserve_batch *b = prepare(L, 40), *c = prepare(L, 40, kOther);
    g_capturing = true;
    EXPECT(relserve_batch_destroy(b) == RELSERVE_OK);   // kept
    EXPECT(relserve_batch_destroy(c) == RELSERVE_OK);   // freed
    EXPECT(relserve_layer_destroy(L) == RELSERVE_OK);   // what was kept
    g_capturing = false;
    EXPECT(!g_capture_broken && g_live.empty() && t_mode == hipStreamCaptureModeGlobal);
    end(layer());
}
void threads() {
    std::vector<std::thread> all;
    for (int t = 0; t < 6; ++t)
        all.emplace_back([] {
            for (int i = 0; i < 300; ++i) {
                relserve_layer* L = layer();
                relserve_batch *b = prepare(L, 40), *c = prepare(L, 60);
                EXPECT(relserve_batch_destroy(b) == RELSERVE_OK);
                if (i % 2) EXPECT(relserve_layer_destroy(L) == RELSERVE_OK);
                EXPECT(relserve_batch_destroy(c) == RELSERVE_OK);
                if (i % 2 == 0) EXPECT(relserve_layer_destroy(L) == RELSERVE_OK);
            }
        });
    for (std::thread& t : all) t.join();
    EXPECT(g_live.empty() && g_misuse == 0);
}
}  // namespace

int main(int argc, char** argv) {
    const std::map<std::string, void (*)()> cases = {
        {"reuse", reuse}, {"other_stream_behind_default", other_stream_behind_default}, {"default_behind_other_stream", default_behind_other_stream},
        {"bounded", bounded}, {"batch_outlives_the_layers", batch_outlives_the_layers}, {"destroy_allocates_nothing", destroy_allocates_nothing},
        {"inside_a_capture", inside_a_capture}, {"threads", threads}};
    for (int i = 1; i < argc; ++i) cases.at(argv[i])();
    std::printf("ok\n");
    return 0;
}
