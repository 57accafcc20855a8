// Host boundary of the layer-step library: validation, descriptor expansion, upload,
// workspace carving and kernel sequencing.  No arithmetic of the method lives here.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>

#include "relserve_internal.h"

using namespace relserve;

namespace {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

const char* const kSlotNames[RELSERVE_PROFILE_SLOTS] = {
    "rmsnorm_in", "gemm_qkv_rope_append", "attn_own_keys", "attn_prefix", "attn_tile", "attn_split",
    "gemm_o",     "rmsnorm_post", "gemm_gate_up", "gemm_down",  "attn_merge", "quantise_attn"};
// the last slot stays empty: the attention kernels store a quantised step's codes themselves (slots and names are part of the interface)
enum { S_NORM1 = 0, S_QKV, S_ATTN_OWN, S_ATTN_PREFIX, S_ATTN_TILE, S_ATTN_SPLIT, S_O, S_NORM2, S_GU, S_DOWN, S_ATTN_MERGE };

struct Workspace {
    char* h;         // [T, H] bf16 (normed activations; reused for the post norm)
    char* q;         // [T, q_dim] bf16 rotated queries
    char* attn;      // [T, q_dim] bf16
    char* x1;        // [T, H] fp32 residual stream after attention
    char* act;       // [T, I] bf16
    float* part_o;   // [T + split slots, n_q, d] fp32
    float* part_ml;  // [T + split slots, n_q, 2] fp32
    float* accum;    // fp32 split-K scratch of the GEMMs
    size_t accum_floats;
    size_t total;
};

Workspace carve(const relserve_layer& L, int64_t T, void* base) {
    Workspace w;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char* p = base ? static_cast<char*>(base) + off : nullptr;
        off += align_up(bytes);
        return p;
    };
    const relserve_layer_config& c = L.cfg;
    w.h = take((size_t)T * c.hidden * 2);
    w.q = take((size_t)T * L.q_dim * 2);
    w.attn = take((size_t)T * L.q_dim * 2);
    w.x1 = take((size_t)T * c.hidden * 4);
    w.act = take((size_t)T * c.mlp_dim * 2);
    const size_t part_rows = (size_t)(T + split_slot_cap(T));
    w.part_o = reinterpret_cast<float*>(take(part_rows * L.q_dim * 4));
    w.part_ml = reinterpret_cast<float*>(take(part_rows * c.n_q_heads * 2 * 4));
    w.accum_floats = (size_t)gemm_scratch_floats(T, std::max({L.qkv_dim, 2 * c.mlp_dim, c.hidden}));
    w.accum = reinterpret_cast<float*>(take(w.accum_floats * 4));
    w.total = off;
    return w;
}

// Cut of a batch of decode rows (see expand_batch): per shared prefix the number and length of its chunks, and the length
// of the chunks of own keys.
struct SlotPlan {
    bool use = false;
    std::vector<int32_t> prefix_chunks, prefix_len;
    int32_t chunk_len = 0;
};

// rows_len: the chunk length of the same rows without slots (0 = uncut, -1 = no row is long enough to cut).
template <typename OwnKeys, typename ChunksOf>
SlotPlan plan_slots(const relserve_layer_config& cfg, const relserve_batch_desc& d, const std::vector<uint8_t>& joint,
                    OwnKeys own_keys, ChunksOf chunks_of, int32_t rows_len) {
    SlotPlan plan;
    const int32_t B = d.num_reqs;
    int64_t own_total = 0;
    for (int32_t r = 0; r < B; ++r) own_total += own_keys(r);
    const double stream_us = (double)own_total * cfg.n_kv_heads * cfg.head_dim * 4.0 / 6.0e6;   // the own keys at about 6 TB/s
    // A prefix chunk should not outlast the own keys (these start behind 8 us of latency): a block of 64 prefix keys takes a
    // workgroup about 2.5 us.
    const int32_t blocks_max = (int32_t)std::min(1e6, std::max(2.0, (8.0 + stream_us) / 2.5));
    plan.prefix_chunks.assign(d.num_prefixes, 0);
    plan.prefix_len.assign(d.num_prefixes, 0);
    bool any = false;
    for (int32_t p = 0; p < d.num_prefixes; ++p) {
        if (!joint[p]) continue;
        any = true;
        const int32_t blocks = (d.prefix_len[p] + 63) / 64, n = (blocks + blocks_max - 1) / blocks_max;
        plan.prefix_len[p] = (blocks + n - 1) / n * 64;
        plan.prefix_chunks[p] = (d.prefix_len[p] + plan.prefix_len[p] - 1) / plan.prefix_len[p];
    }
    // Nor should an item of own keys: beside other rows a wave walks one in about 0.055 us, and an item is up to a chunk and a
    // half.  So the longest chunk of 64 .. 512 keys that takes no longer than the stream, whatever the batch: one long row
    // among short ones is cut as well.  13B layer behind a template of 512 (without slots / now): 100 rows of 60 keys and one
    // of 3000 53 / 37 us, of 8000 73 / 55; 60 rows, ten of them of 8000 285 / 268; 60 rows of 1000 206 / 195; 4 of 1000 47 / 22.
    const double ideal = std::min(512.0, stream_us / 0.08);
    int32_t len = 64;
    while (2 * len <= ideal) len *= 2;
    // Two rounds of waves (256 CUs x 8 resident waves) with much to read: the rows balance by themselves, and a kernel with the
    // tiled items in it holds fewer waves of them than one without (200 rows of 1000: 626 us without slots, 647 with).
    if ((int64_t)B * cfg.n_kv_heads >= 2 * 2048 && stream_us > 200.0) return plan;
    // Without a template slots are only for rows that the workspace's own (2 T) cannot cut about as finely: 4 rows of 1000
    // 33 / 19 us, 2 of 8000 437 / 65; but 24 rows with two of 1500 17 / 21.
    if (!any && (rows_len < 0 || (rows_len > 0 && rows_len < 2 * ideal))) return plan;
    const int64_t cap = scratch_slot_cap(cfg.n_q_heads, cfg.head_dim);
    for (; len <= 1024; len *= 2) {
        int64_t slots = 0;
        bool cut = false;
        for (int32_t r = 0; r < B; ++r) {
            const int32_t pid = d.prefix_id ? d.prefix_id[r] : -1;
            const int32_t n = chunks_of(own_keys(r), len);
            const int32_t parts = n + (pid >= 0 && joint[pid] ? plan.prefix_chunks[pid] : 0);
            if (parts > 1) slots += parts;
            cut |= n > 1;
        }
        if (slots > cap) continue;
        plan.chunk_len = len;
        plan.use = any || cut;
        break;
    }
    return plan;
}

// Where the attention passes of a batch keep partial state: the workspace's own rows, or (slot plans) the GEMM scratch.
struct PartialState { float* o; float* ml; };
PartialState partial_state(const relserve_layer& L, const BatchDev& b, const Workspace& w) {
    if (b.n_scratch_slots == 0) return {w.part_o, w.part_ml};
    return {w.accum, w.accum + (int64_t)b.n_scratch_slots * L.q_dim};
}

// The cut of the attention a step over these pools runs.  A 16-bit output that rounds the other way moves codes of the keys and
// values the next layer appends to its quantised pool, and those move the rest of the stack (3 % of the codes of a third 13B
// layer, 2e-2 of the logits after four), so over quantised pools every entry point takes the cut without slots, whose results
// stacks were recorded with.
const BatchDev& attention_batch(const relserve_batch& b, const relserve_kv_cache& cache) {
    return cache.dtype == RELSERVE_KV_FP8 ? b.dev_no_slots : b.dev;
}

bool is_pow2(int32_t v) { return v > 0 && (v & (v - 1)) == 0; }

// Workspace of relserve_layer_step_static: a fixed array in device memory, one copy per GPU the library runs on,
// held until the process ends.  `scratch` is only a host-side stand-in for the symbol: the device address comes
// from hipGetSymbolAddress, once per device, and only that address is handed to kernels.
constexpr size_t kStaticScratchBytes = (size_t)RELSERVE_STATIC_SCRATCH_BYTES;
__device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

int32_t static_scratch(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return RELSERVE_ERR_NO_DEVICE;
    if (dev < 0 || dev >= kMaxDevices) return RELSERVE_ERR_BAD_ARGUMENT;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return RELSERVE_ERR_HIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return RELSERVE_OK;
}

KvFormat kv_format(const relserve_kv_cache& cache) {
    KvFormat f;
    f.fp8 = cache.dtype == RELSERVE_KV_FP8;
    if (f.fp8) f.k_scale = cache.k_scale, f.v_scale = cache.v_scale;
    return f;
}

int32_t check_cache(const relserve_batch* b, const relserve_kv_cache& cache, bool fp8_ok = true) {
    if (!cache.k_pages || !cache.v_pages) return RELSERVE_ERR_NULL_POINTER;
    if (cache.dtype != RELSERVE_KV_BF16 && cache.dtype != RELSERVE_KV_FP8) return RELSERVE_ERR_BAD_ARGUMENT;
    if (cache.dtype == RELSERVE_KV_FP8) {
        if (!fp8_ok) return RELSERVE_ERR_BAD_ARGUMENT;
        if (!(cache.k_scale > 0.0f) || !(cache.v_scale > 0.0f) || !std::isfinite(cache.k_scale) || !std::isfinite(cache.v_scale))
            return RELSERVE_ERR_BAD_ARGUMENT;
    }
    if (cache.num_pages < b->dev.num_pages) return RELSERVE_ERR_MISMATCH;
    return RELSERVE_OK;
}

// stream: where the caller submits work that reads the batch
int32_t check_pair(const relserve_layer* L, const relserve_batch* b, const void* stream) {
    if (!L || !b) return RELSERVE_ERR_NULL_POINTER;
    if (std::memcmp(&L->cfg, &b->cfg, sizeof(relserve_layer_config)) != 0) return RELSERVE_ERR_MISMATCH;
    if (stream) b->other_stream.store(true, std::memory_order_relaxed);
    return RELSERVE_OK;
}

// Device allocations of destroyed batches, kept for the next ones.  hipFree waits for the whole device and gives the pages back:
// 45 - 75 us of an iteration that prepares and destroys a batch (24 rows, four 13B layers: 820), with the GPU idle.
// A blob comes here only if all work on its batch went to the default stream, where an event recorded as the batch is destroyed
// stands behind it; it is handed out again when that event has passed, so neither side waits.  (Streams of the caller may be gone
// by then; their batches take hipFree.)  At most kSpareBlobs of at most kSpareBlobBytes each, and none without a layer handle: freed when
// the last one goes, and a batch that outlives it keeps nothing.
struct SpareBlob { void* blob; size_t bytes; int device; hipEvent_t idle; };
constexpr int kSpareBlobs = 8;
constexpr size_t kSpareBlobBytes = (size_t)4 << 20;
struct SpareBlobs {   // in place, so that keeping one allocates nothing; nothing to run at the process's end
    std::mutex m;
    SpareBlob blobs[kSpareBlobs];   // oldest first
    int n = 0;
    int layers = 0;                 // handles alive
};
SpareBlobs g_spare;

// Frees a batch's allocation, or one that was kept: also where some stream is being captured.  hipFree ends a capture in global mode on any
// thread of the process (measured, as are the calls beside it), and the one that frees need not know of it -- another thread's, or a
// collector's that runs while a program captures; nothing here becomes part of a graph.
hipError_t free_blob(const SpareBlob& s) {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    if (s.idle) (void)hipEventDestroy(s.idle);
    const hipError_t e = s.blob ? hipFree(s.blob) : hipSuccess;
    if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
    return e;
}

// The i-th leaves the list (g_spare.m is held).
SpareBlob pull_spare_blob(int i) {
    const SpareBlob s = g_spare.blobs[i];
    for (--g_spare.n; i < g_spare.n; ++i) g_spare.blobs[i] = g_spare.blobs[i + 1];
    return s;
}

bool take_spare_blob(size_t bytes, int device, SpareBlob* out) {
    std::lock_guard<std::mutex> lock(g_spare.m);
    for (int i = 0; i < g_spare.n; ++i) {
        if (g_spare.blobs[i].device != device || g_spare.blobs[i].bytes < bytes) continue;
        if (hipEventQuery(g_spare.blobs[i].idle) != hipSuccess) {
            (void)hipGetLastError();   // not ready
            continue;
        }
        *out = pull_spare_blob(i);
        return true;
    }
    return false;
}

// False: it is still the caller's.
bool give_spare_blob(SpareBlob& s) {
    int device = -1;
    if (s.bytes > kSpareBlobBytes || hipGetDevice(&device) != hipSuccess || device != s.device) return false;
    if (!s.idle && hipEventCreateWithFlags(&s.idle, hipEventDisableTiming) != hipSuccess) return false;
    if (hipEventRecord(s.idle, nullptr) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    SpareBlob oldest{};
    {
        std::lock_guard<std::mutex> lock(g_spare.m);
        if (g_spare.layers == 0) return false;
        if (g_spare.n == kSpareBlobs) oldest = pull_spare_blob(0);
        g_spare.blobs[g_spare.n++] = s;
    }
    (void)free_blob(oldest);
    return true;
}

void free_spare_blobs() {
    SpareBlob all[kSpareBlobs];
    int n;
    {
        std::lock_guard<std::mutex> lock(g_spare.m);
        n = g_spare.n;
        std::copy(g_spare.blobs, g_spare.blobs + n, all);
        g_spare.n = 0;
    }
    for (int i = 0; i < n; ++i) (void)free_blob(all[i]);
}

// +1: a handle more; -1: one less.
void count_layer(int by) {
    bool last;
    {
        std::lock_guard<std::mutex> lock(g_spare.m);
        g_spare.layers += by;
        last = g_spare.layers == 0;
    }
    if (last) free_spare_blobs();
}

}  // namespace

// ------------------------------------------------------------------------------------------
// descriptor expansion (host only)
// ------------------------------------------------------------------------------------------
int32_t relserve::expand_batch(const relserve_layer_config& cfg, const relserve_batch_desc& d,
                               bool build_items, HostBatch* out) {
    if (d.num_reqs < 0 || d.max_blocks < 0 || d.num_pages < 0 || d.num_prefixes < 0)
        return RELSERVE_ERR_BAD_ARGUMENT;
    if (!d.q_start) return RELSERVE_ERR_NULL_POINTER;
    if (d.num_reqs > 0 && (!d.ctx_len || !d.block_table)) return RELSERVE_ERR_NULL_POINTER;
    if (d.num_prefixes > 0 && !d.prefix_len) return RELSERVE_ERR_NULL_POINTER;
    const int32_t P = cfg.page_size, B = d.num_reqs;
    if ((int64_t)d.num_pages * P >= (int64_t)1 << 31) return RELSERVE_ERR_TOO_LARGE;
    if (d.q_start[0] != 0) return RELSERVE_ERR_BAD_Q_START;
    for (int32_t r = 0; r < B; ++r)
        if (d.q_start[r + 1] <= d.q_start[r]) return RELSERVE_ERR_BAD_Q_START;
    const int32_t T = d.q_start[B];
    if (T > (1 << 22)) return RELSERVE_ERR_TOO_LARGE;

    for (int32_t p = 0; p < d.num_prefixes; ++p)
        if (d.prefix_len[p] < 0 || d.prefix_len[p] % P != 0) return RELSERVE_ERR_BAD_PREFIX;

    HostBatch hb;
    hb.T = T;
    hb.tok_req.resize(T);
    hb.tok_pos.resize(T);
    hb.tok_slot.resize(T);
    std::vector<int32_t> first_member(d.num_prefixes, -1), members(d.num_prefixes, 0);
    for (int32_t r = 0; r < B; ++r) {
        const int32_t q_len = d.q_start[r + 1] - d.q_start[r];
        const int32_t L = d.ctx_len[r];
        if (L < q_len) return RELSERVE_ERR_BAD_CTX_LEN;
        const int32_t blocks = (L + P - 1) / P;
        if (blocks > d.max_blocks) return RELSERVE_ERR_BLOCK_TABLE_SHORT;
        const int32_t* bt = d.block_table + (size_t)r * d.max_blocks;
        for (int32_t i = 0; i < blocks; ++i)
            if (bt[i] < 0 || bt[i] >= d.num_pages) return RELSERVE_ERR_PAGE_RANGE;
        const int32_t past = L - q_len;
        const int32_t pid = d.prefix_id ? d.prefix_id[r] : -1;
        if (pid < -1 || pid >= d.num_prefixes) return RELSERVE_ERR_BAD_PREFIX;
        if (pid >= 0) {
            const int32_t pl = d.prefix_len[pid];
            if (pl > past) return RELSERVE_ERR_BAD_PREFIX;  // a member never writes a shared page
            if (first_member[pid] < 0) {
                first_member[pid] = r;
            } else {
                const int32_t* bt0 = d.block_table + (size_t)first_member[pid] * d.max_blocks;
                for (int32_t i = 0; i < pl / P; ++i)
                    if (bt[i] != bt0[i]) return RELSERVE_ERR_BAD_PREFIX;
            }
            ++members[pid];
        }
        for (int32_t j = 0; j < q_len; ++j) {
            const int32_t t = d.q_start[r] + j, pos = past + j;
            hb.tok_req[t] = r;
            hb.tok_pos[t] = pos;
            hb.tok_slot[t] = bt[pos / P] * P + pos % P;
        }
    }
    {   // no two appended tokens may land in the same slot
        std::vector<int32_t> s(hb.tok_slot);
        std::sort(s.begin(), s.end());
        for (size_t i = 1; i < s.size(); ++i)
            if (s[i] == s[i - 1]) return RELSERVE_ERR_SLOT_ALIAS;
    }
    {   // and none may land in a page that serves as a shared prefix page
        std::vector<uint8_t> shared(d.num_pages > 0 ? d.num_pages : 1, 0);
        bool any = false;
        for (int32_t p = 0; p < d.num_prefixes; ++p) {
            if (first_member[p] < 0) continue;
            const int32_t* bt0 = d.block_table + (size_t)first_member[p] * d.max_blocks;
            for (int32_t i = 0; i < d.prefix_len[p] / P; ++i) shared[bt0[i]] = 1, any = true;
        }
        if (any)
            for (int32_t t = 0; t < T; ++t)
                if (shared[hb.tok_slot[t] / P]) return RELSERVE_ERR_BAD_PREFIX;
    }

    for (int32_t r = 0; r < B; ++r) (d.q_start[r + 1] - d.q_start[r] == 1 ? hb.n_decode : hb.n_prefill)++;

    auto build = [&](bool slots_allowed, ItemLists& il) {
        hb.n_groups = 0;
        const int32_t group = cfg.n_q_heads / cfg.n_kv_heads;
        const int32_t tile_tok = ATTN_BLOCK_M / group;    // tokens per row-tiled item (rows past tile_tok * group stay idle)
        // a prefix is handled jointly when at least two requests of the batch carry it
        std::vector<uint8_t> joint(d.num_prefixes, 0);
        for (int32_t p = 0; p < d.num_prefixes; ++p)
            joint[p] = (members[p] >= 2 && d.prefix_len[p] > 0);
        auto own_keys = [&](int32_t r) {
            const int32_t pid = d.prefix_id ? d.prefix_id[r] : -1;
            return d.ctx_len[r] - ((pid >= 0 && joint[pid]) ? d.prefix_len[pid] : 0);
        };
        auto chunks_of = [](int32_t own, int32_t len) { return len > 0 ? std::max(1, (own + len / 2) / len) : 1; };

        // Batches of decode rows alone (at most SKINNY_MAX_T): every part of a row's keys is an item of its own -- chunks of
        // the shared prefix for the tiled kernel, chunks of its own keys for the wave kernel -- in ONE launch, each leaving
        // its running state in a slot of the GEMM scratch, and one merge finishes the rows.  The prefix pass of few rows is
        // few workgroups that walk the whole template one block after the other, with the own keys waiting behind it.
        // Attention of a 13B layer, template of 512: 4 rows 13.5 + 11.8 us (prefix pass, own keys) -> 8.7 + 4.5 (launch,
        // merge), 24 rows 14.4 + 14.2 -> 13.9 + 4.7; 70B shape, 256 rows, templates of 768: 26.4 + 76.2 + 5.1 -> 82.0 + 6.5.
        // (Batches with prefill rows: below.)
        // Without slots, decode rows with many own keys are cut into chunks too (one wave item each, merged afterwards), so that
        // one long context does not set the kernel's duration and the waves come in several even rounds.  The chunk length is
        // the smallest of 128 .. 1024 keys whose chunks fit the partial-state slots of the workspace.
        // (with two rounds of waves or more -- 256 CUs x 8 resident waves each -- the rows balance by themselves: cutting
        // the 128 rows x 40 heads of 1024 keys of a 13B decode batch in two left its kernel at 6.5 TB/s and added the merge)
        auto rows_chunk_len = [&]() -> int32_t {   // 0 = uncut, -1 = uncut because no row is longer than a chunk and a half
            if ((int64_t)hb.n_decode * cfg.n_kv_heads >= 2 * 2048) return 0;
            for (int32_t len = 128; len <= 1024; len *= 2) {
                int64_t slots = 0;
                bool any = false;
                for (int32_t r = 0; r < B; ++r)
                    if (d.q_start[r + 1] - d.q_start[r] == 1) {
                        const int32_t n = chunks_of(own_keys(r), len);
                        if (n > 1) slots += n, any = true;
                    }
                if (!any) return len == 128 ? -1 : 0;   // nothing to cut at any larger length
                if (slots <= split_slot_cap(T)) return len;
            }
            return 0;
        };
        // Prefill rows of a group take the shared keys and their own in ONE item: its rows are packed over requests as in a pass of
        // its own over the template, but the running state (n_q (d + 2) floats a row, written and read back) stays in registers.
        // Attention of 65 requests of 50 .. 200 tokens behind 1024 (13B): 266 + 139 us (two passes) -> 337; of 31, 146 + 71 -> 179.
        // Such an item walks the own keys of its requests one after the other, cached ones among them, which the two passes walk at
        // the same time: short requests, and long ones with keys cached behind the template, are faster in two passes.  Both are priced
        // in blocks of 64 keys (about 2 us): a launch takes its longest item and what falls to one of the workgroups the chip holds;
        // an item costs two blocks beyond its own, each request of a joint item one (its rows' sums are kept in memory till
        // then); two passes cost the state's way through memory, and a launch if nothing else needs the pass (two blocks beyond
        // the two of its longest item).  All groups go one way: while one group keeps the pass, the joint items of the others, which walk
        // their templates once more, run behind it (64/8 heads, 15 requests of 30 tokens in three groups behind 768: 50 us in two
        // passes, 51 in joint items, 76 in both).  Decode rows need the pass as well: it stays (pass_stays), or their template's items join the
        // one launch (below) and the merge is as dear as the pass's launch.  The last launch reads the decode rows' own keys beside its
        // tiled items, and the shorter of the two costs about 0.3 of its time: behind a long stream of keys joint items are nearly free.
        // Fitted to the attention of 1660 batches over 16-bit and 1488 over quantised pools (40/40, 64/8, 40/8, 20/4, 16/2, 8/8, 8/4 and 4/2
        // heads; up to 5000 tokens in requests of 2 .. 280 with 0 .. 500 cached keys, two thirds of them with 1 .. 1200 decode rows, behind one to
        // three templates of 64 .. 1024).  1200 other batches, off the faster of the two on average: prefill rows alone 0.3 % (two passes
        // alone 7 %, joint items alone 28 %), beside decode rows over quantised pools 0.5 % (2 and 40 %), over 16-bit ones 0.9 % (7 and 22 %); on
        // average 7, 1 and 6 % faster than two passes throughout, 26 of the 1200 by 3 .. 13 % slower, one by 21.  Batches such as a relQuery's,
        // 40/40, 64/8 and 40/8 heads, 3 .. 24 requests of 30 .. 120 tokens beside 30 .. 250 rows: 19 % faster.  Two passes / joint, us: 40/40 heads
        // behind 256, 400 tokens in requests of 4 52 / 108, of 32 24 / 23, of 32 with 1000 cached 62 / 120; 2000 in requests of 16 82 / 73, of 100
        // 61 / 53, of 100 with 1000 cached 155 / 258; 8-bit pools, 64/8 heads, 8 requests of 7 tokens and 29 decode rows behind 1024 39 / 72;
        // 16-bit, 40/40, 16 requests of 75 and 184 rows behind 512 109 / 97.
        std::vector<int32_t> pre_toks(d.num_prefixes, 0), dec_rows(d.num_prefixes, 0);   // behind each template that is handled jointly
        int64_t behind = 0;                                                              // decode rows behind any of them
        for (int32_t r = 0; r < B; ++r) {
            const int32_t pid = d.prefix_id ? d.prefix_id[r] : -1, q_len = d.q_start[r + 1] - d.q_start[r];
            if (pid < 0 || !joint[pid]) continue;
            if (q_len == 1) ++dec_rows[pid], ++behind;
            else pre_toks[pid] += q_len;
        }
        auto joint_pays = [&](bool pass_stays) {
            struct Launch {
                int64_t longest = 0, total = 0;
                void item(int64_t blocks) { longest = std::max(longest, blocks + 2), total += blocks + 2; }
                double time(int32_t n_kv) const { return (double)longest + (double)total * n_kv / ATTN_WGS; }
            } pass, own, both, dec;
            int64_t state_rows = 0, stream_keys = 0;             // the decode rows' own keys, read beside the last launch's items
            std::vector<int32_t> filled(d.num_prefixes, 0);      // of each group's joint item being filled: its tokens ...
            std::vector<int64_t> packed(d.num_prefixes, 0);      // ... and the blocks of its requests' own keys
            for (int32_t r = 0; r < B; ++r) {
                const int32_t p = d.prefix_id ? d.prefix_id[r] : -1, q_len = d.q_start[r + 1] - d.q_start[r];
                if (q_len == 1) stream_keys += own_keys(r);
                if (p < 0 || !joint[p] || q_len == 1) continue;
                const int32_t cached = d.ctx_len[r] - q_len - d.prefix_len[p];
                for (int32_t o = 0; o < q_len; o += tile_tok) own.item((cached + std::min(q_len, o + tile_tok) + 63) / 64);
                for (int32_t o = 0; o < q_len;) {
                    const int32_t n = std::min(q_len - o, tile_tok - filled[p]);
                    o += n;
                    packed[p] += (cached + o + 63) / 64 + 1;
                    if ((filled[p] += n) == tile_tok) both.item((d.prefix_len[p] + 63) / 64 + packed[p]), filled[p] = 0, packed[p] = 0;
                }
            }
            for (int32_t p = 0; p < d.num_prefixes; ++p) {
                if (!joint[p]) continue;
                const int64_t shared = (d.prefix_len[p] + 63) / 64;
                if (filled[p] > 0) both.item(shared + packed[p]);
                for (int64_t o = 0; o < (int64_t)pre_toks[p] + dec_rows[p]; o += tile_tok) pass.item(shared);
                for (int32_t o = 0; o < dec_rows[p]; o += tile_tok) (pass_stays ? dec : both).item(shared);
                state_rows += pre_toks[p];
            }
            const double state_us = (double)state_rows * cfg.n_q_heads * (cfg.head_dim + 2) * 8 / 5.0e6;   // written and read at 5 TB/s
            const double stream = (double)stream_keys * cfg.n_kv_heads * cfg.head_dim * 4 / 3.0e6 / 2;     // at 3 TB/s of 16-bit pools
            auto beside = [&](double items) { return std::max(items, stream) + 0.3 * std::min(items, stream); };
            const int32_t n_kv = cfg.n_kv_heads;
            return dec.time(n_kv) + beside(both.time(n_kv)) <= pass.time(n_kv) + beside(own.time(n_kv)) + (behind == 0 ? 2 : 0) + state_us / 2;
        };
        const int32_t rows_len = rows_chunk_len();
        SlotPlan plan;
        if (slots_allowed && hb.n_prefill == 0 && T > 0 && T <= SKINNY_MAX_T) plan = plan_slots(cfg, d, joint, own_keys, chunks_of, rows_len);

        // Decode rows behind a template in a batch that prefills too: the template is an item of the one launch as well, its state and
        // those of the rows' own keys in the workspace's slots (T + ..), and the merge finishes the rows.  As a launch of its own
        // it was few workgroups with everything else waiting.  With many rows that launch fills the chip, and the second state of every
        // row and the merge cost more than it: attention of 200 / 500 / 1000 / 2000 rows of about 150 own keys behind 512 beside a
        // chunk of 512 tokens, launch of its own -> one launch, us: 64/8 heads 58 -> 44, 95 -> 98, 155 -> 168, 286 -> 304; 40/40
        // 132 -> 122, 286 -> 287, 532 -> 553, 1042 -> 1098.  So up to 8 MB of state; over 1560 batches of four shapes that is 1.4 % off the
        // faster of the two on average (15 % with none), in twelve of them 2 .. 5 % slower than the launch of its own.
        bool mixed = slots_allowed && hb.n_prefill > 0 && behind > 0 && behind * cfg.n_q_heads * cfg.head_dim <= ATTN_MIXED_FLOATS;
        std::vector<uint8_t> fused(d.num_prefixes, 0);
        auto choose_joint = [&] {
            const bool pays = joint_pays(!mixed);
            for (int32_t p = 0; p < d.num_prefixes; ++p) fused[p] = pays && pre_toks[p] > 0;
        };
        choose_joint();
        if (mixed) {
            plan.prefix_chunks.assign(d.num_prefixes, 1);
            plan.prefix_len.assign(d.prefix_len, d.prefix_len + d.num_prefixes);
            plan.chunk_len = std::max(0, rows_len);
            int64_t slots = 0;
            for (int32_t r = 0; r < B; ++r) {
                const int32_t pid = d.prefix_id ? d.prefix_id[r] : -1;
                const bool grouped = pid >= 0 && joint[pid];
                if (d.q_start[r + 1] - d.q_start[r] > 1) {
                    mixed &= !grouped || fused[pid];     // its rows read a state that an earlier launch has to leave
                } else {
                    const int32_t n = grouped + chunks_of(own_keys(r), plan.chunk_len);
                    if (n > 1) slots += n;
                }
            }
            mixed &= slots <= split_slot_cap(T);
            plan.use = mixed;
            if (!mixed) choose_joint();
        }
        std::vector<int32_t> row_slot;      // per request: its first slot (slot plans only)
        if (plan.use) {
            row_slot.resize(B);
            int32_t slots = 0;
            for (int32_t r = 0; r < B; ++r) {
                if (d.q_start[r + 1] - d.q_start[r] > 1) continue;
                const int32_t pid = d.prefix_id ? d.prefix_id[r] : -1;
                const int32_t n = (pid >= 0 && joint[pid] ? plan.prefix_chunks[pid] : 0) + chunks_of(own_keys(r), plan.chunk_len);
                row_slot[r] = slots;
                if (n > 1) slots += n;
            }
            if (!mixed) il.n_scratch_slots = slots;
        }
        il.in_slots = plan.use;
        auto joint_items = [&](int32_t p) {
            AttnItem it{};
            std::vector<int32_t> runs;   // request, end of keys, first token, tokens
            std::vector<int32_t> toks;
            auto close = [&] {
                if (toks.empty()) return;
                it.tok_off = (int32_t)il.attn_tok.size();
                it.n_tok = (int32_t)toks.size();
                il.attn_tok.insert(il.attn_tok.end(), toks.begin(), toks.end());
                it.bt_req = first_member[p];
                it.key_begin = 0;
                it.key_end = d.prefix_len[p];
                it.flags = ITEM_JOINT;
                it.pad0 = (int32_t)il.attn_tok.size();
                int32_t blocks = (d.prefix_len[p] + 63) / 64;
                for (size_t i = 0; i < runs.size(); i += 4) blocks += (runs[i + 1] - d.prefix_len[p] + 63) / 64;
                il.attn_tok.push_back(blocks);
                il.attn_tok.insert(il.attn_tok.end(), runs.begin(), runs.end());
                il.items_tile.push_back(it);
                runs.clear();
                toks.clear();
            };
            for (int32_t r = 0; r < B; ++r) {
                const int32_t q_len = d.q_start[r + 1] - d.q_start[r];
                if (d.prefix_id[r] != p || q_len == 1) continue;
                for (int32_t o = 0; o < q_len;) {
                    const int32_t n = std::min(q_len - o, tile_tok - (int32_t)toks.size());
                    runs.insert(runs.end(), {r, d.ctx_len[r] - q_len + o + n, (int32_t)toks.size(), n});
                    for (int32_t j = 0; j < n; ++j) toks.push_back(d.q_start[r] + o + j);
                    o += n;
                    if ((int32_t)toks.size() == tile_tok) close();
                }
            }
            close();
        };
        for (int32_t p = 0; p < d.num_prefixes; ++p) {
            if (!joint[p]) continue;
            ++hb.n_groups;
            if (fused[p]) joint_items(p), il.has_joint = true;
            auto in_pass = [&](int32_t r, int32_t p) { return d.prefix_id[r] == p && !(fused[p] && d.q_start[r + 1] - d.q_start[r] > 1); };
            const int32_t start = (int32_t)il.attn_tok.size();
            for (int32_t r = 0; r < B; ++r)
                if (in_pass(r, p))
                    for (int32_t t = d.q_start[r]; t < d.q_start[r + 1]; ++t) il.attn_tok.push_back(t);
            const int32_t n = (int32_t)il.attn_tok.size() - start;
            const int32_t slots = (int32_t)il.attn_tok.size();
            if (plan.use)
                for (int32_t r = 0; r < B; ++r)
                    if (in_pass(r, p)) il.attn_tok.push_back(row_slot[r]);
            const int32_t n_chunks = plan.use ? plan.prefix_chunks[p] : 1;
            const int32_t per = plan.use ? plan.prefix_len[p] : d.prefix_len[p];
            for (int32_t c = 0; c < n_chunks; ++c)
                for (int32_t o = 0; o < n; o += tile_tok) {
                    AttnItem it{};
                    it.tok_off = start + o;
                    it.n_tok = std::min(tile_tok, n - o);
                    it.bt_req = first_member[p];
                    it.key_begin = c * per;
                    it.key_end = std::min((c + 1) * per, d.prefix_len[p]);
                    it.flags = ITEM_WRITE_PARTIAL;
                    if (plan.use) {
                        it.flags |= ITEM_SLOTS;
                        it.pad0 = slots + o;
                        it.pad1 = c;
                    }
                    (mixed ? il.items_tile : il.items_prefix).push_back(it);
                }
        }
        const int32_t chunk_len = plan.use ? plan.chunk_len : std::max(0, rows_len);   // 0 = no row is cut
        int32_t next_slot = 0;
        for (int32_t r = 0; r < B; ++r) {
            const int32_t q_len = d.q_start[r + 1] - d.q_start[r];
            const int32_t pid = d.prefix_id ? d.prefix_id[r] : -1;
            const bool grouped = pid >= 0 && joint[pid];
            const int32_t kb = grouped ? d.prefix_len[pid] : 0;
            const int32_t flags = ITEM_CAUSAL | (grouped && !plan.use ? ITEM_INIT_PARTIAL : 0);
            const int32_t past = d.ctx_len[r] - q_len;
            if (q_len == 1) {
                const int32_t own = d.ctx_len[r] - kb;
                const int32_t n_chunks = chunks_of(own, chunk_len);
                const int32_t n_prefix = plan.use && grouped ? plan.prefix_chunks[pid] : 0;   // parts of the row another item computes
                // chunk boundaries on multiples of 32 keys (the wave kernel's block) counted from the first own key
                const int32_t per = n_chunks > 1 ? ((own + n_chunks - 1) / n_chunks + 31) / 32 * 32 : own;
                const bool parts = n_chunks + n_prefix > 1;
                if (plan.use) next_slot = row_slot[r] + n_prefix;
                if (parts) il.merge_items.push_back(MergeItem{d.q_start[r], plan.use ? row_slot[r] : next_slot, n_prefix, 0});
                for (int32_t c = 0; c < n_chunks; ++c) {
                    const int32_t b0 = kb + c * per, b1 = std::min(kb + (c + 1) * per, d.ctx_len[r]);
                    if (b0 >= b1) break;
                    AttnItem it{};
                    it.tok_off = (int32_t)il.attn_tok.size();
                    il.attn_tok.push_back(d.q_start[r]);
                    it.n_tok = 1;
                    it.pad0 = d.q_start[r];  // the decode kernel takes its single token from here
                    it.bt_req = r;
                    it.key_begin = b0;
                    it.key_end = b1;
                    it.flags = c == 0 ? flags : ITEM_CAUSAL;      // only the first chunk continues from the prefix pass's state
                    if (parts) {
                        it.flags |= ITEM_WRITE_PARTIAL;
                        it.pad1 = next_slot++;
                        ++il.merge_items.back().n_chunks;
                    }
                    il.items_split.push_back(it);
                }
            } else if (!(grouped && fused[pid])) {
                for (int32_t o = 0; o < q_len; o += tile_tok) {
                    AttnItem it{};
                    it.tok_off = (int32_t)il.attn_tok.size();
                    it.n_tok = std::min(tile_tok, q_len - o);
                    for (int32_t j = 0; j < it.n_tok; ++j) il.attn_tok.push_back(d.q_start[r] + o + j);
                    it.bt_req = r;
                    it.key_begin = kb;
                    it.key_end = past + o + it.n_tok;  // the item's last row sees keys up to itself
                    it.flags = flags;
                    il.items_tile.push_back(it);
                }
            }
        }
        // longest first: the tail of the launch then consists of short items
        auto keys = [&](const AttnItem& it) { return it.flags & ITEM_JOINT ? 64 * il.attn_tok[it.pad0] : it.key_end - it.key_begin; };
        auto longer = [&](const AttnItem& a, const AttnItem& b) { return keys(a) > keys(b); };
        std::stable_sort(il.items_tile.begin(), il.items_tile.end(), longer);
        std::stable_sort(il.items_split.begin(), il.items_split.end(), longer);
    };
    if (build_items) {
        build(true, hb.items);
        if (hb.items.in_slots) build(false, hb.no_slots);
    }
    *out = std::move(hb);
    return RELSERVE_OK;
}

// ------------------------------------------------------------------------------------------
// plain entry points
// ------------------------------------------------------------------------------------------
// The launchers report hipGetLastError() after a launch; an error an earlier, unrelated HIP call of this thread left
// behind (the runtime keeps the last one until it is read) must not be taken for theirs.
static inline void drop_stale_hip_error() { (void)hipGetLastError(); }

extern "C" {

int32_t relserve_version(void) { return 100; }

const char* relserve_strerror(int32_t s) {
    switch (s) {
        case RELSERVE_OK: return "ok";
        case RELSERVE_ERR_NULL_POINTER: return "null pointer";
        case RELSERVE_ERR_BAD_CONFIG: return "unsupported layer shape";
        case RELSERVE_ERR_BAD_Q_START: return "q_start must start at 0 and increase strictly";
        case RELSERVE_ERR_BAD_CTX_LEN: return "ctx_len shorter than the request's query tokens";
        case RELSERVE_ERR_BLOCK_TABLE_SHORT: return "block table row too short for ctx_len";
        case RELSERVE_ERR_PAGE_RANGE: return "block table entry outside the page pool";
        case RELSERVE_ERR_BAD_PREFIX: return "shared prefix inconsistent with the block tables";
        case RELSERVE_ERR_SLOT_ALIAS: return "two query tokens map to the same cache slot";
        case RELSERVE_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
        case RELSERVE_ERR_HIP: return "HIP runtime error";
        case RELSERVE_ERR_NO_DEVICE: return "no gfx950 device";
        case RELSERVE_ERR_TOO_LARGE: return "size exceeds 32-bit device indices or the fixed scratch";
        case RELSERVE_ERR_MISMATCH: return "batch / layer / cache do not belong together";
        case RELSERVE_ERR_BAD_ARGUMENT: return "bad argument";
        default: return "unknown status";
    }
}

int32_t relserve_config_validate(const relserve_layer_config* c) {
    if (!c) return RELSERVE_ERR_NULL_POINTER;
    if (c->hidden <= 0 || c->hidden % 8) return RELSERVE_ERR_BAD_CONFIG;
    if (c->mlp_dim <= 0 || c->mlp_dim % 8) return RELSERVE_ERR_BAD_CONFIG;
    if (c->head_dim != 64 && c->head_dim != 128) return RELSERVE_ERR_BAD_CONFIG;
    if (c->n_kv_heads <= 0 || c->n_q_heads <= 0 || c->n_q_heads % c->n_kv_heads) return RELSERVE_ERR_BAD_CONFIG;
    if (c->n_q_heads / c->n_kv_heads > ATTN_SPLIT_ROWS) return RELSERVE_ERR_BAD_CONFIG;  // one wave's query rows
    if (!is_pow2(c->page_size) || c->page_size < 8 || c->page_size > 256) return RELSERVE_ERR_BAD_CONFIG;
    if (!(c->rms_eps >= 0.0f) || !(c->rope_base > 0.0f)) return RELSERVE_ERR_BAD_CONFIG;
    return RELSERVE_OK;
}

int32_t relserve_layer_create(const relserve_layer_config* cfg, relserve_layer** out) {
    if (!cfg || !out) return RELSERVE_ERR_NULL_POINTER;
    *out = nullptr;
    if (int32_t rc = relserve_config_validate(cfg)) return rc;
    relserve_layer* L = new (std::nothrow) relserve_layer();
    if (!L) return RELSERVE_ERR_BAD_ARGUMENT;
    L->cfg = *cfg;
    L->group = cfg->n_q_heads / cfg->n_kv_heads;
    L->q_dim = cfg->n_q_heads * cfg->head_dim;
    L->kv_dim = cfg->n_kv_heads * cfg->head_dim;
    L->qkv_dim = L->q_dim + 2 * L->kv_dim;
    const int half = cfg->head_dim / 2;
    L->inv_freq.resize(half);
    for (int i = 0; i < half; ++i)
        L->inv_freq[i] = (float)std::pow((double)cfg->rope_base, -2.0 * i / (double)cfg->head_dim);
    count_layer(1);
    *out = L;
    return RELSERVE_OK;
}

int32_t relserve_layer_destroy(relserve_layer* L) {
    if (!L) return RELSERVE_OK;
    for (auto& p : L->pending) {
        (void)hipEventDestroy(p.a);
        (void)hipEventDestroy(p.b);
    }
    for (hipEvent_t e : L->event_pool) (void)hipEventDestroy(e);
    delete L;
    count_layer(-1);
    return RELSERVE_OK;
}

int32_t relserve_batch_validate(const relserve_layer_config* cfg, const relserve_batch_desc* desc) {
    if (!cfg || !desc) return RELSERVE_ERR_NULL_POINTER;
    if (int32_t rc = relserve_config_validate(cfg)) return rc;
    HostBatch hb;
    return expand_batch(*cfg, *desc, false, &hb);
}

int32_t relserve_batch_slots(const relserve_layer_config* cfg, const relserve_batch_desc* desc,
                             int32_t* slots_out) {
    if (!cfg || !desc || !slots_out) return RELSERVE_ERR_NULL_POINTER;
    if (int32_t rc = relserve_config_validate(cfg)) return rc;
    HostBatch hb;
    if (int32_t rc = expand_batch(*cfg, *desc, false, &hb)) return rc;
    std::memcpy(slots_out, hb.tok_slot.data(), sizeof(int32_t) * hb.tok_slot.size());
    return RELSERVE_OK;
}

int32_t relserve_batch_prepare(const relserve_layer* L, const relserve_batch_desc* desc, void* stream,
                               relserve_batch** out) {
    drop_stale_hip_error();
    if (!L || !desc || !out) return RELSERVE_ERR_NULL_POINTER;
    *out = nullptr;
    HostBatch hb;
    if (int32_t rc = expand_batch(L->cfg, *desc, true, &hb)) return rc;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev == 0) return RELSERVE_ERR_NO_DEVICE;
    int dev = 0;
    {
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess)
            return RELSERVE_ERR_HIP;
        if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0) return RELSERVE_ERR_NO_DEVICE;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int32_t T = hb.T, B = desc->num_reqs, half = L->cfg.head_dim / 2;

    // one host blob, one device allocation
    size_t off = 0;
    auto reserve = [&](size_t bytes) { size_t o = off; off += align_up(bytes ? bytes : 1); return o; };
    const size_t o_req = reserve(sizeof(int32_t) * T), o_pos = reserve(sizeof(int32_t) * T);
    const size_t o_slot = reserve(sizeof(int32_t) * T);
    const size_t o_last = reserve(sizeof(int32_t) * B);
    const size_t o_bt = reserve(sizeof(int32_t) * (size_t)B * desc->max_blocks);
    struct ListOffsets { size_t tok, prefix, tile, split, merge; };
    auto reserve_lists = [&](const ItemLists& il) {
        ListOffsets o;
        o.tok = reserve(sizeof(int32_t) * il.attn_tok.size());
        o.prefix = reserve(sizeof(AttnItem) * il.items_prefix.size());
        o.tile = reserve(sizeof(AttnItem) * il.items_tile.size());
        o.split = reserve(sizeof(AttnItem) * il.items_split.size());
        o.merge = reserve(sizeof(MergeItem) * il.merge_items.size());
        return o;
    };
    const ListOffsets o_items = reserve_lists(hb.items), o_seq = reserve_lists(hb.no_slots);
    const size_t o_freq = reserve(sizeof(float) * half);
    const size_t host_bytes = off;
    const size_t o_cs = reserve(sizeof(float2) * (size_t)T * half);
    const size_t total = off;

    std::vector<char> host(host_bytes, 0);
    auto put = [&](size_t o, const void* src, size_t bytes) { if (bytes) std::memcpy(host.data() + o, src, bytes); };
    put(o_req, hb.tok_req.data(), sizeof(int32_t) * T);
    put(o_pos, hb.tok_pos.data(), sizeof(int32_t) * T);
    put(o_slot, hb.tok_slot.data(), sizeof(int32_t) * T);
    {
        std::vector<int32_t> last(B);
        for (int32_t r = 0; r < B; ++r) last[r] = desc->q_start[r + 1] - 1;
        put(o_last, last.data(), sizeof(int32_t) * B);
    }
    put(o_bt, desc->block_table, sizeof(int32_t) * (size_t)B * desc->max_blocks);
    auto put_lists = [&](const ListOffsets& o, const ItemLists& il) {
        put(o.tok, il.attn_tok.data(), sizeof(int32_t) * il.attn_tok.size());
        put(o.prefix, il.items_prefix.data(), sizeof(AttnItem) * il.items_prefix.size());
        put(o.tile, il.items_tile.data(), sizeof(AttnItem) * il.items_tile.size());
        put(o.split, il.items_split.data(), sizeof(AttnItem) * il.items_split.size());
        put(o.merge, il.merge_items.data(), sizeof(MergeItem) * il.merge_items.size());
    };
    put_lists(o_items, hb.items);
    put_lists(o_seq, hb.no_slots);
    put(o_freq, L->inv_freq.data(), sizeof(float) * half);

    relserve_batch* b = new (std::nothrow) relserve_batch();
    if (!b) return RELSERVE_ERR_BAD_ARGUMENT;
    b->cfg = L->cfg;
    b->device = dev;
    b->other_stream = stream != nullptr;
    SpareBlob spare{};
    if (take_spare_blob(total, dev, &spare)) {
        b->blob = spare.blob;
        b->blob_bytes = spare.bytes;
        b->idle = spare.idle;
    } else {
        b->blob_bytes = 65536;   // sizes that fit again: powers of two
        while (b->blob_bytes < total) b->blob_bytes *= 2;
        if (b->blob_bytes > kSpareBlobBytes) b->blob_bytes = total;
        hipError_t got = hipMalloc(&b->blob, b->blob_bytes);
        if (got != hipSuccess) {   // the spare ones may be what is missing
            (void)hipGetLastError();
            free_spare_blobs();
            got = hipMalloc(&b->blob, b->blob_bytes);
        }
        if (got != hipSuccess) {
            delete b;
            return RELSERVE_ERR_HIP;
        }
    }
    char* base = static_cast<char*>(b->blob);
    BatchDev& dv = b->dev;
    dv.T = T;
    dv.num_reqs = B;
    dv.max_blocks = desc->max_blocks;
    dv.num_pages = desc->num_pages;
    dv.tok_req = reinterpret_cast<int32_t*>(base + o_req);
    dv.tok_pos = reinterpret_cast<int32_t*>(base + o_pos);
    dv.tok_slot = reinterpret_cast<int32_t*>(base + o_slot);
    dv.last_tok = reinterpret_cast<int32_t*>(base + o_last);
    dv.block_table = reinterpret_cast<int32_t*>(base + o_bt);
    dv.rope_cs = reinterpret_cast<float2*>(base + o_cs);
    auto view_lists = [&](BatchDev& v, const ListOffsets& o, const ItemLists& il) {
        v.attn_tok = reinterpret_cast<int32_t*>(base + o.tok);
        v.items_prefix = reinterpret_cast<AttnItem*>(base + o.prefix);
        v.items_tile = reinterpret_cast<AttnItem*>(base + o.tile);
        v.items_split = reinterpret_cast<AttnItem*>(base + o.split);
        v.merge_items = reinterpret_cast<MergeItem*>(base + o.merge);
        v.n_items_prefix = (int32_t)il.items_prefix.size();
        v.n_items_tile = (int32_t)il.items_tile.size();
        v.n_items_split = (int32_t)il.items_split.size();
        v.n_merge = (int32_t)il.merge_items.size();
        v.has_joint = il.has_joint;
        v.n_scratch_slots = il.n_scratch_slots;
    };
    view_lists(dv, o_items, hb.items);
    b->dev_no_slots = dv;
    if (hb.items.in_slots) view_lists(b->dev_no_slots, o_seq, hb.no_slots);
    b->info = relserve_batch_info{T, B, hb.n_decode, hb.n_prefill, hb.n_groups,
                                  dv.n_items_prefix + dv.n_items_tile + dv.n_items_split};

    hipError_t e = hipMemcpyAsync(b->blob, host.data(), host_bytes, hipMemcpyHostToDevice, s);
    if (e == hipSuccess && T > 0)
        e = launch_rope_table(dv.tok_pos, reinterpret_cast<float*>(base + o_freq), T, half,
                              reinterpret_cast<float2*>(base + o_cs), s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        (void)free_blob(SpareBlob{b->blob, 0, 0, b->idle});
        delete b;
        return RELSERVE_ERR_HIP;
    }
    *out = b;
    return RELSERVE_OK;
}

int32_t relserve_batch_destroy(relserve_batch* b) {
    if (!b) return RELSERVE_OK;
    SpareBlob blob{b->blob, b->blob_bytes, b->device, b->idle};
    const bool kept = b->blob && !b->other_stream.load(std::memory_order_relaxed) && give_spare_blob(blob);
    const hipError_t e = kept ? hipSuccess : free_blob(blob);
    delete b;
    return e == hipSuccess ? RELSERVE_OK : RELSERVE_ERR_HIP;
}

int32_t relserve_batch_get_info(const relserve_batch* b, relserve_batch_info* out) {
    if (!b || !out) return RELSERVE_ERR_NULL_POINTER;
    *out = b->info;
    return RELSERVE_OK;
}

int32_t relserve_workspace_bytes(const relserve_layer* L, int32_t max_tokens, size_t* out) {
    if (!L || !out) return RELSERVE_ERR_NULL_POINTER;
    if (max_tokens < 0) return RELSERVE_ERR_BAD_ARGUMENT;
    *out = carve(*L, max_tokens, nullptr).total + kAlign;
    return RELSERVE_OK;
}

int32_t relserve_kv_append(const relserve_layer* L, const relserve_batch* b, const void* k, const void* v,
                           relserve_kv_cache cache, void* stream) {
    drop_stale_hip_error();
    if (int32_t rc = check_pair(L, b, stream)) return rc;
    if (int32_t rc = check_cache(b, cache, false)) return rc;
    if (b->dev.T == 0) return RELSERVE_OK;
    if (!k || !v) return RELSERVE_ERR_NULL_POINTER;
    hipError_t e = launch_kv_append(b->dev, k, v, cache.k_pages, cache.v_pages, L->kv_dim,
                                    static_cast<hipStream_t>(stream));
    return e == hipSuccess ? RELSERVE_OK : RELSERVE_ERR_HIP;
}

int32_t relserve_rmsnorm(const void* x, int32_t x_is_f32, const void* w, float eps, int32_t n_rows,
                         int32_t hidden, void* out, void* stream) {
    drop_stale_hip_error();
    if (n_rows < 0 || hidden <= 0 || hidden % 8) return RELSERVE_ERR_BAD_ARGUMENT;
    if (n_rows == 0) return RELSERVE_OK;
    if (!x || !w || !out) return RELSERVE_ERR_NULL_POINTER;
    hipError_t e = launch_rmsnorm(x, x_is_f32 != 0, w, eps, n_rows, hidden, out, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? RELSERVE_OK : RELSERVE_ERR_HIP;
}

namespace {
int32_t linear_entry(const void* a, const void* w, int32_t T, int32_t N, int32_t K, int32_t epilogue,
                     const void* residual, void* out, void* stream, bool packed) {
    if (T < 0 || N <= 0 || K <= 0 || K % 8 || epilogue < 0 || epilogue > 3) return RELSERVE_ERR_BAD_ARGUMENT;
    if (epilogue == 3 ? (N % 16) : (N % 4)) return RELSERVE_ERR_BAD_ARGUMENT;
    if (packed && K % 64) return RELSERVE_ERR_BAD_ARGUMENT;
    const int64_t n_rows = packed ? ((int64_t)N + 255) / 256 * 256 : N;
    if ((int64_t)T * K >= ((int64_t)1 << 31) || n_rows * K >= ((int64_t)1 << 31)) return RELSERVE_ERR_TOO_LARGE;
    if (T == 0) return RELSERVE_OK;
    if (!a || !w || !out) return RELSERVE_ERR_NULL_POINTER;
    if (epilogue == 2 && !residual) return RELSERVE_ERR_NULL_POINTER;
    hipError_t e = launch_linear(a, w, T, N, K, epilogue, residual, out, static_cast<hipStream_t>(stream), nullptr, packed);
    return e == hipSuccess ? RELSERVE_OK : RELSERVE_ERR_HIP;
}
}  // namespace

int32_t relserve_linear(const void* a, const void* w, int32_t T, int32_t N, int32_t K, int32_t epilogue,
                        const void* residual, void* out, void* stream) {
    drop_stale_hip_error();
    return linear_entry(a, w, T, N, K, epilogue, residual, out, stream, false);
}

int32_t relserve_linear_packed(const void* a, const void* w_packed, int32_t T, int32_t N, int32_t K, int32_t epilogue,
                               const void* residual, void* out, void* stream) {
    drop_stale_hip_error();
    return linear_entry(a, w_packed, T, N, K, epilogue, residual, out, stream, true);
}

int32_t relserve_packed_weight_elems(int32_t N, int32_t K, int64_t* out) {
    if (!out) return RELSERVE_ERR_NULL_POINTER;
    if (N <= 0 || K <= 0 || K % 64) return RELSERVE_ERR_BAD_ARGUMENT;
    *out = ((int64_t)N + 255) / 256 * 256 * K;
    return *out >= ((int64_t)1 << 31) ? RELSERVE_ERR_TOO_LARGE : RELSERVE_OK;
}

int32_t relserve_pack_weight(const void* w, int32_t N, int32_t K, void* out, void* stream) {
    drop_stale_hip_error();
    int64_t elems = 0;
    if (int32_t rc = relserve_packed_weight_elems(N, K, &elems)) return rc;
    if (!w || !out) return RELSERVE_ERR_NULL_POINTER;
    return launch_pack_weight(w, N, K, out, static_cast<hipStream_t>(stream)) == hipSuccess ? RELSERVE_OK
                                                                                              : RELSERVE_ERR_HIP;
}

int32_t relserve_rope_append(const relserve_layer* L, const relserve_batch* b, void* qkv,
                             relserve_kv_cache cache, void* stream) {
    drop_stale_hip_error();
    if (int32_t rc = check_pair(L, b, stream)) return rc;
    if (int32_t rc = check_cache(b, cache, false)) return rc;
    if (b->dev.T == 0) return RELSERVE_OK;
    if (!qkv) return RELSERVE_ERR_NULL_POINTER;
    hipError_t e = launch_rope_append(b->dev, *L, qkv, cache.k_pages, cache.v_pages, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? RELSERVE_OK : RELSERVE_ERR_HIP;
}

int32_t relserve_qkv_rope_append(const relserve_layer* L, const relserve_batch* b, const void* h, const void* w_qkv,
                                 void* q_out, relserve_kv_cache cache, void* stream) {
    drop_stale_hip_error();
    if (int32_t rc = check_pair(L, b, stream)) return rc;
    if (int32_t rc = check_cache(b, cache)) return rc;
    if (b->dev.T == 0) return RELSERVE_OK;
    if (!h || !w_qkv || !q_out) return RELSERVE_ERR_NULL_POINTER;
    hipError_t e = launch_qkv_rope_append(b->dev, *L, h, w_qkv, q_out, cache.k_pages, cache.v_pages,
                                          static_cast<hipStream_t>(stream), nullptr, false, kv_format(cache));
    return e == hipSuccess ? RELSERVE_OK : RELSERVE_ERR_HIP;
}

int32_t relserve_attention(const relserve_layer* L, const relserve_batch* b, const void* q, int32_t q_pitch,
                           relserve_kv_cache cache, void* out, void* workspace, size_t workspace_bytes,
                           void* stream) {
    drop_stale_hip_error();
    if (int32_t rc = check_pair(L, b, stream)) return rc;
    if (int32_t rc = check_cache(b, cache)) return rc;
    if (b->dev.T == 0) return RELSERVE_OK;
    if (!q || !out) return RELSERVE_ERR_NULL_POINTER;
    if (q_pitch < L->q_dim || q_pitch % 8) return RELSERVE_ERR_BAD_ARGUMENT;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) % kAlign)) return RELSERVE_ERR_WORKSPACE;
    Workspace w = carve(*L, b->dev.T, workspace);
    if (w.total > workspace_bytes) return RELSERVE_ERR_WORKSPACE;
    const BatchDev& batch = attention_batch(*b, cache);
    const PartialState part = partial_state(*L, batch, w);
    hipError_t e = launch_attention(batch, *L, q, q_pitch, cache.k_pages, cache.v_pages, out, part.o,
                                    part.ml, static_cast<hipStream_t>(stream), nullptr, kv_format(cache));
    return e == hipSuccess ? RELSERVE_OK : RELSERVE_ERR_HIP;
}

namespace {
// One layer step.  In a stack, `normed` says that the layer before has already normed this layer's input into the workspace,
// and `next` names the norm that reads this layer's output (its `out` is the workspace's too).
int32_t layer_step(const relserve_layer* L, const relserve_batch* b, const relserve_layer_weights* wt, const void* x, void* y,
                   relserve_kv_cache cache, void* workspace, size_t workspace_bytes, void* stream, bool normed, NextNorm* next) {
    if (int32_t rc = check_pair(L, b, stream)) return rc;
    if (!wt) return RELSERVE_ERR_NULL_POINTER;
    if (int32_t rc = check_cache(b, cache)) return rc;
    const int32_t T = b->dev.T;
    if (T == 0) return RELSERVE_OK;
    if (!x || !y || !wt->w_in_norm || !wt->w_qkv || !wt->w_o || !wt->w_post_norm || !wt->w_gate_up || !wt->w_down)
        return RELSERVE_ERR_NULL_POINTER;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) % kAlign)) return RELSERVE_ERR_WORKSPACE;
    Workspace w = carve(*L, T, workspace);
    if (w.total > workspace_bytes) return RELSERVE_ERR_WORKSPACE;
    const bool packed = wt->packed != 0;
    if (packed && (L->cfg.hidden % 64 || L->q_dim % 64 || L->cfg.mlp_dim % 64)) return RELSERVE_ERR_BAD_ARGUMENT;

    hipStream_t s = static_cast<hipStream_t>(stream);
    const relserve_layer_config& c = L->cfg;
    relserve_layer* prof = L->profile ? const_cast<relserve_layer*>(L) : nullptr;
    hipError_t e = hipSuccess;
    auto run = [&](int slot, auto&& launch) {
        if (e != hipSuccess) return;
        profile_mark(prof, slot, s, true);
        e = launch();
        profile_mark(prof, slot, s, false);
    };
    // the GEMMs split K across workgroups (whole skinny problems, narrow outputs at mid-size T, or the
    // incomplete last round of tiles) through an fp32 scratch that they write before they read
    float* accum = w.accum;
    const BatchDev& batch = attention_batch(*b, cache);
    const PartialState part = partial_state(*L, batch, w);
    const KvFormat kv = kv_format(cache);
    if (!normed) run(S_NORM1, [&] { return launch_rmsnorm(x, false, wt->w_in_norm, c.rms_eps, T, c.hidden, w.h, s); });
    run(S_QKV, [&] {
        return launch_qkv_rope_append(b->dev, *L, w.h, wt->w_qkv, w.q, cache.k_pages, cache.v_pages, s, accum, packed, kv);
    });
    if (e == hipSuccess)
        e = launch_attention(batch, *L, w.q, L->q_dim, cache.k_pages, cache.v_pages, w.attn, part.o, part.ml, s, prof, kv);
    NextNorm post{wt->w_post_norm, c.rms_eps, w.h};
    const CodeScales o{nullptr, 1.0f, 0.0f, &post}, down{nullptr, 1.0f, 0.0f, next};   // 16-bit operands
    run(S_O, [&] { return launch_linear(w.attn, wt->w_o, T, c.hidden, L->q_dim, 1, x, w.x1, s, accum, packed, &o); });
    if (!post.done) run(S_NORM2, [&] { return launch_rmsnorm(w.x1, true, wt->w_post_norm, c.rms_eps, T, c.hidden, w.h, s); });
    run(S_GU, [&] {
        return launch_linear(w.h, wt->w_gate_up, T, 2 * c.mlp_dim, c.hidden, 3, nullptr, w.act, s, accum, packed);
    });
    if (next) next->out = w.h;   // free by now: the gate/up projection has read it
    run(S_DOWN, [&] { return launch_linear(w.act, wt->w_down, T, c.hidden, c.mlp_dim, 2, w.x1, y, s, accum, packed, &down); });
    return e == hipSuccess ? RELSERVE_OK : RELSERVE_ERR_HIP;
}

int32_t layer_step_codes(const relserve_layer* L, const relserve_batch* b, const relserve_layer_weights_w8a8* wt, const void* x, void* y,
                         relserve_kv_cache cache, void* workspace, size_t workspace_bytes, void* stream, bool normed, NextNorm* next) {
    if (int32_t rc = check_pair(L, b, stream)) return rc;
    if (!wt) return RELSERVE_ERR_NULL_POINTER;
    if (int32_t rc = check_cache(b, cache)) return rc;
    const relserve_layer_config& c = L->cfg;
    if (c.hidden % 128 || L->q_dim % 128 || c.mlp_dim % 128) return RELSERVE_ERR_BAD_ARGUMENT;
    for (float a : {wt->a_qkv, wt->a_o, wt->a_gate_up, wt->a_down})
        if (!(a > 0.0f) || !std::isfinite(a)) return RELSERVE_ERR_BAD_ARGUMENT;
    const int32_t T = b->dev.T;
    if (T == 0) return RELSERVE_OK;
    if (!x || !y || !wt->w_in_norm || !wt->w_qkv || !wt->w_o || !wt->w_post_norm || !wt->w_gate_up || !wt->w_down ||
        !wt->s_qkv || !wt->s_o || !wt->s_gate_up || !wt->s_down)
        return RELSERVE_ERR_NULL_POINTER;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) % kAlign)) return RELSERVE_ERR_WORKSPACE;
    Workspace w = carve(*L, T, workspace);   // the 16-bit step's buffers hold the codes too (half of each is used)
    if (w.total > workspace_bytes) return RELSERVE_ERR_WORKSPACE;
    const bool packed = wt->packed != 0;

    hipStream_t s = static_cast<hipStream_t>(stream);
    relserve_layer* prof = L->profile ? const_cast<relserve_layer*>(L) : nullptr;
    hipError_t e = hipSuccess;
    auto run = [&](int slot, auto&& launch) {
        if (e != hipSuccess) return;
        profile_mark(prof, slot, s, true);
        e = launch();
        profile_mark(prof, slot, s, false);
    };
    float* accum = w.accum;
    // Codes amplify: an attention output that rounds differently by 1e-3 moves about 2 % of W_o's inputs to the neighbouring
    // code, and a wide layer's output by up to 7e-3.  The attention is therefore cut as it is over quantised pools.
    const BatchDev& batch = b->dev_no_slots;
    const PartialState part = partial_state(*L, batch, w);
    NextNorm post{wt->w_post_norm, c.rms_eps, w.h, wt->a_gate_up};
    const CodeScales qkv{wt->s_qkv, wt->a_qkv}, o{wt->s_o, wt->a_o, 0.0f, &post}, gu{wt->s_gate_up, wt->a_gate_up, wt->a_down},
        down{wt->s_down, wt->a_down, 0.0f, next};
    KvFormat attn = kv_format(cache);
    attn.out_scale = wt->a_o;
    if (!normed) run(S_NORM1, [&] { return launch_rmsnorm(x, false, wt->w_in_norm, c.rms_eps, T, c.hidden, w.h, s, nullptr, wt->a_qkv); });
    run(S_QKV, [&] {
        return launch_qkv_rope_append(b->dev, *L, w.h, wt->w_qkv, w.q, cache.k_pages, cache.v_pages, s, accum, packed,
                                      kv_format(cache), &qkv);
    });
    if (e == hipSuccess)
        e = launch_attention(batch, *L, w.q, L->q_dim, cache.k_pages, cache.v_pages, w.attn, part.o,
                             part.ml, s, prof, attn);
    run(S_O, [&] { return launch_linear(w.attn, wt->w_o, T, c.hidden, L->q_dim, 1, x, w.x1, s, accum, packed, &o); });
    if (!post.done)
        run(S_NORM2, [&] { return launch_rmsnorm(w.x1, true, wt->w_post_norm, c.rms_eps, T, c.hidden, w.h, s, nullptr, wt->a_gate_up); });
    run(S_GU, [&] {
        return launch_linear(w.h, wt->w_gate_up, T, 2 * c.mlp_dim, c.hidden, 3, nullptr, w.act, s, accum, packed, &gu);
    });
    if (next) next->out = w.h;   // free by now: the gate/up projection has read it
    run(S_DOWN, [&] { return launch_linear(w.act, wt->w_down, T, c.hidden, c.mlp_dim, 2, w.x1, y, s, accum, packed, &down); });
    return e == hipSuccess ? RELSERVE_OK : RELSERVE_ERR_HIP;
}
}  // namespace

int32_t relserve_layer_step(const relserve_layer* L, const relserve_batch* b, const relserve_layer_weights* wt,
                            const void* x, void* y, relserve_kv_cache cache, void* workspace,
                            size_t workspace_bytes, void* stream) {
    drop_stale_hip_error();
    return layer_step(L, b, wt, x, y, cache, workspace, workspace_bytes, stream, false, nullptr);
}

int32_t relserve_layer_step_w8a8(const relserve_layer* L, const relserve_batch* b, const relserve_layer_weights_w8a8* wt,
                                 const void* x, void* y, relserve_kv_cache cache, void* workspace,
                                 size_t workspace_bytes, void* stream) {
    drop_stale_hip_error();
    return layer_step_codes(L, b, wt, x, y, cache, workspace, workspace_bytes, stream, false, nullptr);
}

int32_t relserve_rmsnorm_codes(const void* x, int32_t x_is_f32, const void* w, float eps, int32_t n_rows,
                               int32_t hidden, float scale, void* out, void* stream) {
    drop_stale_hip_error();
    if (n_rows < 0 || hidden <= 0 || hidden % 8 || !(scale > 0.0f) || !std::isfinite(scale)) return RELSERVE_ERR_BAD_ARGUMENT;
    if (n_rows == 0) return RELSERVE_OK;
    if (!x || !w || !out) return RELSERVE_ERR_NULL_POINTER;
    hipError_t e = launch_rmsnorm(x, x_is_f32 != 0, w, eps, n_rows, hidden, out, static_cast<hipStream_t>(stream), nullptr, scale);
    return e == hipSuccess ? RELSERVE_OK : RELSERVE_ERR_HIP;
}

int32_t relserve_quantise_bf16(const void* in, int64_t n, float scale, void* codes, void* stream) {
    drop_stale_hip_error();
    if (n < 0 || n % 8 || !(scale > 0.0f) || !std::isfinite(scale)) return RELSERVE_ERR_BAD_ARGUMENT;
    if (n == 0) return RELSERVE_OK;
    if (!in || !codes) return RELSERVE_ERR_NULL_POINTER;
    return launch_quantise_bf16(in, n, scale, codes, static_cast<hipStream_t>(stream)) == hipSuccess ? RELSERVE_OK : RELSERVE_ERR_HIP;
}

int32_t relserve_linear_w8a8(const void* a, const void* w, const float* w_scale, float a_scale, int32_t T, int32_t N,
                             int32_t K, int32_t epilogue, const void* residual, void* out, float out_scale,
                             int32_t packed, void* stream) {
    drop_stale_hip_error();
    if (T < 0 || N <= 0 || K <= 0 || K % 128 || epilogue < 0 || epilogue > 3) return RELSERVE_ERR_BAD_ARGUMENT;
    if (epilogue != 3 && N % 4) return RELSERVE_ERR_BAD_ARGUMENT;
    if (epilogue == 3 && N % 16) return RELSERVE_ERR_BAD_ARGUMENT;
    if (!(a_scale > 0.0f) || !std::isfinite(a_scale) || out_scale < 0.0f || !std::isfinite(out_scale)) return RELSERVE_ERR_BAD_ARGUMENT;
    if (out_scale > 0.0f && epilogue != 3) return RELSERVE_ERR_BAD_ARGUMENT;
    if (T == 0) return RELSERVE_OK;
    if (!a || !w || !w_scale || !out) return RELSERVE_ERR_NULL_POINTER;
    if (epilogue == 2 && !residual) return RELSERVE_ERR_NULL_POINTER;
    const CodeScales codes{w_scale, a_scale, out_scale};
    hipError_t e = launch_linear(a, w, T, N, K, epilogue, residual, out, static_cast<hipStream_t>(stream), nullptr, packed != 0, &codes);
    return e == hipSuccess ? RELSERVE_OK : RELSERVE_ERR_HIP;
}

int32_t relserve_static_scratch_bytes(size_t* out) {
    if (!out) return RELSERVE_ERR_NULL_POINTER;
    *out = kStaticScratchBytes;
    return RELSERVE_OK;
}

int32_t relserve_layer_step_static(const relserve_layer* L, const relserve_batch* b, const relserve_layer_weights* wt,
                                   const void* x, void* y, relserve_kv_cache cache, void* stream) {
    drop_stale_hip_error();
    if (int32_t rc = check_pair(L, b, stream)) return rc;
    if (carve(*L, b->dev.T, nullptr).total > kStaticScratchBytes) return RELSERVE_ERR_TOO_LARGE;
    void* ws = nullptr;
    if (int32_t rc = static_scratch(&ws)) return rc;
    return relserve_layer_step(L, b, wt, x, y, cache, ws, kStaticScratchBytes, stream);
}

int32_t relserve_model_workspace_bytes(const relserve_layer* L, int32_t max_tokens, int32_t max_reqs, size_t* out) {
    if (!L || !out) return RELSERVE_ERR_NULL_POINTER;
    if (max_tokens < 0 || max_reqs < 0) return RELSERVE_ERR_BAD_ARGUMENT;
    *out = carve(*L, max_tokens, nullptr).total + align_up((size_t)max_tokens * L->cfg.hidden * 2) +
           align_up((size_t)max_reqs * L->cfg.hidden * 2) + kAlign;
    return RELSERVE_OK;
}

namespace {
// q8 != nullptr: every layer runs relserve_layer_step_w8a8 on q8[l] instead of relserve_layer_step on m->layers[l]
int32_t model_step(const relserve_layer* L, const relserve_batch* b, const relserve_model* m,
                   const relserve_layer_weights_w8a8* q8, const int32_t* token_ids, void* logits, void* workspace,
                   size_t workspace_bytes, void* stream) {
    if (int32_t rc = check_pair(L, b, stream)) return rc;
    if (!m) return RELSERVE_ERR_NULL_POINTER;
    if (m->n_layers < 0 || m->vocab <= 0 || m->vocab % 4) return RELSERVE_ERR_BAD_ARGUMENT;
    const int32_t T = b->dev.T, B = b->dev.num_reqs, H = L->cfg.hidden;
    if (T == 0) return RELSERVE_OK;
    if (!token_ids || !logits || !m->embedding || !m->w_final_norm || !m->w_lm_head) return RELSERVE_ERR_NULL_POINTER;
    if (m->n_layers > 0 && ((!q8 && !m->layers) || !m->caches)) return RELSERVE_ERR_NULL_POINTER;
    for (int32_t l = 0; l < m->n_layers; ++l) {
        if (!q8) {
            const relserve_layer_weights& w = m->layers[l];
            if (!w.w_in_norm || !w.w_qkv || !w.w_o || !w.w_post_norm || !w.w_gate_up || !w.w_down)
                return RELSERVE_ERR_NULL_POINTER;
        }
        if (int32_t rc = check_cache(b, m->caches[l])) return rc;
    }
    if ((int64_t)m->vocab * H >= ((int64_t)1 << 31)) return RELSERVE_ERR_TOO_LARGE;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) % kAlign)) return RELSERVE_ERR_WORKSPACE;
    const size_t layer_ws = carve(*L, T, nullptr).total;
    const size_t x_bytes = align_up((size_t)T * H * 2), last_bytes = align_up((size_t)B * H * 2);
    if (layer_ws + x_bytes + last_bytes > workspace_bytes) return RELSERVE_ERR_WORKSPACE;
    char* x = static_cast<char*>(workspace) + layer_ws;
    char* h_last = x + x_bytes;

    hipStream_t s = static_cast<hipStream_t>(stream);
    if (launch_embedding(token_ids, m->embedding, m->vocab, H, T, x, s) != hipSuccess) return RELSERVE_ERR_HIP;
    bool normed = false;
    for (int32_t l = 0; l < m->n_layers; ++l) {   // the residual stream stays in x, rounded to bf16 between layers
        // the next layer's input norm, if that layer can be stepped at all (what is wrong with it is for its own step to say)
        NextNorm nn;
        bool have_next = l + 1 < m->n_layers;
        if (have_next && q8) {
            nn = NextNorm{q8[l + 1].w_in_norm, L->cfg.rms_eps, nullptr, q8[l + 1].a_qkv};
            have_next = nn.w && nn.code_scale > 0.0f && std::isfinite(nn.code_scale);
        } else if (have_next) {
            nn = NextNorm{m->layers[l + 1].w_in_norm, L->cfg.rms_eps};
        }
        NextNorm* next = have_next ? &nn : nullptr;
        const int32_t rc = q8 ? layer_step_codes(L, b, &q8[l], x, x, m->caches[l], workspace, layer_ws, stream, normed, next)
                              : layer_step(L, b, &m->layers[l], x, x, m->caches[l], workspace, layer_ws, stream, normed, next);
        if (rc) return rc;
        normed = nn.done;
    }
    if (launch_rmsnorm(x, false, m->w_final_norm, L->cfg.rms_eps, B, H, h_last, s, b->dev.last_tok) != hipSuccess)
        return RELSERVE_ERR_HIP;
    if (launch_linear(h_last, m->w_lm_head, B, m->vocab, H, 1, nullptr, logits, s) != hipSuccess)
        return RELSERVE_ERR_HIP;
    return RELSERVE_OK;
}
}  // namespace

int32_t relserve_model_step(const relserve_layer* L, const relserve_batch* b, const relserve_model* m,
                            const int32_t* token_ids, void* logits, void* workspace, size_t workspace_bytes,
                            void* stream) {
    drop_stale_hip_error();
    return model_step(L, b, m, nullptr, token_ids, logits, workspace, workspace_bytes, stream);
}

int32_t relserve_model_step_w8a8(const relserve_layer* L, const relserve_batch* b, const relserve_model* m,
                                 const relserve_layer_weights_w8a8* layers, const int32_t* token_ids, void* logits,
                                 void* workspace, size_t workspace_bytes, void* stream) {
    drop_stale_hip_error();
    if (!layers) return RELSERVE_ERR_NULL_POINTER;
    return model_step(L, b, m, layers, token_ids, logits, workspace, workspace_bytes, stream);
}

int32_t relserve_greedy_sample(const void* logits, int32_t n_rows, int32_t vocab, int32_t* next_token, void* stream) {
    drop_stale_hip_error();
    if (n_rows < 0 || vocab <= 0) return RELSERVE_ERR_BAD_ARGUMENT;
    if (n_rows == 0) return RELSERVE_OK;
    if (!logits || !next_token) return RELSERVE_ERR_NULL_POINTER;
    if (reinterpret_cast<uintptr_t>(logits) % 4) return RELSERVE_ERR_BAD_ARGUMENT;
    return launch_greedy_sample(static_cast<const float*>(logits), n_rows, vocab, next_token,
                                static_cast<hipStream_t>(stream)) == hipSuccess
               ? RELSERVE_OK
               : RELSERVE_ERR_HIP;
}

int32_t relserve_peak_probe_mfma(void* sink, int32_t iters, double* flops, void* stream) {
    drop_stale_hip_error();
    if (!sink || !flops) return RELSERVE_ERR_NULL_POINTER;
    if (iters <= 0) return RELSERVE_ERR_BAD_ARGUMENT;
    *flops = 256.0 * 4.0 * iters * 32.0 * 16384.0;
    return launch_peak_mfma(static_cast<float*>(sink), iters, static_cast<hipStream_t>(stream)) == hipSuccess
               ? RELSERVE_OK
               : RELSERVE_ERR_HIP;
}

int32_t relserve_peak_probe_stream(const void* src, size_t bytes, void* sink, void* stream) {
    drop_stale_hip_error();
    if (!src || !sink) return RELSERVE_ERR_NULL_POINTER;
    if (bytes < 16 || (reinterpret_cast<uintptr_t>(src) % 16)) return RELSERVE_ERR_BAD_ARGUMENT;
    return launch_peak_stream(src, (int64_t)bytes, static_cast<uint32_t*>(sink), static_cast<hipStream_t>(stream)) ==
                   hipSuccess
               ? RELSERVE_OK
               : RELSERVE_ERR_HIP;
}

int32_t relserve_peak_probe_stream_pattern(const void* src, size_t bytes, int32_t pattern, void* sink, void* stream) {
    drop_stale_hip_error();
    if (!src || !sink) return RELSERVE_ERR_NULL_POINTER;
    if (bytes < 32768 || (reinterpret_cast<uintptr_t>(src) % 16) || pattern < 0 || pattern > 4) return RELSERVE_ERR_BAD_ARGUMENT;
    return launch_peak_stream_pattern(src, (int64_t)bytes, pattern, static_cast<uint32_t*>(sink), static_cast<hipStream_t>(stream)) ==
                   hipSuccess
               ? RELSERVE_OK
               : RELSERVE_ERR_HIP;
}

int32_t relserve_debug_force_gemm_plan(int32_t tile, int32_t tail_splits) {
    if (tile < -1 || tile > 4 || tail_splits < 0 || tail_splits > 8) return RELSERVE_ERR_BAD_ARGUMENT;
    gemm_force_plan(tile, tail_splits);
    return RELSERVE_OK;
}

// ---- profiling ---------------------------------------------------------------------------
const char* relserve_profile_slot_name(int32_t slot) {
    return (slot >= 0 && slot < RELSERVE_PROFILE_SLOTS) ? kSlotNames[slot] : "";
}

int32_t relserve_profile_enable(relserve_layer* L, int32_t slot_mask) {
    if (!L) return RELSERVE_ERR_NULL_POINTER;
    L->profile = static_cast<uint32_t>(slot_mask);
    return RELSERVE_OK;
}

int32_t relserve_profile_read(relserve_layer* L, double* ms_sum, int64_t* launches, int32_t reset) {
    if (!L) return RELSERVE_ERR_NULL_POINTER;
    int32_t rc = RELSERVE_OK;
    if (!L->pending.empty()) {
        if (hipStreamSynchronize(L->pending_stream) != hipSuccess) rc = RELSERVE_ERR_HIP;
        for (auto& p : L->pending) {
            float ms = 0.f;
            if (rc == RELSERVE_OK && hipEventElapsedTime(&ms, p.a, p.b) == hipSuccess) {
                L->ms_sum[p.slot] += ms;
                L->launches[p.slot] += 1;
            }
            L->event_pool.push_back(p.a);
            L->event_pool.push_back(p.b);
        }
        L->pending.clear();
    }
    for (int i = 0; i < RELSERVE_PROFILE_SLOTS; ++i) {
        if (ms_sum) ms_sum[i] = L->ms_sum[i];
        if (launches) launches[i] = L->launches[i];
        if (reset) L->ms_sum[i] = 0, L->launches[i] = 0;
    }
    return rc;
}

}  // extern "C"

void relserve::profile_mark(relserve_layer* L, int slot, hipStream_t s, bool begin) {
    if (!L || !((L->profile >> slot) & 1u)) return;
    if (begin) {
        relserve_layer::Pending p{slot, nullptr, nullptr};
        auto get = [&](hipEvent_t* e) {
            if (!L->event_pool.empty()) {
                *e = L->event_pool.back();
                L->event_pool.pop_back();
                return true;
            }
            return hipEventCreate(e) == hipSuccess;
        };
        if (!get(&p.a) || !get(&p.b)) return;
        (void)hipEventRecord(p.a, s);
        L->pending.push_back(p);
        L->pending_stream = s;
    } else if (!L->pending.empty() && L->pending.back().slot == slot) {
        (void)hipEventRecord(L->pending.back().b, s);
    }
}
