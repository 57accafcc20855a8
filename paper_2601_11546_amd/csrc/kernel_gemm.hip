// bf16 MFMA GEMM for the dense maps of the layer (Eq. 3, W_o of Eq. 5, gate/up, down):
//   out[T, N] = a[T, K] * w[N, K]^T, fp32 accumulate, fused epilogues.
//
// Both operands are K-contiguous, which is the natural MFMA operand layout: a lane's 8
// consecutive k values are one 16-byte load.  The weight rows take the MFMA row index and
// the tokens the column index, so that an accumulator quad holds 4 consecutive output
// features of one token (one 8/16-byte store; where rows of fp32 are written it is the other way round, see frag_row16).
//
// Workgroup = a grid of 2 x 2 waves over a BM (tokens) x BN (features) tile, BK = 64.
// Main kernel (gemm_dma_kernel, K % 64 == 0): tiles go global -> LDS directly, XOR-swizzled 16-byte
// chunks, two to six stages, one barrier per k iteration, every k step issued in a fixed order that
// slots the refill loads and the next fragment reads between the MFMAs.  Fallback kernel
// (gemm_bf16_kernel): global -> registers -> LDS with zero-filled tails for any K % 8 == 0.
// Workgroup ids are remapped so that each of the 8 XCDs (own L2 each) walks a contiguous run of
// tiles, inside it token tiles fastest within panels of GROUP_M token tiles.
// Launch plans: tile shape by a cost model, or two shapes side by side; the incomplete last round of tiles may split k over
// workgroups; batches of at most 256 tokens, and narrow outputs at a few hundred, split k everywhere.
// Every split but the two ranges of launch_halves writes partial tiles to fp32 slabs that a second kernel sums and finishes.
#include <algorithm>
#include <atomic>
#include <mutex>
#include <type_traits>

#include "device_utils.h"
#include "relserve_internal.h"

namespace relserve {

namespace {

constexpr int BK = 64;
constexpr int NUM_XCD = 8;
constexpr int64_t kTailFloats = GEMM_TAIL_FLOATS;          // fp32 partial tiles (slabs) of the split paths at T > 256

struct GemmArgs {
    const uint16_t* a;
    const uint16_t* w;
    int32_t w_packed;   // weights in the tiled layout of pack_weight_kernel instead of row-major [N, K]
    const void* residual;
    void* out;
    int32_t T, N, K;
    int32_t n_half;  // SwiGLU: gate rows [0, n_half), up rows [n_half, 2 n_half)
    int32_t tiles_m, tiles_n;
    int32_t tile_n0;   // first feature tile of the launch (a launch of columns of tiles: plan_for)
    // fused q/k/v epilogue: rotary embedding + KV append (out = q buffer [T, n_q d])
    const int32_t* tok_slot;
    const float2* rope_cs;
    uint16_t* k_pages;
    uint16_t* v_pages;
    int32_t n_q, n_kv;
    int32_t kv_fp8;          // the pools hold 8-bit codes of x * k_inv / x * v_inv (one byte per element)
    float k_inv, v_inv;
    // split-K (skinny and mid-size T): workgroup b handles tile b % tiles and k steps [split * k_per_split, ...)
    // of that tile and stores its partial sums to slab `split` of accum [n_splits][T, N] fp32; the finish
    // kernel adds the slabs in split order
    float* accum;
    int32_t k_per_split;   // in units of 64; 0 = no split
    int32_t n_splits;
    // tail split (main path): the last tail_tiles tiles (those of the incomplete last round) are each
    // computed by tail_splits workgroups over k_per_split k steps each.  The partial tiles are stored
    // to tail_buf (tail_splits x tail_tiles x BM x BN fp32); a second kernel adds them up and runs the
    // epilogue.
    int32_t tail_tiles, tail_splits;
    float* tail_buf;
    // quantised projections: a and w hold 8-bit codes (one byte per element; K then counts PAIRS of codes, so that a row
    // is K * 2 bytes as in the 16-bit case), the sums are scaled by a_scale * w_scale[n], and a SwiGLU output is
    // stored as codes of value * out_inv
    int32_t f8;
    const float* w_scale;
    float a_scale;
    int32_t out_f8;
    float out_inv;
};

// Test hook (relserve_debug_force_gemm_plan): tile candidate (index into kTiles) and tail splits every launch
// must use; -1 = cost model.  One word, so that a launch on another host thread sees a consistent pair.
std::atomic<int> g_forced_plan{-1};   // -1, or cand | splits << 8
inline int forced_cand() { const int v = g_forced_plan.load(std::memory_order_relaxed); return v < 0 ? -1 : (v & 0xff); }
inline int forced_splits() { const int v = g_forced_plan.load(std::memory_order_relaxed); return v < 0 ? 0 : (v >> 8); }

// The dynamic-LDS limit of a kernel is raised once per process, whichever host thread launches it first.
template <typename Kernel>
hipError_t allow_smem_once(std::once_flag& once, hipError_t& status, Kernel kernel, int bytes) {
    std::call_once(once, [&] {
        status = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    });
    return status;
}

enum { EPI_BF16 = 0, EPI_RES_BF16_OUT_F32 = 1, EPI_RES_F32_OUT_BF16 = 2, EPI_SWIGLU = 3, EPI_QKV_ROPE = 4, EPI_SLAB = 5 };

// Products are 16 x 16 x 32 (on 8-bit codes 16 x 16 x 128).  A chain of them gives the same bits as the chain of twice as many
// 32 x 32 x 16 (measured, k of 32 .. 5120; on codes as 32 x 32 x 64 but for last bits where the codes span their whole range, equally
// far from 64 bits), but a 16 x 16 result passes through the accumulators half as often per product, and the chip is power-limited in
// these kernels: all CUs on register operands alone reach 1.93 PFLOP/s against 1.71 (4.10 against 3.78; profiles/mfma_rates.txt).  T = 7963, 13B: clock 1.70 -> 2.0
// GHz, gate/up 1632 -> 1579 us, W_down 813 -> 776, q/k/v 941 -> 910, the layer 4207 -> 4088.

__device__ __forceinline__ int remap_xcd(int bid, int num) {
    const int per = num / NUM_XCD, rem = num % NUM_XCD;
    const int xcd = bid % NUM_XCD, idx = bid / NUM_XCD;
    return xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
}

// Tile order inside an XCD's run: token tiles fastest within panels of about GROUP_M token tiles, then
// feature tiles, then the next panel.  The ~32 tiles an XCD works on at a time then cover about
// GROUP_M token tiles x 32 / GROUP_M feature tiles, so that its L2 serves ~12 distinct operand
// slices per k step instead of 33 when the batch has many token tiles.  The token tiles are divided
// evenly over the panels (9 token tiles: panels of 5 and 4, not of 8 and 1 -- a panel of one token tile
// shares nothing but its activation slice).
constexpr int GROUP_M = 8;
__device__ __forceinline__ void tile_coords(int t, int tiles_m, int tiles_n, int& tile_m, int& tile_n) {
    const int n_panels = (tiles_m + GROUP_M - 1) / GROUP_M;
    const int base = tiles_m / n_panels, extra = tiles_m % n_panels;   // the first `extra` panels hold base + 1 token tiles
    const int big = (base + 1) * tiles_n;
    int first_m, gsz, in_group;
    if (t < extra * big) {
        gsz = base + 1;
        first_m = (t / big) * gsz;
        in_group = t % big;
    } else {
        const int u = t - extra * big, per = base * tiles_n;
        gsz = base;
        first_m = extra * (base + 1) + (u / per) * base;
        in_group = u % per;
    }
    tile_m = first_m + in_group % gsz;
    tile_n = in_group / gsz;
}

// The small kernel's stores: a unit of 4 consecutive features n_lo .. of token t (lo), or a pair of such quads that the epilogue combines:
// gate and up, or the two halves of a rotated head (its columns n_lo - head D .. and D / 2 further).  oa, ob: what the unit reads besides
// the sums (a quad of the residual; the angles); slot: the token's place in the cache.
template <int EPI, int D>
__device__ __forceinline__ void store_unit(const GemmArgs& p, int t, int n_lo, int head, const float4& lo, const float4& hi, const float4& oa,
                                           const float4& ob, int slot_) {
    constexpr int DH = D > 0 ? D : 64;
    if constexpr (EPI == EPI_QKV_ROPE) {
        const int64_t slot = slot_;
        const int kv_dim = p.n_kv * DH, i = n_lo - head * DH;
        if (head < p.n_q + p.n_kv) {
            float4 rl, rh;
            rotate4(lo, hi, oa, ob, rl, rh);
            if (p.kv_fp8 && head >= p.n_q) {   // quantised cache: one byte per element, quantised from fp32
                uint8_t* dst8 = reinterpret_cast<uint8_t*>(p.k_pages) + slot * kv_dim + (head - p.n_q) * DH + i;
                const float s = p.k_inv;
                *reinterpret_cast<uint32_t*>(dst8) = pack_fp8x4(rl.x * s, rl.y * s, rl.z * s, rl.w * s);
                *reinterpret_cast<uint32_t*>(dst8 + DH / 2) = pack_fp8x4(rh.x * s, rh.y * s, rh.z * s, rh.w * s);
            } else {
                uint16_t* dst = (head < p.n_q ? static_cast<uint16_t*>(p.out) + (int64_t)t * (p.n_q * DH) + head * DH
                                              : p.k_pages + slot * kv_dim + (head - p.n_q) * DH) + i;
                *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf16x2(rl.x, rl.y), pack_bf16x2(rl.z, rl.w));
                *reinterpret_cast<uint2*>(dst + DH / 2) = make_uint2(pack_bf16x2(rh.x, rh.y), pack_bf16x2(rh.z, rh.w));
            }
        } else {
            const int64_t o = slot * kv_dim + (head - p.n_q - p.n_kv) * DH + i;
            if (p.kv_fp8) {
                uint8_t* dst8 = reinterpret_cast<uint8_t*>(p.v_pages) + o;
                const float s = p.v_inv;
                *reinterpret_cast<uint32_t*>(dst8) = pack_fp8x4(lo.x * s, lo.y * s, lo.z * s, lo.w * s);
                *reinterpret_cast<uint32_t*>(dst8 + DH / 2) = pack_fp8x4(hi.x * s, hi.y * s, hi.z * s, hi.w * s);
            } else {
                *reinterpret_cast<uint2*>(p.v_pages + o) = make_uint2(pack_bf16x2(lo.x, lo.y), pack_bf16x2(lo.z, lo.w));
                *reinterpret_cast<uint2*>(p.v_pages + o + DH / 2) = make_uint2(pack_bf16x2(hi.x, hi.y), pack_bf16x2(hi.z, hi.w));
            }
        }
    } else if constexpr (EPI == EPI_SWIGLU) {
        const float o0 = silu_mul(lo.x, hi.x), o1 = silu_mul(lo.y, hi.y), o2 = silu_mul(lo.z, hi.z), o3 = silu_mul(lo.w, hi.w);
        const int64_t o = (int64_t)t * p.n_half + n_lo;
        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(p.out) + o) = make_uint2(pack_bf16x2(o0, o1), pack_bf16x2(o2, o3));
    } else {
        const int64_t o = (int64_t)t * p.N + n_lo;
        if constexpr (EPI == EPI_RES_BF16_OUT_F32) {
            const uint32_t r0 = __float_as_uint(oa.x), r1 = __float_as_uint(oa.y);
            *reinterpret_cast<float4*>(static_cast<float*>(p.out) + o) =
                make_float4(lo.x + bf16_lo(r0), lo.y + bf16_hi(r0), lo.z + bf16_lo(r1), lo.w + bf16_hi(r1));
        } else {
            float4 v = lo;
            if constexpr (EPI == EPI_RES_F32_OUT_BF16) v.x += oa.x, v.y += oa.y, v.z += oa.z, v.w += oa.w;
            *reinterpret_cast<uint2*>(static_cast<uint16_t*>(p.out) + o) = make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
        }
    }
}

constexpr int WGM = 2, WGN = 2;   // grid of waves over a tile

// Which features of a wave's range a weight fragment holds, and how results lie in the lanes.
// Where bf16 or codes are written the weights are the first operand of the products: a lane's results are those of one token, and two
// fragments share 32 features so that it has 8 consecutive ones, the four lanes of a token 64 consecutive bytes.
// Where rows of fp32 are written (ROWS32: the slabs, W_o) the tokens are the first operand (the same products, the same bits): register r
// of a lane is token 4 (lane / 16) + r, and four fragments share 64 features, fragment c the features 4 i + c, so that a lane has four
// consecutive ones and the 16 lanes of a token 256 consecutive bytes, lane behind lane; the residual's bf16 are 128 such bytes.  With
// the weights first here too neighbouring lanes of an access hold pieces of different rows, and the CU's address unit is busy longer (a slab launch of
// 256 x 128 tiles of codes 9.7 million cycles, now 8.3; the L2 sees the same requests of 64 bytes either way, profiles/gemm_epilogue_l2_requests.txt):
// W_o of 8192 x 2048 codes took 57.2 us at T = 2100, now 48.5, of 5120 x 2560 16-bit values 54.8, now 51.3, and a step of a
// quarter of the 70B layer, whose projections all write slabs, at T = 256 210 us, now 202 (on codes 171, 164).
// Neither permutation costs anything: it is which rows of the weights in the LDS a lane reads, and which of eight rows a load puts where.
constexpr bool rows32(int epi) { return epi == EPI_RES_BF16_OUT_F32 || epi == EPI_SLAB; }
// row of the weights in the LDS that lane i of a fragment reads, beside the fragment's first one
template <int EPI>
__device__ __forceinline__ int frag_row16(int i) { return rows32(EPI) ? 8 * (i >> 1) + (i & 1) : 8 * (i >> 2) + (i & 3); }
template <int EPI>
constexpr int frag_base16(int tn) { return rows32(EPI) ? 64 * (tn >> 2) + 2 * (tn & 3) : 32 * (tn >> 1) + 4 * (tn & 1); }
// feature that LDS row `row` holds (ROWS32: 8 a + 2 c + b holds 8 a + 4 b + c, rows of both parities for the 16 lanes of a read)
template <int EPI>
__device__ __forceinline__ int lds_feature(int row) { return rows32(EPI) ? (row & ~7) + ((row >> 1) & 3) + 4 * (row & 1) : row; }
// quads of factors a wave's sums of products of codes need (one for the features a lane writes together)
constexpr int scale_quads(int epi, int tn) { return rows32(epi) ? tn / 4 : tn; }

// The weights' factors w_scale[feature] of a wave's sums of products of codes; loaded ahead of the k loop.
template <int BN, int EPI, int D, int NQ>
__device__ __forceinline__ void load_code_scales(const GemmArgs& p, int tile_n, int wn, int lane, float4 (&sc)[NQ]) {
    constexpr bool SWI = EPI == EPI_SWIGLU;
    constexpr int FEAT = BN / WGN, TN = FEAT / 16;
    static_assert(NQ == scale_quads(EPI, TN), "one quad for the features written together");
    if constexpr (rows32(EPI)) {
        const int n0 = tile_n * BN + wn * FEAT + 4 * (lane & 15);
#pragma unroll
        for (int u = 0; u < NQ; ++u) {
            sc[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (n0 + 64 * u < p.N) sc[u] = *reinterpret_cast<const float4*>(p.w_scale + n0 + 64 * u);
        }
        return;
    }
    const int gq = lane >> 4, cols = SWI ? p.n_half : p.N;
    const int n0 = (SWI ? tile_n * (BN / 2) + wn * (FEAT / 2) : tile_n * BN + wn * FEAT) + 8 * gq;
#pragma unroll
    for (int tn = 0; tn < NQ; ++tn) {
        const int n = n0 + frag_base16<EPI>(SWI ? tn % (TN / 2) : tn);
        sc[tn] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (n < cols) sc[tn] = *reinterpret_cast<const float4*>(p.w_scale + (SWI && tn >= TN / 2 ? p.n_half : 0) + n);
    }
}

// Epilogue of the 16 x 16 kernels, straight from the accumulators: acc[tn][tm] holds fragment tn's features of tokens
// 16 tm .. + 15 (of 32 tm_base on; see frag_row16).  A workgroup has one wave per SIMD, so the epilogue lasts as long as its instructions take to
// issue: there is no pass through the LDS, a row of tiles has one scalar base address and the distances of its accesses are constants,
// and tiles that end inside the matrix (FULL) test nothing per access.  Every access covers runs of 64 bytes (256 of fp32); what a
// row of tiles reads besides the sums is fetched rows ahead.  Cycles of a 256 x 256 tile of bf16 outputs: 13600 through the LDS, 8600
// here, which is what an XCD's 32 CUs, all writing at once, get through to memory (490 bytes a cycle).  8192 x 28672 x 5120 with the k
// loop's fewer instructions (k_step) 1820 -> 1675 us; layer steps, with 16 x 16 products: 13B at T = 7963 4248 -> 3973, 70B at T = 2304
// 3163 -> 2919.  (Workgroups that stay and load their next tile's first stages beside the epilogue gained nothing on this: the next
// tile's first waits then include the stores.)
template <int BM, int BN, int EPI, int D, bool SC, bool FULL, int TN, int TM>
__device__ __forceinline__ void gemm_epilogue16_rows(const f32x4_t (&acc)[TN][TM], const GemmArgs& p, int tile_n, int t0, int wn, int lane,
                                                     const float4 (&sc)[SC ? scale_quads(EPI, TN) : 1]) {
    constexpr int FEAT = BN / WGN;
    static_assert(TN == FEAT / 16, "the wave's features");
    const int l16 = lane & 15, gq = lane >> 4;
    // Rows whose operands are held: what a row waits for are its own loads, and, accesses completing in order, the stores issued before
    // them; with three ahead, of W_o half of a tile's rows (16 registers each), the stores flow.  W_o with all rows loaded first / half /
    // one row ahead: 192 rows, 8192 x 2048 codes at T = 1150 27.6 / 25.9 / 27.0 us, 5120 x 2560 at 1900 30.3 / 28.1 / 29.6; 128 rows, at
    // 1150 23.0 / 22.2 / 22.4; 256 rows 0 - 1 % apart.
    constexpr int R = EPI == EPI_RES_BF16_OUT_F32 ? TM / 2 + 1 : (TM < 4 ? TM : 4);
    auto quad = [&](int tn, int tm) __attribute__((always_inline)) {
        f32x4_t v = acc[tn][tm];
        asm volatile("" : "+v"(v));   // copied here: left to itself the compiler moves all sums to the other register file first, and spills
        return make_float4(v[0], v[1], v[2], v[3]);
    };
    auto scaled = [](float4 v, const float4& s) __attribute__((always_inline)) { return make_float4(v.x * s.x, v.y * s.y, v.z * s.z, v.w * s.w); };
    // a sum and its residual: with a factor one fused multiply-add, written out (left to the compiler it is one in some kernels only)
    auto plus = [](const float4& v, const float4& s, const float4& r) __attribute__((always_inline)) {
        if constexpr (SC)
            return make_float4(__builtin_fmaf(v.x, s.x, r.x), __builtin_fmaf(v.y, s.y, r.y), __builtin_fmaf(v.z, s.z, r.z), __builtin_fmaf(v.w, s.w, r.w));
        else
            return make_float4(v.x + r.x, v.y + r.y, v.z + r.z, v.w + r.w);
    };
    auto pack8 = [](const float4& a, const float4& b) __attribute__((always_inline)) {
        return make_uint4(pack_bf16x2(a.x, a.y), pack_bf16x2(a.z, a.w), pack_bf16x2(b.x, b.y), pack_bf16x2(b.z, b.w));
    };
    auto codes8 = [](const float4& a, const float4& b, float s) __attribute__((always_inline)) {
        return make_uint2(pack_fp8x4(a.x * s, a.y * s, a.z * s, a.w * s), pack_fp8x4(b.x * s, b.y * s, b.z * s, b.w * s));
    };
    // rows of tokens: base (uniform) + this lane's offset; lanes past T take the last token's operands and store nothing
    auto row_off = [&](int tm, int64_t pitch) __attribute__((always_inline)) -> uint32_t {   // bytes from row t0 + 16 tm
        return (uint32_t)(FULL ? l16 : min(l16, max(p.T - 1 - t0 - 16 * tm, 0))) * (uint32_t)pitch;
    };
    if constexpr (rows32(EPI)) {
        constexpr int U = TN / 4;   // groups of 64 features
        constexpr bool RES = EPI == EPI_RES_BF16_OUT_F32;
        const int n0 = tile_n * BN + wn * FEAT;
        auto ok = [&](int u) { return FULL || n0 + 4 * l16 + 64 * u < p.N; };
        const bool add = RES && p.residual != nullptr;   // no residual given: plain fp32 output
        uint2 res[RES ? R : 1][4][U];
        auto fetch = [&](int tm) __attribute__((always_inline)) {
            if constexpr (RES) {
                const int first = min(t0 + 16 * tm, p.T - 1);
                const char* base = static_cast<const char*>(p.residual) + ((int64_t)first * p.N + n0) * 2;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const uint32_t off = (uint32_t)(FULL ? 4 * gq + r : min(4 * gq + r, p.T - 1 - first)) * (uint32_t)p.N * 2 + 8 * l16;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        res[tm % R][r][u] = make_uint2(0, 0);
                        if (add && ok(u)) res[tm % R][r][u] = *reinterpret_cast<const uint2*>(base + off + 128 * u);
                    }
                }
            }
        };
#pragma unroll
        for (int tm = 0; tm < R - 1; ++tm) fetch(tm);
        if constexpr (R == 1) fetch(0);
        const uint32_t off = (uint32_t)(4 * gq) * (uint32_t)p.N * 4 + 16 * l16;
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            if (!FULL && t0 + 16 * tm >= p.T) break;   // padding: nothing of this row of tiles (or the ones behind it) is stored
            __builtin_amdgcn_sched_barrier(0);   // row after row: every register is taken by sums still to be stored
            if (R > 1 && tm + R - 1 < TM) fetch(tm + R - 1);
            char* base = static_cast<char*>(p.out) + ((int64_t)(t0 + 16 * tm) * p.N + n0) * 4;
            float4 q[TN];   // (whole quads: with their elements copied one by one the compiler again moves all sums first)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) q[tn] = quad(tn, tm);
            auto elem = [](const float4& v, int r) { return r == 0 ? v.x : r == 1 ? v.y : r == 2 ? v.z : v.w; };
#pragma unroll
            for (int r = 0; r < 4; ++r, base += (int64_t)p.N * 4) {
                if (!FULL && t0 + 16 * tm + 4 * gq + r >= p.T) continue;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    float4 o = make_float4(elem(q[4 * u], r), elem(q[4 * u + 1], r), elem(q[4 * u + 2], r), elem(q[4 * u + 3], r));
                    if constexpr (RES) {
                        const uint2 x = res[tm % R][r][u];
                        o = plus(o, sc[SC ? u : 0], make_float4(bf16_lo(x.x), bf16_hi(x.x), bf16_lo(x.y), bf16_hi(x.y)));
                    }
                    if (ok(u)) *reinterpret_cast<float4*>(base + off + 256 * u) = o;
                }
            }
        }
    } else if constexpr (EPI == EPI_QKV_ROPE) {
        constexpr int HEADS = FEAT / D, GH = D / 64, TH = D / 16;   // heads of the wave, 8-feature groups of half a head, tiles of a head
        const int head0 = (tile_n * BN + wn * FEAT) / D, kv_dim = p.n_kv * D;
        float4 cs[R][GH][4];
        int slot[R];
        auto fetch = [&](int tm) __attribute__((always_inline)) {
            const int first = min(t0 + 16 * tm, p.T - 1);
            slot[tm % R] = *reinterpret_cast<const int*>(reinterpret_cast<const char*>(p.tok_slot + first) + row_off(tm, 4));
            const char* base = reinterpret_cast<const char*>(p.rope_cs + (int64_t)first * (D / 2));
            const uint32_t off = row_off(tm, D * 4) + 64 * gq;
#pragma unroll
            for (int u = 0; u < GH; ++u)
#pragma unroll
                for (int c = 0; c < 4; ++c) cs[tm % R][u][c] = *reinterpret_cast<const float4*>(base + off + 256 * u + 16 * c);
        };
#pragma unroll
        for (int tm = 0; tm < R - 1; ++tm) fetch(tm);
        if constexpr (R == 1) fetch(0);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            if (!FULL && t0 + 16 * tm >= p.T) break;
            __builtin_amdgcn_sched_barrier(0);
            if (R > 1 && tm + R - 1 < TM) fetch(tm + R - 1);
            if (!FULL && t0 + 16 * tm + l16 >= p.T) continue;
#pragma unroll
            for (int hh = 0; hh < HEADS; ++hh) {
                const int head = __builtin_amdgcn_readfirstlane(head0 + hh);
                if (head >= p.n_q + 2 * p.n_kv) continue;
                const bool is_q = head < p.n_q, is_k = !is_q && head < p.n_q + p.n_kv;
                float4 lo[GH][2], hi[GH][2];
#pragma unroll
                for (int u = 0; u < GH; ++u)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int tl = hh * TH + 2 * u + h, th = tl + TH / 2;
                        lo[u][h] = quad(tl, tm);
                        hi[u][h] = quad(th, tm);
                        if constexpr (SC) lo[u][h] = scaled(lo[u][h], sc[tl]), hi[u][h] = scaled(hi[u][h], sc[th]);
                    }
                if (is_q || is_k) {
#pragma unroll
                    for (int u = 0; u < GH; ++u)
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const float4 a = lo[u][h], b = hi[u][h];
                            rotate4(a, b, cs[tm % R][u][2 * h], cs[tm % R][u][2 * h + 1], lo[u][h], hi[u][h]);
                        }
                }
                if (p.kv_fp8 && !is_q) {   // quantised cache: one byte per element, quantised from fp32
                    uint8_t* dst = reinterpret_cast<uint8_t*>(is_k ? p.k_pages : p.v_pages) + (head - p.n_q - (is_k ? 0 : p.n_kv)) * D +
                                   (int64_t)slot[tm % R] * kv_dim + 8 * gq;
                    const float s = is_k ? p.k_inv : p.v_inv;
#pragma unroll
                    for (int u = 0; u < GH; ++u) {
                        *reinterpret_cast<uint2*>(dst + 32 * u) = codes8(lo[u][0], lo[u][1], s);
                        *reinterpret_cast<uint2*>(dst + 32 * u + D / 2) = codes8(hi[u][0], hi[u][1], s);
                    }
                } else {
                    uint16_t* dst = is_q ? static_cast<uint16_t*>(p.out) + (int64_t)(t0 + 16 * tm + l16) * (p.n_q * D) + head * D
                                         : (is_k ? p.k_pages : p.v_pages) + (head - p.n_q - (is_k ? 0 : p.n_kv)) * D + (int64_t)slot[tm % R] * kv_dim;
                    dst += 8 * gq;
#pragma unroll
                    for (int u = 0; u < GH; ++u) {
                        *reinterpret_cast<uint4*>(dst + 32 * u) = pack8(lo[u][0], lo[u][1]);
                        *reinterpret_cast<uint4*>(dst + 32 * u + D / 2) = pack8(hi[u][0], hi[u][1]);
                    }
                }
            }
        }
    } else {
        // bf16 rows (or codes of a SwiGLU product): groups of 8 features a lane
        constexpr bool SWI = EPI == EPI_SWIGLU;
        constexpr int GROUPS = SWI ? TN / 4 : TN / 2;
        const int cols = SWI ? p.n_half : p.N;
        const int n0 = SWI ? tile_n * (BN / 2) + wn * (FEAT / 2) : tile_n * BN + wn * FEAT;
        auto ok = [&](int u, int h) { return FULL || n0 + 8 * gq + 32 * u + 4 * h < cols; };
        const bool codes = SC && SWI && p.out_f8;   // the down projection reads codes (n_half is a multiple of 8)
        const int esize = codes ? 1 : 2;
        float4 res[R][EPI == EPI_RES_F32_OUT_BF16 ? GROUPS : 1][2];
        auto fetch = [&](int tm) __attribute__((always_inline)) {
            if constexpr (EPI == EPI_RES_F32_OUT_BF16) {
                const char* base = static_cast<const char*>(p.residual) + ((int64_t)min(t0 + 16 * tm, p.T - 1) * p.N + n0) * 4;
                const uint32_t off = row_off(tm, (int64_t)p.N * 4) + 32 * gq;
#pragma unroll
                for (int u = 0; u < GROUPS; ++u)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        if (ok(u, h)) res[tm % R][u][h] = *reinterpret_cast<const float4*>(base + off + 128 * u + 16 * h);
            }
        };
#pragma unroll
        for (int tm = 0; tm < R - 1; ++tm) fetch(tm);
        if constexpr (R == 1) fetch(0);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            if (!FULL && t0 + 16 * tm >= p.T) break;
            __builtin_amdgcn_sched_barrier(0);
            if (R > 1 && tm + R - 1 < TM) fetch(tm + R - 1);
            char* base = static_cast<char*>(p.out) + ((int64_t)(t0 + 16 * tm) * cols + n0) * esize;
            const uint32_t off = row_off(tm, (int64_t)cols * esize) + 8 * gq * esize;
            if (!FULL && t0 + 16 * tm + l16 >= p.T) continue;
#pragma unroll
            for (int u = 0; u < GROUPS; ++u) {
                float4 v[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    v[h] = quad(2 * u + h, tm);
                    if constexpr (EPI == EPI_RES_F32_OUT_BF16)
                        v[h] = plus(v[h], sc[SC ? 2 * u + h : 0], res[tm % R][u][h]);
                    else if constexpr (SC)
                        v[h] = scaled(v[h], sc[2 * u + h]);
                    if constexpr (SWI) {
                        float4 up = quad(TN / 2 + 2 * u + h, tm);
                        if constexpr (SC) up = scaled(up, sc[TN / 2 + 2 * u + h]);
                        v[h] = make_float4(silu_mul(v[h].x, up.x), silu_mul(v[h].y, up.y), silu_mul(v[h].z, up.z), silu_mul(v[h].w, up.w));
                    }
                }
                if (codes) {
                    if (ok(u, 0)) *reinterpret_cast<uint2*>(base + off + 32 * u) = codes8(v[0], v[1], p.out_inv);
                    continue;
                }
                const uint4 b = pack8(v[0], v[1]);
                if constexpr (FULL) {
                    *reinterpret_cast<uint4*>(base + off + 64 * u) = b;
                } else {   // 4 by 4: rows may end inside a group or begin at 8-byte boundaries
                    if (ok(u, 0)) *reinterpret_cast<uint2*>(base + off + 64 * u) = make_uint2(b.x, b.y);
                    if (ok(u, 1)) *reinterpret_cast<uint2*>(base + off + 64 * u + 8) = make_uint2(b.z, b.w);
                }
            }
        }
    }
}

template <int BM, int BN, int EPI, int D, bool SC, int TN, int TM>
__device__ __forceinline__ void gemm_epilogue16(const f32x4_t (&acc)[TN][TM], const GemmArgs& p, int tile_m, int tile_n, int wm, int wn,
                                                int lane, int tm_base, const float4 (&w_scales)[SC ? scale_quads(EPI, TN) : 1] = {}) {
    constexpr int NQ = SC ? scale_quads(EPI, TN) : 1;
    float4 sc[NQ];
#pragma unroll
    for (int i = 0; i < (SC ? NQ : 0); ++i)
        sc[i] = make_float4(w_scales[i].x * p.a_scale, w_scales[i].y * p.a_scale, w_scales[i].z * p.a_scale, w_scales[i].w * p.a_scale);
    const int t0 = tile_m * BM + 32 * tm_base + wm * (BM / WGM);
    const int cols = EPI == EPI_SWIGLU ? p.n_half : p.N, last = (tile_n + 1) * (EPI == EPI_SWIGLU ? BN / 2 : BN);
    const bool aligned = EPI == EPI_QKV_ROPE || rows32(EPI) || (cols % 8 == 0 && reinterpret_cast<uintptr_t>(p.out) % 16 == 0);
    if (t0 + 16 * TM <= p.T && last <= cols && aligned)
        gemm_epilogue16_rows<BM, BN, EPI, D, SC, true>(acc, p, tile_n, t0, wn, lane, sc);
    else if (t0 < p.T)
        gemm_epilogue16_rows<BM, BN, EPI, D, SC, false>(acc, p, tile_n, t0, wn, lane, sc);
}

template <int BM, int BN, int EPI, int D = 0>
__global__ void __launch_bounds__(256) gemm_bf16_kernel(GemmArgs p) {
    constexpr int TM = BM / 32, TN = BN / 32;          // 16x16 MFMA tiles per wave
    constexpr int A_IT = BM / 32, W_IT = BN / 32;      // 16-byte chunks per thread and k step
    constexpr int A_BYTES = BM * BK * 2, W_BYTES = BN * BK * 2, STAGE = A_BYTES + W_BYTES;
    static_assert(EPI != EPI_SWIGLU || TN % 2 == 0, "SwiGLU needs gate and up tiles in one wave");
    static_assert(EPI != EPI_QKV_ROPE || (BN == 256 && (D == 64 || D == 128)), "a wave must own whole heads");
    extern __shared__ __align__(16) unsigned char smem[];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, g = lane >> 4;

    const int tile = remap_xcd(blockIdx.x, p.tiles_m * p.tiles_n);
    int tile_m, tile_n;
    tile_coords(tile, p.tiles_m, p.tiles_n, tile_m, tile_n);
    const int t0 = tile_m * BM;
    const int K = p.K;

    // ---- global -> register staging: element offsets of this thread's chunks (-1 = zero fill)
    const int c8 = (tid & 7) * 8, lrow = tid >> 3;
    int a_off[A_IT], w_off[W_IT];
#pragma unroll
    for (int i = 0; i < A_IT; ++i) {
        const int t = t0 + lrow + 32 * i;
        a_off[i] = t < p.T ? t * K + c8 : -1;
    }
#pragma unroll
    for (int i = 0; i < W_IT; ++i) {
        const int lr = lrow + 32 * i;
        int n;
        bool ok;
        if (EPI == EPI_SWIGLU) {
            constexpr int HALF = BN / 2;
            const int gi = tile_n * HALF + (lr % HALF);
            ok = gi < p.n_half;
            n = lr < HALF ? gi : p.n_half + gi;
        } else {
            n = tile_n * BN + lds_feature<EPI>(lr);
            ok = n < p.N;
        }
        w_off[i] = ok ? n * K + c8 : -1;
    }
    // swizzled LDS store offsets: by row & 7, the weights of ROWS32 by the row's group of 8 (what the 16 lanes of a read differ in)
    auto w_swz = [](int row) { return rows32(EPI) ? (row >> 3) & 7 : row & 7; };
    const int st_off = lrow * 128 + (((tid & 7) ^ (lrow & 7)) << 4);

    uint4 a_reg[A_IT], w_reg[W_IT];
    auto load_global = [&](int k0) {
        const bool k_ok = k0 + c8 < K;
#pragma unroll
        for (int i = 0; i < A_IT; ++i)
            a_reg[i] = (a_off[i] >= 0 && k_ok) ? *reinterpret_cast<const uint4*>(p.a + a_off[i] + k0)
                                               : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < W_IT; ++i)
            w_reg[i] = (w_off[i] >= 0 && k_ok) ? *reinterpret_cast<const uint4*>(p.w + w_off[i] + k0)
                                               : make_uint4(0, 0, 0, 0);
    };
    auto store_lds = [&](int buf) {
        unsigned char* sa = smem + buf * STAGE;
        unsigned char* sw = sa + A_BYTES;
#pragma unroll
        for (int i = 0; i < A_IT; ++i) *reinterpret_cast<uint4*>(sa + i * 32 * 128 + st_off) = a_reg[i];
#pragma unroll
        for (int i = 0; i < W_IT; ++i) {
            const int lr = lrow + 32 * i;
            *reinterpret_cast<uint4*>(sw + lr * 128 + (((tid & 7) ^ w_swz(lr)) << 4)) = w_reg[i];
        }
    };

    // ---- LDS -> MFMA operands: rows l16 of the wave's tokens, frag_row16 of its features
    const int a_row = wm * (BM / 2) + l16, w_lane = frag_row16<EPI>(l16);
    int w_row[TN];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
        const int half = EPI == EPI_SWIGLU && tn >= TN / 2 ? 1 : 0;
        w_row[tn] = half * (BN / 2) + wn * (EPI == EPI_SWIGLU ? BN / 4 : BN / 2) + frag_base16<EPI>(tn - half * (TN / 2)) + w_lane;
    }

    f32x4_t acc[TN][TM];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) acc[tn][tm] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    const int nk = (K + BK - 1) / BK;
    load_global(0);
    store_lds(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const bool more = kt + 1 < nk;
        if (more) load_global((kt + 1) * BK);
        const unsigned char* sa = smem + (kt & 1) * STAGE;
        const unsigned char* sw = sa + A_BYTES;
#pragma unroll
        for (int ks = 0; ks < BK / 32; ++ks) {
            bf16x8_t wf[TN], af[TM];
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
                wf[tn] = as_bf16x8(*reinterpret_cast<const uint4*>(sw + w_row[tn] * 128 + (((4 * ks + g) ^ w_swz(w_row[tn])) << 4)));
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
                af[tm] = as_bf16x8(*reinterpret_cast<const uint4*>(sa + (a_row + 16 * tm) * 128 + (((4 * ks + g) ^ (a_row & 7)) << 4)));
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int tm = 0; tm < TM; ++tm)
                    acc[tn][tm] = rows32(EPI) ? mfma_16x16x32(af[tm], wf[tn], acc[tn][tm]) : mfma_16x16x32(wf[tn], af[tm], acc[tn][tm]);
        }
        if (more) store_lds((kt + 1) & 1);
        __syncthreads();
    }
    gemm_epilogue16<BM, BN, EPI, D, false>(acc, p, tile_m, tile_n, wm, wn, lane, 0);
}

// ------------------------------------------------------------------------------------------
// Main kernel for K % 64 == 0: tiles go global -> LDS directly (global_load_lds_dwordx4, no
// register staging and no LDS store instructions), two LDS stages or more, operand fragments double
// buffered in registers.  The barrier that hands over a stage sits one k step BEFORE the stage
// boundary: the last 16 MFMAs of a stage run while the first fragments of the next stage are
// being read, and the loads of the stage after that are issued at once, so they have a whole
// k iteration to land.
// ------------------------------------------------------------------------------------------
// 64 lanes x 16 bytes from (base + per-lane byte offset) to 1 KB of LDS starting at lds_addr.
// A pointer every lane holds the same value of, moved to scalar registers (the compiler cannot always prove it).
__device__ __forceinline__ const char* uniform_ptr(const char* ptr) {
    const uint64_t v = reinterpret_cast<uint64_t>(ptr);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const char*>(((uint64_t)hi << 32) | lo);
}

// NT = non-temporal: for bytes that are read once (the weights of a batch of one token tile).  A streaming read of
// HBM reaches 7.1-7.4 TB/s with the hint against 6.3-6.4 TB/s without (measured with 32 KB per workgroup in flight);
// operands that other workgroups read again keep the default policy, which lets the L2 hold them.
// In two halves: dma16_to names the LDS address lds_addr + at (the constant) in m0, dma16_from loads; one instruction at least has to
// stand between the two (a load reads m0 too early right behind the scalar instruction that writes it).
__device__ __forceinline__ void dma16_to(uint32_t lds_addr, int at) {
    asm volatile("s_add_u32 m0, %0, %1" ::"s"(lds_addr), "i"(at) : "memory", "scc");
}
template <bool NT = false>
__device__ __forceinline__ void dma16_from(const void* base, uint32_t voff) {
    if (NT)
        asm volatile("global_load_lds_dwordx4 %0, %1 nt" ::"v"(voff), "s"(base) : "memory");
    else
        asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base) : "memory");
}
template <bool NT = false>
__device__ __forceinline__ void dma16(const void* base, uint32_t voff, uint32_t lds_addr, int at) {
    if (NT)
        asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(voff), "s"(base), "s"(lds_addr), "i"(at) : "memory", "scc");
    else
        asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(lds_addr), "i"(at) : "memory", "scc");
}

// BKD = k extent of one LDS stage, NS = stages in the ring (NS - 1 are in flight).
// WNT: the weights are loaded with the non-temporal hint (launches in which no other workgroup reads them again).
// F8: both operands hold 8-bit codes.  Nothing changes in how bytes travel (K counts pairs of codes, a stage row is
// still 128 bytes); a stage is one k step of 16 x 16 x 128 MFMAs, whose operand is the two adjacent 16-byte chunks
// 2 g, 2 g + 1 of the row for k quarter g (both operands alike, so which codes meet which is fixed), and the epilogue applies the scales.
// NSW = stages of the weights' ring: NS, or NS + 1 ("skewed").  Loads of one wave complete in order, so a hand-over of the
// skewed ring issues the activations of stage kt + NS first and the weights of stage kt + NS + 1 behind them: what the next
// hand-over waits for are the activations, and the weights just issued stay in flight for another iteration.
// Tiles of 192 and 256 rows hold two or three stages and leave 16 - 48 KB of the LDS over; two whole stages give a stage hardly
// one iteration from its issue to its use.  With the third stage of weights, one launch, us: 256 x 256, 13B at T = 7963 W_down
// 877 -> 838, W_o 372 -> 356; the 70B gate/up at T = 256, weights from HBM, 220 -> 198; 192 x 256 at T = 640 gate/up 202 -> 174,
// q/k/v 109 -> 98.  Small tiles have four to six whole stages and gain nothing (128 x 128 gate/up 67.6 -> 72).
constexpr int weight_stages(int bm, int bn, int ns) { return bm >= 192 && ns <= 3 && (ns * (bm + bn) + bn) * 128 <= 160 * 1024 ? ns + 1 : ns; }

// HALVES: the tail of a launch of 256-row tiles whose k ranges are two (launch_halves): each of its tiles is two of this kernel's, which
// run over both ranges and add their sums as the finish kernel would.
template <int BM, int BN, int EPI, int D, int BKD, int NS, bool WNT = false, bool F8 = false, int NSW = NS, bool HALVES = false>
__global__ void __launch_bounds__(64 * WGM * WGN) gemm_dma_kernel(GemmArgs p) {
    constexpr bool SKEW = NSW > NS;
    static_assert(NSW == NS || NSW == NS + 1, "weight ring");
    constexpr int NW = WGM * WGN;
    constexpr int TM = BM / (16 * WGM), TN = BN / (16 * WGN);
    constexpr int ROWB = BKD * 2;                        // bytes per LDS row
    constexpr int CPR = BKD / 8;                         // 16-byte chunks per row
    constexpr int RPI = 1024 / ROWB;                     // rows one 1 KB wave load covers
    constexpr int A_IT = BM / (NW * RPI), W_IT = BN / (NW * RPI);
    constexpr int A_BYTES = BM * ROWB, W_BYTES = BN * ROWB, W_LDS = NS * A_BYTES;   // NS stages of activations, then NSW of weights
    constexpr int KSTEPS = F8 ? 1 : BKD / 32;
    constexpr int LOADS = A_IT + W_IT;                   // wave loads per stage
    static_assert(BKD == 64, "stage depth: a slice of the packed weights");
    static_assert(NSW * LOADS < 64, "vmcnt field");
    static_assert(EPI != EPI_SWIGLU || TN % 2 == 0, "SwiGLU needs gate and up tiles in one wave");
    static_assert(EPI != EPI_QKV_ROPE || (BN / WGN == 128 && (D == 64 || D == 128)), "a wave must own whole heads");
    static_assert(BM % (NW * RPI) == 0 && BN % (NW * RPI) == 0, "whole wave loads");
    extern __shared__ __align__(16) unsigned char smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    const int fr = lane % 16, g = lane / 16;             // this lane's row of an operand fragment, and its part of the k step

    const int K = p.K;
    const int n_tiles = p.tiles_m * p.tiles_n, tail_units = p.tail_tiles * p.tail_splits, dp_tiles = n_tiles - p.tail_tiles;
    int tile, split = 0, tail_idx = 0;
    bool tail = false;
    if (HALVES) {   // tiles_m counts 256-row tiles
        tile = dp_tiles + remap_xcd(blockIdx.x, 2 * p.tail_tiles) / 2;
    } else if (EPI == EPI_SLAB) {
        tile = remap_xcd(blockIdx.x % n_tiles, n_tiles);
        split = blockIdx.x / n_tiles;
    } else {
        // the tail units come first in the grid: their short k ranges and slab stores are over before the
        // last whole tiles finish
        tail = (int)blockIdx.x < tail_units;
        if (tail) {
            const int u = remap_xcd(blockIdx.x, tail_units);   // runs of one split, consecutive tiles, per XCD
            split = u / p.tail_tiles;
            tail_idx = u % p.tail_tiles;
            tile = dp_tiles + tail_idx;
        } else {
            tile = remap_xcd(blockIdx.x - tail_units, dp_tiles);
        }
    }
    int tile_m, tile_n;
    tile_coords(tile, p.tiles_m, p.tiles_n, tile_m, tile_n);
    tile_n += p.tile_n0;
    if (HALVES) {
        tile_m = 2 * tile_m + remap_xcd(blockIdx.x, 2 * p.tail_tiles) % 2;
        if (tile_m * BM >= p.T) return;   // the whole workgroup
    }

    // ---- per-lane source offsets: wave load j of this wave fills LDS rows (NW j + wave) * RPI .. ;
    // lane l owns row l / CPR of those and slot l % CPR, which holds the row's chunk slot ^ swz(row).
    // The LDS has 64 four-byte banks and serves a 16-byte-per-lane read 16 lanes at a time, so the
    // 16 consecutive rows those lanes read must cover all 64 banks once: swz = (row >> 1) & 7 (row
    // parity picks the bank half).
    // Rows past the end of a matrix re-read its last row: their products are never stored.
    const uint32_t lrow = lane / CPR;
    const uint32_t row_lo = (uint32_t)(wave * RPI) + lrow;   // LDS row modulo NW * RPI (>= 32): all the swizzle needs
    const uint32_t chunk = (lane % CPR) ^ ((row_lo >> 1) & 7);
    // (the weights are read in rows 0-3, 8-11, 16-19 and 24-27 of 32, or four further on; for fp32 rows in 0, 1, 8, 9, 16, 17 .. of 64:
    // swizzles of their own give those sixteen the same)
    auto w_swz = [](int row) { return rows32(EPI) ? (row >> 3) & 7 : ((row >> 1) & 1) | ((row >> 2) & 6); };
    uint32_t a_voff[A_IT], w_voff[W_IT];
    // row-major: row n starts at n * K; packed: block n / 256 holds, k slice after k slice, 256 rows of 128 bytes
    const uint32_t w_shift = p.w_packed ? 8 : 0, w_block = (uint32_t)K * (p.w_packed ? 512u : 2u), w_mask = p.w_packed ? 255 : 0;
#pragma unroll
    for (int j = 0; j < A_IT; ++j) {
        const int t = min(tile_m * BM + (NW * j + wave) * RPI + (int)lrow, p.T - 1);
        a_voff[j] = ((uint32_t)t * (uint32_t)K + chunk * 8) * 2;
    }
#pragma unroll
    for (int j = 0; j < W_IT; ++j) {
        const int lr = (NW * j + wave) * RPI + (int)lrow;
        uint32_t n;
        if (EPI == EPI_SWIGLU) {
            constexpr int HALF = BN / 2;   // (a wave load's rows lie in one half)
            const int gi = min(tile_n * HALF + (lr % HALF), p.n_half - 1);
            n = NW * j * RPI < HALF ? gi : p.n_half + gi;
        } else {
            n = min(tile_n * BN + lds_feature<EPI>(lr), p.N - 1);
        }
        w_voff[j] = (n >> w_shift) * w_block + (n & w_mask) * 128u + ((lane % CPR) ^ w_swz(lr)) * 16;
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    const int w_stage = p.w_packed ? 32768 : 128;   // bytes from one k slice of the weights to the next

    // ---- LDS -> MFMA operands: this lane's address of the first fragment of a k step inside stage 0; the other fragments lie at
    // constant distances, which the read instruction holds.
    const int swz = (fr >> 1) & 7;
    constexpr int w_wave = EPI == EPI_SWIGLU ? BN / (2 * WGN) : BN / WGN;   // first row of the wave's features (SwiGLU: in either half)
    uint32_t a_lane[KSTEPS], w_lane[KSTEPS];
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
        const int c = F8 ? 2 * g : 4 * ks + g;   // the lane's (first) chunk of a row
        const uint32_t at = lds0 + fr * ROWB + ((c ^ swz) << 4);
        a_lane[ks] = at + wm * (BM / WGM) * ROWB;
        const int row = frag_row16<EPI>(fr);
        w_lane[ks] = lds0 + W_LDS + (wn * w_wave + row) * ROWB + ((c ^ w_swz(row)) << 4);
    }
    auto a_dist = [](int tm) { return 16 * tm * ROWB; };
    auto w_dist = [](int tn) {
        const int half = EPI == EPI_SWIGLU && tn >= TN / 2 ? 1 : 0, i = tn - half * (TN / 2);
        return (half * (BN / 2) + frag_base16<EPI>(i)) * ROWB;
    };

    f32x4_t acc[TN][TM];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) acc[tn][tm] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    using frag_t = std::conditional_t<F8, i32x8_t, bf16x8_t>;
    constexpr bool FIXED = HALVES || (BM * BN >= 6 * 4096 && !(EPI == EPI_SWIGLU && BM == 128));   // issue order: see below
    constexpr bool QUARTERS = F8 && (FIXED || NS == 2);
    constexpr bool EARLY = !FIXED && NS == 2;   // the refill goes out at once: see below
    frag_t wf[QUARTERS ? 1 : 2][TN], af[QUARTERS ? 1 : 2][TM];
    typedef const i32x4_t __attribute__((address_space(3))) * lds_chunk;
    auto read_frag = [&](uint32_t at, int dist) __attribute__((always_inline)) -> frag_t {
        if constexpr (F8) {
            const i32x4_t lo = *(lds_chunk)(uintptr_t)(at + dist), hi = *(lds_chunk)(uintptr_t)((at ^ 16) + dist);
            return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        } else {
            return __builtin_bit_cast(bf16x8_t, *(lds_chunk)(uintptr_t)(at + dist));
        }
    };
    struct Stage { int a, w; };   // indices into the two rings
    struct Source { uint32_t a, w; };
    auto source = [&](Stage st, int ks) __attribute__((always_inline)) {
        Source r{a_lane[ks] + st.a * A_BYTES, w_lane[ks] + st.w * W_BYTES};
        asm("" : "+v"(r.a), "+v"(r.w));   // one sum each, not one for every fragment
        return r;
    };
    auto load_frag_one = [&](int buf, Source src, int i) __attribute__((always_inline)) {   // i-th of the TN + TM fragment reads of a k step
        if (i < TM)   // the first products of a step need all tokens and one row of features
            af[buf][i] = read_frag(src.a, a_dist(i));
        else
            wf[buf][i - TM] = read_frag(src.w, w_dist(i - TM));
    };
    auto load_frags = [&](int buf, Stage st, int ks) __attribute__((always_inline)) {
        const Source src = source(st, ks);
#pragma unroll
        for (int i = 0; i < TN + TM; ++i) load_frag_one(buf, src, i);
    };

    auto mfma_one = [&](int buf, int i) __attribute__((always_inline)) {   // i-th of the TN * TM products of a k step
        const int tn = i / TM, tm = i % TM;
        if constexpr (F8)
            acc[tn][tm] = rows32(EPI) ? mfma_16x16x128_f8(af[buf][tm], wf[buf][tn], acc[tn][tm]) : mfma_16x16x128_f8(wf[buf][tn], af[buf][tm], acc[tn][tm]);
        else
            acc[tn][tm] = rows32(EPI) ? mfma_16x16x32(af[buf][tm], wf[buf][tn], acc[tn][tm]) : mfma_16x16x32(wf[buf][tn], af[buf][tm], acc[tn][tm]);
    };
    // Source of the refill in progress (set at a hand-over): the k slice's first byte in both operands and the
    // freed stages' LDS addresses, so that a load costs its own two instructions plus one scalar add.
    const bool part = EPI == EPI_SLAB || tail;   // k range of this workgroup (the whole K unless the launch splits it)
    const int kbeg = part ? split * p.k_per_split : 0;
    const int nk = part ? min(p.k_per_split, K / BKD - kbeg) : K / BKD;
    const char* rf_a = uniform_ptr(reinterpret_cast<const char*>(p.a) + (size_t)kbeg * ROWB);
    const char* rf_w = uniform_ptr(reinterpret_cast<const char*>(p.w) + (size_t)kbeg * w_stage);
    const uint32_t lds_a0 = __builtin_amdgcn_readfirstlane(lds0 + wave * 1024), lds_w0 = lds_a0 + W_LDS;
    uint32_t rf_la = 0, rf_lw = 0;
    // The i-th of the LOADS wave loads of a refill.  Weights first: they come from further away (HBM) than the activations (L2); the
    // skewed ring has a whole iteration more for them and needs the activations first.
    auto is_w = [](int i) { return SKEW ? i >= A_IT : i < W_IT; };
    auto nth = [](int i) { return SKEW ? (i >= A_IT ? i - A_IT : i) : (i < W_IT ? i : i - W_IT); };   // of its own operand
    auto issue_to = [&](int i) __attribute__((always_inline)) { dma16_to(__builtin_amdgcn_readfirstlane(is_w(i) ? rf_lw : rf_la), nth(i) * (NW * 1024)); };
    auto issue_from = [&](int i) __attribute__((always_inline)) {
        if (is_w(i))
            dma16_from<WNT>(rf_w, w_voff[nth(i)]);
        else
            dma16_from(rf_a, a_voff[nth(i)]);
    };
    auto issue_one = [&](int i) __attribute__((always_inline)) {
        const uint32_t to = __builtin_amdgcn_readfirstlane(is_w(i) ? rf_lw : rf_la);
        if (is_w(i))
            dma16<WNT>(rf_w, w_voff[nth(i)], to, nth(i) * (NW * 1024));
        else
            dma16(rf_a, a_voff[nth(i)], to, nth(i) * (NW * 1024));
    };
    // A flag that is either a run-time bool or std::true_type: the steady-state iterations pass the latter, so their
    // loads sit in straight-line code (a branch and its scalar set-up around each load cost more issue slots than
    // the load itself, and a wave has three slots between two MFMAs).
    auto on = [](auto flag) {
        if constexpr (std::is_same_v<decltype(flag), std::true_type>) return true;
        else return flag;
    };
    constexpr int NM = TN * TM, NF = TN + TM;
    // One k step, issued in a fixed order: MFMA i, then the share of the refill loads and of the next
    // step's fragment reads that falls between MFMA i and i + 1.  A 16 x 16 MFMA lasts 16 cycles, in which a wave issues three
    // other instructions: a read or a load goes behind each (both behind one of an iteration's), a read is one instruction (its address a sum
    // made once a step) and a load two: 93 instructions beside the 128 MFMAs of an iteration, where 136 left 2450 cycles for 2048 of MFMAs, now 2280.  A CU's address unit takes one
    // 1 KB load per ~16 cycles, the time of one MFMA, so the refill loads of a stage (LOADS per wave,
    // four waves) are spread over SPREAD quarters of the iteration (a 16-bit k step is two); issued back
    // to back they would hold up the MFMAs behind them.  The MFMAs sit on ONE control path on purpose: at a join the compiler would make
    // them wait for the newest reads.
    constexpr int STEPS = 2, NMS = NM * KSTEPS / STEPS;                        // steps of an iteration, NMS products each
    constexpr int PARTS = 4, SPREAD = 3, SUB = PARTS / STEPS, NMP = NMS / SUB;   // parts of an iteration; the last before the next hand-over stays free: landing time
    // product number i of step `step` after a hand-over (mfma), with the loads of the refill that fall behind it
    auto slot = [&](int step, int i, auto refill_a, auto refill_w, auto mfma) __attribute__((always_inline)) {
        // share of the stage's loads issued in each part, cumulative, in sixteenths: the weights (first half
        // of the loads) go out at once, the activations (L2 hits, quick to land) trail over two more parts
        constexpr int cut[5] = {0, 8, 13, 16, 16};
        const int part = step * SUB + i / NMP, ip = i % NMP, pc = part < SPREAD ? part : SPREAD;
        // (skewed: the activations at once, the weights over all the parts that remain.  EARLY: a small tile with two stages waits at the
        // next hand-over for what it issues at this one, and its products are over long before: everything in the first part.  Spread
        // over all products, codes with both steps' fragments in registers / this: 5120 x 13824, T = 520 77.4 / 64.0 us, 264 62.1 / 56.5;
        // SwiGLU 2816 x 1024 at 2500 13.0 / 12.4)
        const int d_lo = SKEW ? (part == 0 ? 0 : A_IT + (part - 1) * W_IT / (PARTS - 1)) : EARLY ? (part == 0 ? 0 : LOADS) : cut[pc] * LOADS / 16;
        const int d_n = (SKEW ? A_IT + part * W_IT / (PARTS - 1) : EARLY ? LOADS : cut[pc + 1] * LOADS / 16) - d_lo;
        const int d0 = d_lo + ip * d_n / NMP, d1 = SKEW || part < SPREAD ? d_lo + (ip + 1) * d_n / NMP : d0;   // the slot's loads
        auto wanted = [&](int d) __attribute__((always_inline)) { return SKEW && d >= A_IT ? on(refill_w) : on(refill_a); };
        if (d0 < d1 && wanted(d0)) issue_to(d0);
        __builtin_amdgcn_sched_barrier(0);
        mfma();
        __builtin_amdgcn_sched_barrier(0);
        if (d0 < d1 && wanted(d0)) issue_from(d0);
#pragma unroll
        for (int d = d0 + 1; d < d1; ++d)
            if (wanted(d)) issue_one(d);
    };
    auto k_step = [&](int buf, Stage rd_stage, int rd_ks, int step, auto refill_a, auto refill_w) __attribute__((always_inline)) {
        const Source src = source(rd_stage, rd_ks);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            slot(step, i, refill_a, refill_w, [&]() __attribute__((always_inline)) { mfma_one(buf, i); });
            if (i % 2 == 0 && i / 2 < NF) load_frag_one(buf ^ 1, src, i / 2);   // behind every other MFMA, the refill's loads behind the ones between
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // 8-bit operands on 16 x 16 x 128 products: a stage is one k step, and two buffers of its fragments (256 registers on a 256 x 256
    // tile) do not fit beside the sums (small tiles on deep rings do keep two: 1 % of a step of 24 rows).  The wave's products go quarter by quarter instead, weights' halves lo and hi against tokens'
    // halves h and h' = 1 - h: (lo, h), (lo, h'), (hi, h'), (hi, h), and behind each quarter's products come the four fragments or so
    // that the next one adds, into registers whose last reader is over: tokens h' , weights hi, the next stage's lo and, where tokens h'
    // were, the next stage's tokens h'; so the next stage begins with h'.  Every fragment is read once, at an even rate, and the
    // stage is free (and the next one needed) at the hand-over between the second and third quarter.
    constexpr int WH = TN / 2, AH = TM / 2, NQ = WH * AH;
    auto read_w = [&](Source src, int half, int i) __attribute__((always_inline)) { wf[0][half * WH + i] = read_frag(src.w, w_dist(half * WH + i)); };
    auto read_a = [&](Source src, int half, int i) __attribute__((always_inline)) { af[0][half * AH + i] = read_frag(src.a, a_dist(half * AH + i)); };
    auto half_step = [&](bool second, int h, Stage rd_stage, auto refill_a, auto refill_w) __attribute__((always_inline)) {
        const Source src = source(rd_stage, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 2 * NQ; ++i) {
            const int q = i / NQ, j = i % NQ, a_half = second == (q == 0) ? 1 - h : h;
            slot(second ? 0 : 1, i, refill_a, refill_w, [&]() __attribute__((always_inline)) { mfma_one(0, ((second ? WH : 0) + j / AH) * TM + a_half * AH + j % AH); });
            // behind every other product, or, on tiles of few products, evenly
            const bool rd_w = second == (q == 0);
            const int nf = rd_w ? WH : AH;
            const int f0 = 2 * nf <= NQ + 1 ? (j + 1) / 2 : j * nf / NQ, f1 = 2 * nf <= NQ + 1 ? j / 2 + 1 : (j + 1) * nf / NQ;
#pragma unroll
            for (int f = f0; f < min(f1, nf); ++f) {
                if (rd_w)
                    read_w(src, second ? 0 : 1, f);
                else
                    read_a(src, 1 - h, f);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // Small tiles (two or three workgroups per CU, a handful of MFMAs per k step) do better when the
    // compiler orders the steps between hand-overs and the other resident workgroups fill the gaps;
    // only their hand-over step keeps the fixed order, with the whole refill in it.  Tiles of 6 and 8 products per wave run
    // alone on their CU and take the fixed order too: 13B layer, four projections, 250 -> 239 us at T = 256, 347 -> 329 at 400
    // (q/k/v on 128 x 256 tiles 88 -> 77; on 8-bit operands W_down of the 32B shape at T = 1100 180 -> 173), but the SwiGLU
    // kernel on that tile loses (122 -> 129) and keeps the compiler's.
    // (8-bit operands on 256 x 256 with eight waves, two per SIMD, hide the loads' latency without the skewed ring, but a wave's 64 x 128
    // then reads 96 KB of fragments per k step of 1024 cycles beside the 32 KB that land, all the LDS delivers; four waves read
    // 64 KB.  13B layer at T = 3875 on codes: eight waves 1257 us, with the skewed ring too; four 1231, skewed 1194.)
    static_assert(!HALVES || (!F8 && NSW == NS), "halves of 16-bit tiles");
    static_assert(F8 || !FIXED || 2 * NF <= NM, "a fragment read behind every other MFMA");
    static_assert(TN % 2 == 0 && TM % 2 == 0, "halves");
    static_assert(!SKEW || FIXED, "the skewed ring's weights are issued in the fixed order only");
    Stage cur{0, 0};  // stage being computed
    // One k iteration (one LDS stage).  open_a, open_w: what the refill begun at the previous hand-over still issues (stage
    // kt - 1 + NS of the activations, kt - 1 + NSW of the weights, if there is one); next_a, next_w: what this iteration's
    // hand-over starts (stages kt + NS and kt + NSW).  Without the skew both flags of a pair are the same.
    // H (codes: kt % 2): which half of the tokens the stage begins with, or which buffer its fragments are in.
    auto iteration = [&](int kt, auto H, auto open_a, auto open_w, auto next_a, auto next_w) __attribute__((always_inline)) {
        const Stage nxt{cur.a + 1 == NS ? 0 : cur.a + 1, cur.w + 1 == NSW ? 0 : cur.w + 1};
#pragma unroll
        for (int ks = 0; ks + 1 < (QUARTERS ? 2 : KSTEPS); ++ks) {
            if constexpr (QUARTERS) {
                half_step(false, H.value, cur, open_a, open_w);
            } else if constexpr (FIXED) {
                k_step(ks & 1, cur, ks + 1, ks + 1, open_a, open_w);
            } else {
                load_frags((ks + 1) & 1, cur, ks + 1);
#pragma unroll
                for (int i = 0; i < NM; ++i) mfma_one(ks & 1, i);
            }
        }
        // Last k step of the stage: all its fragments are in registers.  Wait for the next stage (the
        // NS - 2 younger ones may stay in flight), hand over, and start refilling the freed buffer.
        // After the last stage this reads fragments nobody uses.
        constexpr int LB = F8 ? decltype(H)::value : 1;   // the buffer of its fragments
        constexpr bool steady = std::is_same_v<decltype(next_w), std::true_type>;   // then kt + NSW < nk
        if ((NS == 2 && !SKEW) || (!steady && kt + NSW - 1 >= nk))
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        else
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NS - 2) * LOADS + (SKEW ? W_IT : 0)) : "memory");
        __syncthreads();
        rf_a += ROWB;
        rf_w += w_stage;
        rf_la = lds_a0 + cur.a * A_BYTES;
        rf_lw = lds_w0 + cur.w * W_BYTES;
        if constexpr (QUARTERS) {
            half_step(true, H.value, nxt, next_a, next_w);
        } else if constexpr (FIXED) {
            k_step(LB, nxt, 0, 0, next_a, next_w);
        } else {
            const Source src = source(nxt, 0);
            // (16-bit EARLY tiles: within eight products, 128 cycles.  5120 x 13824, T = 520 124.0 -> 122.2 us; 64-row tiles as they were)
            constexpr int AT = EARLY ? 8 : NM;
            static_assert(!F8 || !EARLY, "codes with two stages go quarter by quarter");
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NM; ++i) {
                mfma_one(LB, i);
                __builtin_amdgcn_sched_barrier(0);
                if (on(next_a)) {   // (never skewed)
#pragma unroll
                    for (int d = i * LOADS / AT; d < min((i + 1) * LOADS / AT, LOADS); ++d) issue_one(d);
                }
                if constexpr (F8) {   // the next hand-over waits for these: at once
#pragma unroll
                    for (int f = 2 * i; f < min(2 * i + 2, NF); ++f) load_frag_one(LB ^ 1, src, f);
                } else if (i >= NM / 2) {
#pragma unroll
                    for (int f = (i - NM / 2) * NF / (NM - NM / 2); f < (i + 1 - NM / 2) * NF / (NM - NM / 2); ++f)
                        load_frag_one(LB ^ 1, src, f);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        cur = nxt;
    };
    constexpr bool SC = F8 && EPI != EPI_SLAB;
    float4 w_scales[SC ? scale_quads(EPI, TN) : 1];
    if constexpr (SC) load_code_scales<BN, EPI, D>(p, tile_n, wn, lane, w_scales);
    // fill both rings, wait for stage 0 only
#pragma unroll
    for (int s = 0; s < NSW; ++s) {
        if (s >= nk) break;
        if (s < NS) {
#pragma unroll
            for (int j = 0; j < A_IT; ++j) dma16(rf_a + s * ROWB, a_voff[j], lds_a0, s * A_BYTES + j * (NW * 1024));
        }
#pragma unroll
        for (int j = 0; j < W_IT; ++j) dma16<WNT>(rf_w + s * w_stage, w_voff[j], lds_w0, s * W_BYTES + j * (NW * 1024));
    }
    rf_a += (NS - 1) * ROWB;
    rf_w += (NSW - 1) * w_stage;
    if (nk >= NSW)
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 1) * LOADS + (SKEW ? W_IT : 0)) : "memory");
    else
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if constexpr (QUARTERS) {
        const Source src = source(Stage{0, 0}, 0);
#pragma unroll
        for (int i = 0; i < AH; ++i) read_a(src, 0, i);
#pragma unroll
        for (int i = 0; i < WH; ++i) read_w(src, 0, i);
    } else {
        load_frags(0, Stage{0, 0}, 0);
    }
    // first iteration (nothing to refill yet), steady state (every hand-over refills both rings), drain
    const std::integral_constant<int, 0> even;
    const std::integral_constant<int, 1> odd;
    const std::true_type yes;
    f32x4_t total[HALVES ? TN : 1][HALVES ? TM : 1];
    // behind iteration kt (HALVES): at the end of the first k range, which lies in the steady state, its sums step aside
    auto range_end = [&](int kt) __attribute__((always_inline)) {
        if (!HALVES || kt + 1 != p.k_per_split) return;
#pragma unroll
        for (int tn = 0; tn < (HALVES ? TN : 0); ++tn)
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                total[tn][tm] = f32x4_t{0.f, 0.f, 0.f, 0.f} + acc[tn][tm];
                acc[tn][tm] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            }
    };
    int kt = 0;
    if (nk > 0) {
        iteration(0, even, false, false, NS < nk, NSW < nk);
        kt = 1;
    }
    if constexpr (F8) {
        for (; kt + 1 < nk - NSW; kt += 2) {
            iteration(kt, odd, yes, yes, yes, yes);
            iteration(kt + 1, even, yes, yes, yes, yes);
        }
    } else {
        for (; kt < nk - NSW; ++kt) {
            iteration(kt, even, yes, yes, yes, yes);
            range_end(kt);
        }
    }
    while (kt < nk) {
        iteration(kt, std::integral_constant<int, F8 ? 1 : 0>{}, kt - 1 + NS < nk, kt - 1 + NSW < nk, kt + NS < nk, kt + NSW < nk);
        ++kt;
        if (F8) {   // (kt was odd)
            if (kt == nk) break;
            iteration(kt, even, kt - 1 + NS < nk, kt - 1 + NSW < nk, kt + NS < nk, kt + NSW < nk);
            ++kt;
        }
    }
    if constexpr (HALVES) {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) acc[tn][tm] = total[tn][tm] + acc[tn][tm];
    }
    if (EPI != EPI_SLAB && tail) {
        // Partial tile -> this split's slab (accumulator tile (tn, tm) of thread tid is the 16 bytes at
        // (tn TM + tm) * threads + tid: coalesced).
        // gemm_tail_finish_kernel, launched behind this kernel, adds the slabs of a tile in split order and
        // runs the epilogue; the kernel boundary is what makes the slabs of workgroups on other XCDs
        // (other L2s) visible, so nothing here waits or fences.
        constexpr int AREA4 = BM * BN / 4, NT = 64 * NW;
        f32x4_t* slab = reinterpret_cast<f32x4_t*>(p.tail_buf) + ((size_t)split * p.tail_tiles + tail_idx) * AREA4 + tid;
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) slab[(tn * TM + tm) * NT] = acc[tn][tm];
        return;
    }
    if constexpr (EPI == EPI_SLAB) {   // split-K partial sums -> this split's slab: plain rows of fp32
        p.out = p.accum + (int64_t)split * p.T * p.N;
        gemm_epilogue16<BM, BN, EPI, 0, false>(acc, p, tile_m, tile_n, wm, wn, lane, 0);
    } else {
        gemm_epilogue16<BM, BN, EPI, D, F8>(acc, p, tile_m, tile_n, wm, wn, lane, 0, w_scales);
    }
}

// Second half of a tail split: workgroup (tail tile, row tm of accumulator tiles) has the thread layout of
// the GEMM workgroup that wrote the slabs, adds its part of the tile's slabs in split order (so the sum
// does not depend on scheduling) and runs the GEMM's own epilogue on it.
template <int BM, int BN, int EPI, int D, bool SC = false>
__global__ void __launch_bounds__(64 * WGM * WGN) gemm_tail_finish_kernel(GemmArgs p) {
    constexpr int NW = WGM * WGN, NT = 64 * NW, TM = BM / (16 * WGM), TN = BN / (16 * WGN), AREA4 = BM * BN / 4;
    constexpr int H = 2;   // rows of accumulator tiles a workgroup finishes: 32 tokens per wave
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    const int tail_idx = blockIdx.x / (TM / H), tm_sel = blockIdx.x % (TM / H);
    int tile_m, tile_n;
    tile_coords(p.tiles_m * p.tiles_n - p.tail_tiles + tail_idx, p.tiles_m, p.tiles_n, tile_m, tile_n);
    f32x4_t acc[TN][H];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int h = 0; h < H; ++h) acc[tn][h] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    float4 w_scales[SC ? scale_quads(EPI, TN) : 1];
    if constexpr (SC) load_code_scales<BN, EPI, D>(p, tile_n, wn, lane, w_scales);
    for (int q = 0; q < p.tail_splits; ++q) {
        const f32x4_t* src = reinterpret_cast<const f32x4_t*>(p.tail_buf) + ((size_t)q * p.tail_tiles + tail_idx) * AREA4 + tid;
        f32x4_t v[TN][H];
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int h = 0; h < H; ++h) v[tn][h] = src[(tn * TM + H * tm_sel + h) * NT];
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int h = 0; h < H; ++h) acc[tn][h] += v[tn][h];
    }
    gemm_epilogue16<BM, BN, EPI, D, SC>(acc, p, tile_m, tile_n, wm, wn, lane, tm_sel, w_scales);
}

// ------------------------------------------------------------------------------------------
// Split-K companion kernel: adds the splits' slabs in split order (the sum does not depend on scheduling)
// and applies the same epilogues as the fused path; each thread owns 4 consecutive features of one token.
// ------------------------------------------------------------------------------------------
//
// A thread's work is one chain of memory round trips, and at a few tokens nothing else runs, so the launch costs its longest
// chain: every load of up to eight slabs, and whatever the epilogue reads beside them, is issued before the first addition.
// (One slab after the other was a round trip each, to slabs that other XCDs wrote.)
// One 13B layer with the norms' change (rmsnorm_kernel): four decode rows 140.7 -> 135.4 us.
template <int NV, int N>
__device__ __forceinline__ void slab_add(const float* const (&first)[NV], int64_t slab_stride, float4 (&v)[NV]) {
    float4 w[N][NV];
#pragma unroll
    for (int q = 0; q < N; ++q)
#pragma unroll
        for (int j = 0; j < NV; ++j) w[q][j] = *reinterpret_cast<const float4*>(first[j] + q * slab_stride);
#pragma unroll
    for (int q = 0; q < N; ++q)
#pragma unroll
        for (int j = 0; j < NV; ++j) v[j].x += w[q][j].x, v[j].y += w[q][j].y, v[j].z += w[q][j].z, v[j].w += w[q][j].w;
}

// the sums over n_splits >= 1 slabs, in split order, at NV places of one row (first: the places in slab 0)
template <int NV>
__device__ __forceinline__ void slab_sums(const float* (&first)[NV], int64_t slab_stride, int n_splits, float4 (&v)[NV]) {
#pragma unroll
    for (int j = 0; j < NV; ++j) v[j] = make_float4(-0.0f, -0.0f, -0.0f, -0.0f);   // the identity of the addition, also of -0
    for (; n_splits > 8; n_splits -= 8) {
        slab_add<NV, 8>(first, slab_stride, v);
#pragma unroll
        for (int j = 0; j < NV; ++j) first[j] += 8 * slab_stride;
    }
    switch (n_splits) {
        case 1: return slab_add<NV, 1>(first, slab_stride, v);
        case 2: return slab_add<NV, 2>(first, slab_stride, v);
        case 3: return slab_add<NV, 3>(first, slab_stride, v);
        case 4: return slab_add<NV, 4>(first, slab_stride, v);
        case 5: return slab_add<NV, 5>(first, slab_stride, v);
        case 6: return slab_add<NV, 6>(first, slab_stride, v);
        case 7: return slab_add<NV, 7>(first, slab_stride, v);
        default: return slab_add<NV, 8>(first, slab_stride, v);
    }
}

// factor a_scale * w_scale[n .. n + 3] of sums of products of 8-bit codes (w_scale is null for 16-bit operands)
__device__ __forceinline__ float4 code_factor(const GemmArgs& p, int n) {
    float4 w = make_float4(1.f, 1.f, 1.f, 1.f);
    if (p.w_scale) {
        w = *reinterpret_cast<const float4*>(p.w_scale + n);
        w.x *= p.a_scale; w.y *= p.a_scale; w.z *= p.a_scale; w.w *= p.a_scale;
    }
    return w;
}
__device__ __forceinline__ void code_scale(float4& v, const GemmArgs& p, const float4& f) {
    if (p.w_scale) v.x *= f.x, v.y *= f.y, v.z *= f.z, v.w *= f.w;
}

// A unit: 4 consecutive features, or a pair of such quads that the epilogue combines.  flat_units = 0: blockIdx.y = token, blockIdx.x =
// 256 of its units.  Where a token's units do not fill workgroups (flat_units > 0: their number) the units of all tokens are one run:
// with a workgroup per token, 7980 rows of 256 features took 5.8 us instead of 5.2.
template <int EPI, int D>
__global__ void __launch_bounds__(256) gemm_finish_kernel(GemmArgs p, int flat_units) {
    int t = blockIdx.y, u = blockIdx.x * 256 + threadIdx.x;
    if (flat_units > 0) {
        t = u / flat_units;
        u -= t * flat_units;
        if (t >= p.T) return;
    }
    const int64_t stride = (int64_t)p.T * p.N;
    const float* row = p.accum + (int64_t)t * p.N;
    if (EPI == EPI_SWIGLU) {
        const int c = u * 4;
        if (c >= p.n_half) return;
        const float4 fg = code_factor(p, c), fu = code_factor(p, p.n_half + c);
        const float* src[2] = {row + c, row + p.n_half + c};
        float4 v[2];
        slab_sums(src, stride, p.n_splits, v);
        code_scale(v[0], p, fg);
        code_scale(v[1], p, fu);
        const float4 gt = v[0], up = v[1];
        const float o0 = silu_mul(gt.x, up.x), o1 = silu_mul(gt.y, up.y), o2 = silu_mul(gt.z, up.z), o3 = silu_mul(gt.w, up.w);
        if (p.out_f8) {
            const float sc = p.out_inv;
            *reinterpret_cast<uint32_t*>(static_cast<uint8_t*>(p.out) + (int64_t)t * p.n_half + c) = pack_fp8x4(o0 * sc, o1 * sc, o2 * sc, o3 * sc);
            return;
        }
        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(p.out) + (int64_t)t * p.n_half + c) =
            make_uint2(pack_bf16x2(o0, o1), pack_bf16x2(o2, o3));
    } else if (EPI == EPI_QKV_ROPE) {
        // units per token: rotated heads need (lo, hi) quads: (n_q + n_kv) * D / 8; v heads: n_kv * D / 4
        constexpr int HALF = (D > 0 ? D : 64) / 2;
        const int rot_units = (p.n_q + p.n_kv) * (HALF / 4), v_units = p.n_kv * (2 * HALF / 4);
        if (u >= rot_units + v_units) return;
        const int64_t slot = p.tok_slot[t];
        const int kv_dim = p.n_kv * 2 * HALF;
        if (u < rot_units) {
            const int head = u / (HALF / 4), i0 = (u % (HALF / 4)) * 4, n = head * 2 * HALF + i0;
            const float2* cs = p.rope_cs + (int64_t)t * HALF + i0;
            const float4 c01 = *reinterpret_cast<const float4*>(cs), c23 = *reinterpret_cast<const float4*>(cs + 2);
            const float4 f_lo = code_factor(p, n), f_hi = code_factor(p, n + HALF);
            const float* src[2] = {row + n, row + n + HALF};
            float4 v[2];
            slab_sums(src, stride, p.n_splits, v);
            code_scale(v[0], p, f_lo);
            code_scale(v[1], p, f_hi);
            float4 rl, rh;
            rotate4(v[0], v[1], c01, c23, rl, rh);
            if (p.kv_fp8 && head >= p.n_q) {
                uint8_t* dst8 = reinterpret_cast<uint8_t*>(p.k_pages) + slot * kv_dim + (head - p.n_q) * 2 * HALF + i0;
                const float s = p.k_inv;
                *reinterpret_cast<uint32_t*>(dst8) = pack_fp8x4(rl.x * s, rl.y * s, rl.z * s, rl.w * s);
                *reinterpret_cast<uint32_t*>(dst8 + HALF) = pack_fp8x4(rh.x * s, rh.y * s, rh.z * s, rh.w * s);
                return;
            }
            uint16_t* dst = head < p.n_q ? static_cast<uint16_t*>(p.out) + (int64_t)t * (p.n_q * 2 * HALF) + head * 2 * HALF
                                         : p.k_pages + slot * kv_dim + (head - p.n_q) * 2 * HALF;
            *reinterpret_cast<uint2*>(dst + i0) = make_uint2(pack_bf16x2(rl.x, rl.y), pack_bf16x2(rl.z, rl.w));
            *reinterpret_cast<uint2*>(dst + HALF + i0) = make_uint2(pack_bf16x2(rh.x, rh.y), pack_bf16x2(rh.z, rh.w));
        } else {
            const int c = (u - rot_units) * 4, n = (p.n_q + p.n_kv) * 2 * HALF + c;
            const float4 f = code_factor(p, n);
            const float* src[1] = {row + n};
            float4 v1[1];
            slab_sums(src, stride, p.n_splits, v1);
            code_scale(v1[0], p, f);
            const float4 v = v1[0];
            if (p.kv_fp8) {
                const float s = p.v_inv;
                *reinterpret_cast<uint32_t*>(reinterpret_cast<uint8_t*>(p.v_pages) + slot * kv_dim + c) =
                    pack_fp8x4(v.x * s, v.y * s, v.z * s, v.w * s);
            } else {
                *reinterpret_cast<uint2*>(p.v_pages + slot * kv_dim + c) = make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
            }
        }
    } else {
        const int c = u * 4;
        if (c >= p.N) return;
        const int64_t o = (int64_t)t * p.N + c;
        uint2 rb = make_uint2(0, 0);
        float4 rf = make_float4(0.f, 0.f, 0.f, 0.f);
        if (EPI == EPI_RES_BF16_OUT_F32 && p.residual) rb = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(p.residual) + o);
        if (EPI == EPI_RES_F32_OUT_BF16) rf = *reinterpret_cast<const float4*>(static_cast<const float*>(p.residual) + o);
        const float4 f = code_factor(p, c);
        const float* src[1] = {row + c};
        float4 v1[1];
        slab_sums(src, stride, p.n_splits, v1);
        code_scale(v1[0], p, f);
        float4 v = v1[0];
        if (EPI == EPI_RES_BF16_OUT_F32) {
            if (p.residual) v.x += bf16_lo(rb.x), v.y += bf16_hi(rb.x), v.z += bf16_lo(rb.y), v.w += bf16_hi(rb.y);
            *reinterpret_cast<float4*>(static_cast<float*>(p.out) + o) = v;
        } else {
            if (EPI == EPI_RES_F32_OUT_BF16) v.x += rf.x, v.y += rf.y, v.z += rf.z, v.w += rf.w;
            *reinterpret_cast<uint2*>(static_cast<uint16_t*>(p.out) + o) = make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
        }
    }
}

// The finish kernel of a projection whose output rows an RMSNorm reads next (W_o into the post-attention norm; W_down into the
// next layer's input norm): a workgroup per token adds the slabs of its whole row, writes the row and norms it.  What is saved
// is a launch and its chain of round trips: 24 rows of 5120 3.9 + 4.6 -> 4.9 us, 256 rows of 8192 8.4 + 5.3 -> 10.8, a layer of 128
// rows on 8-bit operands 330.2 -> 326.2 (with the attention's own codes), four layers of 24 rows 857 -> 819 (with the step before).
// The row's place in the LDS has its own length: with 32 KB for every row 128 decode rows and a 512-token chunk took 1 % longer.
// A thread owns one chunk of 8 features (N <= 8192).  The sum of squares runs in rmsnorm_kernel's order -- 256 threads, chunk
// after chunk, from the row in LDS -- so that the normed values have the same bits on both paths.
// Narrow rows leave most of a workgroup's threads (256 at least) without a chunk, which counts once the rows fill the chip.  A layer step,
// finish + norm / fused, us: 1000 rows of 128 56.3 / 54.8, 256 62.0 / 60.5, 512 72.4 / 70.8, 1024 84.5 / 82.8; 1500 69.5 / 69.7, 67.8 / 68.2,
// 76.6 / 76.4, 88.5 / 89.2; 2500 68.6 / 69.9, 75.4 / 76.2, 86.7 / 87.5, 102.7 / 102.6.  (3500: 72.7 / 75.3, 82.6 / 84.7, 93.6 / 95.3,
// 114.8 / 113.4: of 1024 features on it would still pay.)
constexpr int FINISH_NORM_MAX_N = 8192;
constexpr int finish_norm_max_rows(int n) { return n >= 1024 ? 2560 : 1280; }
template <int EPI>
__global__ void __launch_bounds__(1024) gemm_finish_norm_kernel(GemmArgs p, const uint16_t* __restrict__ norm_w, float eps,
                                                                uint16_t* __restrict__ norm_out, float code_inv) {
    static_assert(EPI == EPI_RES_BF16_OUT_F32 || EPI == EPI_RES_F32_OUT_BF16, "epilogues with whole rows of the residual stream");
    extern __shared__ __align__(16) unsigned char smem[];   // the row; its own length, so that narrow rows leave room for more workgroups
    float* const vals = reinterpret_cast<float*>(smem);
    __shared__ float red[4];
    const int t = blockIdx.x, tid = threadIdx.x, chunks = p.N / 8;
    const bool on = tid < chunks;
    const int n = 8 * min(tid, chunks - 1);   // threads past the row: the last chunk again, nothing of it stored
    const int64_t o = (int64_t)t * p.N + n;
    const uint4 wu = *reinterpret_cast<const uint4*>(norm_w + n);
    uint4 rb = make_uint4(0, 0, 0, 0);
    float4 rf[2] = {};
    if (EPI == EPI_RES_BF16_OUT_F32) {
        if (p.residual) rb = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(p.residual) + o);
    } else {
        rf[0] = *reinterpret_cast<const float4*>(static_cast<const float*>(p.residual) + o);
        rf[1] = *reinterpret_cast<const float4*>(static_cast<const float*>(p.residual) + o + 4);
    }
    const float4 f0 = code_factor(p, n), f1 = code_factor(p, n + 4);
    const float* src[2] = {p.accum + o, p.accum + o + 4};
    float4 s[2];
    slab_sums(src, (int64_t)p.T * p.N, p.n_splits, s);
    code_scale(s[0], p, f0);
    code_scale(s[1], p, f1);
    float v[8] = {s[0].x, s[0].y, s[0].z, s[0].w, s[1].x, s[1].y, s[1].z, s[1].w};
    if (EPI == EPI_RES_BF16_OUT_F32) {
        if (p.residual) {
            v[0] += bf16_lo(rb.x); v[1] += bf16_hi(rb.x); v[2] += bf16_lo(rb.y); v[3] += bf16_hi(rb.y);
            v[4] += bf16_lo(rb.z); v[5] += bf16_hi(rb.z); v[6] += bf16_lo(rb.w); v[7] += bf16_hi(rb.w);
        }
        if (on) {
            float4* x1 = reinterpret_cast<float4*>(static_cast<float*>(p.out) + o);
            x1[0] = make_float4(v[0], v[1], v[2], v[3]);
            x1[1] = make_float4(v[4], v[5], v[6], v[7]);
        }
    } else {   // the norm reads the row as it was stored, rounded to bf16
        v[0] += rf[0].x; v[1] += rf[0].y; v[2] += rf[0].z; v[3] += rf[0].w;
        v[4] += rf[1].x; v[5] += rf[1].y; v[6] += rf[1].z; v[7] += rf[1].w;
        const uint4 y = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
        if (on) *reinterpret_cast<uint4*>(static_cast<uint16_t*>(p.out) + o) = y;
        v[0] = bf16_lo(y.x); v[1] = bf16_hi(y.x); v[2] = bf16_lo(y.y); v[3] = bf16_hi(y.y);
        v[4] = bf16_lo(y.z); v[5] = bf16_hi(y.z); v[6] = bf16_lo(y.w); v[7] = bf16_hi(y.w);
    }
    if (on) {
        *reinterpret_cast<float4*>(vals + n) = make_float4(v[0], v[1], v[2], v[3]);
        *reinterpret_cast<float4*>(vals + n + 4) = make_float4(v[4], v[5], v[6], v[7]);
    }
    __syncthreads();
    if (tid < 256) {
        float ss = 0.f;
        for (int c = tid; c < chunks; c += 256) {
            const float4 a = *reinterpret_cast<const float4*>(vals + 8 * c), b = *reinterpret_cast<const float4*>(vals + 8 * c + 4);
            ss = __builtin_fmaf(a.x, a.x, ss); ss = __builtin_fmaf(a.y, a.y, ss); ss = __builtin_fmaf(a.z, a.z, ss); ss = __builtin_fmaf(a.w, a.w, ss);
            ss = __builtin_fmaf(b.x, b.x, ss); ss = __builtin_fmaf(b.y, b.y, ss); ss = __builtin_fmaf(b.z, b.z, ss); ss = __builtin_fmaf(b.w, b.w, ss);
        }
        ss = wave_sum(ss);
        if ((tid & 63) == 0) red[tid >> 6] = ss;
    }
    __syncthreads();
    const float inv = 1.0f / sqrtf((red[0] + red[1] + red[2] + red[3]) / (float)p.N + eps);
    if (on) norm_store8(v, inv, wu, code_inv, norm_out, o);
}

// Small problems: one WAVE per tile of 32 tokens x 32 features (two such feature tiles where the epilogue combines pairs), operands
// straight from global memory to registers.  A projection of a narrow layer at a few hundred tokens is a few dozen MFMAs per
// wave and bound by latencies: the launch, the first touch of every operand, and the instruction fetch of code that runs once (the
// tiled kernels' unrolled loops and epilogue are 10 - 40 KB, this one 2 - 4).  So there is no LDS, no barrier and no ring to fill:
// eight k steps of 16 are in flight behind the eight being multiplied, and what the epilogue reads is fetched first.
// The sums run over k in the tiled kernels' order: same bits.  Tiny layer (hidden 256, 134 tokens): q/k/v 10.4 -> 4.6 us, W_o
// 4.9 -> 3.5, W_down (k = 688) 10.1 -> 4.8, the step 47.8 -> 30.2.
template <int EPI, int D = 0>
__global__ void __launch_bounds__(64) gemm_small_kernel(GemmArgs p) {
    constexpr bool PAIRED = EPI == EPI_SWIGLU || EPI == EPI_QKV_ROPE;
    constexpr int NT = PAIRED ? 2 : 1, U = 8;
    constexpr int DH = D > 0 ? D : 64;
    const int lane = threadIdx.x, l32 = lane & 31, g = lane >> 5;
    const int unit = blockIdx.x / p.tiles_m, t = (int)(blockIdx.x % p.tiles_m) * 32 + l32, tc = min(t, p.T - 1);
    int head = 0, n0[NT], rows[NT];   // first feature of each tile, and how many rows of the weight matrix it has from there
    if (EPI == EPI_QKV_ROPE) {
        head = unit / (DH / 64);
        n0[0] = head * DH + unit % (DH / 64) * 32;
        n0[NT - 1] = n0[0] + DH / 2;
        rows[0] = rows[NT - 1] = 32;
    } else if (EPI == EPI_SWIGLU) {
        n0[0] = unit * 32;
        n0[NT - 1] = p.n_half + n0[0];
        rows[0] = rows[NT - 1] = min(32, p.n_half - n0[0]);
    } else {
        n0[0] = unit * 32;
        rows[0] = min(32, p.N - n0[0]);
    }
    // what the epilogue reads besides the sums: quad q = features 8 q + 4 g ..
    float4 oa[4], ob[4];
    int slot = 0;
    if (EPI == EPI_QKV_ROPE) slot = p.tok_slot[tc];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int f = 8 * q + 4 * g;
        oa[q] = ob[q] = make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (EPI == EPI_QKV_ROPE) {
            const float4* cs = reinterpret_cast<const float4*>(p.rope_cs + (int64_t)tc * (DH / 2) + n0[0] - head * DH + f);
            oa[q] = cs[0];
            ob[q] = cs[1];
        } else if constexpr (EPI == EPI_RES_BF16_OUT_F32) {
            if (p.residual && f < rows[0]) {   // no residual given: plain fp32 output
                const uint2 r = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(p.residual) + (int64_t)tc * p.N + n0[0] + f);
                oa[q].x = __uint_as_float(r.x);
                oa[q].y = __uint_as_float(r.y);
            }
        } else if constexpr (EPI == EPI_RES_F32_OUT_BF16) {
            if (f < rows[0]) oa[q] = *reinterpret_cast<const float4*>(static_cast<const float*>(p.residual) + (int64_t)tc * p.N + n0[0] + f);
        }
    }
    // operands: k step s is 32 bytes of every row, this lane's half of them 16 (g)
    const char* const ab = reinterpret_cast<const char*>(p.a);
    const char* const wb = reinterpret_cast<const char*>(p.w);
    const uint32_t a_off = ((uint32_t)tc * (uint32_t)p.K + 8 * g) * 2;
    const int w_slice = p.w_packed ? 32768 : 128;   // from one 64-k slice of a row to the next
    uint32_t w_off[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const uint32_t n = n0[j] + min(l32, rows[j] - 1);   // rows past the end: the last one again, never stored
        w_off[j] = (p.w_packed ? (n >> 8) * (uint32_t)p.K * 512u + (n & 255) * 128u : n * (uint32_t)p.K * 2u) + 16 * g;
    }
    const int steps = p.K / 16;
    uint4 a[2][U], w[2][U][NT];
    auto load = [&](int buf, int s0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = min(s0 + u, steps - 1);
            a[buf][u] = *reinterpret_cast<const uint4*>(ab + s * 32 + a_off);
#pragma unroll
            for (int j = 0; j < NT; ++j) w[buf][u][j] = *reinterpret_cast<const uint4*>(wb + (size_t)(s >> 2) * w_slice + (s & 3) * 32 + w_off[j]);
        }
    };
    f32x16_t acc[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
    auto step = [&](int buf, int u) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[j] = mfma_32x32x16(as_bf16x8(w[buf][u][j]), as_bf16x8(a[buf][u]), acc[j]);
    };
    auto batch = [&](int buf, int s0) __attribute__((always_inline)) {
        if (s0 + U <= steps) {
#pragma unroll
            for (int u = 0; u < U; ++u) step(buf, u);
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (s0 + u < steps) step(buf, u);
        }
    };
    load(0, 0);
    for (int s0 = 0; s0 < steps; s0 += 2 * U) {
        if (s0 + U < steps) load(1, s0 + U);
        batch(0, s0);
        if (s0 + U < steps) {
            if (s0 + 2 * U < steps) load(0, s0 + 2 * U);
            batch(1, s0 + U);
        }
    }
    if (t >= p.T) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int f = 8 * q + 4 * g;
        if (f >= rows[0]) break;   // rows are a multiple of 4 (of 8 in pairs)
        const float4 lo = make_float4(acc[0][4 * q], acc[0][4 * q + 1], acc[0][4 * q + 2], acc[0][4 * q + 3]);
        const float4 hi = make_float4(acc[NT - 1][4 * q], acc[NT - 1][4 * q + 1], acc[NT - 1][4 * q + 2], acc[NT - 1][4 * q + 3]);
        store_unit<EPI, D>(p, t, n0[0] + f, head, lo, hi, oa[q], ob[q], slot);
    }
}

template <int EPI, int D = 0>
hipError_t launch_small(GemmArgs p, hipStream_t s) {
    p.tiles_m = (p.T + 31) / 32;
    p.tiles_n = EPI == EPI_QKV_ROPE ? (p.n_q + 2 * p.n_kv) * (D / 64) : ((EPI == EPI_SWIGLU ? p.n_half : p.N) + 31) / 32;
    gemm_small_kernel<EPI, D><<<dim3(p.tiles_m * p.tiles_n), dim3(64), 0, s>>>(p);
    return hipGetLastError();
}

// Skinny path: T <= 256.  The weights are streamed once; to fill 256 CUs the k range of every
// BM x BN tile (64 / 128 / 192 / 256 tokens x 128 features; x 256 for split_rows) is split over several workgroups, each
// storing its partial tile to its split's slab.  The LDS ring is as deep as 160 KB allow (one workgroup
// per CU); all stages but the one being computed are in flight.
template <int BM, int EPI, int D, int BN = 256, bool WNT = false>
hipError_t launch_split(GemmArgs p, int splits, hipStream_t s, NextNorm* next = nullptr) {
    constexpr int NS = BM + BN <= 192 ? 6 : BM + BN <= 256 ? 4 : BM + BN <= 320 ? 4 : BM + BN <= 384 ? 3 : 2;
    constexpr int NSW = weight_stages(BM, BN, NS);
    constexpr int smem = (NS * BM + NSW * BN) * 64 * 2;
    static_assert(smem <= 160 * 1024, "ring exceeds the LDS");
    p.tiles_m = (p.T + BM - 1) / BM;
    p.tiles_n = (p.N + BN - 1) / BN;
    const int nk = p.K / 64;
    p.k_per_split = (nk + splits - 1) / splits;
    splits = (nk + p.k_per_split - 1) / p.k_per_split;   // no empty split: the finish kernel reads every slab
    p.n_splits = splits;
    // the slabs [split][T, N] have to fit what the workspace reserves (a lower bound of it: this projection's own N)
    if ((int64_t)splits * p.T * p.N > gemm_scratch_floats(p.T, p.N)) return hipErrorInvalidValue;
    auto go = [&](auto f8) -> hipError_t {
        constexpr bool F8 = decltype(f8)::value;
        static std::once_flag once;
        static hipError_t attr_status = hipSuccess;
        if (hipError_t e = allow_smem_once(once, attr_status, &gemm_dma_kernel<BM, BN, EPI_SLAB, 0, 64, NS, WNT, F8, NSW>, smem)) return e;
        gemm_dma_kernel<BM, BN, EPI_SLAB, 0, 64, NS, WNT, F8, NSW><<<dim3(p.tiles_m * p.tiles_n * splits), dim3(256), smem, s>>>(p);
        return hipGetLastError();
    };
    hipError_t e = p.f8 ? go(std::true_type{}) : go(std::false_type{});
    if (e != hipSuccess) return e;
    if constexpr (EPI == EPI_RES_BF16_OUT_F32 || EPI == EPI_RES_F32_OUT_BF16) {
        if (next && p.N % 8 == 0 && p.N <= FINISH_NORM_MAX_N && p.T <= finish_norm_max_rows(p.N)) {
            const int threads = std::max(256, (p.N / 8 + 63) / 64 * 64);
            const float code_inv = next->code_scale > 0.0f ? (float)(1.0 / (double)next->code_scale) : 0.0f;   // as launch_rmsnorm
            gemm_finish_norm_kernel<EPI><<<dim3(p.T), dim3(threads), p.N * sizeof(float), s>>>(p, static_cast<const uint16_t*>(next->w), next->eps,
                                                                             static_cast<uint16_t*>(next->out), code_inv);
            next->done = true;
            return hipGetLastError();
        }
    }
    int units;   // of a token
    if (EPI == EPI_SWIGLU)
        units = p.n_half / 4;
    else if (EPI == EPI_QKV_ROPE)
        units = (p.n_q + p.n_kv) * (D / 8) + p.n_kv * (D / 4);
    else
        units = p.N / 4;
    const bool flat = units % 256 != 0;   // (the split paths bound tokens x features by 2^24)
    gemm_finish_kernel<EPI, D><<<flat ? dim3((unsigned)(((int64_t)p.T * units + 255) / 256)) : dim3(units / 256, p.T), dim3(256), 0, s>>>(
        p, flat ? units : 0);
    return hipGetLastError();
}

// Number of k splits for a skinny GEMM: enough workgroups for every CU, at least 4 k steps each.
int choose_splits(int T, int N, int K, int BM, int BN = 256) {
    const int tiles = ((T + BM - 1) / BM) * ((N + BN - 1) / BN);
    const int nk = K / 64;
    int splits = 256 / tiles;   // one workgroup per CU: a single full round
    splits = std::min(splits, std::max(1, nk / 4));
    return std::max(1, splits);
}

// The fused kernel on 128-feature tiles with a deep ring, one workgroup per CU: for a skinny GEMM whose
// tiles fill the CUs without any k split (the gate/up projection), so no slabs and no finish kernel.
template <int BM, int EPI, int D = 0, int BN = 128, bool WNT = true>
hipError_t launch_skinny_whole(GemmArgs p, hipStream_t s) {
    // (256 x 256 tiles have room for two 64-k stages and a third of the weights; four 32-k stages measured no faster)
    constexpr int BKD = 64;
    constexpr int NS = BM + BN <= 192 ? 6 : BM + BN <= 256 ? 4 : BM + BN <= 384 ? 3 : 2;
    constexpr int NSW = weight_stages(BM, BN, NS);
    constexpr int smem = (NS * BM + NSW * BN) * BKD * 2;
    static_assert(smem <= 160 * 1024, "ring exceeds the LDS");
    p.tiles_m = (p.T + BM - 1) / BM;
    p.tiles_n = EPI == EPI_SWIGLU ? (p.n_half + BN / 2 - 1) / (BN / 2) : (p.N + BN - 1) / BN;
    p.tail_tiles = 0;
    p.tail_splits = 1;
    auto go = [&](auto f8) -> hipError_t {
        constexpr bool F8 = decltype(f8)::value;
        static std::once_flag once;
        static hipError_t attr_status = hipSuccess;
        if (hipError_t e = allow_smem_once(once, attr_status, &gemm_dma_kernel<BM, BN, EPI, D, BKD, NS, WNT, F8, NSW>, smem)) return e;
        gemm_dma_kernel<BM, BN, EPI, D, BKD, NS, WNT, F8, NSW><<<dim3(p.tiles_m * p.tiles_n), dim3(256), smem, s>>>(p);
        return hipGetLastError();
    };
    return p.f8 ? go(std::true_type{}) : go(std::false_type{});
}

template <int EPI, int D>
hipError_t launch_skinny(const GemmArgs& p, hipStream_t s, NextNorm* next = nullptr) {
    if (p.T <= 128) {
        // One token tile: the MFMA work is small next to the weight stream, so 128-feature tiles cost nothing
        // and need half the k splits (half the slab traffic); the gate/up projection has enough of them to
        // fill the CUs unsplit and runs the fused kernel.
        if constexpr (EPI == EPI_SWIGLU) {
            const int tiles = (p.n_half + 63) / 64, rounds = (tiles + 255) / 256;
            if (tiles >= 0.8 * 256 * rounds)
                return p.T <= 64 ? launch_skinny_whole<64, EPI>(p, s) : launch_skinny_whole<128, EPI>(p, s);
        }
        if (p.T <= 64) return launch_split<64, EPI, D, 128, true>(p, choose_splits(p.T, p.N, p.K, 64, 128), s, next);
        return launch_split<128, EPI, D, 128, true>(p, choose_splits(p.T, p.N, p.K, 128, 128), s, next);
    }
    // 129 .. 256 tokens: one token tile of 192 or 256 rows x 128 features, so that every weight is read once (two tiles of
    // 128 rows read them twice; what the CUs draw from the L2 is the bound here, weights and activations together).
    // A projection that fills the CUs without a k split runs whole.  13B layer, its four projections, before -> now:
    // 248 -> 208 us at T = 160, 253 -> 232 at 200, 265 -> 239 at 256 (with an event pair per launch).
    // The k ranges are those of 128 x 256 tiles (never fewer tiles than these): how often a sum is cut does not depend on
    // the tile that computes it.
    const int splits = choose_splits(p.T, p.N, p.K, 128);
    if (splits == 1) {
        // wide enough that one 256 x 256 tile per CU is (nearly) a full round: half the activation reads again
        const int tiles256 = EPI == EPI_SWIGLU ? (p.n_half + 127) / 128 : (p.N + 255) / 256;
        if (p.T > 192 && tiles256 >= 200 && tiles256 <= 256) return launch_skinny_whole<256, EPI, D, 256>(p, s);
        if constexpr (EPI == EPI_QKV_ROPE)   // the fused rotation needs 128 features per wave
            return launch_skinny_whole<128, EPI, D, 256>(p, s);
        else
            return p.T <= 192 ? launch_skinny_whole<192, EPI>(p, s) : launch_skinny_whole<256, EPI>(p, s);
    }
    return p.T <= 192 ? launch_split<192, EPI, D, 128, true>(p, splits, s, next) : launch_split<256, EPI, D, 128, true>(p, splits, s, next);
}

// The output layer of a decode batch: at most 256 rows against a weight matrix far larger than the activations, with no
// scratch to split k into.  Wide enough that 128-feature tiles fill the CUs, it runs as ONE token tile on a deep ring, so
// that the weights are read once; the general plan takes 64 x 128 tiles with one stage in flight and, beyond 64 rows, reads
// the weights once per 64 rows.  32000 x 5120: 24 rows 86 -> 54 us, 129 rows 112 -> 77.
// The deep ring pays where a tile is long against filling it: not for k below 512 (32000 x 256, 100 rows: 9 -> 10 us), nor, one
// workgroup per CU, for several rounds of short tiles (60000 x 2048: 160 rows 66 -> 73).  At 65 .. 128 rows of several rounds
// the general plan's three workgroups per CU are faster (128256 x 5120, 100 rows: 252 against 293).
bool wide_whole_applies(const GemmArgs& p) {
    const int tiles = (p.N + 127) / 128, rounds = (tiles + 255) / 256;
    if (p.accum || p.T > SKINNY_MAX_T || p.K % 64 || tiles < 0.8 * 256 * rounds || forced_cand() >= 0) return false;
    return rounds == 1 ? p.K >= 512 : p.K >= 3072 && (p.T <= 64 || p.T > 128);
}

template <int EPI>
hipError_t launch_wide_whole(const GemmArgs& p, hipStream_t s) {
    if (p.T <= 64) return launch_skinny_whole<64, EPI>(p, s);
    if (p.T <= 128) return launch_skinny_whole<128, EPI>(p, s);
    if (p.T <= 192) return launch_skinny_whole<192, EPI>(p, s);
    return launch_skinny_whole<256, EPI>(p, s);
}

bool skinny_applies(int T, int N, int K, const float* accum) {
    return accum != nullptr && T <= SKINNY_MAX_T && K % 64 == 0 && N % 4 == 0;
}

// Mid-size batches on a narrow output (W_o and W_down at a few hundred tokens): whole tiles are too few
// for 256 CUs and splitting them through the fenced partial-tile protocol costs more than it gains, so
// these run like the skinny path (k ranges stored to slabs, then the finish kernel) on tiles
// of 128 rows while every tile gets at least two k ranges, or of 256 rows while it gets at least three
// and k is long.  Returns the tile rows, 0 = not this path.  The slabs (at most 256 units x 256 x 256
// floats) use the tail scratch.
int split_rows(int T, int N, int K, bool has_accum) {
    if (!has_accum || T <= SKINNY_MAX_T || K % 64 || N % 4 || forced_cand() >= 0) return 0;
    const int tn = (N + 255) / 256;
    if (((T + 127) / 128) * tn <= 128) return 128;
    if (((T + 255) / 256) * tn <= 85 && K >= 8192) return 256;
    return 0;
}

// k too short to cut (below 512): one k range leaves the sums of whole tiles, and the fused epilogue the bits of the finish kernel
// (on codes it rounds once less), a launch and a pass over the slab less.  Gate/up of the tiny layer (hidden 256) with its finish kernel at
// T = 482 / 1308 / 1947 14.8 / 14.9 / 17.0 us, whole 5.1 / 5.8 / 6.4; W_o at 1947 13.6, 6.0.
bool one_range(const GemmArgs& p, int bm) { return !p.f8 && choose_splits(p.T, p.N, p.K, bm) == 1; }

template <int EPI>
hipError_t launch_mid_split(GemmArgs p, int bm, hipStream_t s, NextNorm* next) {
    if (bm == 128) return launch_split<128, EPI, 0>(p, choose_splits(p.T, p.N, p.K, 128), s, next);
    return launch_split<256, EPI, 0>(p, choose_splits(p.T, p.N, p.K, 256), s, next);
}

// Which problems take the small kernel: those whose k the general paths never cut (the cut fixes the order of the sums), up to
// one wave per CU: a second wave on a CU doubles what its L1 has to deliver, and the tiled kernels read an operand once per tile.
// 16-bit, us, general path -> small kernel: 256 x 256 5.0 -> 3.5 at 200 waves, 5.1 -> 4.5 at 304 and 5.3 -> 5.8 at 752; 256 x 512
// 6.2 -> 4.8 at 200, 6.3 -> 6.5 at 304; 1024 x 320 4.7 -> 4.1 at 256, 4.7 -> 5.3 at 320; gate/up 1376 x 256 4.5 -> 4.4 at 220,
// 4.6 -> 5.7 at 352; 512 x 1024 7.9 -> 7.3 at 256.  Where the general path has only its 256-feature tiles (q/k/v) or the fallback
// for k of no multiple of 64, up to three waves per CU: q/k/v 768 x 256 10.6 -> 4.7 at 192 waves, 10.9 -> 8.4 at 756, 11.3 -> 13.0
// at 1128; W_down 256 x 688 10.2 -> 4.9 at 200, 10.3 -> 8.1 at 752, 10.6 -> 16.3 at 1000.
bool small_applies(const GemmArgs& p, int epi, int head_dim = 0) {
    if (p.f8 || p.K % 16 || p.K > 1024 || forced_cand() >= 0) return false;
    if (p.accum && p.K % 64 == 0 && p.K >= 512) return false;   // from eight k steps on the general paths may cut k
    const int64_t units = epi == EPI_QKV_ROPE ? (p.n_q + 2 * p.n_kv) * (head_dim / 64) : ((epi == EPI_SWIGLU ? p.n_half : p.N) + 31) / 32;
    return (p.T + 31) / 32 * units <= (epi == EPI_QKV_ROPE || p.K % 64 ? 768 : 256);
}

// What a launch does beyond whole tiles: the last tail_tiles tiles split their k range over `splits` workgroups; or, where nothing is
// split, the first cols1 columns of tiles run as cand1 and the others as cand2 (cols1 = 0: all as cand).
struct Plan { int cand, tail_tiles, splits, cols1 = 0, cand1 = 0, cand2 = 0; };

// 256 x 256 tiles whose incomplete last round is cut into two k ranges: the whole tiles, then the tail as twice as many tiles of 128 rows,
// each over both ranges with the sums of either in registers of its own (HALVES).  As many workgroups with as much to multiply, and
// the finish kernel's sums bit for bit, without 256 KB of partial sums to memory and back per range, nor its launch.  (On codes the
// second set of sums does not fit beside the fragments.)
// The line: tiles of 128 rows load more per product, which grows with k while what is saved does not, and run as a launch behind the whole
// tiles instead of beside them.  Finish / halves, 154 projections of eight layers at 408 .. 8950 tokens: k of 4096 .. 8192 beside whole tiles
// 1.016 on average (0.98 .. 1.06; W_o of the 13B layer at T = 8061 341 / 324 us, q/k/v of the 70B layer at 5394 692 / 678), k of 13824 and
// 14336 0.98 (0.92 .. 1.03; W_down of the 13B layer at 7553 768 / 782).  Without whole tiles the ranges of the other way run alone on the chip, at a higher clock the
// fewer they are, so there it pays where the halves nearly fill it: k of 8192, 120 tiles 1.035 (q/k/v of the 70B layer at 667 118 / 112), 96 .. 112 tiles 0.98
// (0.93 .. 1.05); of 13824, 120 tiles 0.98.
constexpr int kHalvesMaxK = 8192, kHalvesAloneTiles = 116;
bool in_halves(int64_t tiles, int64_t tail_tiles, int tail_splits, int K, bool f8) {
    return tail_splits == 2 && K >= 1024 && K <= kHalvesMaxK && !f8 && (tiles > tail_tiles || tail_tiles >= kHalvesAloneTiles);
}
template <int EPI, int D>
hipError_t launch_halves(const GemmArgs& base, hipStream_t s) {
    GemmArgs p = base;
    p.tail_splits = 0;   // the first launch ends with the whole tiles
    const int whole = p.tiles_m * p.tiles_n - p.tail_tiles;
    constexpr int NSW = weight_stages(256, 256, 2), smem = (2 * 256 + NSW * 256) * 128, half_smem = 3 * (128 + 256) * 128;
    auto* const tiles = &gemm_dma_kernel<256, 256, EPI, D, 64, 2, false, false, NSW>;
    auto* const halves = &gemm_dma_kernel<128, 256, EPI, D, 64, 3, false, false, 3, true>;
    static std::once_flag once, once_halves;
    static hipError_t st = hipSuccess, st_halves = hipSuccess;
    if (hipError_t e = allow_smem_once(once, st, tiles, smem)) return e;
    if (hipError_t e = allow_smem_once(once_halves, st_halves, halves, half_smem)) return e;
    if (whole > 0) {
        tiles<<<dim3(whole), dim3(64 * WGM * WGN), smem, s>>>(p);
        if (hipError_t e = hipGetLastError()) return e;
    }
    halves<<<dim3(2 * p.tail_tiles), dim3(64 * WGM * WGN), half_smem, s>>>(p);
    return hipGetLastError();
}

template <int BM, int BN, int EPI, int D = 0>
hipError_t launch_cfg(const GemmArgs& base, hipStream_t s, const Plan& plan = Plan{0, 0, 1}, int col0 = 0, int cols = 0) {
    GemmArgs p = base;
    p.tiles_m = (p.T + BM - 1) / BM;
    p.tiles_n = EPI == EPI_SWIGLU ? (p.n_half + BN / 2 - 1) / (BN / 2) : (p.N + BN - 1) / BN;
    if (cols > 0) {   // columns [col0, col0 + cols) of tiles
        p.tile_n0 = col0;
        p.tiles_n = std::min(cols, p.tiles_n - col0);
    }
    constexpr int smem = 2 * (BM + BN) * BK * 2;
    // 128 x 256 tiles are one workgroup per CU either way, so they take the third stage that fits (144 KB)
    constexpr int DMA_BK = 64, DMA_NS = (BM == 128 && BN == 256) ? 3 : 2, DMA_NSW = weight_stages(BM, BN, DMA_NS);
    constexpr int dma_smem = (DMA_NS * BM + DMA_NSW * BN) * DMA_BK * 2;
    const int tiles = p.tiles_m * p.tiles_n;
    if (p.K % 64 != 0) {
        if (p.f8) return hipErrorInvalidValue;   // codes go through the direct-to-LDS kernel only
        static std::once_flag once_generic;
        static hipError_t st_generic = hipSuccess;
        if (hipError_t e = allow_smem_once(once_generic, st_generic, &gemm_bf16_kernel<BM, BN, EPI, D>, smem)) return e;
        gemm_bf16_kernel<BM, BN, EPI, D><<<dim3(tiles), dim3(256), smem, s>>>(p);
        return hipGetLastError();
    }
    int grid = tiles;
    if (plan.tail_tiles > 0 && plan.splits > 1 && p.accum && p.T > SKINNY_MAX_T) {
        const int nk = p.K / 64;
        p.k_per_split = (nk + plan.splits - 1) / plan.splits;
        p.tail_splits = (nk + p.k_per_split - 1) / p.k_per_split;   // no empty split
        p.tail_tiles = std::min(plan.tail_tiles, tiles);
        if constexpr (BM == 256 && BN == 256) {
            if (in_halves(tiles, p.tail_tiles, p.tail_splits, p.K, p.f8)) return launch_halves<EPI, D>(p, s);
        }
        p.tail_buf = p.accum;
        if ((int64_t)p.tail_tiles * p.tail_splits * BM * BN > kTailFloats)
            return hipErrorInvalidValue;   // a plan that does not fit the scratch: choose_cut never makes one
        grid = tiles - p.tail_tiles + p.tail_tiles * p.tail_splits;
    }
    auto go = [&](auto f8) -> hipError_t {
        constexpr bool F8 = decltype(f8)::value;
        static std::once_flag once_dma;
        static hipError_t st_dma = hipSuccess;
        if (hipError_t e = allow_smem_once(once_dma, st_dma, &gemm_dma_kernel<BM, BN, EPI, D, DMA_BK, DMA_NS, false, F8, DMA_NSW>, dma_smem))
            return e;
        gemm_dma_kernel<BM, BN, EPI, D, DMA_BK, DMA_NS, false, F8, DMA_NSW>
            <<<dim3(grid), dim3(64 * WGM * WGN), dma_smem, s>>>(p);
        if (p.tail_tiles > 0) {
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
            gemm_tail_finish_kernel<BM, BN, EPI, D, F8>
                <<<dim3(p.tail_tiles * (BM / (32 * WGM))), dim3(64 * WGM * WGN), 0, s>>>(p);
        }
        return hipGetLastError();
    };
    return p.f8 ? go(std::true_type{}) : go(std::false_type{});
}

// Tile choice, in two steps.
//
// 1. The cut: which tiles split their k range, and how often.  Of a launch of ceil(tiles / resident workgroups) rounds the
// tiles of the incomplete last one (the tail) may split it, so that the round takes 1 / splits of a tile time; the price is
// that every partial tile is written to memory and read back by the kernel that finishes the tile.  The cut fixes the order
// of every sum, and a last-bit difference does not stay small: a few layers on it decides between near-equal next tokens,
// and a code on the other side of its rounding boundary moves many in the next layer (2e-2 of the logits of four quantised
// layers).  So the cut depends on the sizes alone, for every kind of operand, and these constants are kept as they are: a
// refit of them for 16-bit operands changed a next token in 129 (four 13B layers, 128 decode rows and a 512-token chunk).
//
// 2. The shape of whole tiles: any gives the same bits, so where nothing is split the fastest one runs (whole_tile).  For the
// SwiGLU projection of a k (in 2-byte units) below swiglu_fit_k that is the shape the cut's own model names.  Distance from the fastest of the five
// shapes, on average, with that shape / with whole_tile's (profiles/gemm_whole_tiles.txt, ten layer shapes at 19 token counts): more than 256
// tokens, k from 2560 on 1.4 / 0.1 % (16-bit), 0.9 / 0.4 (codes), below 0.2 / 3.1 and 0.4 / 3.6; at most 256 tokens (without scratch, as
// relserve_linear runs them), k from 5120 on 4.1 / 0.9, 2560 .. 4096 0.8 / 3.8, below 0.0 / 1.4.
struct TileCand { int bm, bn, wg_per_cu; float eff_cut, eff, eff_swiglu; bool qkv; };   // qkv: usable by the fused q/k/v epilogue (128 features per wave)
constexpr int swiglu_fit_k(int T) { return T > SKINNY_MAX_T ? 2560 : 5120; }
constexpr TileCand kTiles[] = {
    // eff: fitted to the times of every whole tile shape, forced, of the other projections that split nothing, five layer shapes
    // at 18 token counts of 264 .. 4200, 16-bit and 8-bit.  Distance of the choice from the fastest shape, on average: 0.03 % in
    // 16 bits, 0.1 % in 8 (eff_cut's shape: 5 and 7 %); at hidden sizes of 256 .. 3072, which the fit had not seen, 0.2 and
    // 1.1 % (16 and 11 %).  W_o of the 13B layer at T = 1152 86 -> 74 us; 8-bit q/k/v of the 32B one at T = 806 59 -> 43.
    // With the third stage of weights 192 x 256 gained most (0.88 before): measured again at 17 token counts, 0.0 % off the fastest in
    // 16 bits (0.13 % with 0.88) and 0.4 % in 8; q/k/v of the 70B layer at T = 2304 322 (128 x 256) -> 308 us, 7168 x 8192 at 2700 289 -> 280.
    // With 16 x 16 products all of it was measured once more (profiles/gemm_whole_tiles.txt): 0.00 % off the fastest in 16 bits and 0.3 % on
    // codes at hidden sizes of 5120 and more, 0.1 and 1.4 % at 256 .. 3072.  eff_swiglu: the SwiGLU projection, whose 128 x 256 tile has the
    // compiler's order and lags: 0.00 and 0.5 %.
    {256, 256, 1, 1.00f, 1.00f, 1.00f, true}, {192, 256, 1, 0.92f, 0.98f, 0.96f, true}, {128, 256, 1, 0.68f, 0.90f, 0.75f, true},
    {128, 128, 2, 0.76f, 0.50f, 0.45f, false}, {64, 128, 3, 0.60f, 0.40f, 0.40f, false}};
constexpr int kTileCount = (int)(sizeof(kTiles) / sizeof(kTiles[0]));

constexpr double kCuFlops = 5.2e12;          // sustained MFMA rate of one CU inside a 256 x 256 tile
constexpr double kSlabBytesPerSec = 3.0e12;  // partial tiles through memory (written by the GEMM, read by the finish kernel)
constexpr double kTailFinishSec = 6e-6;      // the finish kernel's launch and ramp
constexpr double kRoundSec = 5e-6;           // what a round of whole tiles costs whatever the tile: first loads and last stores

int64_t tile_count(const TileCand& c, int T, int64_t n_eff) { return (int64_t)((T + c.bm - 1) / c.bm) * ((n_eff + c.bn - 1) / c.bn); }
double tile_sec(const TileCand& c, int K, double eff) { return 2.0 * c.bm * c.bn * (double)K / (eff * kCuFlops); }
// a launch that leaves CUs idle runs its big tiles faster (the chip is power-limited: up to 2.2 GHz instead of ~1.9);
// the small ones are bound by L2 traffic and gain nothing
double idle_boost(int64_t tiles, int64_t slots) { return tiles < slots ? 1.0 + 0.25 * (1.0 - (double)tiles / (double)slots) : 1.0; }

// need_bn256: the fused q/k/v epilogue's tiles only
Plan choose_cut(int T, int64_t n_eff, int K, bool need_bn256, bool allow_tail) {
    Plan best{0, 0, 1};
    double best_cost = 1e300;
    for (int i = 0; i < kTileCount; ++i) {
        const TileCand& c = kTiles[i];
        if (need_bn256 && !c.qkv) continue;
        const int64_t tiles = tile_count(c, T, n_eff), slots = 256 * c.wg_per_cu;
        // resident workgroups of a CU share its MFMA pipes: a round of wg_per_cu tiles costs wg_per_cu tile times
        double t_round = c.wg_per_cu * tile_sec(c, K, c.eff_cut);
        if (c.bm >= 192) t_round /= idle_boost(tiles, slots);
        const int64_t full = tiles / slots, rem = tiles % slots;
        const double whole = (double)(full + (rem ? 1 : 0)) * t_round;
        if (whole < best_cost) best_cost = whole, best = Plan{i, 0, 1};
        const int nk = K / 64;
        // tiles that share a CU (two or three workgroups) gained nothing from split tails in any measured case
        const bool can_tail = allow_tail && rem > 0 && K % 64 == 0 && c.wg_per_cu == 1;
        for (int sp = 2; can_tail && sp <= 8 && nk / sp >= 8; ++sp) {
            const int64_t units = rem * sp;
            if (units * c.bm * c.bn > kTailFloats) break;
            const double rounds = (double)((units + slots - 1) / slots);
            const double slabs = (double)units * c.bm * c.bn * 4.0 * 2.0 / kSlabBytesPerSec;
            const double cost = full * t_round + rounds * t_round / sp + slabs + kTailFinishSec;
            if (cost < best_cost) best_cost = cost, best = Plan{i, (int)rem, sp};
        }
    }
    return best;
}

// The cost of a round is the tile's MFMA work over the shape's in-tile efficiency (relative to 256 x 256) plus kRoundSec;
// this trades tile quantisation in T (padding to BM), the incomplete round, and the efficiency against each other.
int whole_tile(int T, int64_t n_eff, int K, bool need_bn256, bool swiglu) {
    int best = 0;
    double best_cost = 1e300;
    for (int i = 0; i < kTileCount; ++i) {
        const TileCand& c = kTiles[i];
        if (need_bn256 && !c.qkv) continue;
        const int64_t tiles = tile_count(c, T, n_eff), slots = 256 * c.wg_per_cu, rounds = (tiles + slots - 1) / slots;
        const double t_tile = tile_sec(c, K, swiglu ? c.eff_swiglu : c.eff);
        double cost;
        if (c.wg_per_cu > 1)   // tiles of an incomplete round share fewer CUs' pipes
            cost = (double)((tiles + 255) / 256) * t_tile + (double)rounds * kRoundSec;
        else
            cost = (double)rounds * (t_tile + kRoundSec) / (c.bm >= 256 ? idle_boost(tiles, slots) : 1.0);
        if (cost < best_cost) best_cost = cost, best = i;
    }
    return best;
}

// Whole tiles of two shapes: the last round of a launch is half empty on average, and what it leaves idle can be had by giving its
// columns of tiles to a launch of smaller tiles that fill one round more evenly (any shape gives the same bits).  For each number of
// full rounds of each 256-feature shape: as many columns as they hold, the rest on another; taken where the model that
// whole_tile uses sees a gain of kTwoShapesGain beyond kSecondLaunchSec.  One launch / two, us, measured in turn: gate/up of the 32B layer on
// codes at T = 806 219 / 197, of its 16-bit half 217 / 190, 70B at 577 503 / 466, 13B at 1409 315 / 303; q/k/v of the 13B layer at 2500
// on codes 163 / 154, W_o at 3875 162 / 152; of 65 sizes of ten layer shapes that take it 5.7 % on average (-0.8 .. 13.5;
// profiles/gemm_whole_tiles.txt), of 70 more at k (in 2-byte units) of 768 .. 2304 4.7 % and one loss of 2.6.  (Below a modelled gain of
// 4 % the second launch lost 1 - 3 % as often as it won them.)
constexpr double kSecondLaunchSec = 6e-6, kTwoShapesGain = 0.04;
void two_shapes(int T, int64_t n_eff, int K, bool swiglu, Plan* plan) {
    const int cols = (int)((n_eff + 255) / 256);
    auto cost = [&](int cand, int c) {
        const TileCand& t = kTiles[cand];
        const int64_t tiles = (int64_t)((T + t.bm - 1) / t.bm) * c, rounds = (tiles + 255) / 256;
        return (double)rounds * (tile_sec(t, K, swiglu ? t.eff_swiglu : t.eff) + kRoundSec) / (t.bm >= 256 ? idle_boost(tiles, 256) : 1.0);
    };
    if (plan->cand > 2) return;
    double best = cost(plan->cand, cols) * (1.0 - kTwoShapesGain) - kSecondLaunchSec;
    for (int a = 0; a < 3; ++a) {
        const int rows = (T + kTiles[a].bm - 1) / kTiles[a].bm;
        for (int rounds = 1; rounds * 256 / rows < cols; ++rounds) {
            const int c = rounds * 256 / rows;
            if (c == 0) continue;
            for (int b = 0; b < 3; ++b) {
                if (b == a) continue;
                const double t = cost(a, c) + cost(b, cols - c);
                if (t < best) best = t, plan->cols1 = c, plan->cand1 = a, plan->cand2 = b;
            }
        }
    }
}

// Test hook: the forced tile, or the nearest one the epilogue can run on; its whole incomplete round split if asked for.
bool forced_plan(int T, int64_t n_eff, int K, bool need_bn256, bool allow_tail, Plan* out) {
    const int cand = forced_cand(), splits = forced_splits();
    if (cand < 0 || cand >= kTileCount) return false;
    if (need_bn256 && !kTiles[cand].qkv) {   // whole tiles of the best shape that can
        *out = Plan{whole_tile(T, n_eff, K, true, false), 0, 1};
        return true;
    }
    const TileCand& c = kTiles[cand];
    const int64_t rem = tile_count(c, T, n_eff) % (256 * c.wg_per_cu);
    const bool tail = allow_tail && splits > 1 && splits <= 8 && rem > 0 && K % 64 == 0 && K / 64 / splits >= 8 &&
                      rem * splits * c.bm * c.bn <= kTailFloats;
    *out = tail ? Plan{cand, (int)rem, splits} : Plan{cand, 0, 1};
    return true;
}

Plan plan_for(int T, int64_t n_eff, int K, bool need_bn256, bool allow_tail, bool swiglu) {
    Plan plan;
    if (forced_plan(T, n_eff, K, need_bn256, allow_tail, &plan)) return plan;
    plan = choose_cut(T, n_eff, K, need_bn256, allow_tail);
    if (plan.tail_tiles == 0 && !(swiglu && K < swiglu_fit_k(T))) plan.cand = whole_tile(T, n_eff, K, need_bn256, swiglu);
    if (plan.tail_tiles == 0 && K % 64 == 0) two_shapes(T, n_eff, K, swiglu, &plan);   // (the kernel for other k knows no columns)
    return plan;
}

// The plan's launch, or two.
template <typename Launch>   // launch(candidate, first column, columns; 0: all)
hipError_t run_plan(const Plan& plan, Launch launch) {
    if (plan.cols1 == 0) return launch(plan.cand, 0, 0);
    if (hipError_t e = launch(plan.cand1, 0, plan.cols1)) return e;
    return launch(plan.cand2, plan.cols1, 1 << 30);
}

template <int EPI>
hipError_t launch_epi(const GemmArgs& p, hipStream_t s) {
    const int64_t n_eff = EPI == EPI_SWIGLU ? 2 * (int64_t)p.n_half : p.N;
    const Plan plan = plan_for(p.T, n_eff, p.K, false, p.accum != nullptr, EPI == EPI_SWIGLU);
    return run_plan(plan, [&](int cand, int col0, int cols) {
        switch (cand) {
            case 0: return launch_cfg<256, 256, EPI>(p, s, plan, col0, cols);
            case 1: return launch_cfg<192, 256, EPI>(p, s, plan, col0, cols);
            case 2: return launch_cfg<128, 256, EPI>(p, s, plan, col0, cols);
            case 3: return launch_cfg<128, 128, EPI>(p, s, plan);
            default: return launch_cfg<64, 128, EPI>(p, s, plan);
        }
    });
}

}  // namespace

void gemm_force_plan(int cand, int splits) {
    g_forced_plan.store(cand < 0 ? -1 : (cand | (splits << 8)), std::memory_order_relaxed);
}

GemmPlan gemm_plan(int32_t T, int64_t features, int32_t K, bool qkv, bool swiglu, bool scratch) {
    const Plan p = plan_for(T, features, K, qkv, scratch, swiglu);
    GemmPlan g{kTiles[p.cand].bm, kTiles[p.cand].bn, p.tail_tiles, p.splits, p.cols1, 0, 0, false};
    if (p.cols1 > 0) g.rows1 = kTiles[p.cand1].bm, g.rows2 = kTiles[p.cand2].bm;
    g.halves = p.cand == 0 && p.tail_tiles > 0 && in_halves(tile_count(kTiles[0], T, features), p.tail_tiles, p.splits, K, false);
    return g;
}

int64_t gemm_scratch_floats(int64_t T, int64_t n_max) {
    // skinny: one slab per split, at most 256 units of 128 x 256 floats, or a single slab of T x N
    return T <= SKINNY_MAX_T ? std::max<int64_t>(T * n_max, GEMM_SKINNY_FLOATS) : kTailFloats;
}


// Tiled weight layout for streaming: out[n / 256][k / 64][n % 256][k % 64], rows past N are zeros.  One k
// slice of 256 rows is 32 KB of consecutive memory, so a stage of the GEMM reads whole DRAM pages
// instead of 128-byte pieces 2 K bytes apart.
__global__ void pack_weight_kernel(const uint4* w, uint4* out, int32_t N, int32_t K, int64_t n_chunks) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;   // 16-byte chunk of the output
    if (i >= n_chunks) return;
    const int c = (int)(i & 7), r = (int)((i >> 3) & 255);
    const int64_t slice = i >> 11;                                       // (block, k slice)
    const int ks = (int)(slice % (K / 64));
    const int64_t n = (slice / (K / 64)) * 256 + r;
    out[i] = n < N ? w[(n * K + ks * 64) / 8 + c] : make_uint4(0, 0, 0, 0);
}

hipError_t launch_pack_weight(const void* w, int32_t N, int32_t K, void* out, hipStream_t s) {
    const int64_t n_chunks = (int64_t)((N + 255) / 256) * 256 * K / 8;
    if (n_chunks == 0) return hipSuccess;
    pack_weight_kernel<<<dim3((unsigned)((n_chunks + 255) / 256)), dim3(256), 0, s>>>(
        static_cast<const uint4*>(w), static_cast<uint4*>(out), N, K, n_chunks);
    return hipGetLastError();
}


// 8-bit operands: the kernels see rows of K / 2 two-byte units (same bytes, same layouts) and the scales
static hipError_t set_codes(GemmArgs& p, const CodeScales* codes) {
    if (!codes || !codes->w_scale) return hipSuccess;
    if (p.K % 128 || !(codes->a_scale > 0.0f)) return hipErrorInvalidValue;
    p.f8 = 1;
    p.K /= 2;
    p.w_scale = codes->w_scale;
    p.a_scale = codes->a_scale;
    p.out_f8 = codes->out_scale > 0.0f ? 1 : 0;
    p.out_inv = p.out_f8 ? (float)(1.0 / (double)codes->out_scale) : 0.0f;   // reciprocal in double, rounded once
    return hipSuccess;
}

hipError_t launch_linear(const void* a, const void* w, int32_t T, int32_t N, int32_t K, int32_t epilogue,
                         const void* residual, void* out, hipStream_t s, float* accum, bool w_packed, const CodeScales* codes) {
    if (T == 0) return hipSuccess;
    if ((int64_t)T * K >= ((int64_t)1 << 31) || (int64_t)N * K >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    if (epilogue != EPI_SWIGLU && (N % 4)) return hipErrorInvalidValue;
    if (epilogue == EPI_SWIGLU && ((N / 2) % 8)) return hipErrorInvalidValue;
    if (w_packed && K % 64) return hipErrorInvalidValue;   // only the direct-to-LDS kernel reads it
    GemmArgs p{};
    p.w_packed = w_packed;
    p.a = static_cast<const uint16_t*>(a);
    p.w = static_cast<const uint16_t*>(w);
    p.residual = residual;
    p.out = out;
    p.T = T;
    p.N = N;
    p.K = K;
    p.n_half = N / 2;
    p.accum = accum;
    if (hipError_t e = set_codes(p, codes)) return e;
    K = p.K;
    NextNorm* next = codes ? codes->next : nullptr;
    if (small_applies(p, epilogue)) {
        switch (epilogue) {
            case EPI_BF16: return launch_small<EPI_BF16>(p, s);
            case EPI_RES_BF16_OUT_F32: return launch_small<EPI_RES_BF16_OUT_F32>(p, s);
            case EPI_RES_F32_OUT_BF16: return launch_small<EPI_RES_F32_OUT_BF16>(p, s);
            case EPI_SWIGLU: return launch_small<EPI_SWIGLU>(p, s);
            default: return hipErrorInvalidValue;
        }
    }
    if (skinny_applies(T, N, K, accum)) {
        switch (epilogue) {
            case EPI_BF16: return launch_skinny<EPI_BF16, 0>(p, s);
            case EPI_RES_BF16_OUT_F32: return launch_skinny<EPI_RES_BF16_OUT_F32, 0>(p, s, next);
            case EPI_RES_F32_OUT_BF16: return launch_skinny<EPI_RES_F32_OUT_BF16, 0>(p, s, next);
            case EPI_SWIGLU: return launch_skinny<EPI_SWIGLU, 0>(p, s);
            default: return hipErrorInvalidValue;
        }
    }
    const int bm = split_rows(T, N, K, accum != nullptr);
    if (bm && !one_range(p, bm)) {
        switch (epilogue) {
            case EPI_BF16: return launch_mid_split<EPI_BF16>(p, bm, s, next);
            case EPI_RES_BF16_OUT_F32: return launch_mid_split<EPI_RES_BF16_OUT_F32>(p, bm, s, next);
            case EPI_RES_F32_OUT_BF16: return launch_mid_split<EPI_RES_F32_OUT_BF16>(p, bm, s, next);
            case EPI_SWIGLU: return launch_mid_split<EPI_SWIGLU>(p, bm, s, next);
            default: return hipErrorInvalidValue;
        }
    }
    if (epilogue == EPI_RES_BF16_OUT_F32 && wide_whole_applies(p)) return launch_wide_whole<EPI_RES_BF16_OUT_F32>(p, s);
    switch (epilogue) {
        case EPI_BF16: return launch_epi<EPI_BF16>(p, s);
        case EPI_RES_BF16_OUT_F32: return launch_epi<EPI_RES_BF16_OUT_F32>(p, s);
        case EPI_RES_F32_OUT_BF16: return launch_epi<EPI_RES_F32_OUT_BF16>(p, s);
        case EPI_SWIGLU: return launch_epi<EPI_SWIGLU>(p, s);
        default: return hipErrorInvalidValue;
    }
}

namespace {
template <int D>
hipError_t launch_qkv_d(const GemmArgs& p, hipStream_t s) {
    if (p.T <= 64) return launch_cfg<64, 256, EPI_QKV_ROPE, D>(p, s);
    const Plan plan = plan_for(p.T, p.N, p.K, true, p.accum != nullptr, false);   // the rotation needs 128 features per wave
    return run_plan(plan, [&](int cand, int col0, int cols) {
        switch (cand) {
            case 0: return launch_cfg<256, 256, EPI_QKV_ROPE, D>(p, s, plan, col0, cols);
            case 1: return launch_cfg<192, 256, EPI_QKV_ROPE, D>(p, s, plan, col0, cols);
            default: return launch_cfg<128, 256, EPI_QKV_ROPE, D>(p, s, plan, col0, cols);
        }
    });
}
}  // namespace

hipError_t launch_qkv_rope_append(const BatchDev& b, const relserve_layer& L, const void* h, const void* w_qkv,
                                  void* q_out, void* k_pages, void* v_pages, hipStream_t s, float* accum,
                                  bool w_packed, KvFormat kv, const CodeScales* codes) {
    if (b.T == 0) return hipSuccess;
    const int32_t K = L.cfg.hidden;
    if ((int64_t)b.T * K >= ((int64_t)1 << 31) || (int64_t)L.qkv_dim * K >= ((int64_t)1 << 31))
        return hipErrorInvalidValue;
    GemmArgs p{};
    if (w_packed && K % 64) return hipErrorInvalidValue;
    p.w_packed = w_packed;
    p.a = static_cast<const uint16_t*>(h);
    p.w = static_cast<const uint16_t*>(w_qkv);
    p.out = q_out;
    p.T = b.T;
    p.N = L.qkv_dim;
    p.K = K;
    p.tok_slot = b.tok_slot;
    p.rope_cs = b.rope_cs;
    p.k_pages = static_cast<uint16_t*>(k_pages);
    p.v_pages = static_cast<uint16_t*>(v_pages);
    p.n_q = L.cfg.n_q_heads;
    p.n_kv = L.cfg.n_kv_heads;
    p.kv_fp8 = kv.fp8 ? 1 : 0;
    p.k_inv = (float)(1.0 / (double)kv.k_scale);      // reciprocal in double, rounded once
    p.v_inv = (float)(1.0 / (double)kv.v_scale);
    p.accum = accum;
    if (hipError_t e = set_codes(p, codes)) return e;
    if (small_applies(p, EPI_QKV_ROPE, L.cfg.head_dim))
        return L.cfg.head_dim == 128 ? launch_small<EPI_QKV_ROPE, 128>(p, s) : launch_small<EPI_QKV_ROPE, 64>(p, s);
    if (skinny_applies(p.T, p.N, p.K, accum))
        return L.cfg.head_dim == 128 ? launch_skinny<EPI_QKV_ROPE, 128>(p, s) : launch_skinny<EPI_QKV_ROPE, 64>(p, s);
    return L.cfg.head_dim == 128 ? launch_qkv_d<128>(p, s) : launch_qkv_d<64>(p, s);
}

}  // namespace relserve
