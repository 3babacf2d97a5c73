// gfx950 kernels of libmlastep: latent append and mixed-step latent attention
// (decode rows and chunked-prefill rows of one step in one launch).
//
// The step is the one a decode node runs when it serves deflected prefill
// chunks next to its in-flight decodes (section 2.3; section 4.3.1, Eq. 4 of
// the paper); the head shapes are those of the served model's absorbed latent
// attention (DeepSeek-V2-Lite, section 6).
//
// Work decomposition (one persistent launch for all rows of a step: one
// 8-wavefront workgroup per CU runs a first work item fixed by its index, then
// takes items from two atomic counters, one per kind; the workgroups the host
// plans as decode-first start on the decode items, the others on the chunk
// items, and each moves to the other kind when its own runs out):
//   * chunk rows (c > 1): an item is a block of 8 query tokens (one per
//     wave, 16 head rows each) times a range of its causal keys.  32-key
//     tiles stream through a 3-slot global -> LDS DMA ring; scores on bf16
//     MFMA against a fixed reference max, probabilities to LDS as fp16, and
//     each wave accumulates P*V for its 64 value dims of all 8 tokens on fp16
//     MFMA, V read with transposing LDS reads and converted in registers.
//   * decode rows (c = 1): the decode tiles (32 keys each) of all decode
//     requests form one list cut into equal units; an item is a pair of
//     units, one per 4-wave group of the workgroup, each streaming its tiles
//     through its own 2-slot ring.
// Rows whose keys are split across items leave fp32 partials (the
// unnormalised sum, the max and sum in log2 units); a second, small merge
// kernel combines them in a fixed order.  Results are therefore run-to-run
// deterministic and do not depend on the physical page order.
#include "mla_kernels.h"

#include <limits.h>
#include <math.h>

#include <mutex>

// Scratch of the no-allocation entry point (mixed_step_noalloc): the
// attention workspace (work-queue counters, then split partials) for callers
// that cannot allocate.  Each device holds its own copy until the process
// ends; host code reaches it only through the address that
// hipGetSymbolAddress returns on that device (noalloc_scratch below).
static __device__ __align__(256) unsigned char scratch[mla::kNoAllocScratchBytes];


namespace mla {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int kChunksPerRow = kRowBytes / 16;  // 72 16-byte chunks per latent
// decode path
constexpr int kDecKeys = kKeysPerTile;  // 32
constexpr int kDecTileBytes = kDecKeys * kRowBytes;  // 36864
constexpr int kDecRing = 2;                                   // ring slots of each decode wave group
constexpr int kDecGroupBytes = kDecRing * kDecTileBytes;
constexpr int kDecXBytes = 4 * kHeads * 20 * 4;               // partial score blocks of a group
constexpr int kDecLds = 2 * kDecGroupBytes + 2 * kDecXBytes;  // two groups: rings, then score blocks
// chunk path
constexpr int kChunkKeys = kKeysPerTile;  // 32
constexpr int kChunkTileBytes = kChunkKeys * kRowBytes;  // 36864

constexpr float kNegInf = -INFINITY;

// Optional per-workgroup timeline for profiling builds (-DMLA_TRACE): slot k
// of workgroup b records the 100 MHz real-time counter at point k.
#ifdef MLA_TRACE
// Trace builds only: per work item, 16 stamps (slot = the item's queue index).
__device__ unsigned long long g_trace[1 << 20];
__shared__ int s_trace_item;
#define TRACE_ITEM(item)                                                                  \
    do {                                                                                  \
        if (threadIdx.x == 0) {                                                           \
            s_trace_item = (item);                                                        \
            unsigned xcc, hw;                                                             \
            asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));           \
            asm volatile("s_getreg_b32 %0, hwreg(HW_REG_HW_ID)" : "=s"(hw));             \
            if ((item) < (1 << 16)) {                                                     \
                g_trace[(size_t)(item) * 16 + 0] = __builtin_amdgcn_s_memrealtime();      \
                g_trace[(size_t)(item) * 16 + 9] = ((unsigned long long)xcc << 32) | hw;  \
            }                                                                             \
        }                                                                                 \
    } while (0)
#define TRACE(k)                                                                          \
    do {                                                                                  \
        if (threadIdx.x == 0 && s_trace_item < (1 << 16))                                 \
            g_trace[(size_t)s_trace_item * 16 + (k)] = __builtin_amdgcn_s_memrealtime();  \
    } while (0)
#define TRACE_VAL(k, v)                                                                   \
    do {                                                                                  \
        if (threadIdx.x == 0 && s_trace_item < (1 << 16)) g_trace[(size_t)s_trace_item * 16 + (k)] = (v); \
    } while (0)
// shader-clock stamps inside the third tile of an item (slots 10..15)
#define TRACE_TILE(t, k)                                                                  \
    do {                                                                                  \
        if ((t) == 2 && threadIdx.x == 0 && s_trace_item < (1 << 16))                     \
            g_trace[(size_t)s_trace_item * 16 + (k)] = __builtin_amdgcn_s_memtime();      \
    } while (0)
#else
#define TRACE_ITEM(item) \
    do {                 \
    } while (0)
#define TRACE_TILE(t, k) \
    do {                 \
    } while (0)
#define TRACE(k) \
    do {         \
    } while (0)
#define TRACE_VAL(k, v) \
    do {                \
    } while (0)
#endif

constexpr float kLn2 = 0.69314718055994530942f;

// Sticky error flags of the kernels on this device (MLA_FLAG_* of
// mla_step.h): raised on the rare error paths only, read and cleared by the
// host (mla_device_flags).
__device__ int g_flags;

__device__ __forceinline__ void raise_flag(int f) {
    __hip_atomic_fetch_or(&g_flags, f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------- helpers
__device__ __forceinline__ int ceil_div(int a, int b) { return (a + b - 1) / b; }

__device__ __forceinline__ float bf16_bits_to_float(uint32_t b) { return __uint_as_float(b << 16); }

__device__ __forceinline__ uint32_t bf16_bits(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }

__device__ __forceinline__ uint32_t lds_addr(const void *p) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>(p));
}

// One 16-byte global -> LDS DMA per lane: lane i writes LDS bytes
// [base + 16 i, base + 16 i + 16).  `base` must be wave-uniform.  Issued with
// inline assembly so that the compiler does not drain the whole ring before
// every barrier; completion is tracked by hand (vmcnt).
__device__ __forceinline__ void lds_dma16(const void *gsrc, uint32_t lds_base) {
    asm volatile(
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, off\n\t"
        :
        : "{m0}"(lds_base), "v"(gsrc)
        : "memory");
}

__device__ __forceinline__ void wait_dma_all() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_f16(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a),
                                                  __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// Reductions over lanes l, l^16, l^32, l^48 (the four row groups of a
// 16-column MFMA tile) with the gfx950 cross-row swaps: permlane32_swap pairs
// lane l with l +- 32, permlane16_swap pairs row groups 0-1 and 2-3.
__device__ __forceinline__ float wave_max16(float v) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float wave_sum16(float v) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// LDS byte offset of 16-byte chunk c of key k inside a decode tile (keys
// row-major, 72 chunks each).  Chunk positions are xor-swizzled inside
// aligned groups of 8 chunks with the key's low 3 bits, so 8 lanes that read
// the same chunk of 8 consecutive keys hit 8 different bank groups.  Chunk
// tiles use their own octet layout (see the chunk section).
__device__ __forceinline__ int tile_swz(int k) { return k & 7; }
__device__ __forceinline__ int tile_off(int k, int c) { return (k * kChunksPerRow + (c ^ tile_swz(k))) * 16; }

// One v_max3_f32.  Written with fmaxf and not as inline assembly: its operands
// are MFMA results, and the wait states such a read needs are only inserted for
// instructions the compiler knows.
__device__ __forceinline__ float max3(float x, float y, float z) { return fmaxf(fmaxf(x, y), z); }

// Transposing LDS read (gfx950): inside each 16-lane group, lane i receives
// element (i & 3) of the 8 bytes read by lane 4 j + (i >> 2), j = 0..3.
__device__ __forceinline__ u32x2 lds_read_tr16(const char *p) {
    const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p));
    return __builtin_bit_cast(u32x2, v);
}

// threadIdx.x behind an empty asm: values derived from it inside a work item
// are then computed per item instead of being hoisted out of the persistent
// loop, where they would stay live across both paths and spill to scratch (a
// scratch reload waits on vmcnt, i.e. on every DMA in flight).
__device__ __forceinline__ int item_tid() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// ------------------------------------------------------ work-item lookup
// Items of one kind are numbered request by request; request r owns
// count(r) consecutive items.  Every wavefront looks its item up by itself: no
// barrier and no LDS exchange stands between the load of the lengths and the
// item's own loads (a lookup is mostly the latency of that load).  It takes up
// to 64 requests in one step, larger batches 256 a step (four lengths a lane,
// their prefix sums independent) with the next 256 already
// loading.  (64 a step with shuffles for the sums: 4000 rows of 16 to 256 keys
// 307.9 -> 288.6 us, 1000 rows of 64 to 2048 keys 285.7 -> 281.1, 4 rows 18.8 ->
// 18.2; the lane addresses of the shuffles were also held across the items, which
// cost the chunk tiles registers: 20 spilled, now none.)
struct ReqLens {
    const int32_t *cu_q;
    const int32_t *prefix;
    bool rev;  // number the items from the last request to the first
};

struct Located {
    int r, local, p, row0, c;
};

struct LenRow {
    int row0, next, p;
};

// Lengths of request r (all zero outside [0, num_reqs)).
__device__ __forceinline__ LenRow load_lens(const int32_t *cu_q, const int32_t *prefix, int r, int num_reqs) {
    LenRow l{0, 0, 0};
    if ((unsigned)r < (unsigned)num_reqs) l = LenRow{cu_q[r], cu_q[r + 1], prefix[r]};
    return l;
}

// Inclusive prefix sum over the lanes of a wavefront, all of them active: inside
// rows of 16 lanes by shifts, then the last lane of row 0 (2) added to row 1
// (3) and lane 31 to rows 2 and 3, all in the vector unit (DPP).
__device__ __forceinline__ int wave_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
    return v;
}

constexpr int kLookupQ = 4;  // lengths a lane and step of a lookup over more than 64 requests

// End of a lookup: its loads, which nothing reads any more, count as landed.
// (Left in flight as far as the compiler knows, it waits for them where it next
// writes their registers, and there for every load issued in between.)
__device__ __forceinline__ void end_lookup() { __builtin_amdgcn_s_waitcnt(0x0F70); }  // vmcnt(0), the others left alone

template <int Q, typename CountFn>
__device__ __forceinline__ bool locate_in(int target, int num_reqs, const ReqLens &rl, CountFn count, Located &loc) {
    const int lane = item_tid() & 63;
    const auto req = [&](int i) { return rl.rev ? num_reqs - 1 - i : i; };
    LenRow cur[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) cur[q] = load_lens(rl.cu_q, rl.prefix, req(64 * q + lane), num_reqs);
    int running = 0;
    for (int base = 0; base < num_reqs; base += 64 * Q) {
        LenRow nxt[Q];
        if constexpr (Q > 1) {
#pragma unroll
            for (int q = 0; q < Q; ++q) nxt[q] = load_lens(rl.cu_q, rl.prefix, req(base + 64 * (Q + q) + lane), num_reqs);
        }
        int cnt[Q], inc[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            cnt[q] = base + 64 * q + lane < num_reqs ? count(cur[q].p, cur[q].next - cur[q].row0) : 0;
            inc[q] = wave_scan(cnt[q]);
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int end = running + inc[q], first = end - cnt[q];
            const uint64_t hit = __builtin_amdgcn_ballot_w64(cnt[q] > 0 && target >= first && target < end);
            if (hit != 0) {
                const int l = __builtin_ctzll(hit);
                loc = Located{req(base + 64 * q + l), target - __builtin_amdgcn_readlane(first, l),
                              __builtin_amdgcn_readlane(cur[q].p, l), __builtin_amdgcn_readlane(cur[q].row0, l),
                              __builtin_amdgcn_readlane(cur[q].next - cur[q].row0, l)};
                return true;
            }
            running = __builtin_amdgcn_readlane(end, 63);
        }
        if constexpr (Q == 1) break;  // at most 64 requests
#pragma unroll
        for (int q = 0; q < Q; ++q) cur[q] = nxt[q];
    }
    return false;
}

template <typename CountFn>
__device__ bool locate_item(int target, int num_reqs, const ReqLens &rl, CountFn count, Located &loc) {
    const bool found = num_reqs <= 64 ? locate_in<1>(target, num_reqs, rl, count, loc) : locate_in<kLookupQ>(target, num_reqs, rl, count, loc);
    end_lookup();
    return found;
}

struct ChunkCount {
    int ks;
    ChunkRoute route;
    __device__ int operator()(int p, int c) const {
        return c > 1 && !route.multi_head(p, c) ? ceil_div(c, kChunkBlockTokens) * ceil_div(p + c, ks) : 0;
    }
};

struct ChunkItem {
    int r, p, c, row0, i0, i1, k0, k1, ks, nks_eff;
};

// Item `local` of a chunk request: every block of 8 query tokens (the
// longest rows first) takes nks = ceil((p + c) / ks_chunk) queue slots.  The
// block's keys (0 .. p + i1 - 1, its causal limit klim) are cut into
// ceil(klim / ks_chunk) ranges of equal length, rounded up to a multiple of
// 64 keys (at most ks_chunk); the remaining slots are empty items.  A block
// whose keys fit one range writes its rows directly.
__device__ __forceinline__ ChunkItem decode_chunk_item(const AttnArgs &a, const Located &lc) {
    ChunkItem it;
    it.r = lc.r;
    it.p = lc.p;
    it.row0 = lc.row0;
    it.c = lc.c;
    const int nrb = ceil_div(it.c, kChunkBlockTokens);
    const int nks = ceil_div(it.p + it.c, a.ks_chunk);
    const int rb = nrb - 1 - lc.local / nks;  // longest rows first
    it.ks = lc.local % nks;
    it.i0 = rb * kChunkBlockTokens;
    it.i1 = min(it.i0 + kChunkBlockTokens, it.c);
    const int klim = it.p + it.i1;
    const int kp = ceil_div(ceil_div(klim, ceil_div(klim, a.ks_chunk)), 64) * 64;  // keys per range (<= ks_chunk)
    it.nks_eff = ceil_div(klim, kp);
    it.k0 = it.ks * kp;
    it.k1 = min(klim, it.k0 + kp);
    return it;
}

// DMA of a 32-key tile that lies inside one page: a uniform source base (the
// tile's first key) in SGPRs plus per-lane offsets fixed for all tiles.
// Round i of wave wv fills LDS chunk u = 256 i + 64 wv + lane of the tile,
// which holds source chunk (u % 72) ^ swz(key) of key u / 72.
constexpr int kTileDma = kKeysPerTile * kRowBytes / (kThreads * 16);  // 9 rounds per tile
// Offsets (< 2^16) packed two per register: round i in the half i & 1 of word i / 2.
__device__ __forceinline__ void tile_dma_offsets(int wv, int lane, uint32_t (&off)[(kTileDma + 1) / 2]) {
#pragma unroll
    for (int w = 0; w < (kTileDma + 1) / 2; ++w) off[w] = 0;
#pragma unroll
    for (int i = 0; i < kTileDma; ++i) {
        const int u = (i * 4 + wv) * 64 + lane;
        const int kk = u / kChunksPerRow;
        const int c = (u - kk * kChunksPerRow) ^ tile_swz(kk);
        off[i / 2] |= (uint32_t)(kk * kRowBytes + c * 16) << (16 * (i & 1));
    }
}

__device__ __forceinline__ void lds_dma16_sbase(const void *sbase, uint32_t voff, uint32_t lds_base) {
    asm volatile(
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %0, %1\n\t"
        :
        : "v"(voff), "s"(sbase), "{m0}"(lds_base)
        : "memory");
}

// Fused append: copy n new latents (rows row0 .. of a.new_kv, keys key0 .. of
// request r) into their cache slots; the whole workgroup takes part.  Slots
// with a page id outside the pool are skipped.
__device__ __forceinline__ void append_rows(const AttnArgs &a, int r, int key0, int row0, int n) {
    const int32_t *btr = a.bt + (size_t)r * a.max_pages;
    for (int x = threadIdx.x; x < n * kChunksPerRow; x += blockDim.x) {
        const int i = x / kChunksPerRow, c = x - i * kChunksPerRow;
        const int key = key0 + i;
        const int lp = key >> a.log2_page;
        const int page = lp < a.max_pages ? btr[lp] : -1;
        if ((unsigned)page >= (unsigned)a.num_pages) {
            raise_flag(kFlagBadPage);
            continue;
        }
        const u32x4 v = *reinterpret_cast<const u32x4 *>(a.new_kv + (size_t)(row0 + i) * kDqk + c * 8);
        *reinterpret_cast<u32x4 *>(a.kv_out + ((size_t)page * a.page_size + (key & (a.page_size - 1))) * kDqk +
                                   c * 8) = v;
    }
}

// The same for one 256-thread group of a larger workgroup (gtid = thread index in it).
__device__ __forceinline__ void append_rows_group(const AttnArgs &a, int r, int key0, int row0, int n, int gtid) {
    const int32_t *btr = a.bt + (size_t)r * a.max_pages;
    for (int x = gtid; x < n * kChunksPerRow; x += kThreads) {
        const int i = x / kChunksPerRow, c = x - i * kChunksPerRow;
        const int key = key0 + i;
        const int lp = key >> a.log2_page;
        const int page = lp < a.max_pages ? btr[lp] : -1;
        if ((unsigned)page >= (unsigned)a.num_pages) {
            raise_flag(kFlagBadPage);
            continue;
        }
        const u32x4 v = *reinterpret_cast<const u32x4 *>(a.new_kv + (size_t)(row0 + i) * kDqk + c * 8);
        *reinterpret_cast<u32x4 *>(a.kv_out + ((size_t)page * a.page_size + (key & (a.page_size - 1))) * kDqk +
                                   c * 8) = v;
    }
}

// Store 4 consecutive dims of one (row, head) output, fp32 or bf16.
__device__ __forceinline__ void store_out4(const AttnArgs &a, int row, int head, int dv, f32x4 v) {
    const size_t off = ((size_t)row * kHeads + head) * kDv + dv;
    if (a.out_bf16) {
        const uint32_t w0 = bf16_bits(v[0]) | (bf16_bits(v[1]) << 16);
        const uint32_t w1 = bf16_bits(v[2]) | (bf16_bits(v[3]) << 16);
        *reinterpret_cast<u32x2 *>(reinterpret_cast<uint16_t *>(a.out) + off) = u32x2{w0, w1};
    } else {
        *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(a.out) + off) = v;
    }
}

// ------------------------------------------------------------------ merge
// Merge the key-split partials of output rows.  Split s holds an
// unnormalised output o_s (16 heads x 512 dims) with its max m_s and sum l_s
// in log2 units; slot(s) gives pointers to both.  A wavefront takes one head
// and every SW-th split of it, lane l holding dims 4 l .. + 3 and 256 + 4 l ..;
// the SW wavefronts of a head meet in LDS, in a fixed order.
//
// Bound by latency: the partials are small (0.1 .. 35 MB a call) and were just
// written by other XCDs, so every load is a round trip past the L2 and what
// counts is how many such rounds follow one another.  All loads of a batch
// of splits go out together, and rows cut into many parts spread over
// more wavefronts, so a row takes one or two rounds.  (One thread loop per head
// and row before, a block-wide scan of the lengths in front: 18.2 us for 4 rows
// of 75 parts, now 8.3; 16.5 -> 12.2 us for 128 rows of up to 23 parts.  More
// workgroups per row of few parts cost more in launches than they overlap: 256
// rows of 2 to 4 parts take 10.5 us with 4 workgroups a row, 15.6 with 8.)
// Chunk rows of up to 4 parts take one workgroup, four heads a wavefront one
// after the other: 20.9 -> 9.8 us for 1069 of them and 37 decode rows.  With more
// parts that chain loses, so they are spread as decode rows are: 8 rows of 65
// parts 62.0 us before, 71.9 with the chain, 7.8 spread; 64 rows of 9 parts 12.6,
// 15.1 and 6.9; 2048 rows of 7 parts 136.9, 119.7 and 94.3.  Only rows that have
// partials get workgroups (the chain's launch had one per item and block row).
struct SplitRef {
    const float *o, *ml;
};

// o, M, den += splits s0, s0 + SW, .. of head hh (B of them in flight).
template <int B, int SW, typename Slot>
__device__ __forceinline__ void merge_splits(int s0, int nsplit, int hh, int lane, Slot slot, f32x4 (&o)[2], float &M,
                                             float &den) {
    for (; s0 < nsplit; s0 += B * SW) {
        float ms[B], ls[B];
        f32x4 v[B][2];
#pragma unroll
        for (int q = 0; q < B; ++q) {
            ms[q] = kNegInf;
            ls[q] = 0.f;
            v[q][0] = v[q][1] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (s0 + q * SW < nsplit) {
                const SplitRef sr = slot(s0 + q * SW);
                ms[q] = sr.ml[hh * 2];
                ls[q] = sr.ml[hh * 2 + 1];
                const f32x4 *src = reinterpret_cast<const f32x4 *>(sr.o + hh * kDv) + lane;
                v[q][0] = src[0];
                v[q][1] = src[64];
            }
        }
        float m_new = M;
#pragma unroll
        for (int q = 0; q < B; ++q) m_new = fmaxf(m_new, ms[q]);
        const float c_old = (M == kNegInf) ? 0.f : exp2f(M - m_new);
        den *= c_old;
#pragma unroll
        for (int k = 0; k < 2; ++k) o[k] = o[k] * c_old;
#pragma unroll
        for (int q = 0; q < B; ++q) {
            if (ms[q] == kNegInf) continue;  // a split that saw no key of this row
            const float c = exp2f(ms[q] - m_new);
            den += ls[q] * c;
#pragma unroll
            for (int k = 0; k < 2; ++k) o[k] = o[k] + v[q][k] * c;
        }
        M = m_new;
    }
}

__device__ __forceinline__ void store_merged(const AttnArgs &a, int row, int hh, int lane, const f32x4 (&o)[2], float M,
                                             float den) {
    const float inv = 1.f / den;
#pragma unroll
    for (int k = 0; k < 2; ++k) store_out4(a, row, hh, 4 * lane + 256 * k, o[k] * inv);
    if (a.lse && lane == 0) a.lse[(size_t)row * kHeads + hh] = (M + log2f(den)) * kLn2;
}

// Heads hh0 .. hh0 + 4 / SW - 1 of a row with many splits; s_o holds 4 x 512 floats, s_ml 4 x 2.
template <int B, int SW, typename Slot>
__device__ void merge_heads(const AttnArgs &a, int row, int hh0, int nsplit, Slot slot, float *s_o, float *s_ml) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int hh = hh0 + wv / SW, part = wv % SW;
    f32x4 o[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    float M = kNegInf, den = 0.f;
    merge_splits<B, SW>(part, nsplit, hh, lane, slot, o, M, den);
    if constexpr (SW > 1) {
        if (part != 0) {
            f32x4 *dst = reinterpret_cast<f32x4 *>(s_o + wv * kDv) + lane;
            dst[0] = o[0];
            dst[64] = o[1];
            if (lane == 0) {
                s_ml[2 * wv] = M;
                s_ml[2 * wv + 1] = den;
            }
        }
        __syncthreads();
        if (part != 0) return;
#pragma unroll
        for (int w = 1; w < SW; ++w) {
            const float m = s_ml[2 * (wv + w)], l = s_ml[2 * (wv + w) + 1];
            if (m == kNegInf) continue;  // fewer splits than wavefronts
            const float m_new = fmaxf(M, m);
            const float c_old = (M == kNegInf) ? 0.f : exp2f(M - m_new), c = exp2f(m - m_new);
            const f32x4 *src = reinterpret_cast<const f32x4 *>(s_o + (wv + w) * kDv) + lane;
            den = den * c_old + l * c;
            o[0] = o[0] * c_old + src[0] * c;
            o[1] = o[1] * c_old + src[64] * c;
            M = m_new;
        }
    }
    store_merged(a, row, hh, lane, o, M, den);
}

// A whole row of few parts, four heads per wavefront.
template <typename Slot>
__device__ void merge_row(const AttnArgs &a, int row, int nsplit, Slot slot) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < kHeads / 4; ++k) {
        const int hh = wv * (kHeads / 4) + k;
        f32x4 o[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
        float M = kNegInf, den = 0.f;
        merge_splits<2, 1>(0, nsplit, hh, lane, slot, o, M, den);
        store_merged(a, row, hh, lane, o, M, den);
    }
}

// ------------------------------------------------------------ decode path
// The 32-key tiles of all decode requests, request after request, form one
// list cut into units of S tiles; unit v owns tiles [v S, (v + 1) S), and a
// decode item is a pair of units, one per 4-wave group of the workgroup
// (the groups run independently, synchronised by LDS arrival counters).  A
// unit's share splits into segments, one per request it touches.  A segment
// streams its query block and then its tiles through the group's 2-slot
// global -> LDS DMA ring, so prefetch runs on across request boundaries and
// the start-up latency is paid once per unit.  Per tile, wave w scores 16
// keys over half of the 576 latent dims (the four partial 16 x 16 score
// blocks meet in LDS), then accumulates its 128-wide slice of the value dims
// over all 32 keys.  A request spread over several units leaves fp32
// partials (slot 2 v for unit v's first segment, 2 v + 1 for its last) that
// the merge kernel combines.
constexpr int kMaxSeg = kMaxDecSegments;
constexpr int kXStride = 20;  // floats per head row of a partial score block (16 + pad)

struct DecSeg {
    int r, p, row, t0, t1, pw, lp0;  // tiles t0 .. t1-1 of request r; page window offset / first page
};

__device__ __forceinline__ int dec_tiles(int p, int c) { return c == 1 ? ceil_div(p + 1, kDecKeys) : 0; }

// Segments (request order) of the decode tile range [R0, R1), with the page
// window each needs; returns their count.  Every wavefront of a group finds
// them by itself (as a lookup does) and `writer` stores them.
template <int Q>
__device__ __forceinline__ int find_unit_in(const AttnArgs &a, int R0, int R1, DecSeg *s_seg, bool writer) {
    const int lane = item_tid() & 63;
    int running = 0, nseg = 0, pages = 0;
    LenRow cur[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) cur[q] = load_lens(a.cu_q, a.prefix, 64 * q + lane, a.num_reqs);
    for (int base = 0; base < a.num_reqs && running < R1; base += 64 * Q) {
        LenRow nxt[Q];
        if constexpr (Q > 1) {
#pragma unroll
            for (int q = 0; q < Q; ++q) nxt[q] = load_lens(a.cu_q, a.prefix, base + 64 * (Q + q) + lane, a.num_reqs);
        }
        int nt[Q], inc[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            // rows outside [0, T) only arise from device lengths that disagree with the host's
            const bool row_ok = base + 64 * q + lane < a.num_reqs && cur[q].p >= 0 && cur[q].row0 >= 0 && cur[q].row0 < a.num_rows;
            nt[q] = row_ok ? dec_tiles(cur[q].p, cur[q].next - cur[q].row0) : 0;
            inc[q] = wave_scan(nt[q]);
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int end = running + inc[q], T = end - nt[q];
            const bool ov = nt[q] > 0 && T < R1 && end > R0;
            const uint64_t m = __builtin_amdgcn_ballot_w64(ov);
            if (m != 0) {
                const int t0 = max(R0 - T, 0), t1 = min(R1 - T, nt[q]);
                const int lp0 = (t0 * kDecKeys) >> a.log2_page;
                const int np = ov ? ((min(t1 * kDecKeys, cur[q].p + 1) - 1) >> a.log2_page) - lp0 + 1 : 0;
                const int pend = pages + wave_scan(np);
                const int j = nseg + __builtin_popcountll(m & ((1ull << lane) - 1));
                if (ov && writer && j < kMaxSeg)
                    s_seg[j] = DecSeg{base + 64 * q + lane, cur[q].p, cur[q].row0, t0, t1, pend - np, lp0};
                nseg += __builtin_popcountll(m);
                pages = __builtin_amdgcn_readlane(pend, 63);
            }
            running = __builtin_amdgcn_readlane(end, 63);
        }
        if constexpr (Q == 1) break;  // at most 64 requests
#pragma unroll
        for (int q = 0; q < Q; ++q) cur[q] = nxt[q];
    }
    return min(nseg, kMaxSeg);
}
__device__ int find_unit(const AttnArgs &a, int R0, int R1, DecSeg *s_seg, bool writer) {
    const int nseg = a.num_reqs <= 64 ? find_unit_in<1>(a, R0, R1, s_seg, writer) : find_unit_in<kLookupQ>(a, R0, R1, s_seg, writer);
    end_lookup();
    return nseg;
}

// Unit cursor of a group's stream: segment j, tile t (t < 0: the query block).
// The segment is kept in scalar registers and read from LDS only when it
// changes, so that no LDS round trip stands before a tile's loads (256 rows of
// up to 16384 keys 465.1 -> 461.7 us, 19 rows of about 5430 keys 62.8 -> 61.8).
struct Cursor {
    int j, t;
    DecSeg sg;
};
__device__ __forceinline__ DecSeg load_seg(const DecSeg *s_seg, int j) {
    const DecSeg d = s_seg[j];
    return DecSeg{__builtin_amdgcn_readfirstlane(d.r),  __builtin_amdgcn_readfirstlane(d.p),
                  __builtin_amdgcn_readfirstlane(d.row), __builtin_amdgcn_readfirstlane(d.t0),
                  __builtin_amdgcn_readfirstlane(d.t1), __builtin_amdgcn_readfirstlane(d.pw),
                  __builtin_amdgcn_readfirstlane(d.lp0)};
}
__device__ __forceinline__ void advance(Cursor &c, const DecSeg *s_seg, int nseg) {
    c.t = c.t < 0 ? c.sg.t0 : c.t + 1;
    if (c.t >= c.sg.t1) {
        ++c.j;
        c.t = -1;
        if (c.j < nseg) c.sg = load_seg(s_seg, c.j);
    }
}

// DMA of one stream unit into a 36 KB ring slot.  A query block (16 heads x
// 576 dims, 18 KB) is copied twice over so every unit takes 9 DMA rounds.  A
// full tile inside one page uses the uniform-base form (offsets `dma_off`).
__device__ __forceinline__ void issue_unit(const AttnArgs &a, const DecSeg &sg, int t, const int *s_pages,
                                           uint32_t slot, int wv, int lane,
                                           const uint32_t (&dma_off)[(kTileDma + 1) / 2]) {
    constexpr int kDma = kDecTileBytes / (kThreads * 16);  // 9
    const int kbase = t * kDecKeys;
    const int last_cached = a.new_kv != nullptr ? sg.p - 1 : sg.p;  // key p is the new latent when fused
    if (t >= 0 && a.page_size >= kDecKeys && kbase + kDecKeys - 1 <= last_cached) {
        const int page = s_pages[min(sg.pw + (kbase >> a.log2_page) - sg.lp0, kPageWindow - 1)];
        const char *src = reinterpret_cast<const char *>(a.kv) +
                          ((size_t)__builtin_amdgcn_readfirstlane(page) * a.page_size + (kbase & (a.page_size - 1))) *
                              kRowBytes;
#pragma unroll
        for (int i = 0; i < kDma; ++i)
            lds_dma16_sbase(src, (dma_off[i / 2] >> (16 * (i & 1))) & 0xffffu,
                            __builtin_amdgcn_readfirstlane(slot + (i * 4 + wv) * 1024));
        return;
    }
    const char *src[kDma];
    if (t < 0) {
        const char *qb = reinterpret_cast<const char *>(a.q + (size_t)sg.row * kHeads * kDqk);
#pragma unroll
        for (int i = 0; i < kDma; ++i) {
            const int u = (i * 4 + wv) * 64 + lane;
            src[i] = qb + (u % (kHeads * kChunksPerRow)) * 16;
        }
    } else {
        const char *kv = reinterpret_cast<const char *>(a.kv);
        const int klast = sg.p;
#pragma unroll
        for (int i = 0; i < kDma; ++i) {
            const int u = (i * 4 + wv) * 64 + lane;
            const int kk = u / kChunksPerRow;
            const int c = (u - kk * kChunksPerRow) ^ (kk & 7);
            const int key = min(kbase + kk, klast);
            const int page = s_pages[min(sg.pw + (key >> a.log2_page) - sg.lp0, kPageWindow - 1)];
            src[i] = (a.new_kv != nullptr && key == klast)
                         ? reinterpret_cast<const char *>(a.new_kv) + (size_t)sg.row * kRowBytes + c * 16
                         : kv + ((size_t)page * a.page_size + (key & (a.page_size - 1))) * kRowBytes + c * 16;
        }
    }
#pragma unroll
    for (int i = 0; i < kDma; ++i) lds_dma16(src[i], __builtin_amdgcn_readfirstlane(slot + (i * 4 + wv) * 1024));
}

// Barrier of the four wavefronts of one wave group, through an arrival
// counter in LDS; epoch (wave-uniform) counts the group's barriers so far.
// Each wave first waits for its own LDS accesses, so what it wrote before the
// barrier is visible to the group after it.  The wait is bounded (far beyond
// any real skew): a broken count cannot hang the kernel; an expired wait
// raises kFlagWaitExpired (that call's results are then undefined).
__device__ __forceinline__ void group_barrier(int *ctr, int &epoch, int spin_limit) {
    ++epoch;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if ((threadIdx.x & 63) == 0) __hip_atomic_fetch_add(ctr, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    const int target = 4 * epoch;
    int spin = 0;
    for (; spin < spin_limit; ++spin) {
        const int seen = __builtin_amdgcn_readfirstlane(__hip_atomic_load(ctr, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP));
        if (seen >= target) break;
        __builtin_amdgcn_s_sleep(1);
    }
    if (spin == spin_limit && (threadIdx.x & 63) == 0) raise_flag(kFlagWaitExpired);
    asm volatile("" ::: "memory");
}

// Barrier of the workgroup for LDS contents only: loads may stay in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ void decode_wg(const AttnArgs &a, int w, char *smem, int (*s_pages_g)[kPageWindow],
                          DecSeg (*s_seg_g)[kMaxSeg], int *s_gbar) {
    const int tid = item_tid(), lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wv >> 2, gw = wv & 3, gtid = tid & 255;  // wave group, wave and thread inside it
    const int g = lane >> 4, h = lane & 15;
    const int S = a.dec_unit_tiles;
    // Item w is the pair of decode units 2 w and 2 w + 1 (S tiles each), one per
    // wave group.  A unit of a tile or two is mostly start-up, a chain of round
    // trips to memory: the lengths, then the query block and the page ids at
    // once, then the first tile beside the fused append.
    const int v = 2 * w + grp;  // this group's unit
    const int R0 = v * S, R1 = min(R0 + S, a.dec_total_tiles);
    DecSeg *const s_seg = s_seg_g[grp];
    int *const s_pages = s_pages_g[grp];
    const int nseg = R0 < R1 ? find_unit(a, R0, R1, s_seg, gw == 0) : 0;
    const int n_units = nseg > 0 ? nseg + (R1 - R0) : 0;
    if (tid < 2) s_gbar[tid] = 0;
    TRACE(1);
    __syncthreads();
    uint32_t dma_off[(kTileDma + 1) / 2];
    tile_dma_offsets(gw, lane, dma_off);
    const uint32_t ring = lds_addr(smem) + grp * kDecGroupBytes;
    float *s_X = reinterpret_cast<float *>(smem + 2 * kDecGroupBytes + grp * kDecXBytes);
    Cursor prod{0, -1, DecSeg{}};
    if (n_units > 0) prod.sg = load_seg(s_seg, 0);
    Cursor cons = prod;
    if (n_units > 0) {
        issue_unit(a, prod.sg, -1, s_pages, ring, gw, lane, dma_off);  // the first query block
        advance(prod, s_seg, nseg);
        // page window: entry gtid belongs to the last segment that starts at or before it
        static_assert(kPageWindow == kThreads, "one window entry per thread of the group");
        int j = 0;
        for (int k = 1; k < nseg; ++k) j = s_seg[k].pw <= gtid ? k : j;
        const DecSeg sg = s_seg[j];
        const int i = gtid - sg.pw;
        if (i < ((min(sg.t1 * kDecKeys, sg.p + 1) - 1) >> a.log2_page) - sg.lp0 + 1) {
            const int lp = sg.lp0 + i;
            const int pg = lp < a.max_pages ? a.bt[(size_t)sg.r * a.max_pages + lp] : 0;
            const bool ok = (unsigned)pg < (unsigned)a.num_pages;
            if (!ok) raise_flag(kFlagBadPage);
            s_pages[gtid] = ok ? pg : 0;
        }
    }
    __syncthreads();
    if (n_units == 0) return;  // this group has no unit (the other one may)
    if (n_units > 1) {
        issue_unit(a, prod.sg, prod.t, s_pages, ring + kDecTileBytes, gw, lane, dma_off);
        advance(prod, s_seg, nseg);
    }
    if (a.new_kv != nullptr) {  // fused append: the group holding a request's last tile writes its latent
        for (int j = 0; j < nseg; ++j) {
            const DecSeg sg = s_seg[j];
            if (sg.t1 == dec_tiles(sg.p, 1)) append_rows_group(a, sg.r, sg.p, sg.row, 1, gtid);
        }
    }
    int epoch = 0;
    int *const gbar = s_gbar + grp;
    TRACE(2);
    TRACE_VAL(8, 1000000ull * 2 + n_units);

    u32x4 qreg[9];  // this wave's half of the query operand: steps 9 (gw >> 1) .. + 9
    f32x4 acc[8];
#pragma unroll
    for (int mt = 0; mt < 8; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_ref = kNegInf, l_run = 0.f;
    const int hf = gw >> 1;
    const int kq = 16 * (gw & 1) + (lane & 15);             // key this lane scores
    const int tr_key = 4 * g + ((lane & 15) >> 2);          // transposing-read source row
    const int tr_dv = gw * 128 + 4 * (lane & 3);            // and its first value dim

    TRACE(3);
    // The two groups run independently, each with barriers of its own four
    // wavefronts (two per unit).
    for (int u = 0; u < n_units; ++u) {
        TRACE_TILE(u, 10);
        wait_dma_all();                // unit u (the first two are issued together)
        group_barrier(gbar, epoch, a.spin_limit);    // unit u landed; slot (u + 1) % 2 is free
        bool tile_unit = false;
        const DecSeg sg = cons.sg;
        const char *slot = smem + grp * kDecGroupBytes + (u % kDecRing) * kDecTileBytes;
        {
            if (u > 0 && prod.j < nseg) {
                issue_unit(a, prod.sg, prod.t, s_pages, ring + ((u + 1) % kDecRing) * kDecTileBytes, gw, lane, dma_off);
                advance(prod, s_seg, nseg);
            }
            if (cons.t < 0) {  // a new request: its query block
#pragma unroll
                for (int s2 = 0; s2 < 9; ++s2)
                    qreg[s2] = *reinterpret_cast<const u32x4 *>(slot + (h * kChunksPerRow + (9 * hf + s2) * 4 + g) * 16);
                advance(cons, s_seg, nseg);
            } else {
                tile_unit = true;
                TRACE_TILE(u, 11);
                // partial scores: keys 16 (gw & 1) .. + 16, dims of steps 9 hf .. 9 hf + 8
                f32x4 sa = {0.f, 0.f, 0.f, 0.f}, sb = {0.f, 0.f, 0.f, 0.f};
                u32x4 av[9];
#pragma unroll
                for (int s2 = 0; s2 < 9; ++s2)
                    av[s2] = *reinterpret_cast<const u32x4 *>(slot + tile_off(kq, (9 * hf + s2) * 4 + g));
#pragma unroll
                for (int s2 = 0; s2 < 9; s2 += 2) {
                    sa = mfma_bf16(av[s2], qreg[s2], sa);
                    if (s2 + 1 < 9) sb = mfma_bf16(av[s2 + 1], qreg[s2 + 1], sb);
                }
                *reinterpret_cast<f32x4 *>(s_X + (gw * kHeads + h) * kXStride + 4 * g) = sa + sb;
            }
        }
        if (!tile_unit) continue;
        group_barrier(gbar, epoch, a.spin_limit);  // partial score blocks complete
        TRACE_TILE(u, 12);
        const int kbase = cons.t * kDecKeys;
        // full scores of this lane's head: x[kt][i] = key 16 kt + 4 g + i (kt = 0, 1)
        f32x4 x[2];
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
            const f32x4 lo = *reinterpret_cast<const f32x4 *>(s_X + (kt * kHeads + h) * kXStride + 4 * g);
            const f32x4 hi = *reinterpret_cast<const f32x4 *>(s_X + ((kt + 2) * kHeads + h) * kXStride + 4 * g);
            x[kt] = lo + hi;
        }
        float mt = kNegInf;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[kt][i] = (kbase + 16 * kt + 4 * g + i <= sg.p) ? x[kt][i] * a.scale_log2 : kNegInf;
                mt = fmaxf(mt, x[kt][i]);
            }
        }
        mt = wave_max16(mt);
        // Lazy rescale (the same decision in every wave of the group): keep the
        // reference max unless the tile max exceeds it by more than 2^8.
        if (__builtin_amdgcn_ballot_w64(mt > m_ref + 8.f) != 0) {
            const float m_new = fmaxf(m_ref, mt);
            const float alpha = (m_ref == kNegInf) ? 0.f : exp2f(m_ref - m_new);
#pragma unroll
            for (int mt2 = 0; mt2 < 8; ++mt2) acc[mt2] = acc[mt2] * alpha;
            l_run *= alpha;
            m_ref = m_new;
        }
        // probabilities, split into bf16 hi + lo so that P*V keeps ~16 bits;
        // slot 8 g + 4 kt + i of the B operand holds key 16 kt + 4 g + i
        uint32_t bh[4], bl[4];
        float ps = 0.f;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
            for (int i = 0; i < 4; i += 2) {
                const float p0 = (x[kt][i] == kNegInf) ? 0.f : exp2f(x[kt][i] - m_ref);
                const float p1 = (x[kt][i + 1] == kNegInf) ? 0.f : exp2f(x[kt][i + 1] - m_ref);
                ps += p0 + p1;
                const uint32_t h0 = bf16_bits(p0), h1 = bf16_bits(p1);
                bh[kt * 2 + (i >> 1)] = h0 | (h1 << 16);
                bl[kt * 2 + (i >> 1)] = bf16_bits(p0 - bf16_bits_to_float(h0)) |
                                        (bf16_bits(p1 - bf16_bits_to_float(h1)) << 16);
            }
        }
        l_run += ps;
        TRACE_TILE(u, 13);
        u32x4 vop[8];
#pragma unroll
        for (int mt2 = 0; mt2 < 8; ++mt2) {
            const int dv = tr_dv + mt2 * 16;
            const int byte = ((dv >> 2) & 1) * 8;
            const u32x2 lo = lds_read_tr16(slot + tile_off(tr_key, dv >> 3) + byte);
            const u32x2 hi = lds_read_tr16(slot + tile_off(tr_key + 16, dv >> 3) + byte);
            vop[mt2] = u32x4{lo[0], lo[1], hi[0], hi[1]};
        }
        const u32x4 opb_h = {bh[0], bh[1], bh[2], bh[3]};
        const u32x4 opb_l = {bl[0], bl[1], bl[2], bl[3]};
#pragma unroll
        for (int mt2 = 0; mt2 < 8; ++mt2) acc[mt2] = mfma_bf16(vop[mt2], opb_h, acc[mt2]);
#pragma unroll
        for (int mt2 = 0; mt2 < 8; ++mt2) acc[mt2] = mfma_bf16(vop[mt2], opb_l, acc[mt2]);

        TRACE_TILE(u, 14);
        const int jseg = cons.j;
        advance(cons, s_seg, nseg);
        if (cons.j != jseg) {  // the segment's last tile: finish it
            const float l_tot = wave_sum16(l_run);
            if (sg.t0 == 0 && sg.t1 == dec_tiles(sg.p, 1)) {
                const float inv = 1.f / l_tot;
#pragma unroll
                for (int mt2 = 0; mt2 < 8; ++mt2)
                    store_out4(a, sg.row, h, gw * 128 + mt2 * 16 + 4 * g, acc[mt2] * inv);
                if (a.lse && gw == 0 && g == 0) a.lse[(size_t)sg.row * kHeads + h] = (m_ref + log2f(l_tot)) * kLn2;
            } else if (a.ws_dec_o != nullptr) {
                const size_t slot_id = 2 * (size_t)v + (jseg == 0 ? 0 : 1);
                float *po = a.ws_dec_o + (slot_id * kHeads + h) * kDv;
#pragma unroll
                for (int mt2 = 0; mt2 < 8; ++mt2)
                    *reinterpret_cast<f32x4 *>(po + gw * 128 + mt2 * 16 + 4 * g) = acc[mt2];
                if (gw == 0 && g == 0) {
                    a.ws_dec_ml[(slot_id * kHeads + h) * 2 + 0] = m_ref;
                    a.ws_dec_ml[(slot_id * kHeads + h) * 2 + 1] = l_tot;
                }
            }
#pragma unroll
            for (int mt2 = 0; mt2 < 8; ++mt2) acc[mt2] = f32x4{0.f, 0.f, 0.f, 0.f};
            m_ref = kNegInf;
            l_run = 0.f;
        }
    }
    TRACE(4);
}

// Merge kernel side.  A decode row is split when its tiles span several decode
// units; unit v keeps its first segment in slot 2 v and its last one in slot
// 2 v + 1.  The k-th split row, in request order, found as a lookup does:
struct SplitRow {
    int row, T, nt;  // output row, decode tiles before its own, its own
};
template <int Q>
__device__ __forceinline__ bool find_split_in(const AttnArgs &a, int k, SplitRow &sr) {
    const int lane = threadIdx.x & 63, S = a.dec_unit_tiles;
    int tiles = 0, splits = 0;  // of the requests before this step's
    LenRow cur[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) cur[q] = load_lens(a.cu_q, a.prefix, 64 * q + lane, a.num_reqs);
    for (int base = 0; base < a.num_reqs; base += 64 * Q) {
        LenRow nxt[Q];
        if constexpr (Q > 1) {
#pragma unroll
            for (int q = 0; q < Q; ++q) nxt[q] = load_lens(a.cu_q, a.prefix, base + 64 * (Q + q) + lane, a.num_reqs);
        }
        int nt[Q], inc[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const bool row_ok = base + 64 * q + lane < a.num_reqs && cur[q].p >= 0 && cur[q].row0 >= 0 && cur[q].row0 < a.num_rows;
            nt[q] = row_ok ? dec_tiles(cur[q].p, cur[q].next - cur[q].row0) : 0;
            inc[q] = wave_scan(nt[q]);
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int T = tiles + inc[q] - nt[q];
            const bool split = nt[q] > 0 && T / S != (T + nt[q] - 1) / S;
            const uint64_t m = __builtin_amdgcn_ballot_w64(split);
            const uint64_t hit = __builtin_amdgcn_ballot_w64(
                split && splits + __builtin_popcountll(m & ((1ull << lane) - 1)) == k);
            if (hit != 0) {
                const int l = __builtin_ctzll(hit);
                sr = SplitRow{__builtin_amdgcn_readlane(cur[q].row0, l), __builtin_amdgcn_readlane(T, l),
                              __builtin_amdgcn_readlane(nt[q], l)};
                return true;
            }
            splits += __builtin_popcountll(m);
            tiles = __builtin_amdgcn_readlane(T + nt[q], 63);
        }
        if constexpr (Q == 1) break;  // at most 64 requests
#pragma unroll
        for (int q = 0; q < Q; ++q) cur[q] = nxt[q];
    }
    return false;
}

// Workgroup `part` of split row k merges its share of the heads.
template <bool MANY>
__device__ void decode_merge(const AttnArgs &a, int k, int part, float *s_o, float *s_ml) {
    SplitRow sr;
    if (!(a.num_reqs <= 64 ? find_split_in<1>(a, k, sr) : find_split_in<kLookupQ>(a, k, sr))) return;
    end_lookup();
    const int S = a.dec_unit_tiles, T = sr.T, row = sr.row;
    const int w0 = T / S, w1 = (T + sr.nt - 1) / S;
    if (T + sr.nt > a.dec_total_tiles) return;  // device lengths beyond the host's: no such unit
    auto slot = [&](int s) {
        const int v = w0 + s;
        const size_t sl = 2 * (size_t)v + ((v == w0 && T != w0 * S) ? 1 : 0);
        return SplitRef{a.ws_dec_o + sl * kHeads * kDv, a.ws_dec_ml + sl * kHeads * 2};
    };
    const int n = w1 - w0 + 1;
    if (MANY && a.merge_many)
        merge_heads<8, 4>(a, row, part, n, slot, s_o, s_ml);
    else
        merge_heads<4, 1>(a, row, 4 * part, n, slot, s_o, s_ml);
}

// The k-th row of the chunk requests whose keys are cut into ranges (requests
// in item order): its request and the number of items of the requests before.
struct ChunkRow {
    Located lc;  // local: the row's index in its request
    int items;
};
template <int Q>
__device__ __forceinline__ bool find_chunk_row_in(const AttnArgs &a, int k, ChunkRow &cr) {
    const int lane = threadIdx.x & 63;
    const auto req = [&](int i) { return a.chunk_rev != 0 ? a.num_reqs - 1 - i : i; };
    const ChunkCount count{a.ks_chunk, a.route};
    int rows = 0, items = 0;  // of the requests before this step's
    LenRow cur[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) cur[q] = load_lens(a.cu_q, a.prefix, req(64 * q + lane), a.num_reqs);
    for (int base = 0; base < a.num_reqs; base += 64 * Q) {
        LenRow nxt[Q];
        if constexpr (Q > 1) {
#pragma unroll
            for (int q = 0; q < Q; ++q) nxt[q] = load_lens(a.cu_q, a.prefix, req(base + 64 * (Q + q) + lane), a.num_reqs);
        }
        int ni[Q], nr[Q], inc_i[Q], inc_r[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int c = cur[q].next - cur[q].row0;
            ni[q] = base + 64 * q + lane < a.num_reqs ? count(cur[q].p, c) : 0;
            nr[q] = ni[q] > ceil_div(c, kChunkBlockTokens) ? c : 0;  // more items than blocks: cut into ranges
            inc_i[q] = wave_scan(ni[q]);
            inc_r[q] = wave_scan(nr[q]);
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int end = rows + inc_r[q], first = end - nr[q];
            const uint64_t hit = __builtin_amdgcn_ballot_w64(nr[q] > 0 && k >= first && k < end);
            if (hit != 0) {
                const int l = __builtin_ctzll(hit);
                cr.lc = Located{req(base + 64 * q + l), k - __builtin_amdgcn_readlane(first, l),
                                __builtin_amdgcn_readlane(cur[q].p, l), __builtin_amdgcn_readlane(cur[q].row0, l),
                                __builtin_amdgcn_readlane(cur[q].next - cur[q].row0, l)};
                cr.items = items + __builtin_amdgcn_readlane(inc_i[q] - ni[q], l);
                return true;
            }
            rows = __builtin_amdgcn_readlane(end, 63);
            items += __builtin_amdgcn_readlane(inc_i[q], 63);
        }
        if constexpr (Q == 1) break;  // at most 64 requests
#pragma unroll
        for (int q = 0; q < Q; ++q) cur[q] = nxt[q];
    }
    return false;
}

// Workgroup `part` of row k of the split chunk requests.
template <bool MANY>
__device__ void chunk_merge(const AttnArgs &a, int k, int part, float *s_o, float *s_ml) {
    ChunkRow cr;
    if (!(a.num_reqs <= 64 ? find_chunk_row_in<1>(a, k, cr) : find_chunk_row_in<kLookupQ>(a, k, cr))) return;
    end_lookup();
    // the row's block: its item of key range 0, and ranges 1, 2, .. behind it
    Located lc = cr.lc;
    const int nks = ceil_div(lc.p + lc.c, a.ks_chunk), j = lc.local % kChunkBlockTokens;
    lc.local = (ceil_div(lc.c, kChunkBlockTokens) - 1 - lc.local / kChunkBlockTokens) * nks;
    const ChunkItem it = decode_chunk_item(a, lc);
    const int item = cr.items + lc.local;
    if (it.nks_eff <= 1 || item + it.nks_eff > a.n_chunk_items) return;
    if (it.p < 0 || it.row0 < 0 || it.row0 + it.i1 > a.num_rows) return;
    const auto slot = [&](int ks) {
        const size_t prow = (size_t)(item + ks) * kChunkBlockTokens + j;
        return SplitRef{a.ws_chunk_o + prow * kPartialFloats, a.ws_chunk_ml + prow * kPartialStats};
    };
    const int row = it.row0 + it.i0 + j;
    if (MANY && a.chunk_merge_wgs == kHeads)
        merge_heads<8, 4>(a, row, part, it.nks_eff, slot, s_o, s_ml);
    else if (a.chunk_merge_wgs == kHeads / 4)
        merge_heads<4, 1>(a, row, 4 * part, it.nks_eff, slot, s_o, s_ml);
    else
        merge_row(a, row, it.nks_eff, slot);
}

// ------------------------------------------------------------- chunk path
// Chunk rows: one workgroup of 8 wavefronts (two per SIMD) per block of 8
// query tokens (128 rows of 16 heads) and a key range of ks_chunk keys;
// 32-key tiles stream through a 3-slot global -> LDS DMA ring.  Two
// wavefronts per SIMD let one issue matrix work while the other waits on LDS
// or runs its softmax.
//  * Scores.  Wave w holds the query of token w (16 heads) over all 576
//    latent dims (18 operands of 32 dims) and forms S^T = K Q^T for two
//    16-key blocks with 16x16x32 MFMAs; nothing is exchanged between waves.
//  * Softmax.  Probabilities against a fixed reference max (no rescaling; see
//    the passes below), written to LDS as fp16 in the B-operand order of P*V:
//    slot 8 g + 4 kt + i of lane (g, head) holds key 16 kt + 4 g + i, which
//    is exactly what the lane's own scores hold, so each lane stores 16 bytes.
//  * P*V.  Wave w accumulates value dims 64 w .. 64 w + 63 of all 8 tokens
//    (4 dim blocks x 8 tokens of 16x16 accumulators); V^T comes from
//    transposing LDS reads with the same key order, converted bf16 -> fp16 in
//    registers (exact for |v| in [2^-14, 65504]).
// Per tile: one barrier.  After it, the P*V of tile t and the scores of tile
// t+1 run back to back (their operands come from different ring slots and P
// buffers), then the softmax of tile t+1 fills the other P buffer.
// A tile takes about 4,600 shader clocks, 2,176 of them the products; both
// waves of a SIMD stand at the same point of it, so what lies between the
// barrier and the first product, or between two products of a chain, is idle
// time of the matrix unit.  Hence V is read and converted before the barrier
// (beside the softmax) and not after it, and the redo test is one comparison
// per item instead of one per tile: 2048 tokens at prefix 6144 beside 128
// decode rows 570 -> 551 us, four 1024-token chunks beside 64 rows 547 -> 535.
// (Waves 4..7 half a tile ahead of the others, with a barrier per half: 561
// and 548 us.  K operands three steps ahead instead of two, or the rope query
// operands read ahead of their products: registers spill in the loop, 569 and
// 560, 620 and 644 us.)

// bf16 pairs -> fp16 pairs (exact for |v| in [2^-14, 65504]; larger values
// clamp to +-65504, smaller ones round toward zero).
__device__ __forceinline__ uint32_t bf16x2_to_f16x2(uint32_t w) {
    const auto h = __builtin_amdgcn_cvt_pkrtz(__uint_as_float(w << 16), __uint_as_float(w & 0xffff0000u));
    return __builtin_bit_cast(uint32_t, h);
}

__device__ __forceinline__ uint32_t f16x2_bits(float a, float b) {
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    const f16x2 v = {(_Float16)a, (_Float16)b};  // round to nearest even
    return __builtin_bit_cast(uint32_t, v);
}

constexpr int kCT = kChunkBlockTokens;                 // 8 tokens per item, one per wave
constexpr int kQSteps = kDqk / 32;                     // 18 query operands of 32 dims
constexpr int kQRegSteps = 16;                         // the first 16 stay in registers, the rope ones in LDS
constexpr int kChunkRing = 3;
constexpr int kPTile = kCT * 64 * 16;                  // fp16 P of one tile: [token][lane] 16 bytes
constexpr int kQLdsBytes = (kQSteps - kQRegSteps) * kCT * 64 * 16;  // rope query operands: [step][token][lane]
constexpr int kChunkLds = kChunkRing * kChunkTileBytes + 2 * kPTile + kQLdsBytes + 2 * kCT * kHeads * 4 + 16;
// Largest exponent (log2 units) a probability may take against the reference
// max: 2^15 stays inside fp16.
constexpr float kMaxPExp = 15.f;

// Chunk tiles are laid out by octets of chunks: 16-byte chunk c (8 latent
// dims) of tile key k (0..31) sits at position 256 (c >> 3) + 8 k +
// ((c & 7) ^ (k & 7)), i.e. the eight chunks (128 bytes) of a key that share
// an octet stay together, xor-swizzled with the key's low three bits.  One
// DMA round (64 positions) then reads eight keys' 128-byte pieces, one cache
// line per key, and the 16-key operand reads keep the bank pattern of a
// row-major tile (conflict-free).  Round j fills octet j >> 2, keys
// 8 (j & 3) .. + 7: lane l loads chunk 8 (j >> 2) + ((l & 7) ^ ((l >> 3) & 7))
// of key 8 (j & 3) + (l >> 3).
// The instruction offset OFF moves the LDS destination as well as the
// global source, so M0 is set to lds_base - OFF.
template <int OFF>
__device__ __forceinline__ void lds_dma16_imm(const void *gsrc, uint32_t lds_base) {
    asm volatile(
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, off offset:%2\n\t"
        :
        : "{m0}"(lds_base - OFF), "v"(gsrc), "i"(OFF)
        : "memory");
}
template <int OFF>
__device__ __forceinline__ void lds_dma16_sbase_imm(const void *sbase, uint32_t voff, uint32_t lds_base) {
    asm volatile(
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %0, %1 offset:%3\n\t"
        :
        : "v"(voff), "s"(sbase), "{m0}"(lds_base - OFF), "i"(OFF)
        : "memory");
}

// Passes of a chunk item.  The reference max of each row is fixed for the
// whole key range, so the accumulators are never rescaled:
//   main    reference = max of the first tile.  Each lane also tracks the max
//           of every score it sees.  If a later score exceeds the reference by
//           more than 2^15, the pass still runs to the end and its products
//           are discarded;
//   exact   then the item runs again against the exact max.

// Returns true when the main pass was abandoned: the caller then runs the
// item again with exact = true (the exact maxima wait in LDS).
__device__ bool chunk_item(const AttnArgs &a, int item, char *smem, int *s_pages, bool exact) {
    Located lc;
    if (!locate_item(item, a.num_reqs, ReqLens{a.cu_q, a.prefix, a.chunk_rev != 0}, ChunkCount{a.ks_chunk, a.route}, lc)) return false;
    const ChunkItem it = decode_chunk_item(a, lc);
    TRACE(1);
    const int r = it.r;
    if (it.k0 >= it.k1) return false;  // key range past this block's causal limit
    if (it.p < 0 || it.row0 < 0 || it.row0 + it.i1 > a.num_rows) return false;
    if (it.nks_eff > 1 && a.ws_chunk_o == nullptr) return false;
    const int tid = item_tid(), lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, hd = lane & 15;
    const int nt = it.i1 - it.i0;  // tokens of this block (1 .. 8)
    const int ntiles = ceil_div(it.k1 - it.k0, kChunkKeys);
    const int lp0 = it.k0 >> a.log2_page;
    // This wave's token (an idle token repeats the last one; its results are
    // not stored).  Query operands: lane l holds dims 32 s + 8 g .. + 7 of
    // head hd, s = 0..17.
    const int tk = min(wv, nt - 1);
    // Page ids (needed first, by the tile DMAs), then the queries go out, and
    // the DMAs follow while the queries are still on their way: one round trip
    // less before an item's first tile (32 + 512 rows 43.1 -> 42.3 us).
    const int npages = ((it.k1 - 1) >> a.log2_page) - lp0 + 1;
    static_assert(kPageWindow <= kAttnThreads, "one window entry per thread");
    int pg = 0;
    if (tid < min(npages, kPageWindow) && lp0 + tid < a.max_pages) pg = a.bt[(size_t)r * a.max_pages + lp0 + tid];
    u32x4 qreg[kQRegSteps], qr[kQSteps - kQRegSteps];
    char *const s_q = smem + kChunkRing * kChunkTileBytes + 2 * kPTile;  // rope query operands
    {
        const uint16_t *qp = a.q + ((size_t)(it.row0 + it.i0 + tk) * kHeads + hd) * kDqk + 8 * g;
#pragma unroll
        for (int s = 0; s < kQRegSteps; ++s) qreg[s] = *reinterpret_cast<const u32x4 *>(qp + 32 * s);
#pragma unroll
        for (int s = kQRegSteps; s < kQSteps; ++s) qr[s - kQRegSteps] = *reinterpret_cast<const u32x4 *>(qp + 32 * s);
    }
    if (tid < min(npages, kPageWindow)) {
        const bool ok = (unsigned)pg < (unsigned)a.num_pages;
        if (!ok) raise_flag(kFlagBadPage);
        s_pages[tid] = ok ? pg : 0;
    }
    TRACE(2);
    TRACE_VAL(8, 1000000ull * 1 + ntiles);

    const uint32_t ring = lds_addr(smem);
    char *const s_pbuf = smem + kChunkRing * kChunkTileBytes;           // [2][token][lane] 16 bytes
    float *const s_l = reinterpret_cast<float *>(s_q + kQLdsBytes);     // [token][head] row sums
    float *const s_mx = s_l + kCT * kHeads;                            // [token][head] exact maxima
    int *const s_abort = reinterpret_cast<int *>(s_mx + kCT * kHeads);

    // Causal limit of this wave's token (absolute key index, clipped to the
    // item's key range); wave-uniform.
    const int lim = __builtin_amdgcn_readfirstlane(min(it.p + it.i0 + tk, it.k1 - 1));

    // K operand of key block kb, step s (keys 16 kb + hd, dims 32 s + 8 g ..):
    // chunk 4 s + g, at kq_off[s & 1] + 2048 kb + 4096 (s >> 1).
    int kq_off[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) kq_off[e] = 128 * hd + 16 * ((4 * e + g) ^ (hd & 7));
    // V^T operand of value block db (dims 64 wv + 16 db + (lane & 15)): two
    // transposing reads of keys tr_key .. + 3 and tr_key + 16 .. + 3 at dims
    // 64 wv + 16 db + 4 (lane & 3) .. + 3, i.e. chunk 8 wv + 2 db + b with
    // b = (lane >> 1) & 1: vt_off[db] (+ 2048 for the second read).
    const int tr_key = 4 * g + ((lane & 15) >> 2);
    int vt_off[4];
#pragma unroll
    for (int db = 0; db < 4; ++db)
        vt_off[db] = 4096 * wv + 128 * tr_key + 16 * ((2 * db + ((lane >> 1) & 1)) ^ (tr_key & 7)) + 8 * (lane & 1);

    // DMA of tile t into its ring slot, issued by waves 4..7 only (the first tile by
    // waves 0..3; nine rounds each: round i = (wv & 3) + 4 j).  Issuing stalls a wave for a while; the
    // other wave of the same SIMD meanwhile runs ahead on its matrix work, so
    // the two wavefronts of a SIMD drift apart by about that much and the
    // softmax of one overlaps the products of the other.  A full tile inside
    // one page takes a uniform (scalar) base; any other tile (small pages, the
    // last partial tile, new latents of a fused append) one address per lane.
    const bool dma_wave = wv >= 4;
    const int dw = wv & 3;
    const int dkey = 8 * dw + (lane >> 3);  // this lane's key in every round of this wave
    const uint32_t dvoff = dkey * kRowBytes + 16 * ((lane & 7) ^ ((lane >> 3) & 7));
    const bool in_page = a.page_size >= kChunkKeys;
    const int cached_end = a.new_kv != nullptr ? min(it.k1, it.p) : it.k1;
    auto page_of = [&](int t) {
        return s_pages[min(((it.k0 + t * kChunkKeys) >> a.log2_page) - lp0, kPageWindow - 1)];
    };
    auto issue = [&](int t, int slot, int page) {
        const int kbase = it.k0 + t * kChunkKeys;
        const uint32_t dst = ring + slot * kChunkTileBytes + dw * 1024;  // round r = dw + 4 r'
        if (in_page && kbase + kChunkKeys <= cached_end) {
            const char *src = reinterpret_cast<const char *>(a.kv) +
                              ((size_t)__builtin_amdgcn_readfirstlane(page) * a.page_size +
                               (kbase & (a.page_size - 1))) * kRowBytes;
#define MLA_CHUNK_DMA_S(r) lds_dma16_sbase_imm<128 * (r)>(src, dvoff, __builtin_amdgcn_readfirstlane(dst + 4096 * (r)))
            MLA_CHUNK_DMA_S(0); MLA_CHUNK_DMA_S(1); MLA_CHUNK_DMA_S(2); MLA_CHUNK_DMA_S(3); MLA_CHUNK_DMA_S(4);
            MLA_CHUNK_DMA_S(5); MLA_CHUNK_DMA_S(6); MLA_CHUNK_DMA_S(7); MLA_CHUNK_DMA_S(8);
#undef MLA_CHUNK_DMA_S
        } else {
            // keys past the item's range repeat its last key (a finite cached latent)
            const int key = min(kbase + dkey, it.k1 - 1);
            const char *gs;
            if (a.new_kv != nullptr && key >= it.p) {
                gs = reinterpret_cast<const char *>(a.new_kv) + (size_t)(it.row0 + key - it.p) * kRowBytes;
            } else {
                const int pg = s_pages[min((key >> a.log2_page) - lp0, kPageWindow - 1)];
                gs = reinterpret_cast<const char *>(a.kv) +
                     ((size_t)pg * a.page_size + (key & (a.page_size - 1))) * kRowBytes;
            }
            gs += 16 * ((lane & 7) ^ ((lane >> 3) & 7));
#define MLA_CHUNK_DMA_V(r) lds_dma16_imm<128 * (r)>(gs, __builtin_amdgcn_readfirstlane(dst + 4096 * (r)))
            MLA_CHUNK_DMA_V(0); MLA_CHUNK_DMA_V(1); MLA_CHUNK_DMA_V(2); MLA_CHUNK_DMA_V(3); MLA_CHUNK_DMA_V(4);
            MLA_CHUNK_DMA_V(5); MLA_CHUNK_DMA_V(6); MLA_CHUNK_DMA_V(7); MLA_CHUNK_DMA_V(8);
#undef MLA_CHUNK_DMA_V
        }
    };

    float m_ref = kNegInf, m_lane = kNegInf, l_run = 0.f;
    f32x4 acc[kCT][4];  // [token][value block db]

    // S^T of tile t for this wave's token: lane l, element i of block kb =
    // key 16 kb + 4 g + i of the tile, head hd.  Two accumulation chains.
    auto scores = [&](int slot, f32x4 (&s)[2]) {
        const char *tile = smem + __builtin_amdgcn_readfirstlane(slot * kChunkTileBytes);
        s[0] = s[1] = f32x4{0.f, 0.f, 0.f, 0.f};
        constexpr int D = 2;  // steps whose K operands are in flight
        u32x4 av[D][2];
#pragma unroll
        for (int st = 0; st < D; ++st)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
                av[st][kb] = *reinterpret_cast<const u32x4 *>(tile + kq_off[st & 1] + 2048 * kb + 4096 * (st >> 1));
#pragma unroll
        for (int st = 0; st < kQSteps; ++st) {
            u32x4 cur[2] = {av[st % D][0], av[st % D][1]};
            if (st + D < kQSteps) {
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
                    av[st % D][kb] = *reinterpret_cast<const u32x4 *>(tile + kq_off[(st + D) & 1] + 2048 * kb +
                                                                      4096 * ((st + D) >> 1));
            }
            u32x4 qb;
            if (st < kQRegSteps)
                qb = qreg[st];
            else
                qb = *reinterpret_cast<const u32x4 *>(s_q + (((st - kQRegSteps) * kCT + wv) * 64 + lane) * 16);
            s[0] = mfma_bf16(cur[0], qb, s[0]);
            s[1] = mfma_bf16(cur[1], qb, s[1]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // masked raw scores of tile t
    auto masked = [&](int t, const f32x4 (&s)[2], float (&x)[8]) {
        const int kbase = it.k0 + t * kChunkKeys;
        if (kbase + kChunkKeys - 1 <= lim) {
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = s[e >> 2][e & 3];
        } else {
            const int rel = lim - kbase - 4 * g;
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = (16 * (e >> 2) + (e & 3) <= rel) ? s[e >> 2][e & 3] : kNegInf;
        }
    };
    auto lane_max = [&](const float (&x)[8], float m) {
        return max3(max3(max3(max3(m, x[0], x[1]), x[2], x[3]), x[4], x[5]), x[6], x[7]);
    };
    auto softmax = [&](int t, int pbuf, const f32x4 (&s)[2]) {
        float x[8];
        masked(t, s, x);
        m_lane = lane_max(x, m_lane);
        // the scaled score is rounded before the max is subtracted, so the max
        // key gets p = 1 exactly; masked scores give p = 0
        const float mref = m_ref == kNegInf ? 0.f : m_ref;
        float p[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
#pragma clang fp contract(off)
            p[e] = __builtin_amdgcn_exp2f(x[e] * a.scale_log2 - mref);
        }
        l_run += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
        *reinterpret_cast<u32x4 *>(s_pbuf + __builtin_amdgcn_readfirstlane(pbuf * kPTile) + (wv * 64 + lane) * 16) =
            u32x4{f16x2_bits(p[0], p[1]), f16x2_bits(p[2], p[3]), f16x2_bits(p[4], p[5]), f16x2_bits(p[6], p[7])};
    };
    // V^T operands of a tile for this wave's value dims, converted to fp16.
    // They are read and converted before the barrier that P waits for, so
    // that only the P reads stand between it and the first product.
    u32x4 av[4];
    auto vload = [&](int slot) {
        const char *tile = smem + __builtin_amdgcn_readfirstlane(slot * kChunkTileBytes);
#pragma unroll
        for (int db = 0; db < 4; ++db) {
            const u32x2 lo = lds_read_tr16(tile + vt_off[db]);
            const u32x2 hi = lds_read_tr16(tile + vt_off[db] + 2048);
            av[db] = u32x4{lo[0], lo[1], hi[0], hi[1]};
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto vconv = [&] {
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int i = 0; i < 4; ++i) av[db][i] = bf16x2_to_f16x2(av[db][i]);
    };
    // O^T += V^T P^T for tile t (P from buffer t & 1)
    auto pv = [&](int pbuf) {
        const char *pb = s_pbuf + __builtin_amdgcn_readfirstlane(pbuf * kPTile) + lane * 16;
        constexpr int PD = 3;  // P operands in flight
        u32x4 bp[PD];
#pragma unroll
        for (int tb = 0; tb < PD; ++tb) bp[tb] = *reinterpret_cast<const u32x4 *>(pb + tb * 64 * 16);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int tb = 0; tb < kCT; ++tb) {
            const u32x4 cur = bp[tb % PD];
            if (tb + PD < kCT) bp[tb % PD] = *reinterpret_cast<const u32x4 *>(pb + (tb + PD) * 64 * 16);
#pragma unroll
            for (int db = 0; db < 4; ++db) acc[tb][db] = mfma_f16(av[db], cur, acc[tb][db]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    TRACE(3);
    const bool main_pass = !exact;
    if (exact) m_ref = s_mx[wv * kHeads + hd];
    if (tid == 0) *s_abort = 0;
    lds_barrier();  // page window and abort flag ready; the ring is idle
    // Waves 0..3 issue tile 0 at once, beside their queries; waves 4..7 issue
    // tile 1 when theirs have landed.  The compiler does not count the
    // DMAs, so a wait of its own for a query load would wait for every DMA the
    // wave has issued since: this way it only waits for tile 0, which the barrier
    // waits for anyway, and tile 1 stays in flight across it.  (Both tiles from
    // waves 4..7, the queries awaited behind them: 5 + 32 rows 22.6 -> 22.3 us, 32 +
    // 512 rows 41.0 -> 40.4, ragged chunks in two calls 85.0 -> 84.1.)
    if (!dma_wave) issue(0, 0, page_of(0));
#pragma unroll
    for (int s = 0; s < kQRegSteps; ++s) asm volatile("" : "+v"(qreg[s]));
#pragma unroll
    for (int s = 0; s < kQSteps - kQRegSteps; ++s) asm volatile("" : "+v"(qr[s]));
    wait_dma_all();
    if (dma_wave && ntiles > 1) issue(1, 1, page_of(1));
#pragma unroll
    for (int s = 0; s < kQSteps - kQRegSteps; ++s)
        *reinterpret_cast<u32x4 *>(s_q + ((s * kCT + wv) * 64 + lane) * 16) = qr[s];
    __syncthreads();  // queries and tile 0 landed
#pragma unroll
    for (int tb = 0; tb < kCT; ++tb)
#pragma unroll
        for (int db = 0; db < 4; ++db) acc[tb][db] = f32x4{0.f, 0.f, 0.f, 0.f};

    // tile 0: scores, the reference max, probabilities
    TRACE_TILE(0, 11);
    {
        f32x4 s0[2];
        scores(0, s0);
        if (main_pass) {
            float x[8];
            masked(0, s0, x);
            m_ref = wave_max16(lane_max(x, kNegInf) * a.scale_log2);
        }
        vload(0);
        softmax(0, 0, s0);
        vconv();
    }
    int slot = 0;  // ring slot of tile t (t % 3)
    // steady state: after the barrier, P*V of tile t and the scores of t + 1,
    // then the softmax of t + 1
    for (int t = 0; t < ntiles; ++t) {
        TRACE_TILE(t, 11);
        const int next_page = page_of(min(t + 2, ntiles - 1));
        if (t + 1 < ntiles) wait_dma_all();  // tile t + 1 (this wave's part)
        __syncthreads();  // tile t + 1 and P of tile t complete; slot (t + 2) % 3 and P buffer (t + 1) & 1 free
        TRACE_TILE(t, 12);
        const int slot1 = slot == kChunkRing - 1 ? 0 : slot + 1;
        const int slot2 = slot1 == kChunkRing - 1 ? 0 : slot1 + 1;
        if (dma_wave && t + 2 < ntiles) issue(t + 2, slot2, next_page);
        TRACE_TILE(t, 14);
        pv(t & 1);
        TRACE_TILE(t, 15);
        if (t + 1 < ntiles) {
            f32x4 s1[2];
            scores(slot1, s1);
            vload(slot1);
            softmax(t + 1, (t + 1) & 1, s1);
            vconv();
        }
        slot = slot1;
        TRACE_TILE(t, 13);
    }
    // a score that exceeds the reference by more than P may hold (also a first
    // visible key after the first tile): the products are discarded
    m_lane *= a.scale_log2;
    if (main_pass && __builtin_amdgcn_ballot_w64(m_lane - m_ref > kMaxPExp) != 0 && lane == 0) *s_abort = 1;
    __syncthreads();  // every wave's flag write and P*V reads are done
    if (main_pass && __builtin_amdgcn_readfirstlane(*s_abort) != 0) {
        // abandoned: publish the exact maxima for the exact pass
        const float mx = wave_max16(m_lane);
        if (g == 0) s_mx[wv * kHeads + hd] = mx;
        __syncthreads();
        return true;
    }

    TRACE(4);
    // row sums of this wave's token
    {
        const float lt = wave_sum16(l_run);
        if (g == 0) s_l[wv * kHeads + hd] = lt;
    }
    __syncthreads();
    TRACE(6);
    // acc[tb][db] element i: value dim 64 wv + 16 db + 4 g + i of token tb, head hd
#pragma unroll
    for (int tb = 0; tb < kCT; ++tb) {
        if (tb >= nt) break;
        const int row = it.row0 + it.i0 + tb;
        if (it.nks_eff == 1) {
            const float inv = 1.f / s_l[tb * kHeads + hd];
#pragma unroll
            for (int db = 0; db < 4; ++db) store_out4(a, row, hd, 64 * wv + 16 * db + 4 * g, acc[tb][db] * inv);
        } else {
            const size_t prow = (size_t)item * kCT + tb;
            float *po = a.ws_chunk_o + (prow * kHeads + hd) * kDv + 64 * wv + 4 * g;
#pragma unroll
            for (int db = 0; db < 4; ++db) *reinterpret_cast<f32x4 *>(po + 16 * db) = acc[tb][db];
        }
    }
    if (g == 0 && wv < nt) {
        const int row = it.row0 + it.i0 + wv;
        const float l = s_l[wv * kHeads + hd];
        if (it.nks_eff == 1) {
            if (a.lse) a.lse[(size_t)row * kHeads + hd] = (m_ref + log2f(l)) * kLn2;
        } else {
            const size_t prow = (size_t)item * kCT + wv;
            a.ws_chunk_ml[(prow * kHeads + hd) * 2 + 0] = m_ref;
            a.ws_chunk_ml[(prow * kHeads + hd) * 2 + 1] = l;
        }
    }
    // fused append: split 0 of a block writes the block's own new latents
    // (nothing in this launch reads those slots, so it can come last)
    if (a.new_kv != nullptr && it.ks == 0) append_rows(a, r, it.p + it.i0, it.row0 + it.i0, it.i1 - it.i0);
    TRACE(5);
    return false;
}

constexpr int kMainLds = kDecLds > kChunkLds ? kDecLds : kChunkLds;

// Persistent workgroups (one per CU) take work items from two counters in
// the workspace, one per queue: the chunk items (largest blocks first) and
// the decode items.  Workgroups below dec_first_wgs start on the decode
// queue, the others on the chunk queue, and each moves to the other queue
// once its own is empty: with no decode-first workgroups the decode units
// fill the tail after the chunk items; with some, decode streaming runs
// beside the chunk tiles from the start.  An item's results and partial
// slots depend only on its index, so the schedule never changes the output
// bits.  The last workgroup to finish zeroes the counters for the next call.
// Every workgroup's first item is fixed (first_item), and the counters deal out
// what is left: a step with no more items than workgroups makes no atomic at
// all.  (With every item taken from the counters, a workgroup of such a step
// waited for up to five round trips to memory.  With the shorter decode
// start-up: 4 decode rows of 842 to 3569 keys 28.6 -> 19.6 us, 68 rows of about
// 205 keys 31.3 -> 23.6, 256 rows of up to 16384 keys 475 -> 465.)
__global__ __launch_bounds__(kAttnThreads, 1) void attention_kernel(AttnArgs a) {
    __shared__ __attribute__((aligned(16))) char smem[kMainLds];
    __shared__ int s_pages[2][kPageWindow];  // chunk items use the first window
    __shared__ DecSeg s_seg[2][kMaxSeg];
    __shared__ int s_gbar[2];
    __shared__ int s_item;
    int item = first_item(a.n_chunk_items, a.n_dec_units, a.dec_first_wgs, a.grid, (int)blockIdx.x);
    bool on_dec = item >= a.n_chunk_items;  // thread 0's current queue
    for (;;) {
        TRACE_ITEM(item);
        if (item < a.n_chunk_items) {
            // a second, exact pass only if the main one was abandoned
            for (int pass = 0; pass < 2; ++pass) {
                if (!chunk_item(a, item, smem, s_pages[0], pass != 0)) break;
                __syncthreads();
            }
        }
        else
            decode_wg(a, item - a.n_chunk_items, smem, s_pages, s_seg, s_gbar);
        TRACE(7);
        int grid = a.grid;
        asm volatile("" : "+s"(grid));  // (computed again per item: kept across the items it would take registers from their loops)
        if (a.n_chunk_items + a.n_dec_units <= grid) return;
        if (threadIdx.x == 0) {
            const int fixed_chunk = first_chunk_items(a.n_chunk_items, a.n_dec_units, a.dec_first_wgs, grid);
            // the current queue, then the other one: -1 once both are empty
            int it = -1;
            for (int k = 0; k < 2 && it < 0; ++k) {
                if (on_dec) {
                    const int d = grid - fixed_chunk + __hip_atomic_fetch_add(a.work + 2, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (d < a.n_dec_units) it = a.n_chunk_items + d;
                } else {
                    const int c = fixed_chunk + __hip_atomic_fetch_add(a.work, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (c < a.n_chunk_items) it = c;
                }
                if (it < 0) on_dec = !on_dec;
            }
            s_item = it;
        }
        __syncthreads();  // LDS free for the next item, whose index is known
        item = __builtin_amdgcn_readfirstlane(s_item);
        if (item < 0) break;
        __syncthreads();  // s_item read
    }
    if (threadIdx.x == 0) {
        const int done = __hip_atomic_fetch_add(a.work + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (done == a.grid - 1) {  // every workgroup has taken its last item
            __hip_atomic_store(a.work, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(a.work + 1, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(a.work + 2, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// Merge workgroups of the split decode rows.  (One set per request, split or
// not: 4000 rows of 16 to 256 keys, most of them whole, 288.6 -> 250.5 us,
// one row of 32000 keys beside 255 short ones 45.9 -> 42.7.)
__host__ __device__ __forceinline__ int merge_dec_wgs(const AttnArgs &a) {
    return a.ws_dec_o != nullptr ? a.n_split_rows * merge_wgs(a) : 0;
}

// Split merges, after the attention kernel (the kernel boundary makes every
// partial visible): first merge_wgs workgroups per split decode row, then
// chunk_merge_wgs per row of the split chunk requests.  MANY: some rows take a
// workgroup per head.
template <bool MANY>
__global__ __launch_bounds__(kThreads, MANY ? 4 : 5) void combine_kernel(AttnArgs a) {
    __shared__ __attribute__((aligned(16))) float s_o[4 * kDv];
    __shared__ float s_ml[8];
    const int b = blockIdx.x;
    const int n_dec = merge_dec_wgs(a);
    if (b < n_dec)
        decode_merge<MANY>(a, b / merge_wgs(a), b % merge_wgs(a), s_o, s_ml);
    else
        chunk_merge<MANY>(a, (b - n_dec) / a.chunk_merge_wgs, (b - n_dec) % a.chunk_merge_wgs, s_o, s_ml);
}

// ----------------------------------------------------------------- append
// Request of a global row: wave-parallel 64-ary search of cu_q.
__device__ __forceinline__ int find_request(const int32_t *cu_q, int num_reqs, int row, int lane) {
    int lo = 0, hi = num_reqs;  // cu_q[lo] <= row < cu_q[hi]
    while (hi - lo > 1) {
        const int step = ceil_div(hi - lo, 64);
        const int idx = lo + lane * step;
        const bool le = idx < hi && cu_q[idx] <= row;
        const uint64_t m = __builtin_amdgcn_ballot_w64(le);
        if (m == 0) break;
        const int last = 63 - __builtin_clzll(m);
        lo = lo + last * step;
        hi = min(hi, lo + step);
    }
    return lo;
}

// One wavefront copies one row (the 64 + 8 16-byte chunks of a latent).  A
// chunk's few hundred rows move less than a megabyte, so the call is bound by
// the chain lengths -> page id -> store and by how many rows run it at once:
// a wavefront per row keeps every CU busy from about a thousand rows on.  (Eight
// rows a wavefront, sharing one lookup: 14.3 us for 1104 rows on 35 workgroups.)
// The row itself and, for up to 64 requests, every length load go out at once.
__global__ __launch_bounds__(kThreads) void append_kernel(AppendArgs a) {
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * (kThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (row >= a.num_rows) return;
    const u32x4 *src = reinterpret_cast<const u32x4 *>(a.src + (size_t)row * kDqk);
    const u32x4 va = src[lane];
    u32x4 vb = {0u, 0u, 0u, 0u};
    if (lane < kChunksPerRow - 64) vb = src[64 + lane];
    // rows past the device's last request (device lengths shorter than the
    // host's) belong to nobody: skipped, with the flag raised
    const int total = a.cu_q[a.num_reqs];
    int r, start, pr;
    if (a.num_reqs <= 64) {
        const int cw = lane < a.num_reqs ? a.cu_q[lane] : INT_MAX;
        const int pw = lane < a.num_reqs ? a.prefix[lane] : 0;
        // cu_q[0] = 0 <= row: at least one lane holds (the last of them owns the row)
        r = max(__builtin_popcountll(__builtin_amdgcn_ballot_w64(cw <= row)) - 1, 0);
        start = __shfl(cw, r, 64);
        pr = __shfl(pw, r, 64);
    } else {
        r = find_request(a.cu_q, a.num_reqs, row, lane);
        start = a.cu_q[r];
        pr = a.prefix[r];
    }
    const int t = pr + (row - start);
    const int lp = t >> a.log2_page;
    const int page = row < total && t >= 0 && lp < a.max_pages ? a.bt[(size_t)r * a.max_pages + lp] : -1;
    if ((unsigned)page >= (unsigned)a.num_pages) {
        raise_flag(kFlagBadPage);
        return;
    }
    u32x4 *dst = reinterpret_cast<u32x4 *>(a.kv + ((size_t)page * a.page_size + (t & (a.page_size - 1))) * kDqk);
    dst[lane] = va;
    if (lane < kChunksPerRow - 64) dst[64 + lane] = vb;
}

}  // namespace

#ifdef MLA_TRACE
extern "C" int mla_trace_read(void *dst, size_t bytes) {
    return (int)hipMemcpyFromSymbol(dst, HIP_SYMBOL(g_trace), bytes, 0, hipMemcpyDeviceToHost);
}
#endif

hipError_t noalloc_scratch(void **ptr) {
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (addr[dev] == nullptr) {
        // once per device, with that device current: its copy's address, and
        // the work-queue counters cleared (every completed call leaves them zero)
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        static const unsigned char zeros[256] = {};
        e = hipMemcpy(p, zeros, sizeof zeros, hipMemcpyHostToDevice);
        if (e != hipSuccess) return e;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}

hipError_t read_flags(int *flags, bool clear) {
    hipError_t e = hipMemcpyFromSymbol(flags, HIP_SYMBOL(g_flags), sizeof(int), 0, hipMemcpyDeviceToHost);
    if (e != hipSuccess || !clear || *flags == 0) return e;
    const int zero = 0;
    return hipMemcpyToSymbol(HIP_SYMBOL(g_flags), &zero, sizeof(int), 0, hipMemcpyHostToDevice);
}

hipError_t launch_append(const AppendArgs &a, hipStream_t s) {
    const int rows_per_block = kThreads / 64;
    const int grid = (a.num_rows + rows_per_block - 1) / rows_per_block;
    if (grid == 0) return hipSuccess;
    hipLaunchKernelGGL(append_kernel, dim3(grid), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_attention(const AttnArgs &a, hipStream_t s) {
    const int grid = a.grid;
    if (grid == 0) return hipSuccess;
    hipLaunchKernelGGL(attention_kernel, dim3(grid), dim3(kAttnThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_combine(const AttnArgs &a, hipStream_t s) {
    // only the rows that left partials get workgroups
    const long long grid_ll =
        (long long)merge_dec_wgs(a) + (a.ws_chunk_o != nullptr ? (long long)a.n_split_chunk_rows * a.chunk_merge_wgs : 0);
    if (grid_ll > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    const int grid = (int)grid_ll;
    if (grid == 0) return hipSuccess;
    if (a.merge_many || a.chunk_merge_wgs == kHeads)
        hipLaunchKernelGGL(combine_kernel<true>, dim3(grid), dim3(kThreads), 0, s, a);
    else
        hipLaunchKernelGGL(combine_kernel<false>, dim3(grid), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace mla
