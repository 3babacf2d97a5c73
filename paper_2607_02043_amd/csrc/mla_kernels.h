// Launch-side description of the kernels of libmlastep (host <-> device).
#pragma once
#include "chunk_route.h"
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mla {

constexpr int kHeads = 16;
constexpr int kDqk = 576;   // latent: 512 compressed + 64 rope dims
constexpr int kDv = 512;    // value: first 512 latent dims
constexpr int kRowBytes = kDqk * 2;
constexpr int kKeysPerTile = 32;
constexpr int kPageWindow = 256;   // page ids one work item may touch
constexpr int kThreads = 256;      // 4 wavefronts of 64 (merge, append; DMA rounds of the attention kernel)
constexpr int kAttnThreads = 512;  // attention kernel: 8 wavefronts, two per SIMD
constexpr int kChunkBlockTokens = 8;                        // tokens per chunk work item
constexpr int kPartialFloats = kHeads * kDv;                // one row's partial output
constexpr int kPartialStats = kHeads * 2;                   // one row's (max, sum) per head
constexpr int kMaxDecSegments = 64;                         // requests one decode workgroup may touch
constexpr int kFlagBadPage = 1;       // a block-table entry outside [0, num_pages) was met (MLA_FLAG_BAD_PAGE)
constexpr int kFlagWaitExpired = 2;   // a bounded wait inside a kernel gave up (MLA_FLAG_WAIT_EXPIRED)
constexpr int kSpinLimit = 1 << 16;   // sleeps of a bounded wait before it gives up
constexpr size_t kNoAllocScratchBytes = size_t(128) << 20;  // scratch of mixed_step_noalloc, per device
constexpr int kMaxDevices = 64;

struct AttnArgs {
    const uint16_t *q;
    const uint16_t *kv;
    // Fused append (both null otherwise): the step's new latents, read in place
    // of their cache slots, and the cache they are written into.
    const uint16_t *new_kv;
    uint16_t *kv_out;
    const int32_t *cu_q;
    const int32_t *prefix;
    const int32_t *bt;
    void *out;
    float *lse;
    float *ws_chunk_o;    // [n_chunk_items][block tokens][16][512]
    float *ws_chunk_ml;   // [n_chunk_items][block tokens][16][2]
    float *ws_dec_o;      // [2 units][16][512]: first / last segment of each decode unit
    float *ws_dec_ml;     // [2 units][16][2]
    int32_t *work;        // [3]: next chunk item, workgroups done, next decode item; zero between calls
    int32_t num_reqs;
    int32_t num_rows;
    int32_t page_size;
    int32_t log2_page;
    int32_t max_pages;
    int32_t num_pages;
    float scale_log2;     // softmax scale * log2(e)
    int32_t ks_chunk;          // chunk blocks are cut into ceil((p + c) / ks_chunk) key ranges (a multiple of 64)
    int32_t chunk_rev;         // chunk items numbered from the last request to the first
    int32_t n_chunk_items;     // work items 0 .. n_chunk_items - 1
    int32_t n_dec_units;       // then the decode items: pairs of units (slices of the flattened decode
                               // tile list), one unit per wave group
    int32_t dec_unit_tiles;    // 32-key decode tiles per unit
    int32_t dec_total_tiles;
    int32_t grid;              // persistent workgroups of the attention launch
    int32_t dec_first_wgs;     // workgroups 0 .. dec_first_wgs - 1 take decode items before chunk items
    int32_t n_split_rows;      // decode rows cut across units: the merge launches workgroups for these alone
    int32_t merge_many;        // 1: some decode row is cut into more than kMergeFewParts parts
    int32_t n_split_chunk_rows;  // rows of the chunk requests whose keys are cut into ranges
    int32_t chunk_merge_wgs;     // merge workgroups of each of them (chunk_merge_wgs())
    int32_t out_bf16;
    int32_t spin_limit;        // sleeps of a bounded wait before it gives up (kSpinLimit)
    ChunkRoute route;          // chunk requests it sends to the multi-head path are left out of this launch
};

// The fixed first items of the attention launch's G workgroups (G at most the
// number of items).  Workgroup b < D takes decode item b, the others take
// chunk items 0, 1, ..; a workgroup whose kind has run out takes the next item
// of the other kind.  Each kind's first items are then its lowest indexes:
// first_chunk_items chunk items and G minus that many decode items.
__host__ __device__ inline int first_chunk_items(int n_chunk, int n_dec, int D, int G) {
    const int n = G - D + (D > n_dec ? D - n_dec : 0);
    return n < n_chunk ? n : n_chunk;
}
// Item of workgroup b: a chunk item, or n_chunk + a decode item.
__host__ __device__ inline int first_item(int n_chunk, int n_dec, int D, int G, int b) {
    if (b < D) return b < n_dec ? n_chunk + b : (G - D) + (b - n_dec);
    const int k = b - D;
    return k < n_chunk ? k : n_chunk + (D < n_dec ? D : n_dec) + (k - n_chunk);
}

// Merge workgroups of a split decode row: of four heads each, or of one head
// (four wavefronts on every fourth part) when rows have many parts.
constexpr int kMergeFewParts = 16;
__host__ __device__ inline int merge_wgs(const AttnArgs &a) { return a.merge_many ? kHeads : kHeads / 4; }
// Merge workgroups of a split chunk row of at most `parts` parts: one for the
// whole row (four heads a wavefront, one after the other), or as a decode row
// where the chain of its loads would be long.
constexpr int kChunkMergeFewParts = 4;
inline int chunk_merge_wgs(long long parts) {
    return parts > kMergeFewParts ? kHeads : parts > kChunkMergeFewParts ? kHeads / 4 : 1;
}

struct AppendArgs {
    const uint16_t *src;
    uint16_t *kv;
    const int32_t *cu_q;
    const int32_t *prefix;
    const int32_t *bt;
    int32_t num_reqs;
    int32_t num_rows;
    int32_t page_size;
    int32_t log2_page;
    int32_t max_pages;
    int32_t num_pages;
};

hipError_t launch_append(const AppendArgs &a, hipStream_t s);
// Reads the device's sticky kernel error flags (kFlag*), and clears them if asked.
hipError_t read_flags(int *flags, bool clear);
// Device address of the current device's no-allocation scratch
// (kNoAllocScratchBytes bytes, counters zero on first use); set up once per device.
hipError_t noalloc_scratch(void **ptr);
hipError_t launch_attention(const AttnArgs &a, hipStream_t s);
hipError_t launch_combine(const AttnArgs &a, hipStream_t s);

}  // namespace mla
