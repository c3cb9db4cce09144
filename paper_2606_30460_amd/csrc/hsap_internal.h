// Internal declarations shared by the libhsap translation units (not installed).
#pragma once

#include <cstdint>
#include <cstdio>
#include <string>

#include "../../include/hsap.h"

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define HSAP_HD __host__ __device__
#else
#define HSAP_HD
#endif

namespace hsap {

// ---------------------------------------------------------------------------
// error reporting (thread-local message behind hsap_last_error)
// ---------------------------------------------------------------------------
void set_error(const char* fmt, ...) __attribute__((format(printf, 1, 2)));
void clear_error();

#define HSAP_FAIL(code, ...)        \
  do {                              \
    ::hsap::set_error(__VA_ARGS__); \
    return code;                    \
  } while (0)

// ---------------------------------------------------------------------------
// shard geometry
//
// A batch of B packed sequences of Ns tokens each, concatenated (sequence b
// holds positions b*Ns .. b*Ns+Ns-1), every sequence split P ways.  Shard
// (or chunk) x holds ns = Ns/P positions of each sequence; its local rows are
// b*ns + l.  CONTIGUOUS: position b*Ns + x*ns + l.  ZIGZAG: each sequence is
// cut into 2P pieces of m = Ns/(2P); rows l < m are piece x, rows m..2m-1 are
// piece 2P-1-x.
// ---------------------------------------------------------------------------
struct Geom {
  int64_t N;   // positions over the batch (B * Ns)
  int64_t n;   // rows per shard over the batch (B * ns)
  int64_t m;   // rows per piece of one sequence (ns for CONTIGUOUS, ns/2 for ZIGZAG)
  int64_t Ns;  // tokens per sequence
  int64_t ns;  // rows per shard of one sequence
  int32_t P;
  int32_t layout;
  int32_t B;
};

HSAP_HD inline int64_t global_pos(const Geom& g, int32_t shard, int64_t local) {
  int64_t base = 0;
  if (g.B > 1) {  // rows and positions stay below 2^31 (checked with the descriptor)
    const uint32_t b = (uint32_t)local / (uint32_t)g.ns;
    base = (int64_t)b * g.Ns;
    local -= (int64_t)b * g.ns;
  }
  if (g.layout == HSAP_LAYOUT_CONTIGUOUS) return base + (int64_t)shard * g.ns + local;
  return base + (local < g.m ? (int64_t)shard * g.m + local : (int64_t)(2 * g.P - 1 - shard) * g.m + (local - g.m));
}

// Validates N, P, layout, shard id and tile sizes; fills `g`.
hsap_status check_shard(const hsap_shard_desc* d, Geom* g);

// Validates an attention descriptor (shard part plus heads, head_dim, scale).
hsap_status check_attn(const hsap_attn_desc* d, Geom* g);

// Whether the backward kernels exist for the descriptor's (head_dim, BM, BN); the descriptor
// must already pass check_attn.
bool backward_supported(const hsap_attn_desc* d);

// Key streams per workgroup of the forward and dQ kernels (their KS): the waves of a q-tile are
// repeated KS times, each set takes every KS-th 64-key step of the run and the results are combined
// in LDS at the end, so a run's chain of steps is KS times shorter at the same work.  That pays while
// the grid leaves the chip idle.  The choice depends on the shape alone -- `items`, the (q-tile, head)
// pairs of the call (times the chunks for the partial forward, whose runs are one per chunk) -- so that
// calls over the same tiles give the same bits however their lists are cut.  Measured on one
// document, forward / dQ in us, one stream -> KS (runs of at most 8 steps gain nothing: 13.9 / 20.0 ->
// 13.8 / 19.2 at 512 keys, and a step of 128-key chunks lost 1.5 %; `keys` is the most a run can have):
//   head_dim 64, 64-row q-tiles:  256 items of 16 tiles 29.5 / 34.0 -> 16.0 / 18.5 (four streams),
//     512 items 30.7 / 35.8 -> 20.8 / 25.7 (two), 1024 items of 4 tiles 13.0 / 22.5 -> 16.2 / 23.3 (two)
//   head_dim 64, 128-row:  256 items 31.9 / 35.4 -> 25.0 / 28.7, 512 items of 5 tiles 13.9 / 20.9 -> 16.7 / 22.8
//   head_dim 128, 128-row: 128 items 36.6 / 55.0 -> 32.1 / 45.7, 256 items of 2.5 tiles 15.7 / 23.5 -> 15.7 / 23.8,
//     512 items 23.0 / 31.7 -> 29.5 / 42.2
//   head_dim 128, 64-row:  256 items 41.8 / 53.1 -> 29.7 / 36.0, 512 items of 2.5 tiles 17.0 / 23.1 -> 19.8 / 25.6
constexpr int64_t kComputeUnits = 256;
inline int key_streams(int head_dim, int block_m, int64_t items, int64_t keys) {
  if (block_m > 128 || keys < 1024) return 1;
  if (head_dim == 64 && block_m == 64) return items <= kComputeUnits ? 4 : items <= 2 * kComputeUnits ? 2 : 1;
  return items <= (head_dim == 128 && block_m == 128 ? 3 * kComputeUnits / 4 : kComputeUnits) ? 2 : 1;
}

// The direct-to-LDS forward packs a tile descriptor as k_tile | chunk << 23 | kind << 31.
constexpr int kMaxDlChunks = 256;
constexpr int64_t kMaxDlKTiles = int64_t(1) << 23;
inline bool dl_packed(const Geom& g, int block_n) { return g.P <= kMaxDlChunks && g.n / block_n < kMaxDlKTiles; }

// The same for the partial forward, whose runs each cover one chunk.
inline int fwd_key_streams(int head_dim, int block_m, int block_n, int heads_q, const Geom& g) {
  return dl_packed(g, block_n) ? key_streams(head_dim, block_m, g.n / block_m * heads_q * g.P, g.ns) : 1;
}

#if defined(__HIPCC__)
// First index i of tiles[0 .. num - 1] (sorted by q_tile) with tiles[i].q_tile >= key, for the
// tile-list entry points (one chunk's tiles in the planner's order).  Wave-wide: each round
// narrows the range 64-fold with one strided probe per lane, the last compares a window of at
// most 64 entries; every probe stays inside the list (num <= 2^30).  The result is the same on
// every lane.
__device__ inline int32_t lower_bound_q_tile(const hsap_tile* tiles, int32_t num, int32_t key, int lane) {
  if (num <= 0) return 0;
  int32_t lo = 0, len = num;
  while (len > 64) {
    const int32_t stride = (len + 63) >> 6;
    const int32_t idx = min(lo + lane * stride, lo + len - 1);
    const bool below = lo + lane * stride < lo + len && tiles[idx].q_tile < key;
    const int32_t cnt = __popcll(__builtin_amdgcn_ballot_w64(below));
    if (cnt == 0) return lo;  // tiles[lo] is already >= key
    const int32_t next = lo + (cnt - 1) * stride + 1;
    len = min(lo + cnt * stride, lo + len) - next;
    lo = next;
  }
  const bool below = lane < len && tiles[min(lo + lane, num - 1)].q_tile < key;
  return lo + __popcll(__builtin_amdgcn_ballot_w64(below));
}

// Workgroup bid of a (run, query head) grid -> its run and query head.  Workgroups are dispatched
// to the eight XCDs round-robin (workgroup i on XCD i % 8), and each XCD has its own L2.  When the
// K/V heads split evenly over the XCDs, the query heads that read one K/V head are placed on one
// XCD (K/V head g on XCD g % 8), so the K/V tiles they share are fetched into one L2 instead of
// `group` of them.  Runs keep their order (longest first) on every XCD.  Without grouped heads
// (hq == hkv) this is the plain run-major order, head fastest.
__device__ inline void run_and_head(int bid, int hq, int hkv, int& run, int& h) {
  if (hkv % 8 == 0 && hq != hkv) {
    const int per = hq >> 3;  // query heads per XCD
    const int group = hq / hkv;
    const int x = bid & 7, y = bid >> 3;
    run = y / per;
    const int lh = y - run * per;  // the XCD's lh-th query head: K/V head 8 j + x, member i
    const int j = lh / group, i = lh - j * group;
    h = (8 * j + x) * group + i;
  } else {
    run = bid / hq;
    h = bid - run * hq;
  }
}

// Document start of this lane's query (global position gq), in two parts so the memory access
// is issued at kernel start and consumed after the prologue.  With per-position starts it is one
// load.  From the cumulative lengths instead: a wave's 32 queries (lanes 0..31; lane l ^ 32 holds
// the query of lane l) are 32 consecutive positions -- every piece of a shard is a multiple of
// the 64-, 128- or 256-row q-tile -- so at most 31 documents with tokens begin after lane 0's position
// g_lo, up to lane 31's position g_hi.  The wave loads 64 consecutive entries
// of cu_seqlens, starting at most 31 entries before the document of g_lo (a 64-way search in
// rounds narrows the start when there are more than 32 entries), and each lane takes the largest
// entry not above its position with ballots and lane reads: no further memory access.  Repeated entries
// (documents without tokens) can outnumber the window; then each lane searches the entries.
struct DocWindow {
  int32_t w;           // cu[base + lane], or this lane's start when per-position starts are given
  int32_t g_lo, g_hi;  // positions of the wave's first and last query
};

__device__ __forceinline__ DocWindow doc_window(const int32_t* doc_start, const int32_t* cu, int32_t num_docs, int32_t gq,
                                                int lane) {
  DocWindow r{};
  if (!cu) {
    r.w = doc_start[gq];
    return r;
  }
  r.g_lo = __builtin_amdgcn_readlane(gq, 0);
  r.g_hi = __builtin_amdgcn_readlane(gq, 31);
  const int32_t nd = num_docs;
  int32_t base = 0, len = nd + 1;  // the document of g_lo is one of base .. base + len - 1
  while (len > 32) {
    const int32_t stride = (len + 63) >> 6;
    const int32_t v = cu[min(base + lane * stride, nd)];
    base += stride * (__popcll(__builtin_amdgcn_ballot_w64(v <= r.g_lo)) - 1);
    len = stride;
  }
  r.w = cu[min(base + lane, nd)];
  return r;
}

__device__ __forceinline__ int32_t doc_window_start(const int32_t* cu, int32_t num_docs, const DocWindow& r, int32_t gq) {
  if (!cu) return r.w;
  const int32_t lo = __popcll(__builtin_amdgcn_ballot_w64(r.w <= r.g_lo)) - 1;    // document of g_lo
  const int32_t last = __popcll(__builtin_amdgcn_ballot_w64(r.w <= r.g_hi)) - 1;  // last boundary <= g_hi
  int32_t start = __builtin_amdgcn_readlane(r.w, lo);
  if (last >= 63) {  // more entries than the window holds: documents without tokens among them
    int32_t l = 0, h = num_docs;
    while (h - l > 1) {
      const int32_t mid = (l + h) >> 1;
      if (cu[mid] <= gq) l = mid;
      else h = mid;
    }
    return cu[l];
  }
  for (int32_t j = lo + 1; j <= last; ++j) {
    const int32_t b = __builtin_amdgcn_readlane(r.w, j);
    if (gq >= b) start = b;
  }
  return start;
}

// The run of q-tile qt in a sorted tile list: {slot 0, qt, first, count}.
__device__ inline hsap_run q_tile_run(const hsap_tile* tiles, int32_t num, int32_t qt, int lane) {
  const int32_t first = lower_bound_q_tile(tiles, num, qt, lane);
  const int32_t end = lower_bound_q_tile(tiles, num, qt + 1, lane);
  return hsap_run{0, qt, first, end - first};
}

// Workgroups of the bf16 partial forward resident on one compute unit for the descriptor's shape
// (the runtime's occupancy of the kernel that runs); 0 when there is none.
int fwd_resident_per_cu(const hsap_attn_desc* d);
#endif

#if defined(__HIPCC__)
// Copies `bytes` (a multiple of 16) from pinned, device-mapped host memory to dst, both 16-byte
// aligned, with one launch.
hsap_status upload(void* dst, const void* pinned, size_t bytes, hipStream_t stream);

// Zeroes tiles tiles[0 .. num_tiles-1] (device int32) of both a and b, tile t being the byte
// range [t * tile_bytes, (t + 1) * tile_bytes); tile_bytes a multiple of 16, a and b 16-byte
// aligned.  Nothing is launched for an empty list.
hsap_status zero_tiles(void* a, void* b, const int32_t* tiles, int32_t num_tiles, int64_t tile_bytes,
                       hipStream_t stream);

// hsap_lse_merge over the rows of the BM-row q-tiles listed in tiles[0 .. num_tiles-1] (device
// int32), or over every row when tiles is NULL; rows of other q-tiles are neither read nor written.
hsap_status lse_merge(int32_t num_parts, const float* const* o_parts, const float* const* lse_parts, int64_t n,
                      int32_t heads_q, int32_t head_dim, void* o_out, float* lse_out, const int32_t* tiles,
                      int32_t num_tiles, int32_t block_m, hipStream_t stream);

// The executor's forwards.  Document starts come from the cumulative lengths cu_seqlens
// [num_docs + 1] on the device (no per-position start array).  fused: hsap_attn_fwd_fused over
// runs that span every chunk.  Otherwise hsap_partial_attn_fwd_runs, where runs whose slot is
// kFinalSlot write the final bf16 O and LSE of their q-tile to o_out / lse_out (the q-tile's
// only part: nothing to merge).
constexpr int32_t kFinalSlot = -2;

// hsap_attn_bwd_bf16 with the backward preprocess folded into the dQ kernel: delta (device fp32
// [Hq, n], written) is computed there from o and d_o, and read by the dK/dV kernel launched after, and so
// are the document starts of the shard's rows, from cu_seqlens [num_docs + 1], written to doc_start
// [N] at the rows' positions.
hsap_status attn_bwd_bf16_delta(const hsap_attn_desc* desc, const void* q, const void* k, const void* v,
                                const void* d_o, const void* o, const float* lse, float* delta,
                                const int32_t* cu_seqlens, int32_t num_docs, int32_t* doc_start,
                                const hsap_tile* tiles_k, const hsap_run* runs_k, int64_t num_runs_k,
                                const hsap_tile* tiles_q, const hsap_run* runs_q, int64_t num_runs_q, void* dq,
                                void* dk, void* dv, int key_blocks, hipStream_t stream);

// Key blocks of 32 per dK/dV workgroup (attn_bwd_bf16_delta's key_blocks) for all k-major runs of a plan, longest
// first (host), with num_tiles tiles in all.
int plan_key_blocks(const hsap_attn_desc& d, const Geom& g, const hsap_run* runs, int64_t num_runs, int64_t num_tiles);
hsap_status executor_forward(const hsap_attn_desc* desc, bool fused, const void* q, const void* k, const void* v,
                             const int32_t* cu_seqlens, int32_t num_docs, const hsap_tile* tiles,
                             const hsap_run* runs, int64_t num_runs, float* o_part, float* lse_part,
                             int32_t num_slots, void* o_out, float* lse_out, hipStream_t stream);
#endif

}  // namespace hsap
