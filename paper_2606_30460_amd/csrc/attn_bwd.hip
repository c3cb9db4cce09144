// Partial attention backward: gradients of one shard's attention with
// respect to its queries and to the listed k-tiles of each K/V chunk (the
// backward "computing" whose results the paper's per-rank code returns as dq
// and dkv messages, instruction table of the SAP section).  P is recomputed
// from the final (merged) LSE, so no attention matrix is stored between
// forward and backward.  Two kernels share the work, so that neither needs
// atomics per k-tile:
//
// dK/dV kernels: one workgroup per (k-major run, K/V head).  A run is one
// (chunk, k-tile) with the q-tiles listed against it; the workgroup keeps the
// k-tile's K and V rows (as MFMA B operands) and its dK, dV accumulators in
// registers for the whole run, looping over the query heads of its K/V head
// group and over the listed q-tiles in sub-tiles of 64 or 32 rows.  Per sub-tile:
//   S  = Q K^T, dP = dO V^T           (lane = key, registers = queries)
//   P  = exp2(S * scale*log2e - LSE*log2e) on allowed pairs, dS = P (dP - delta)
//   dV += P^T dO, dK += dS^T Q        (A operands from registers; dO and Q
//                                      read transposed from LDS)
// Each 32-key block belongs to two waves on one SIMD, one forming S, P and dV,
// the other dP, dS and dK (P handed over through LDS).  Q and dO sub-tiles sit
// in XOR-swizzled LDS tiles (mfma.h).  Each (chunk, key block, K/V head) of
// dK/dV has one owner.
//
// dQ kernel: one workgroup per (q-major run, query head), shaped like the
// forward; it forms S and dP again for its own pairs (described below).
//
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "hsap_internal.h"
#include "mfma.h"

namespace hsap {

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

struct BwdArgs {
  const __bf16* q;
  const __bf16* k;
  const __bf16* v;
  const __bf16* d_o;
  const float* lse;
  const float* delta;
  const __bf16* o;     // when set, the dQ kernel computes delta from O and dO itself, writing delta_out
  float* delta_out;
  const int32_t* doc_start;
  const int32_t* cu;      // when set, the dQ kernel finds document starts here, writing them to start_out
  int32_t num_docs;
  int32_t* start_out;
  const hsap_tile* tiles;
  const hsap_run* runs;
  float* dq;       // fp32 accumulators (+=), or
  float* dk;
  float* dv;
  __bf16* dq16;    // final bf16 gradients (written once)
  __bf16* dk16;
  __bf16* dv16;
  Geom geom;
  int32_t shard;
  int32_t hq;
  int32_t hkv;
  int32_t group;
  int32_t bm;
  int32_t bn;
  int32_t parts;         // dK/dV: workgroups per k-tile (BN / keys of a workgroup)
  int32_t wide_kv;       // dK/dV: both outputs 16-byte aligned (16-byte accesses)
  float scale;
  float scale_log2;
  int32_t num_tiles;     // tile-list mode: entries of tiles (one chunk's, sorted by q_tile)
  int32_t chunk;         // tile-list mode: the chunk of every tile
};

// Tile-list mode of the dK/dV kernel: at most this many q-tiles (n / BM) per k-tile.
constexpr int kMaxListQTiles = 2048;

// ---------------------------------------------------------------------------
// dK/dV kernel with split roles: eight waves in four pairs, each pair on one SIMD
// (wave w and wave w + 4 share one: waves are placed round-robin).  A pair owns
// 32 keys of the k-tile: its S wave holds the block's K rows as MFMA B operands
// and its dV accumulators, its dP wave the V rows and the dK accumulators.  Per
// sub-tile of SUB query rows:
//   scores    S wave:  S = Q K^T, P = exp2(S * scale*log2e - LSE*log2e) on
//                      allowed pairs; P to LDS for its partner
//             dP wave: dP = dO V^T
//   products  S wave:  dV += P^T dO             (dO read transposed)
//             dP wave: P from LDS, dS = P (dP - delta), dK += dS^T Q
//                      (Q read transposed)
// software-pipelined by one sub-tile: iteration t runs the products of t and
// the scores of t + 1 while later Q and dO rows go from global memory straight
// into LDS (global_load_lds).  One wave's exponentials (or dS arithmetic) run
// while the other wave's products occupy the matrix core; S and dP are formed
// once.
//
// The workgroup covers KB key blocks (32 KB keys) with QS = 4 / KB streams of
// sub-tiles: pair p works on key block p % KB and takes every QS-th sub-tile of
// the run; the streams' gradients are summed in LDS at the end, in stream
// order.  KB = 4: one 128-key tile, 64-row sub-tiles, each staged row feeding
// four key blocks.  KB = 2: 64 keys.  KB = 1: 32 keys; four times the
// workgroups of KB = 4 with chains a quarter as long, for grids too small to
// fill the chip, at four times the staging traffic.
//
// The two roles are two loops of their own.  Bound by the matrix cores and the LDS
// reads of the operands, of which neither is saturated (latency of each wave's chain
// LDS read -> MFMA -> exponentials; MFMA busy 0.50 at head_dim 128, 0.30 at 64).  Measured, the
// kernel alone: head_dim 128, 4096 rows of one document x 32 heads, 305 -> 290 us against
// one loop with a role test per product; against one wave per 32 keys doing all four
// products, P in fp32: head_dim 64, 8192 rows x 32 heads over 8, 602 -> 448 us; tile-list call,
// 4096 rows x 12 heads over 4, 498 -> 156 us (four streams of 32 keys).
//
// LDS ring: three sub-tiles (t: products, t + 1: scores, t + 2: in flight) and
// one barrier per iteration; KB = 1 at head_dim 128 has room for two only
// (sub-tile t + 1 is moved during the products of t, with a barrier between
// the products and the scores).
// ---------------------------------------------------------------------------
// WIDE: Q rows of so many heads that 32 of them do not fit 32-bit byte offsets (the transfers take
// 64-bit addresses per lane).
// P32: P handed over in fp32, otherwise in fp16.
template <int D, int KB, bool BF16OUT, bool LIST, bool WIDE = false, bool P32 = KB < 4 || LIST>
__global__ __launch_bounds__(512, D == 64 && KB == 2 ? 4 : 2) void attn_bwd_dkdv_kernel(BwdArgs a) {
  static_assert(!LIST || !BF16OUT, "the tile-list mode accumulates fp32");
  static_assert((D == 128 || D == 64) && (KB == 4 || KB == 2 || KB == 1), "shapes with a kernel");
  constexpr int QS = 4 / KB;                    // sub-tile streams
  constexpr int SUB = KB == 4 ? 64 : 32;        // query rows per sub-tile
  constexpr int QB = SUB / 32;
  constexpr int RING = D == 128 && KB == 1 ? 2 : 3;
  constexpr int CPR = D / 8;
  constexpr int MB = D / 32;
  constexpr int WCH = SUB * CPR / (2 * KB);     // 16-byte chunks of a Q (or dO) sub-tile a wave moves
  constexpr int U = WCH / 64;                   // transfer instructions per wave per sub-tile and tensor
  static_assert(WCH % 64 == 0, "a wave moves whole instructions of a sub-tile");
  constexpr float LOG2E = 1.44269504088896340736f;
  // LDS: the ring of Q and dO sub-tiles per stream and the P hand-off, used again for the
  // accumulators at the end (rows padded by 8 floats: the two lane halves of a store, four rows
  // apart, hit different banks)
  constexpr int TILE = SUB * D;                                  // elements of one sub-tile
  constexpr int RING_BYTES = QS * RING * 2 * TILE * 2;
  // P per pair and 32-query block: lane l's 16 values as 16-byte pieces at [piece][l] (consecutive
  // lanes at consecutive 16 bytes: no bank conflict).  KB = 4 over the runs of more than 1024 key blocks: fp16,
  // two buffers (P of t + 1 is written while the dP wave reads P of t).  Else fp32, one buffer in the same
  // room: in the three-slot ring, whose iterations have one barrier, a pair's S wave overwrites P of t once its
  // dP wave has counted it as taken.  (fp32 for KB = 4 over all runs costs 4 %: 131072-token step 13.96 ->
  // 14.53 ms; elsewhere fp16 would gain 1..6 %, layer 32k of head_dim 64 871 -> 820 us, but dS would be
  // formed from 11 bits of P.)
  constexpr int PIECES = 4 * QB * (P32 ? 4 : 2);  // of 64 x 16 bytes, the four pairs' P of one sub-tile
  constexpr int P_BYTES = PIECES * 64 * 16 * (P32 ? 1 : 2);
  constexpr int ACC_STRIDE = D + 8;
  constexpr int ACC_BYTES = 8 * 32 * ACC_STRIDE * 4;
  // (tile-list mode: and this k-tile's q-tiles, q_tile | kind << 31, behind the hand-off)
  constexpr int LOOP_BYTES = RING_BYTES + P_BYTES + (LIST ? 4 * kMaxListQTiles : 0);
  constexpr int LDS_BYTES = LOOP_BYTES > ACC_BYTES ? LOOP_BYTES : ACC_BYTES;
  __shared__ __attribute__((aligned(16))) unsigned char raw[LDS_BYTES];
  __shared__ __attribute__((aligned(16))) float lse_s[QS][RING][SUB];
  __shared__ __attribute__((aligned(16))) float ndelta_s[QS][RING][SUB];  // -delta
  __shared__ __attribute__((aligned(16))) int32_t start_s[QS][RING][SUB];
  __shared__ int32_t wave_hits[LIST ? 8 : 1];
  __shared__ int32_t taken[4];  // fp32 hand-off, per pair: sub-tiles whose P the dP wave has read
  uint32_t* const qlist = (uint32_t*)(raw + RING_BYTES + P_BYTES);
  typedef __attribute__((address_space(3))) void* lds_void;

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
  const bool s_wave = w < 4;                // role of the wave
  const int pair = w & 3;
  const int kb = pair % KB, qs = pair / KB; // key block, stream
  __bf16* const ring = (__bf16*)raw + qs * RING * 2 * TILE;  // this stream's [RING][Q | dO]
  using P16 = std::conditional_t<P32, f32x4, h16x8>;  // 16 bytes of P
  P16* const px = (P16*)(raw + RING_BYTES) + pair * (PIECES / 4) * 64 + lane;
  auto q_tile = [&](int b) { return ring + b * 2 * TILE; };
  auto o_tile = [&](int b) { return ring + b * 2 * TILE + TILE; };

  // workgroup -> (run, 32 KB-key part of its k-tile, K/V head), heads fastest
  const int rest = blockIdx.x / a.hkv;
  const int g = blockIdx.x - rest * a.hkv;
  const int run_idx = rest / a.parts;
  const int part = rest - run_idx * a.parts;
  // Run mode: a k-major run from hsap_plan_runs (never empty).  Tile-list mode: k-tile run_idx of
  // chunk a.chunk; the workgroup gathers the tiles with that k_tile from the list (sorted by
  // q_tile) into LDS, in list order, 64 per wave per pass.
  const hsap_run run = LIST ? hsap_run{a.chunk, run_idx, 0, 0} : a.runs[run_idx];
  const int c = LIST ? a.chunk : a.tiles[run.first].chunk;
  int count = run.count;
  if constexpr (LIST) {
    int found = 0;
    for (int base = 0; base < a.num_tiles; base += 512) {
      const int i = base + tid;
      bool hit = false;
      uint32_t packed = 0u;
      if (i < a.num_tiles) {
        const hsap_tile t = a.tiles[i];
        hit = t.k_tile == run.tile;
        packed = (uint32_t)t.q_tile | ((uint32_t)t.kind << 31);
      }
      const uint64_t m = __builtin_amdgcn_ballot_w64(hit);
      const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
      if (lane == 0) wave_hits[w] = __popcll(m);
      __syncthreads();
      int off = found, all = 0;
      for (int x = 0; x < 8; ++x) {
        off += x < w ? wave_hits[x] : 0;
        all += wave_hits[x];
      }
      if (hit && off + rank < kMaxListQTiles) qlist[off + rank] = packed;
      found += all;
      __syncthreads();  // wave_hits is rewritten by the next pass; qlist is complete after the last
    }
    count = __builtin_amdgcn_readfirstlane(min(found, kMaxListQTiles));
    if (count == 0) return;  // no query of the shard reaches this k-tile in the chunk: nothing to add
  }
  const int64_t n = a.geom.n;
  const int64_t krow0 = (int64_t)run.tile * a.bn + part * (32 * KB);
  const int32_t gk = (int32_t)global_pos(a.geom, c, krow0 + 32 * kb + l32);  // this lane's key position
  const int64_t kvrow = (int64_t)c * n + krow0;                            // first row in the sharded K/V buffers

  // ---- LDS offsets (elements) as lane constants + compile-time immediates -------------
  // Row reads (row 32 qb + l32, chunk 2 kk + hi) of a swizzled [rows][D] tile:
  //   offset = 32 qb * D + rowoff[kk]
  // Transpose reads (rows rb + tr_row with rb = 8 k (mod 16), columns 32 mb + tr_col):
  //   offset = rb * D + troff[mb][k]      (the swizzle of rb + tr_row depends on k only)
  const int tr_row = 4 * hi + ((lane & 15) >> 2);
  const int tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  int rowoff[D / 16], troff[MB][2];
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) rowoff[kk] = swz<CPR>(l32, 16 * kk + 8 * hi);
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int k = 0; k < 2; ++k) troff[mb][k] = swz<CPR>(8 * k + tr_row, 32 * mb + tr_col) - 8 * k * D;

  const int nsub = a.bm / SUB;
  const int total = (a.group * count * nsub + QS - 1) / QS;  // iterations over the streams' sub-tiles
  uint32_t win0 = 0u, win1 = 0u;
  int win_lo = 0, win_hi = -1;
  // The run's q-tiles, packed one per lane (q_tile | kind << 31) in windows of 64 tiles, read
  // with v_readlane: the next sub-tile's address never waits on a memory load.  Window v lives
  // in win0 (v even) or win1 (v odd); sub-tiles visit the run's tiles in order once per query
  // head, so the window is reloaded when the tile index leaves it.
  auto load_window = [&](int v) {
    const int i = 64 * v + lane;
    uint32_t p = 0;
    if (i < count) {
      if constexpr (LIST) {
        p = qlist[i];
      } else {
        const hsap_tile t = a.tiles[run.first + i];
        p = (uint32_t)t.q_tile | ((uint32_t)t.kind << 31);
      }
    }
    if (v & 1) win1 = p;
    else win0 = p;
  };
  auto ensure_window = [&](int v) {  // v is the window of the next tile index needed
    if (v >= win_lo && v <= win_hi) return;
    load_window(v);
    if (v == win_hi + 1 && v - 1 >= win_lo) win_lo = v - 1;
    else win_lo = v;
    win_hi = v;
  };
  // Sub-tile position as counters (no division in the loop): query head h, tile index idx in the
  // run, SUB-row slice sb of the tile; with its position and kind once it has been loaded.  Stream qs
  // takes the slices qs, qs + QS, ... of every tile or, of tiles with fewer slices (64-row q-tiles,
  // four streams), slice qs % nsub of every other tile; there its last iteration lies past the run's
  // end when the tiles are odd in number: it moves the last sub-tile once more and leaves its
  // products out (`past`; P = 0 would turn an infinite dO of that sub-tile into NaN).
  struct Pos {
    int h, idx, sb;
    bool masked;
    int32_t gq0;
  };
  const bool past = QS > 2 && nsub < QS && qs >= nsub && (a.group * count) % 2 != 0;
  auto fold = [&](Pos p) {  // tile indexes past the run's end continue with the next query head
    if (p.idx >= count) {
      p.idx -= count;
      ++p.h;
      if (QS > 2 && p.idx >= count) {
        p.idx -= count;
        ++p.h;
      }
    }
    if (QS > 2 && p.h >= a.group) {
      p.h = a.group - 1;
      p.idx = count - 1;
    }
    return p;
  };
  auto advance = [&](Pos p) {
    if (QS <= 2 || nsub >= QS) {  // (a q-tile has at least 64 rows: two slices of 32)
      p.sb += QS;
      if (p.sb >= nsub) {
        p.sb -= nsub;
        ++p.idx;
      }
    } else {
      p.idx += QS / 2;
    }
    return fold(p);
  };
  auto tile_at = [&](const Pos& p) -> uint32_t {
    return __builtin_amdgcn_readlane(((p.idx >> 6) & 1) ? win1 : win0, p.idx & 63);
  };

  // Q and dO sub-tiles by direct-to-LDS transfers: instruction u of the stream's wave x fills chunk
  // positions p = WCH x + 64 u + lane of the swizzled tile; the lane's source is the chunk the
  // swizzle places there, a 32-bit byte offset from the sub-tile's scalar base (Q and dO rows have
  // the same stride)
  const int x = kb + (s_wave ? 0 : KB);
  using Offset = std::conditional_t<WIDE, uint64_t, uint32_t>;
  Offset gsrc[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int p = WCH * x + 64 * u + lane, row = p / CPR;
    gsrc[u] = 2u * ((Offset)row * a.hq * D + swz_chunk<CPR>(row, p % CPR) * 8);
  }
  auto stage = [&](const __bf16* src, __bf16* dst) {
    const uint32_t lds = (uint32_t)(uintptr_t)(lds_void)dst + (uint32_t)(WCH * x * 16);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if constexpr (WIDE)
        asm volatile("global_load_lds_dwordx4 %0, off" ::"v"((const char*)src + gsrc[u]), "{m0}"(lds + 64 * 16 * u));
      else
        asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(gsrc[u]), "s"(src), "{m0}"(lds + 64 * 16 * u));
  };
  // One role's whole run (S: K rows and dV; otherwise V rows and dK).  The two loops are separate
  // code, so each is one straight-line block per iteration for the compiler to order.
  auto work = [&](auto role) __attribute__((always_inline)) {
    constexpr bool S = decltype(role)::value;
    // this lane's key row of K (S) or V as MFMA B operands
    bf16x8 kv[D / 16];
    {
      const __bf16* src = S ? a.k : a.v;
      const int64_t off = ((kvrow + 32 * kb + l32) * a.hkv + g) * D + 8 * hi;
#pragma unroll
      for (int kk = 0; kk < D / 16; ++kk) kv[kk] = *(const bf16x8*)(src + off + 16 * kk);
    }
    f32x16 acc[MB];  // dV (S) or dK
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[mb] = f32x16{};

    float lreg = 0.f, dreg = 0.f;
    int32_t sreg = 0;
    const bool row_lane = S && kb == 0 && lane < SUB;  // this stream's lanes that bring the per-row values
    // the sub-tile's Q and dO into buffer buf (transfers), its LSE, delta and document starts into
    // registers of SUB lanes (written to LDS by store_sub)
    auto load_sub = [&](Pos& ps, int buf) {
      // (uniform across the wave, which the transfers' scalar bases need the compiler to know)
      const int h = __builtin_amdgcn_readfirstlane(g * a.group + ps.h);
      ensure_window(ps.idx >> 6);
      const uint32_t t = tile_at(ps);
      const int64_t q0 = __builtin_amdgcn_readfirstlane((int)(t & 0x7FFFFFFFu) * a.bm + ps.sb * SUB);
      ps.masked = (t >> 31) != 0;
      ps.gq0 = (int32_t)global_pos(a.geom, a.shard, q0);
      const int64_t base = (q0 * a.hq + h) * D;
      stage(a.q + base, q_tile(buf));
      stage(a.d_o + base, o_tile(buf));
      if (row_lane) {
        lreg = a.lse[(int64_t)h * n + q0 + lane];
        dreg = a.delta[(int64_t)h * n + q0 + lane];
        sreg = a.doc_start[ps.gq0 + lane];
      }
    };
    auto store_sub = [&](int buf) {
      if (row_lane) {
        lse_s[qs][buf][lane] = lreg == -__builtin_inff() ? __builtin_inff() : lreg * LOG2E;  // no key: P = 0
        ndelta_s[qs][buf][lane] = -dreg;
        start_s[qs][buf][lane] = sreg;
      }
    };

    // Scores of a sub-tile from its rows (buffer rb): S = Q K^T or dP = dO V^T into sp, the latter
    // accumulated onto -delta of each query (register j = 4 cq + e), so the chain ends with
    // dP - delta and dS takes one multiply per element.
    auto scores = [&](int rb, f32x16 (&sp)[QB]) __attribute__((always_inline)) {
      const __bf16* R = S ? q_tile(rb) : o_tile(rb);
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        bf16x8 ra[D / 16];
#pragma unroll
        for (int kk = 0; kk < D / 16; ++kk) ra[kk] = *(const bf16x8*)(R + 32 * qb * D + rowoff[kk]);
        if constexpr (S) {
          sp[qb] = f32x16{};
        } else {
          f32x16 init;
#pragma unroll
          for (int cq = 0; cq < 4; ++cq) {
            const f32x4 d4 = *(const f32x4*)(&ndelta_s[qs][rb][32 * qb + 8 * cq + 4 * hi]);
#pragma unroll
            for (int e = 0; e < 4; ++e) init[4 * cq + e] = d4[e];
          }
          sp[qb] = init;
        }
#pragma unroll
        for (int kk = 0; kk < D / 16; ++kk) sp[qb] = mfma32(ra[kk], kv[kk], sp[qb]);
      }
    };
    // P of a sub-tile (register j = 4 grp + e holds query q4 + e, q4 = 32 qb + 8 grp + 4 hi;
    // P = exp2(S * scale*log2e - LSE*log2e), masked in one uniform branch): in bf16 as this wave's
    // next A operand, in fp32 or fp16 to the dP wave.
    auto probs = [&](int rb, f32x16 (&sp)[QB]) __attribute__((always_inline)) {
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int grp = 0; grp < 4; ++grp) {
          const f32x4 l4 = *(const f32x4*)(&lse_s[qs][rb][32 * qb + 8 * grp + 4 * hi]);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            sp[qb][4 * grp + e] = fast_exp2(__builtin_fmaf(sp[qb][4 * grp + e], a.scale_log2, -l4[e]));
        }
    };
    auto hand_over = [&](int rb, int t, const Pos& ps, f32x16 (&sp)[QB], bf16x8 (&opnd)[QB][2])
                         __attribute__((always_inline)) {
      if (ps.masked) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
          for (int grp = 0; grp < 4; ++grp) {
            const int q4 = 32 * qb + 8 * grp + 4 * hi;
            const i32x4 s4 = *(const i32x4*)(&start_s[qs][rb][q4]);
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if ((uint32_t)(gk - s4[e]) > (uint32_t)(ps.gq0 + q4 + e - s4[e])) sp[qb][4 * grp + e] = 0.f;
          }
      }
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        if constexpr (P32) {
#pragma unroll
          for (int grp = 0; grp < 4; ++grp)
            px[(qb * 4 + grp) * 64] =
                f32x4{sp[qb][4 * grp], sp[qb][4 * grp + 1], sp[qb][4 * grp + 2], sp[qb][4 * grp + 3]};
        } else {
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            h16x8 ph;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const auto pk = __builtin_amdgcn_cvt_pkrtz(sp[qb][8 * half + 2 * i], sp[qb][8 * half + 2 * i + 1]);
              ph[2 * i] = pk[0];
              ph[2 * i + 1] = pk[1];
            }
            px[((t & 1) * PIECES + qb * 2 + half) * 64] = ph;
          }
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) opnd[qb][j >> 3][j & 7] = (__bf16)sp[qb][j];
      }
    };
    // dS = P (dP - delta) of sub-tile t (fp16: one mixed-precision multiply per element).  An fp32 P
    // counts as taken once it is read: a wave's LDS operations are carried out in the order they are
    // issued, which the empty asm keeps, so no wait stands between.
    auto take_over = [&](int t, const f32x16 (&sp)[QB], bf16x8 (&opnd)[QB][2]) __attribute__((always_inline)) {
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        if constexpr (P32) {
#pragma unroll
          for (int grp = 0; grp < 4; ++grp) {
            const f32x4 p = px[(qb * 4 + grp) * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int j = 4 * grp + e;
              opnd[qb][j >> 3][j & 7] = (__bf16)(p[e] * sp[qb][j]);
            }
          }
        } else {
          const h16x8 ph[2] = {px[((t & 1) * PIECES + qb * 2) * 64], px[((t & 1) * PIECES + qb * 2 + 1) * 64]};
#pragma unroll
          for (int j = 0; j < 16; ++j)
            opnd[qb][j >> 3][j & 7] = (__bf16)__builtin_fmaf((float)ph[j >> 3][j & 7], sp[qb][j], 0.f);
        }
      }
      if constexpr (P32 && RING == 3) {
        asm volatile("" ::: "memory");
        __hip_atomic_store(&taken[pair], t + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        asm volatile("" ::: "memory");
      }
    };
    auto taken_now = [&] { return __hip_atomic_load(&taken[pair], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
    // Gradient products of a sub-tile (buffer tb): dV += P^T dO or dK += dS^T Q, dO and Q read
    // transposed, 16 queries per MFMA
    auto products = [&](int tb, const bf16x8 (&opnd)[QB][2]) __attribute__((always_inline)) {
      const __bf16* T = S ? o_tile(tb) : q_tile(tb);
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const int rb = (32 * qb + 16 * half) * D;
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) {
            const bf16x8 bt = cat4(ds_read_tr16(T + rb + troff[mb][0]), ds_read_tr16(T + rb + 8 * D + troff[mb][1]));
            acc[mb] = mfma32(opnd[qb][half], bt, acc[mb]);
          }
        }
    };
    // prologue: the first sub-tiles staged, the scores of sub-tile 0
    if (P32 && S && lane == 0) taken[pair] = 0;
    ensure_window(0);
    Pos cur{0, 0, qs, false, 0};
    if (QS > 2 && nsub < QS) {
      cur.sb = qs % 2;
      cur.idx = qs / 2;
      cur = fold(cur);
    }
    Pos nx1 = advance(cur);
    load_sub(cur, 0);
    store_sub(0);
    if (RING == 3 && total > 1) {
      load_sub(nx1, 1);
      store_sub(1);
    }
    // The compiler does not see the waits inside asm statements: without a use of the K (or V) rows
    // here it would wait for their loads at their first use inside the loop, in every iteration,
    // and since the counter also counts the transfers, each iteration would wait for the next
    // sub-tiles before its first product.
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) asm volatile("" ::"v"(kv[kk]));
    asm volatile("s_waitcnt vmcnt(0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    f32x16 sp[QB];
    bf16x8 opnd[QB][2];  // A operands of the gradient products: P (S) or dS
    scores(0, sp);
    if constexpr (S) {
      probs(0, sp);
      hand_over(0, 0, cur, sp, opnd);
    }
    hsap_lds_barrier();  // P of sub-tile 0 is in LDS

    if constexpr (RING == 3) {
      // Iteration t: the gradient products of sub-tile t and the scores of sub-tile t + 1, while
      // sub-tile t + 2 is moved into the third buffer; one barrier.
      int b0 = 0;  // t % 3
      for (int t = 0; t + 1 < total; ++t) {
        const int b1 = b0 == 2 ? 0 : b0 + 1, b2 = b1 == 2 ? 0 : b1 + 1;
        Pos nx2 = advance(nx1);
        const bool more = t + 2 < total;
        if (more) load_sub(nx2, b2);  // buffer b2 was last read before the previous barrier
        if constexpr (S) {
          int32_t seen = P32 ? taken_now() : 0;
          products(b0, opnd);
          if constexpr (P32) {
            // P of t is taken at the start of the partner's iteration, before any barrier of its own:
            // mostly done by now, and the wait ends whatever the order of the two waves
            while (__builtin_amdgcn_readfirstlane(seen) <= t) seen = taken_now();
            asm volatile("" ::: "memory");
          }
          scores(b1, sp);
          probs(b1, sp);
          hand_over(b1, t + 1, nx1, sp, opnd);
        } else {
          // dS leaves sp, so the dP products of t + 1 go first: their row reads and the dS
          // arithmetic fill the shadow of the S wave's products, and dK follows (against dK first:
          // 131072-token step 14.71 -> 14.43 ms, 32768-token step 624 -> 615 us)
          take_over(t, sp, opnd);
          scores(b1, sp);
          products(b0, opnd);
        }
        if (more) store_sub(b2);
        // sub-tile t + 2 has landed and is staged; P of t + 1 is in LDS; buffer b0 is free
        asm volatile("s_waitcnt vmcnt(0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        nx1 = nx2;
        b0 = b1;
      }
      if (!past) {
        if constexpr (!S) take_over(total - 1, sp, opnd);
        products(b0, opnd);
      }
    } else {
      // Two buffers: sub-tile t + 1 moves into the buffer of t - 1 while the products of t run.
      for (int t = 0; t + 1 < total; ++t) {
        const int b0 = t & 1, b1 = b0 ^ 1;
        load_sub(nx1, b1);
        if constexpr (!S) take_over(t, sp, opnd);
        products(b0, opnd);
        store_sub(b1);
        asm volatile("s_waitcnt vmcnt(0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        scores(b1, sp);
        if constexpr (S) {
          probs(b1, sp);
          hand_over(b1, t + 1, nx1, sp, opnd);
        }
        hsap_lds_barrier();  // P of t + 1 is in LDS; every read of buffer b0 is done
        nx1 = advance(nx1);
      }
      if (!past) {
        if constexpr (!S) take_over(total - 1, sp, opnd);
        products((total - 1) & 1, opnd);
      }
    }

    // the accumulators to LDS, once no wave reads the ring or P any more
    hsap_lds_barrier();
    float* const mine = (float*)raw + w * 32 * ACC_STRIDE;
    const float mul = S ? 1.f : a.scale;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int j = 0; j < 16; ++j) mine[c_row(j, hi) * ACC_STRIDE + 32 * mb + l32] = acc[mb][j] * mul;
    hsap_lds_barrier();
  };
  if (s_wave) work(std::true_type{});
  else work(std::false_type{});

  // whole rows out: this workgroup owns rows [krow0, krow0 + 32 KB) of chunk c for K/V head g,
  // summed over the streams in order, 8 values per thread
  constexpr int OUT = 2 * 32 * KB * CPR;  // 8-value pieces: dV rows, then dK rows
#pragma unroll
  for (int i0 = 0; i0 < OUT; i0 += 512) {
    const int i = i0 + tid;
    if (OUT % 512 != 0 && i >= OUT) break;
    const int tensor = i / (32 * KB * CPR), r = i / CPR % (32 * KB), col = 8 * (i % CPR);
    const float* src = (const float*)raw + ((4 * tensor + r / 32) * 32 + (r & 31)) * ACC_STRIDE + col;
    f32x4 lo = *(const f32x4*)src, up = *(const f32x4*)(src + 4);
#pragma unroll
    for (int s = 1; s < QS; ++s) {
      lo += *(const f32x4*)(src + s * KB * 32 * ACC_STRIDE);
      up += *(const f32x4*)(src + s * KB * 32 * ACC_STRIDE + 4);
    }
    const int64_t idx = ((kvrow + r) * a.hkv + g) * D + col;
    if constexpr (BF16OUT) {
      __bf16* dst = (tensor ? a.dk16 : a.dv16) + idx;
      const bf16x8 val{(__bf16)lo[0], (__bf16)lo[1], (__bf16)lo[2], (__bf16)lo[3],
                       (__bf16)up[0], (__bf16)up[1], (__bf16)up[2], (__bf16)up[3]};
      if (a.wide_kv) {
        *(bf16x8*)dst = val;
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) dst[e] = val[e];
      }
    } else {
      float* dst = (tensor ? a.dk : a.dv) + idx;
      if (a.wide_kv) {
        *(f32x4*)dst += lo;
        *(f32x4*)(dst + 4) += up;
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) dst[e] += e < 4 ? lo[e] : up[e - 4];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// dQ kernel: one workgroup per (q-major run, query head), shaped like the
// forward.  Wave w owns 32 query rows; in the transposed orientation
// S^T = K Q^T and dP^T = V dO^T a lane holds one query, so its LSE and delta
// are scalars of the lane.  Per step of 64 keys:
//   P^T = exp2(S^T * scale*log2e - LSE*log2e), dS^T = P^T o (dP^T - delta),
//   dQ^T += K^T dS^T (K^T read transposed from the [key][d] tile).
// A run may span several chunks (tile by tile), so one run per q-tile covers
// every chunk; dQ stays in registers for the whole run and is written once at
// the end, by the q-tile's only run: a plain read-add-write of the fp32
// accumulator, or a store of the final bf16 value.  KS key streams (small grids,
// key_streams()): WAVES x KS waves, stream ks with a ring and a sum of its own
// over the steps ks, ks + KS, ..., added in LDS in stream order.
// ---------------------------------------------------------------------------
template <int D, int BN, int WAVES, bool BF16OUT, bool LIST = false, int KS = 1>
__global__ __launch_bounds__(64 * WAVES * KS, 2) void attn_bwd_dq_kernel(BwdArgs a) {
  static_assert(!LIST || !BF16OUT, "the tile-list mode accumulates fp32");
  constexpr int KB = 64;                     // keys per step
  constexpr int SUBS = BN / KB;
  constexpr int CPR = D / 8;
  constexpr int MB = D / 32;
  constexpr int CHUNKS = KB * CPR;           // 16-byte chunks per K (or V) step
  static_assert(KS == 1 || WAVES * KS <= 8, "at most eight waves with key streams");
  constexpr float LOG2E = 1.44269504088896340736f;
  constexpr float NEG_INF = -__builtin_inff();
  // the streams' rings of swizzled [key][d] tiles; with several streams used again for their sums
  constexpr int TILE = KB * D;
  __shared__ __attribute__((aligned(16))) __bf16 rings[KS][4 * TILE];

  const int tid = threadIdx.x;
  const int lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
  // wave -> (32-row slice of the q-tile, key stream)
  const int w = KS == 1 ? tid >> 6 : __builtin_amdgcn_readfirstlane(tid >> 6) % WAVES;
  const int ks = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6) / WAVES;
  auto Ks = [&](int slot) { return &rings[ks][slot * TILE]; };
  auto Vs = [&](int slot) { return &rings[ks][(2 + slot) * TILE]; };
  int run_idx, h;
  run_and_head(blockIdx.x, a.hq, a.hkv, run_idx, h);
  // LIST: the tile-list mode, this workgroup's q-tile found in one chunk's list (last q-tiles first:
  // under the causal mask they have the most keys)
  if (LIST) run_idx = (int)(a.geom.n / (32 * WAVES)) - 1 - run_idx;
  const hsap_run run = LIST ? q_tile_run(a.tiles, a.num_tiles, run_idx, lane) : a.runs[run_idx];
  const int g = h / a.group;
  const int64_t n = a.geom.n;
  const int64_t qrow = (int64_t)run.tile * (32 * WAVES) + 32 * w + l32;
  if (run.count == 0) {  // no key for this q-tile: dQ = 0
    if (BF16OUT) {
      bf16x4* dst = (bf16x4*)(a.dq16 + (qrow * a.hq + h) * D + 4 * hi);
#pragma unroll
      for (int e = 0; e < D / 8; ++e) dst[2 * e] = bf16x4{};
    }
    return;
  }
  const int32_t gq = (int32_t)global_pos(a.geom, a.shard, qrow);
  const DocWindow docw = doc_window(a.doc_start, a.cu, a.num_docs, gq, lane);
  const float lse_raw = a.lse[(int64_t)h * n + qrow];
  const float lse2 = lse_raw == NEG_INF ? __builtin_inff() : lse_raw * LOG2E;  // no key: P = 0
  bf16x8 qf[D / 16], of[D / 16];
  float dlt;
  {
    const int64_t off = (qrow * a.hq + h) * D + 8 * hi;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) {
      qf[kk] = *(const bf16x8*)(a.q + off + 16 * kk);
      of[kk] = *(const bf16x8*)(a.d_o + off + 16 * kk);
    }
    if (a.o) {
      // the backward preprocess for this row, delta = sum_d dO O, summed in the order of
      // hsap_attn_bwd_preprocess (so both give the same bits): a sum per 8-element chunk, then a
      // tree over the chunk index from its highest bit down.  The lane holds chunks 2 kk + hi, so
      // the tree runs over kk within the lane and ends with the lane l ^ 32 (chunk bit 0).
      float p[D / 16];
#pragma unroll
      for (int kk = 0; kk < D / 16; ++kk) {
        const bf16x8 ov = *(const bf16x8*)(a.o + off + 16 * kk);
        p[kk] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) p[kk] = __builtin_fmaf((float)ov[e], (float)of[kk][e], p[kk]);
      }
#pragma unroll
      for (int wdt = D / 32; wdt >= 1; wdt >>= 1)
#pragma unroll
        for (int kk = 0; kk < wdt; ++kk) p[kk] = p[kk] + p[kk + wdt];
      dlt = p[0] + __shfl_xor(p[0], 32);
      if (hi == 0 && ks == 0) a.delta_out[(int64_t)h * n + qrow] = dlt;  // read by the dK/dV kernel, launched after
    } else {
      dlt = a.delta[(int64_t)h * n + qrow];
    }
  }
  f32x16 ndlt;
#pragma unroll
  for (int j = 0; j < 16; ++j) ndlt[j] = -dlt;
  const int tr_row = 4 * hi + ((lane & 15) >> 2);
  const int tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  int rowoff[D / 16], troff[MB][2];
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) rowoff[kk] = swz<CPR>(l32, 16 * kk + 8 * hi);
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int k = 0; k < 2; ++k) troff[mb][k] = swz<CPR>(8 * k + tr_row, 32 * mb + tr_col) - 8 * k * D;

  const int64_t rstride = (int64_t)a.hkv * D;
  // Stream ks takes the steps ks, ks + KS, ... of the run: its step i is the run's step KS i + ks.
  const int run_steps = run.count * SUBS;
  const int total = KS == 1 ? run_steps : (run_steps - ks + KS - 1) / KS;  // this stream's steps
  auto at = [&](int i) { return KS == 1 ? i : KS * i + ks; };
  // The run's tile descriptors, packed one per lane (k_tile | chunk << 23 | kind << 31) in windows
  // of 64 tiles (window v in win0 or win1 by parity), read with v_readlane: the loop issues no
  // vector load besides the transfers (one would wait for every transfer in flight).
  uint32_t win0 = 0u, win1 = 0u;
  int win_hi = -1;
  auto load_window = [&](int v) {
    const int i = 64 * v + lane;
    uint32_t p = 0;
    if (i < run.count) {
      const hsap_tile t = a.tiles[run.first + i];
      p = (uint32_t)t.k_tile | ((uint32_t)t.chunk << 23) | ((uint32_t)t.kind << 31);
    }
    if (v & 1) win1 = p;
    else win0 = p;
    win_hi = v;
  };
  auto tile_at = [&](int s) -> uint32_t {
    const int idx = at(s) / SUBS;
    return __builtin_amdgcn_readlane(((idx >> 6) & 1) ? win1 : win0, idx & 63);
  };
  auto chunk_of = [](uint32_t p) { return (int32_t)((p >> 23) & 0xFFu); };
  auto step_row0 = [&](uint32_t p, int s) { return (int64_t)(p & 0x7FFFFFu) * BN + (at(s) % SUBS) * KB; };
  // the step's first row in the sharded K/V buffers: chunk of the tile, K/V head g
  auto step_off = [&](uint32_t p, int s) { return (((int64_t)chunk_of(p) * n + step_row0(p, s)) * a.hkv + g) * D; };
  load_window(0);

  // K and V steps go from global memory straight into LDS (global_load_lds) in a two-slot ring of
  // swizzled tiles: the next step's transfers are issued at the start of a step into the slot the
  // previous step read, and have landed at the step's closing barrier.  Instruction u of wave w
  // fills chunk positions p = WCH w + 64 u + lane; the lane's source is the chunk the swizzle
  // places there, a 32-bit byte offset from the step's scalar base.
  constexpr int WCH = CHUNKS / WAVES, U = WCH / 64;
  static_assert(WCH % 64 == 0, "a wave moves whole instructions of a tile");
  uint32_t gsrc[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int p = WCH * w + 64 * u + lane, row = p / CPR;
    gsrc[u] = (uint32_t)((row * rstride + swz_chunk<CPR>(row, p % CPR) * 8) * 2);
  }
  typedef __attribute__((address_space(3))) void* lds_void;
  const int wu = __builtin_amdgcn_readfirstlane(w);
  auto stage = [&](const __bf16* src, __bf16* dst) {
    const uint32_t lds = (uint32_t)(uintptr_t)(lds_void)dst + (uint32_t)(WCH * wu * 16);
#pragma unroll
    for (int u = 0; u < U; ++u)
      asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(gsrc[u]), "s"(src), "{m0}"(lds + 64 * 16 * u));
  };

  f32x16 dq[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) dq[mb] = f32x16{};

  if (KS == 1 || total > 0) {
    const int64_t off = step_off(tile_at(0), 0);
    stage(a.k + off, Ks(0));
    stage(a.v + off, Vs(0));
  }
  // The compiler does not see the waits inside asm statements: without a use of Q and dO here it
  // would wait for their loads at their first use inside the loop, in every step, and since the
  // counter also counts the step's transfers, each step would wait for the next step's K and V.
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) asm volatile("" ::"v"(qf[kk]), "v"(of[kk]));
  const int32_t qstart = doc_window_start(a.cu, a.num_docs, docw, gq);
  const uint32_t span = (uint32_t)(gq - qstart);
  if (a.start_out && h == 0 && hi == 0 && ks == 0) a.start_out[gq] = qstart;  // read by the dK/dV kernel, launched after
  asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");

  // one 64-key step from slot PAR (= s % 2, a compile-time constant, so every slot address is an
  // immediate); the next step's transfers go to the other slot
  auto step = [&](int s, auto par) __attribute__((always_inline)) {
    constexpr int PAR = decltype(par)::value;
    if (s + 1 < total && (at(s + 1) / SUBS) >> 6 > win_hi) load_window(win_hi + 1);
    const uint32_t tile = tile_at(s);
    if (s + 1 < total) {
      const int64_t off = step_off(tile_at(s + 1), s + 1);
      stage(a.k + off, Ks(PAR ^ 1));
      stage(a.v + off, Vs(PAR ^ 1));
    }
    const __bf16* K = Ks(PAR);
    const __bf16* V = Vs(PAR);
    // Masked tile: a step whose keys no query of the wave may see contributes nothing (skipped);
    // one whose keys every query of the wave may see needs no per-element mask.
    bool live = true, need_mask = false;
    int32_t rel0 = 0;  // key row of register j: rel0 + 32 nb + c_row(j, 0)
    if (tile >> 31) {
      const int32_t r = (int32_t)global_pos(a.geom, chunk_of(tile), step_row0(tile, s)) - qstart;
      const bool none = r > (int32_t)span || r + (KB - 1) < 0;
      const bool all = r >= 0 && r + (KB - 1) <= (int32_t)span;
      live = __builtin_amdgcn_ballot_w64(!none) != 0;
      need_mask = live && __builtin_amdgcn_ballot_w64(!all) != 0;
      rel0 = r + 4 * hi;
    }
    if (live) {
#pragma unroll
      for (int nb = 0; nb < KB / 32; ++nb) {
        // dP^T accumulates onto -delta (ndlt), so the chain ends with dP^T - delta
        f32x16 st{}, dpt = ndlt;
#pragma unroll
        for (int kk = 0; kk < D / 16; ++kk) {
          st = mfma32(*(const bf16x8*)(K + 32 * nb * D + rowoff[kk]), qf[kk], st);
          dpt = mfma32(*(const bf16x8*)(V + 32 * nb * D + rowoff[kk]), of[kk], dpt);
        }
        float p[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) p[j] = fast_exp2(__builtin_fmaf(st[j], a.scale_log2, -lse2));
        if (need_mask) {  // uniform branch: the mask costs nothing on steps that need none
#pragma unroll
          for (int j = 0; j < 16; ++j)
            if ((uint32_t)(rel0 + (32 * nb + c_row(j, 0))) > span) p[j] = 0.f;
        }
        bf16x8 sb[2];
#pragma unroll
        for (int j = 0; j < 16; ++j) sb[j >> 3][j & 7] = (__bf16)(p[j] * dpt[j]);
        // dQ^T += K^T dS^T, 16 keys per MFMA
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const int rb = (32 * nb + 16 * half) * D;
#pragma unroll
          for (int mb = 0; mb < MB; ++mb) {
            const bf16x8 ka = cat4(ds_read_tr16(K + rb + troff[mb][0]), ds_read_tr16(K + rb + 8 * D + troff[mb][1]));
            dq[mb] = mfma32(ka, sb[half], dq[mb]);
          }
        }
      }
    }
    // every read of slot PAR is done and the transfers into slot PAR ^ 1 have landed
    asm volatile("s_waitcnt vmcnt(0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  };
  if constexpr (KS == 1) {
    for (int s = 0; s < total; s += 2) {
      step(s, std::integral_constant<int, 0>{});
      if (s + 1 < total) step(s + 1, std::integral_constant<int, 1>{});
    }
  } else {
    // every stream takes part in the barriers of the longest one (the first)
    const int most = (run_steps + KS - 1) / KS;
    for (int s = 0; s < most; s += 2) {
      if (s < total) step(s, std::integral_constant<int, 0>{});
      else vm_wait_barrier<0>();
      if (s + 1 < most) {
        if (s + 1 < total) step(s + 1, std::integral_constant<int, 1>{});
        else vm_wait_barrier<0>();
      }
    }
    // the streams' sums to LDS (register by register; the loop ended with a barrier and no transfer is
    // in flight), added in stream order
    float* const res = (float*)rings;
    static_assert(KS * 4 * TILE * 2 >= (KS - 1) * WAVES * (D / 2) * 256, "room for the streams' sums");
    if (ks > 0) {
      float* const mine = res + ((ks - 1) * WAVES + w) * (D / 2) * 64 + lane;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int j = 0; j < 16; ++j) mine[(16 * mb + j) * 64] = dq[mb][j];
    }
    hsap_lds_barrier();
    if (ks > 0) return;
    for (int x = 1; x < KS; ++x) {
      const float* const other = res + ((x - 1) * WAVES + w) * (D / 2) * 64 + lane;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int j = 0; j < 16; ++j) dq[mb][j] += other[(16 * mb + j) * 64];
    }
  }

  // dQ^T: this lane's query, d = 32 mb + 8 grp + 4 hi + e for register j = 4 grp + e
  const int64_t base = (qrow * a.hq + h) * D + 4 * hi;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int grp = 0; grp < 4; ++grp) {
      const f32x4 val{dq[mb][4 * grp] * a.scale, dq[mb][4 * grp + 1] * a.scale, dq[mb][4 * grp + 2] * a.scale,
                      dq[mb][4 * grp + 3] * a.scale};
      if (BF16OUT) {
        *(bf16x4*)(a.dq16 + base + 32 * mb + 8 * grp) = bf16x4{(__bf16)val[0], (__bf16)val[1], (__bf16)val[2],
                                                               (__bf16)val[3]};
      } else {
        f32x4* dst = (f32x4*)(a.dq + base + 32 * mb + 8 * grp);
        *dst = *dst + val;
      }
    }
}

template <int D, int KB, bool BF16OUT, bool LIST, bool WIDE = false, bool P32 = KB < 4 || LIST>
static hsap_status launch_dkdv_kb(BwdArgs a, int64_t num_runs, hipStream_t stream) {
  a.parts = a.bn / (32 * KB);
  const int64_t blocks = num_runs * a.parts * a.hkv;
  if (blocks > INT32_MAX) HSAP_FAIL(HSAP_ERR_INVALID_ARG, "too many runs x heads");
  hipLaunchKernelGGL((attn_bwd_dkdv_kernel<D, KB, BF16OUT, LIST, WIDE, P32>), dim3((unsigned)blocks), dim3(512), 0, stream, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) HSAP_FAIL(HSAP_ERR_HIP, "attn_bwd_dkdv launch: %s", hipGetErrorString(e));
  return HSAP_OK;
}

// Key blocks of 32, times K/V heads, that the shard's queries can reach under the causal mask (all their
// documents being one): per sequence, the k-tiles up to the shard's last row.
static int64_t reachable_key_blocks(const hsap_attn_desc& d, const Geom& g) {
  const int64_t keys = (g.layout == HSAP_LAYOUT_CONTIGUOUS ? d.shard.shard_id + 1 : 2 * g.P - d.shard.shard_id) * g.m;
  return g.B * ((keys + d.shard.block_n - 1) / d.shard.block_n) * (d.shard.block_n / 32) * d.heads_kv;
}

// Most key blocks of 32 a dK/dV workgroup can take.
static int most_key_blocks(const hsap_attn_desc& d) {
  // (a 64-row sub-tile has to fit 32-bit byte offsets)
  return d.head_dim == 128 && d.shard.block_n == 128 && (int64_t)d.heads_q * d.head_dim * 64 <= INT32_MAX ? 4 : 2;
}

// Key blocks of 32 per dK/dV workgroup (one workgroup per CU is resident, at head_dim 64 two of 64 keys).
// Fewer key blocks per workgroup give more, shorter workgroups at more staging traffic per product,
// which pays while the grid leaves the chip idle.  In the entry points the choice depends on the descriptor alone --
// the key blocks the shard can reach (tile-list call: those of its chunk) -- so that calls over the same tiles give
// the same bits however their lists are cut and whichever other tiles share the call.  Over 600 random
// backwards (dQ included; geometric mean of the gain against one wave per 32 keys at 64-key tiles, 128
// keys per workgroup at 128-key tiles; in brackets the worst of them):
//   128-key tiles, 128 or 32 keys a workgroup:  32 up to 512 reachable blocks 1.21 (0.97), 640 1.22 (0.97), 768 1.23
//     (0.86), 1024 1.22 (0.75).  (64 keys from 513 to 1024 blocks: down to 0.86, two workgroups in turn on most CUs)
//   64-key tiles, 64 or 32 keys:  512 blocks 1.44 / 1.51 at head_dim 128 / 64, 768 1.45 / 1.53 (0.98), 1024 1.45 / 1.53,
//     1536 1.44 / 1.52 (0.90)
// Tile-list calls at one causal document, head_dim 128 (us for 128 / 64 / 32 keys): 512 blocks 111.9 / 84.1 / 62.4,
// 1024 blocks 115.4 / 98.9 / 120.2, 2048 blocks 152.3 / 194.2 / 247.3; head_dim 64 (64 / 32 keys): 512 blocks
// 66.3 / 46.2, 1024 blocks 71.5 / 88.6.
static int key_blocks(const hsap_attn_desc& d, int64_t blocks) {
  return blocks <= (d.shard.block_n == 128 ? 640 : 768) ? 1 : most_key_blocks(d);
}

static int list_key_blocks(const hsap_attn_desc& d, int64_t blocks) {
  return blocks <= 512 ? 1 : blocks <= 1024 ? 2 : most_key_blocks(d);
}

// Up to this many key blocks 128 keys per workgroup take P in fp32, as fewer keys do.
constexpr int64_t kFp32Blocks = 1024;

// The same for all k-major runs of a plan, whose lengths the executor has on the host: the choice of least estimated
// time, sqrt(chain^2 + work^2), where the chain is that of the longest workgroup or, beyond one workgroup per slot, of
// the two that share the last slot, and the work is per slot.  The descriptor's choice stands unless another saves
// 0.5 us.  Fitted over 2500 random backwards (20..2000 us) run with every choice, and within 0.2 % of the best of them
// in the geometric mean.  The whole backward's gain against one wave per 32 keys (64-key tiles) or 128 keys per
// workgroup (128-key tiles), by the descriptor / by the plan (the worst of the latter): 128-key tiles 1.21 / 1.27
// (0.96), 64-key tiles at head_dim 128 1.41 / 1.44 (0.93), at 64 1.50 / 1.56 (1.05).  What the descriptor does not show is
// how few k-tiles of those in reach have tiles: 544 -> 312 us (716 tiles, 8 heads of 64 over one, 26880 tokens over 7).
int plan_key_blocks(const hsap_attn_desc& d, const Geom& g, const hsap_run* runs, int64_t num_runs, int64_t num_tiles) {
  struct Cost {
    double step, wave, work, fixed;  // us: 32 rows of a chain; per slot a workgroup, and 32 rows; a constant
  };
  const int by_desc = key_blocks(d, reachable_key_blocks(d, g)), most = most_key_blocks(d);
  const int64_t blocks = num_runs * (d.shard.block_n / 32) * d.heads_kv;
  if (num_runs <= 0) return by_desc;
  const double slices = (double)(d.heads_q / d.heads_kv) * d.shard.block_m / 32;  // 32-row slices per q-tile of a run
  auto time = [&](int kb) {
    const Cost c = d.head_dim == 64        ? (kb == 1 ? Cost{0.20, 2.23, 0.241, -0.27} : Cost{0.504, 0.0, 0.448, 0.0})
                   : d.shard.block_n == 64 ? (kb == 1 ? Cost{0.325, 2.23, 0.494, -0.63} : Cost{0.605, 0.0, 0.814, 0.0})
                   : kb == 1               ? Cost{0.271, 3.32, 0.381, -2.2}
                   : kb == 2               ? Cost{0.543, 2.38, 0.579, -1.15}
                   : blocks <= kFp32Blocks ? Cost{0.897, 0.0, 0.758, -0.44}
                                           : Cost{0.74, 0.0, 0.696, 0.0};
    const int64_t slots = kComputeUnits * (d.head_dim == 64 && kb == 2 ? 2 : 1);
    const int64_t each = (int64_t)(d.shard.block_n / (32 * kb)) * d.heads_kv;  // workgroups per run (longest runs first)
    int64_t chain = runs[0].count;
    if (num_runs * each > slots) chain = std::max<int64_t>(chain, runs[(slots - 1) / each].count + runs[slots / each].count);
    const double a = c.step * slices * chain;
    const double b = (c.work * slices * num_tiles + c.wave * num_runs) * each / slots;
    return std::sqrt(a * a + b * b) + c.fixed;
  };
  int best = by_desc;
  double least = time(by_desc) - 0.5;
  for (int kb = 1; kb <= most; kb *= 2) {
    if (kb == by_desc) continue;
    const double t = time(kb);
    if (t < least) {
      least = t;
      best = kb;
    }
  }
  return best;
}

template <bool BF16OUT, bool LIST = false>
static hsap_status launch_dkdv(const BwdArgs& a, int d, int kb, int64_t blocks, int64_t num_runs, hipStream_t stream) {
  if ((int64_t)a.hq * d * 32 > INT32_MAX)
    return d == 64 ? launch_dkdv_kb<64, 2, BF16OUT, LIST, true>(a, num_runs, stream)
                   : launch_dkdv_kb<128, 2, BF16OUT, LIST, true>(a, num_runs, stream);
  if (d == 64) {
    if (kb == 1) return launch_dkdv_kb<64, 1, BF16OUT, LIST>(a, num_runs, stream);
    return launch_dkdv_kb<64, 2, BF16OUT, LIST>(a, num_runs, stream);
  }
  if (kb == 1) return launch_dkdv_kb<128, 1, BF16OUT, LIST>(a, num_runs, stream);
  if (kb == 2) return launch_dkdv_kb<128, 2, BF16OUT, LIST>(a, num_runs, stream);
  if (blocks <= kFp32Blocks) return launch_dkdv_kb<128, 4, BF16OUT, LIST, false, true>(a, num_runs, stream);
  return launch_dkdv_kb<128, 4, BF16OUT, LIST>(a, num_runs, stream);
}

template <int D, int BN, int WAVES, bool BF16OUT, bool LIST, int KS>
static hsap_status launch_dq_ks(const BwdArgs& a, int64_t num_runs, hipStream_t stream) {
  const int64_t blocks = num_runs * a.hq;
  if (blocks > INT32_MAX) HSAP_FAIL(HSAP_ERR_INVALID_ARG, "too many runs x heads");
  hipLaunchKernelGGL((attn_bwd_dq_kernel<D, BN, WAVES, BF16OUT, LIST, KS>), dim3((unsigned)blocks),
                     dim3(64 * WAVES * KS), 0, stream, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) HSAP_FAIL(HSAP_ERR_HIP, "attn_bwd_dq launch: %s", hipGetErrorString(e));
  return HSAP_OK;
}

template <int D, int BN, int WAVES, bool BF16OUT, bool LIST = false>
static hsap_status launch_dq(const BwdArgs& a, int64_t num_runs, hipStream_t stream) {
  if constexpr (WAVES < 8) {
    const int ks = key_streams(D, 32 * WAVES, a.geom.n / (32 * WAVES) * a.hq, LIST ? a.geom.ns : a.geom.Ns);
    if constexpr (D == 64 && WAVES == 2)
      if (ks == 4) return launch_dq_ks<D, BN, WAVES, BF16OUT, LIST, 4>(a, num_runs, stream);
    if (ks >= 2) return launch_dq_ks<D, BN, WAVES, BF16OUT, LIST, 2>(a, num_runs, stream);
  }
  return launch_dq_ks<D, BN, WAVES, BF16OUT, LIST, 1>(a, num_runs, stream);
}

// Packed tile descriptors of the dQ kernel: chunks below 256, k-tiles below 2^23.
constexpr int kMaxDqChunks = 256;
constexpr int64_t kMaxDqKTiles = int64_t(1) << 23;

}  // namespace hsap

// (head_dim, BM, BN) combinations with both backward kernels: the dK/dV kernel takes any BM that is a multiple
// of 64 (its sub-tiles have 64 or 32 rows) and BN = 64 or, at head_dim 128, 128; the dQ kernel BM = 32 x waves.
bool hsap::backward_supported(const hsap_attn_desc* desc) {
  const int bm = desc->shard.block_m, bn = desc->shard.block_n, d = desc->head_dim;
  const bool dkdv_ok = bm % 64 == 0 && ((d == 128 && (bn == 128 || bn == 64)) || (d == 64 && bn == 64));
  const bool dq_ok = (bm == 128 || bm == 64 || (bm == 256 && d == 128)) && (bn == 128 || bn == 64);
  return dkdv_ok && dq_ok;
}

namespace hsap {

// shared checks and dispatch of the fp32-accumulating and the bf16-storing backward
template <bool BF16OUT>
// o == NULL: delta and doc_start are inputs.  Otherwise the dQ kernel computes delta from o and d_o into
// delta_out and the rows' document starts from cu into doc_start (as the forwards find them), and the
// dK/dV kernel (launched after it) reads both there.
static hsap_status backward(const hsap_attn_desc* desc, const void* q, const void* k, const void* v, const void* d_o,
                            const void* o, const float* lse, const float* delta, float* delta_out,
                            const int32_t* cu, int32_t num_docs, const int32_t* doc_start, const hsap_tile* tiles_k, const hsap_run* runs_k,
                            int64_t num_runs_k, const hsap_tile* tiles_q, const hsap_run* runs_q,
                            int64_t num_runs_q, void* dq, void* dk, void* dv, int kb, hipStream_t s) {
  Geom geom;
  hsap_status st = check_attn(desc, &geom);
  if (st != HSAP_OK) return st;
  if (num_runs_k < 0 || num_runs_q < 0) HSAP_FAIL(HSAP_ERR_INVALID_ARG, "negative run count");
  const int bm = desc->shard.block_m, bn = desc->shard.block_n, d = desc->head_dim;
  if (!backward_supported(desc))
    HSAP_FAIL(HSAP_ERR_UNSUPPORTED, "no backward kernel for head_dim=%d BM=%d BN=%d", d, bm, bn);
  if ((int64_t)desc->heads_kv * d * 64 > INT32_MAX) HSAP_FAIL(HSAP_ERR_UNSUPPORTED, "heads_kv too large");
  // the dQ kernel packs a tile descriptor as k_tile | chunk << 23 | kind << 31
  if (num_runs_q > 0 && (geom.P > kMaxDqChunks || geom.n / bn >= kMaxDqKTiles))
    HSAP_FAIL(HSAP_ERR_UNSUPPORTED, "the dQ kernel needs sp_degree <= %d and fewer than 2^23 k-tiles per chunk "
              "(sp_degree %d)", kMaxDqChunks, geom.P);
  if (num_runs_k == 0 && num_runs_q == 0) return HSAP_OK;
  if (!q || !k || !v || !d_o || !lse || !(o ? delta_out : delta) || !doc_start || !dq || !dk || !dv ||
      (num_runs_k > 0 && (!tiles_k || !runs_k)) || (num_runs_q > 0 && (!tiles_q || !runs_q)))
    HSAP_FAIL(HSAP_ERR_INVALID_ARG, "NULL pointer argument");
  if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)d_o | (uintptr_t)o) & 15)
    HSAP_FAIL(HSAP_ERR_INVALID_ARG, "q, k, v, d_o and o must be 16-byte aligned");
  if (o && num_runs_k > 0 && num_runs_q == 0)
    HSAP_FAIL(HSAP_ERR_INVALID_ARG, "delta from o needs the q-major runs (the dQ kernel computes it)");
  if ((uintptr_t)dq & (BF16OUT ? 7 : 15))
    HSAP_FAIL(HSAP_ERR_INVALID_ARG, "dq must be %d-byte aligned", BF16OUT ? 8 : 16);
  BwdArgs a = {};
  a.q = (const __bf16*)q;
  a.k = (const __bf16*)k;
  a.v = (const __bf16*)v;
  a.d_o = (const __bf16*)d_o;
  a.lse = lse;
  a.delta = o ? delta_out : delta;
  a.o = (const __bf16*)o;
  a.delta_out = delta_out;
  a.doc_start = doc_start;
  if (o) {
    a.cu = cu;
    a.num_docs = num_docs;
    a.start_out = const_cast<int32_t*>(doc_start);
  }
  if (BF16OUT) {
    a.dq16 = (__bf16*)dq;
    a.dk16 = (__bf16*)dk;
    a.dv16 = (__bf16*)dv;
  } else {
    a.dq = (float*)dq;
    a.dk = (float*)dk;
    a.dv = (float*)dv;
  }
  a.geom = geom;
  a.shard = desc->shard.shard_id;
  a.hq = desc->heads_q;
  a.hkv = desc->heads_kv;
  a.group = desc->heads_q / desc->heads_kv;
  a.bm = bm;
  a.bn = bn;
  a.wide_kv = (((uintptr_t)dk | (uintptr_t)dv) & 15) == 0;
  a.scale = desc->softmax_scale;
  a.scale_log2 = desc->softmax_scale * 1.44269504088896340736f;
  if (num_runs_q > 0) {
    a.tiles = tiles_q;
    a.runs = runs_q;
#define HSAP_DQ_CASE(D_, BN_, W_) \
  if (d == D_ && bn == BN_ && bm == 32 * W_) st = launch_dq<D_, BN_, W_, BF16OUT>(a, num_runs_q, s);
    HSAP_DQ_CASE(128, 128, 8)
    else HSAP_DQ_CASE(128, 64, 8)
    else HSAP_DQ_CASE(128, 128, 4)
    else HSAP_DQ_CASE(128, 64, 4)
    else HSAP_DQ_CASE(128, 128, 2)
    else HSAP_DQ_CASE(128, 64, 2)
    else HSAP_DQ_CASE(64, 128, 4)
    else HSAP_DQ_CASE(64, 64, 4)
    else HSAP_DQ_CASE(64, 128, 2)
    else HSAP_DQ_CASE(64, 64, 2)
#undef HSAP_DQ_CASE
    if (st != HSAP_OK) return st;
    a.o = nullptr;  // the dK/dV kernel reads delta
  }
  if (num_runs_k > 0) {
    a.tiles = tiles_k;
    a.runs = runs_k;
    // (kb: the executor's choice for its plan, whose runs these are)
    const int64_t blocks = kb > 0 ? num_runs_k * (bn / 32) * desc->heads_kv : reachable_key_blocks(*desc, geom);
    st = launch_dkdv<BF16OUT>(a, d, kb > 0 ? kb : key_blocks(*desc, blocks), blocks, num_runs_k, s);
    if (st != HSAP_OK) return st;
  }
  return HSAP_OK;
}

// hsap_partial_attn_bwd: both kernels in tile-list mode over one chunk's tiles (fp32 accumulators).
static hsap_status backward_tile_list(const hsap_attn_desc* desc, const void* q, const void* k, const void* v,
                                      const void* d_o, const float* lse, const float* delta,
                                      const int32_t* doc_start, const hsap_tile* tiles, int64_t num_tiles,
                                      float* dq, float* dk, float* dv, hipStream_t s) {
  Geom geom;
  hsap_status st = check_attn(desc, &geom);
  if (st != HSAP_OK) return st;
  const int bm = desc->shard.block_m, bn = desc->shard.block_n, d = desc->head_dim;
  if (!backward_supported(desc))
    HSAP_FAIL(HSAP_ERR_UNSUPPORTED, "no backward kernel for head_dim=%d BM=%d BN=%d", d, bm, bn);
  if ((int64_t)desc->heads_kv * d * 64 > INT32_MAX) HSAP_FAIL(HSAP_ERR_UNSUPPORTED, "heads_kv too large");
  if (desc->chunk_id < 0 || desc->chunk_id >= geom.P)
    HSAP_FAIL(HSAP_ERR_INVALID_ARG, "chunk_id %d outside [0, %d)", desc->chunk_id, geom.P);
  if (num_tiles < 0 || num_tiles > (int64_t(1) << 30))
    HSAP_FAIL(HSAP_ERR_INVALID_ARG, "bad num_tiles %lld", (long long)num_tiles);
  if (geom.n / bm > kMaxListQTiles)
    HSAP_FAIL(HSAP_ERR_UNSUPPORTED, "the tile-list backward needs n / BM <= %d (%lld)", kMaxListQTiles,
              (long long)(geom.n / bm));
  if (geom.n / bn >= kMaxDqKTiles) HSAP_FAIL(HSAP_ERR_UNSUPPORTED, "too many k-tiles per chunk");
  if (!q || !k || !v || !d_o || !lse || !delta || !doc_start || !dq || !dk || !dv || (num_tiles > 0 && !tiles))
    HSAP_FAIL(HSAP_ERR_INVALID_ARG, "NULL pointer argument");
  if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)d_o | (uintptr_t)dq) & 15)
    HSAP_FAIL(HSAP_ERR_INVALID_ARG, "q, k, v, d_o and dq_acc must be 16-byte aligned");
  if (num_tiles == 0) return HSAP_OK;  // no pair of this shard and chunk: every gradient term is 0
  BwdArgs a = {};
  a.q = (const __bf16*)q;
  a.k = (const __bf16*)k;
  a.v = (const __bf16*)v;
  a.d_o = (const __bf16*)d_o;
  a.lse = lse;
  a.delta = delta;
  a.doc_start = doc_start;
  a.dq = dq;
  a.dk = dk;
  a.dv = dv;
  a.geom = geom;
  a.shard = desc->shard.shard_id;
  a.hq = desc->heads_q;
  a.hkv = desc->heads_kv;
  a.group = desc->heads_q / desc->heads_kv;
  a.bm = bm;
  a.bn = bn;
  a.wide_kv = (((uintptr_t)dk | (uintptr_t)dv) & 15) == 0;
  a.scale = desc->softmax_scale;
  a.scale_log2 = desc->softmax_scale * 1.44269504088896340736f;
  a.tiles = tiles;
  a.runs = nullptr;
  a.num_tiles = (int32_t)num_tiles;
  a.chunk = desc->chunk_id;
  const int64_t q_tiles = geom.n / bm, k_tiles = geom.n / bn;
#define HSAP_DQ_CASE(D_, BN_, W_) \
  if (d == D_ && bn == BN_ && bm == 32 * W_) st = launch_dq<D_, BN_, W_, false, true>(a, q_tiles, s);
  HSAP_DQ_CASE(128, 128, 8)
  else HSAP_DQ_CASE(128, 64, 8)
  else HSAP_DQ_CASE(128, 128, 4)
  else HSAP_DQ_CASE(128, 64, 4)
  else HSAP_DQ_CASE(128, 128, 2)
  else HSAP_DQ_CASE(128, 64, 2)
  else HSAP_DQ_CASE(64, 128, 4)
  else HSAP_DQ_CASE(64, 64, 4)
  else HSAP_DQ_CASE(64, 128, 2)
  else HSAP_DQ_CASE(64, 64, 2)
#undef HSAP_DQ_CASE
  if (st != HSAP_OK) return st;
  const int64_t blocks = k_tiles * (bn / 32) * desc->heads_kv;
  return launch_dkdv<false, true>(a, d, list_key_blocks(*desc, blocks), blocks, k_tiles, s);
}

}  // namespace hsap

using namespace hsap;

extern "C" hsap_status hsap_partial_attn_bwd(const hsap_attn_desc* desc, const void* q, const void* k, const void* v,
                                             const void* d_o, const float* lse, const float* delta,
                                             const int32_t* doc_start, const hsap_tile* tiles, int64_t num_tiles,
                                             float* dq_acc, float* dk_acc, float* dv_acc, void* hip_stream) {
  clear_error();
  return backward_tile_list(desc, q, k, v, d_o, lse, delta, doc_start, tiles, num_tiles, dq_acc, dk_acc, dv_acc,
                            (hipStream_t)hip_stream);
}

extern "C" hsap_status hsap_partial_attn_bwd_runs(const hsap_attn_desc* desc, const void* q, const void* k, const void* v,
                                             const void* d_o, const float* lse, const float* delta,
                                             const int32_t* doc_start, const hsap_tile* tiles_k,
                                             const hsap_run* runs_k, int64_t num_runs_k, const hsap_tile* tiles_q,
                                             const hsap_run* runs_q, int64_t num_runs_q, float* dq_acc,
                                             float* dk_acc, float* dv_acc, void* hip_stream) {
  clear_error();
  return backward<false>(desc, q, k, v, d_o, nullptr, lse, delta, nullptr, nullptr, 0, doc_start, tiles_k, runs_k, num_runs_k,
                         tiles_q, runs_q, num_runs_q, dq_acc, dk_acc, dv_acc, 0, (hipStream_t)hip_stream);
}

extern "C" hsap_status hsap_attn_bwd_bf16(const hsap_attn_desc* desc, const void* q, const void* k, const void* v,
                                          const void* d_o, const float* lse, const float* delta,
                                          const int32_t* doc_start, const hsap_tile* tiles_k, const hsap_run* runs_k,
                                          int64_t num_runs_k, const hsap_tile* tiles_q, const hsap_run* runs_q,
                                          int64_t num_runs_q, void* dq, void* dk, void* dv, void* hip_stream) {
  clear_error();
  return backward<true>(desc, q, k, v, d_o, nullptr, lse, delta, nullptr, nullptr, 0, doc_start, tiles_k, runs_k, num_runs_k,
                        tiles_q, runs_q, num_runs_q, dq, dk, dv, 0, (hipStream_t)hip_stream);
}

namespace hsap {
hsap_status attn_bwd_bf16_delta(const hsap_attn_desc* desc, const void* q, const void* k, const void* v,
                                const void* d_o, const void* o, const float* lse, float* delta,
                                const int32_t* cu_seqlens, int32_t num_docs, int32_t* doc_start,
                                const hsap_tile* tiles_k, const hsap_run* runs_k, int64_t num_runs_k,
                                const hsap_tile* tiles_q, const hsap_run* runs_q, int64_t num_runs_q, void* dq,
                                void* dk, void* dv, int key_blocks, hipStream_t stream) {
  if (!o || !cu_seqlens || num_docs < 1) HSAP_FAIL(HSAP_ERR_INVALID_ARG, "NULL o or no cumulative lengths");
  return backward<true>(desc, q, k, v, d_o, o, lse, nullptr, delta, cu_seqlens, num_docs, doc_start, tiles_k, runs_k,
                        num_runs_k, tiles_q, runs_q, num_runs_q, dq, dk, dv, key_blocks, stream);
}
}  // namespace hsap
