// Tile-streaming pieces shared by the attention kernels (forward and backward).
#pragma once

#include "bd_common.hpp"

namespace bd {

template <bool B>
struct BoolTag { static constexpr bool value = B; };

// One 16-byte direct-to-LDS load (global_load_lds_dwordx4): lane l's bytes land at the
// wave's LDS base + 16*l.
__device__ inline void dma16(const uint16_t* g, uint8_t* l) {
  __builtin_amdgcn_global_load_lds((const void*)g, (__attribute__((address_space(3))) void*)l, 16, 0, 0);
}
// The same with the non-temporal policy (nt), for data read once per call.
constexpr int kPolicyNt = 2;
__device__ inline void dma16_nt(const uint16_t* g, uint8_t* l) {
  __builtin_amdgcn_global_load_lds((const void*)g, (__attribute__((address_space(3))) void*)l, 16, 0, kPolicyNt);
}

// The same issued by hand, at an LDS address: the compiler's wait analysis does not see it, so ordinary LDS
// reads beside it wait for LDS alone (it would otherwise wait for every such load in flight before any LDS
// read).  The kernel waits for its tiles explicitly.  M0 (the load's LDS base) is named as clobbered: the
// compiler reuses it between the loads that it places itself, and one of those after a load of these would go
// to the other's address.  It warns that M0 is reserved; it keeps no value of its own there that must survive.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ inline void dma16_hidden(const uint16_t* g, uint32_t lds) {
  asm volatile(
      "s_mov_b32 m0, %0\n"
      "s_nop 0\n"
      "global_load_lds_dwordx4 %1, off"
      :
      : "s"(lds), "v"(g)
      : "memory", "m0");
}
// The same with a uniform base and a byte offset per lane (32 bits).
__device__ inline void dma16_hidden(const uint16_t* base, uint32_t voff, uint32_t lds) {
  asm volatile(
      "s_mov_b32 m0, %0\n"
      "s_nop 0\n"
      "global_load_lds_dwordx4 %1, %2"
      :
      : "s"(lds), "v"(voff), "s"(base)
      : "memory", "m0");
}
#pragma clang diagnostic pop

// Where tiles are read by rows alone (scores): chunk c (16 bytes) of row m of a 16-row sub-tile sits at position
// c ^ k_swizzle(m), which differs for all 16 rows.
__device__ inline int k_swizzle(int m) { return ((m & 7) << 1) | (m >> 3); }

// ---- 32-row tiles for v_mfma_f32_32x32x16_bf16 ---------------------------------
//
// A tile of 32 rows of 128 bf16 (8 KiB) that serves both kinds of operand reads.  Load (h, i), 0 <= h < 2,
// 0 <= i < 4, of lane l brings 16 bytes of row 16h + 4*(l/16) + i to byte 1024*(4h + i) + 16*l, so a load
// covers four whole 256-byte rows.  Chunk c (16 bytes) of row m sits at position c ^ w32_swizzle(m % 16).
// Every row starts on the same LDS bank; the swizzle takes all 16 values over 16 rows (the row operand:
// lanes read the same chunk of different rows) and its upper two bits differ over four rows with the same
// m / 4 (the transposing read: 32 lanes read 64 bytes of each of four rows), so neither read meets a bank
// twice.
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
constexpr int kW32TileBytes = 8192;
__device__ inline int w32_swizzle(int m) { return ((m & 3) << 2) | (m >> 2); }
// chunk that lane l's load (h, i) fetches of its row: w32_swizzle(4*(l/16) + i) = 4i | l/16
__device__ inline int w32_dma_chunk(int lane, int i) { return (lane & 15) ^ (lane >> 4) ^ (4 * i); }
// Row operand: byte of chunk 8*(l/32) of row l%32; chunk + j (the contraction's step j) is at this ^ 16*j.
// Lane half l/32 holds the head dimension's half l/32 (the order of a contraction does not matter).
__device__ inline uint32_t w32_row_off(int lane) {
  const int m = lane & 31;
  return 4096u * (uint32_t)(m >> 4) + 1024u * (uint32_t)(m & 3) + 256u * (uint32_t)((m >> 2) & 3) +
         16u * (uint32_t)((8 * (lane >> 5)) ^ w32_swizzle(m & 15));
}
// Transposed operand (M = d, contraction over the tile's rows) of d-tile dt (d = 32*dt + l%32) and step ks:
// slots 0..3 hold rows 16ks + 4*(l/32) + 0..3, slots 4..7 rows 8 further, which is the order in which
// v_mfma_f32_32x32x16 leaves a 32-row result in lane l's registers 8ks .. 8ks+7.  Byte for dt = 0, slots
// 0..3, ks = 0; ks adds 4096, dt flips 64*dt, slots 4..7 add 512 and flip 32.
__device__ inline uint32_t w32_tr_off(int lane) {
  const int r = (lane >> 2) & 3, hf = lane >> 5;       // row r of the four, d = 16*((l/16)%2) + 4*(l%4)
  const int c = (2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ hf;
  return 1024u * (uint32_t)r + 256u * (uint32_t)hf + 16u * (uint32_t)((4 * r) ^ c) + 8u * (uint32_t)(lane & 1);
}
__device__ inline bf16x8 w32_read_row(const uint8_t* tile, uint32_t row_off, int j) {
  return *reinterpret_cast<const bf16x8*>(tile + (row_off ^ (16u * (uint32_t)j)));
}
__device__ inline bf16x8 w32_read_tr(const uint8_t* tile, uint32_t tr_off, int dt, int ks) {
  typedef __attribute__((address_space(3))) bf16x4* lds_ptr;
  const uint32_t a = (tr_off ^ (64u * (uint32_t)dt)) + 4096u * (uint32_t)ks;
  const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr)(tile + a));
  const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr)(tile + ((a ^ 32u) + 512u)));
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}
// Row of register i of a 32x32 result: 8*(i/4) + 4*(l/32) + i%4.
__device__ inline int w32_result_row(int i, int hf) { return 8 * (i >> 2) + 4 * hf + (i & 3); }

// Scheduling of a phase: N products, each followed by up to V vector instructions (transcendentals
// included), so that the in-order issue of one wave alternates between the two units.
template <int N, int V>
__device__ inline void interleave_mfma_valu() {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x402, V, 0);
  }
}

// Transposed operand for d-tile dt from 8 rows of 16 bytes per lane (row slot i = register i,
// bytes 16*(lane%16) of the row): slot i of the result holds row i's element 8*(lane%16) + dt.
// An 8x8 bf16 block transposed in registers with byte permutes.
__device__ inline bf16x8 vt_operand(const u32x4 (&v)[8], int dt) {
  const int w = dt >> 1;
  const uint32_t sel = (dt & 1) ? 0x07060302u : 0x05040100u;
  u32x4 r;
  r[0] = __builtin_amdgcn_perm(v[1][w], v[0][w], sel);
  r[1] = __builtin_amdgcn_perm(v[3][w], v[2][w], sel);
  r[2] = __builtin_amdgcn_perm(v[5][w], v[4][w], sel);
  r[3] = __builtin_amdgcn_perm(v[7][w], v[6][w], sel);
  return as_bf16x8(r);
}

// A tile of 32 key rows kept row-major for the transposing reads: load q (0..7) of lane l brings
// row 4*q + l/16, its 16-byte chunk (l%16) ^ (l/16), to byte rm_block_off(q) + 256*(l/16) +
// 16*(l%16), so chunk c of row r sits at position c ^ (r % 4) and a 16-lane group's reads cover
// 32 distinct banks.  The LDS serves a transposing read 32 lanes (64 banks of 4 bytes) at a time,
// and lanes 0-15 and 16-31 read rows of consecutive blocks (1 KiB, rows 4q .. 4q+3).  At a 1 KiB
// pitch both lane groups meet on the same 32 banks: an in-bounds probe measured every read 2-way
// conflicted.  So odd blocks start 8 bytes past a 16-byte boundary (the other 32 banks), and every
// pair of blocks takes 16 bytes more so that the shifted block does not run into the next: block q
// at 1024*q + 8*(q%2) + 16*(q/2).  The probe then read every element where the layout below says
// and measured no conflict (40% less time).  Rows 16..31 (blocks 4..7) lie 4128 bytes past rows 0..15.
constexpr int kRmTileBytes = 8256;
constexpr int kRmHighRows = 4128;
__device__ inline uint32_t rm_block_off(int q) {
  return 1024u * (uint32_t)q + 8u * (uint32_t)(q & 1) + 16u * (uint32_t)(q >> 1);
}
__device__ inline int rm_row(int q, int lane) { return 4 * q + (lane >> 4); }
__device__ inline int rm_chunk(int lane) { return (lane & 15) ^ (lane >> 4); }
// This lane's transposing-read addresses relative to such a tile: rows 4*(lane/16) + (lane%16)/4 (k-slots
// 0..3; +kRmHighRows for 4..7), d from 32*(lane%4) + 8*j, at the swizzled chunk position.
__device__ inline uint32_t tr_lane_off(int lane, int j) {
  const int lg = lane >> 4, lr = lane & 15;
  return rm_block_off(lg) + 256u * (uint32_t)(lr >> 2) + 16u * (uint32_t)((4 * (lr & 3) + j) ^ (lr >> 2));
}

// The transposing LDS read ds_read_b64_tr_b16 forms the transposed operands (V^T in the forward's block mode)
// of all 8 d-tiles straight from such a tile.  Within each 16-lane group that read hands lane i, element j,
// element i%4 of the 8 bytes that lane 4j + i/4 addressed.  Addresses a[j] = tile + tr_lane_off(lane, j)
// serve d-tiles 2j and 2j+1, k-slots 0..3; +8 selects the odd d-tile, +kRmHighRows (4128) the k-slots 4..7
// (tile rows 16..31).  Result vt[dt], slot k of lane l: row[key slot 16*(k/4) + 4*(l/16) + k%4]
// [d = 32*((l%16)/4) + 4*dt + l%4], so accumulator register r of d-tile dt in lane l holds
// d = 32*(l/16) + 4*dt + r.
static_assert(kRmHighRows == 4128, "the kernels' read offsets are kRmHighRows and kRmHighRows + 8");

// Slot table of one split for the block-mode kernels: row offset (16-byte units) and position of
// every key slot in [0, nslots), entries e_begin .. e_end-1 of the key list (gathered idx entries,
// or cache rows when idx_row is NULL) followed by padding slots (position -1, offset 0).  Keys
// outside [0, L) and rows whose page is outside the pool become padding too.  All idx and
// page-table loads are issued before any result is used.
template <bool PAGED, int kThreadsT, int kCap>
__device__ inline void fill_slot_table(const KvView& kv, int s, int g, int L, const int32_t* idx_row, int e_begin,
                                       int e_end, int nslots, int32_t* roff, int32_t* tpos, int tid) {
  constexpr int kPer = (kCap + kThreadsT - 1) / kThreadsT;
  int tv[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int e = e_begin + tid + k * kThreadsT;
    int t = -1;
    if (e < e_end) t = idx_row ? idx_row[e] : e;
    tv[k] = (t >= 0 && t < L) ? t : -1;
  }
  int pg[kPer];
  if constexpr (PAGED) {
#pragma unroll
    for (int k = 0; k < kPer; ++k)
      pg[k] = tv[k] >= 0 ? kv.page_table[(int64_t)s * kv.max_pages_per_seq + tv[k] / kv.page_size] : 0;
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = tid + k * kThreadsT;
    if (i < nslots && i < kCap) {
      int t = tv[k];
      int64_t o;
      if constexpr (PAGED) {
        o = (unsigned)pg[k] < (unsigned)kv.num_pages
                ? (int64_t)pg[k] * kv.stride_page + (int64_t)g * kv.stride_head +
                      (int64_t)(t % kv.page_size) * kv.stride_tok
                : -1;
      } else {
        o = (int64_t)s * kv.stride_seq + (int64_t)g * kv.stride_head + (int64_t)t * kv.stride_tok;
      }
      if (t < 0 || o < 0) { t = -1; o = 0; }
      roff[i] = (int)(o >> 3);
      tpos[i] = t;
    }
  }
}

// How a (sequence, KV head, row group) unit's key stream (the views' entry lists, then the full
// branch's cache rows) is cut among its nW workgroups: equal shares of weighted work, a gathered
// view entry weighing WG and a cache row of the full branch WF (gathered tiles cost more per tile).
// Views come first, so stream position x (vt = the views' total) weighs WG*x up to vt and WF per
// row after.  A share weighs at least WG*32, so every workgroup below the stream's end gets entries
// and the workgroups that meet a branch are consecutive.  Each kernel has weights of its own (the
// forward 5 and 4, dQ 1 and 1 in whole tiles); none relies on the shares of another.
// ROUND: the share's weight is rounded up to a multiple of ROUND (with WG = WF = 1 and ROUND = 32,
// equal shares that start on whole tiles of the stream).
template <int WG, int WF, int ROUND = 1>
struct StreamCut {
  int vt, total, chunk;   // chunk: weight per workgroup
  __host__ __device__ StreamCut(int vt_, int total_, int nW) : vt(vt_), total(total_) {
    const int tw = WG * vt + WF * (total - vt);
    int c = (tw + nW - 1) / nW;
    c = (c + ROUND - 1) / ROUND * ROUND;
    chunk = c > WG * 32 ? c : WG * 32;
  }
  __host__ __device__ int weight(int x) const { return x <= vt ? WG * x : WG * vt + WF * (x - vt); }
  // workgroup whose share holds stream position x
  __host__ __device__ int wg_of(int x) const { return weight(x) / chunk; }
  // first stream position of workgroup w's share (clamped to the stream's end)
  __host__ __device__ int start_of(int w) const {
    const int t = w * chunk;
    const int x = t <= WG * vt ? (t + WG - 1) / WG : vt + (t - WG * vt + WF - 1) / WF;
    return x < total ? x : total;
  }
};
// Workgroups per unit for `units` streams of at most `weight` each (weighted as StreamCut weighs them),
// between nw_lo (no share overflows its slot table) and nw_hi (each share leaves records in scratch, which the
// merge reads).  A CU holds
// one workgroup of these kernels, so a launch of more than kCus workgroups runs in rounds, and one
// that just exceeds a multiple leaves its last round nearly empty: 24 units at ceil(256 / 24) = 11
// each are 264 workgroups, two rounds of a 1/11 share, where 10 each take one round of a 1/10 share
// (3 sequences x 8 KV heads at 8K, C = 64, four views: forward 90 -> 57 us, training pass 287 -> 215 us).
// So the count that ends first is taken: rounds x (a share + the fixed cost of a workgroup).
constexpr int64_t kCus = 256;
inline int64_t plan_stream_workgroups(int64_t units, int64_t nw_lo, int64_t nw_hi, int64_t weight, int64_t fixed) {
  if (nw_lo < 1) nw_lo = 1;
  if (nw_hi < nw_lo) nw_hi = nw_lo;
  int64_t best = nw_lo, best_cost = INT64_MAX;
  // only the largest counts of 1, 2, ... whole rounds can be best
  for (int64_t r = (units * nw_lo + kCus - 1) / kCus, tries = 0; tries < 16; ++r, ++tries) {
    int64_t nw = kCus * r / units;
    if (nw < nw_lo) nw = nw_lo;
    if (nw > nw_hi) nw = nw_hi;
    const int64_t rounds = (units * nw + kCus - 1) / kCus;
    const int64_t cost = rounds * ((weight + nw - 1) / nw + fixed);
    if (cost < best_cost) { best_cost = cost; best = nw; }
    if (nw == nw_hi) break;
  }
  return best;
}

}  // namespace bd
