// Budgeted KV selection (Alg. 2 "sparsify"; Sec. 3.4: keep the entries with
// the largest cumulative attention weight).
//
// Three launches:
//   1. score pass 1 (skipped when the caller gives the window rows'
//      log-sum-exp): every (sequence, KV head, row block, key split) computes
//      the running max and sum of exp of each observation row over its keys;
//   2. score pass 2: merges those statistics into each row's log-sum-exp and
//      streams K again, adding every row's normalised weight of every key
//      into that key's column sum (complete within a row block, so no atomics);
//   3. top-B: one 1024-thread workgroup per (sequence, KV head) sums the row
//      blocks, max-pools the prefix (or sums its chunks), finds the K-th
//      largest candidate score with a radix select over the float bit patterns
//      (digits of 8, 11 and 12 bits; scores are non-negative, so the bits order
//      like the values), and compacts the chosen positions in ascending order;
//      ties at the threshold take the lowest positions, then the window is
//      appended.
//
// The scoring product is a real dense contraction ((W*G) x 128 x L per
// (s, g)), so it runs on MFMA (v_mfma_f32_32x32x16_bf16) with keys on the M side
// and observation rows on the N side: D element (8*(i/4) + 4*(l/32) + i%4, l%32)
// sits in lane l, register i.  Lane l then holds 16 keys of row l%32: row
// statistics stay lane-local, and a key's column sum is a reduction over the
// 32 lanes of its half.

#include <type_traits>

#include "bd_common.hpp"
#include "bd_kernels.hpp"
#include "attn_tile.hpp"

namespace bd {
namespace {

constexpr int kWaves = 8;                        // two per SIMD: one wave's MFMA and loads overlap another's VALU
constexpr int kThreads = kWaves * kWave;
constexpr int kTile = 32;                        // keys per wave iteration
constexpr int kTileLoads = 8;                    // 16-byte loads per lane per tile
constexpr int kTileBytes = kTileLoads * kWave * 16;
constexpr int kRing = 2;                         // tile slots per wave: one in flight while one is computed
constexpr int kMaxPagedKeys = 4096;              // keys per workgroup through the paged slot table
constexpr int kSlotCap = kMaxPagedKeys + kRing * kWaves * kTile;
constexpr int kStatRows = 128;                   // stats record stride (rows); the most rows of a block
constexpr int kTargetBlocks = 256;               // one workgroup per CU
constexpr int kTopkThreads = 1024;
constexpr int kMaxPerThread = BD_SELECT_MAX_PREFIX / kTopkThreads;   // 32
constexpr int kHistWords = 4096;                // radix histogram words: bins x copies of each digit
// Radix digits of the top-B keys, most significant first (bits, lowest bit, histogram copies).
constexpr int kDigits = 3;
__device__ inline int digit_bits(int i) { return i == 0 ? 8 : (i == 1 ? 11 : 12); }
__device__ inline int digit_shift(int i) { return i == 0 ? 23 : (i == 1 ? 12 : 0); }
__device__ inline int digit_copies(int i) { return i == 0 ? 16 : (i == 1 ? 2 : 1); }
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kRaiseSum = 4096.f;              // pass 1: a lane's 16 weights of a row may sum to this before its reference is raised
constexpr float kNoRef = -3.0e38f;               // pass 1: reference of a row that has seen no key

__device__ inline void merge_ml(float& m, float& l, float m2, float l2) {
  const float M = fmaxf(m, m2);
  if (M == -INFINITY) { m = M; l = 0.f; return; }
  l = l * exp2f(m - M) + l2 * exp2f(m2 - M);
  m = M;
}

// Every kernel argument requested at entry: fetched where first used they took four or five round
// trips in a row before the first data load.  The statements touch no memory and return 0, which
// the caller adds to its block index.
__device__ inline int fetch_select_args(const SelectParams& p) {
  int z0, z1, z2;
  asm("s_mov_b32 %0, 0" : "=s"(z0) : "s"(p.kv.k), "s"(p.kv.seq_lens), "s"(p.kv.page_table), "s"(p.kv.stride_seq),
      "s"(p.kv.stride_head), "s"(p.kv.stride_tok), "s"(p.kv.stride_page), "s"(p.kv.max_seq_len), "s"(p.kv.page_size),
      "s"(p.kv.max_pages_per_seq), "s"(p.kv.num_pages));
  asm("s_mov_b32 %0, 0" : "=s"(z1) : "s"(z0), "s"(p.q_win), "s"(p.lse_win), "s"(p.S), "s"(p.Hkv), "s"(p.Hq), "s"(p.G),
      "s"(p.W), "s"(p.budget), "s"(p.pool_kernel), "s"(p.chunk), "s"(p.keep), "s"(p.ld), "s"(p.R), "s"(p.n_rb));
  asm("s_mov_b32 %0, 0" : "=s"(z2) : "s"(z1), "s"(p.nsplit), "s"(p.kps), "s"(p.max_L), "s"(p.scale_log2),
      "s"(p.max_roff), "s"(p.stats), "s"(p.raw_part), "s"(p.raw), "s"(p.idx_out), "s"(p.nsel_out), "s"(p.page_arith));
  return z2;
}

template <int RT, bool PAGED>
struct ScoreSmem {
  alignas(64) uint8_t ring[kWaves][kRing][kTileBytes];   // per-wave K tile slots filled by DMA
  alignas(16) int32_t roff[PAGED ? kSlotCap : 4];        // paged: row offset (16-byte units) per key slot
  float m[kWaves][32 * RT];
  float l[kWaves][32 * RT];
  float lse2[32 * RT];
};

// Direct-to-LDS loads of one K tile: load (h, i) brings the four whole rows 16h + 4*(lane/16) + i to
// dst + (4h + i) KiB, 16 bytes a lane; r[h][i] are the lane's rows (16-byte units, clamped to the
// layout).  Chunk c (16 bytes) of row m lands at position c ^ k_swizzle(m % 16) of its 256 bytes: all
// rows start on the same LDS bank, and the swizzle puts the rows of a score read on different ones.
__device__ inline void dma_ktile(const uint16_t* k, const u32x4 (&r)[2], uint32_t max_roff, uint32_t dst, int lane) {
  const int kc = (lane & 15) ^ k_swizzle(4 * (lane >> 4));
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t ro = r[h][i] < max_roff ? r[h][i] : max_roff;
      dma16_hidden(k + ((uint64_t)ro << 3) + 8 * (kc ^ (2 * i)), dst + (4 * h + i) * 1024);   // swizzle of row 4*lg + i
    }
}
// Byte offset in a tile of chunk 8*(lane/32) of row lane%32; chunk + j is at this ^ 16*j.
__device__ inline uint32_t k_lane_off(int lane) {
  const int m = lane & 31;
  return 4096u * (uint32_t)(m >> 4) + 1024u * (uint32_t)(m & 3) + 256u * (uint32_t)((m >> 2) & 3) +
         16u * (uint32_t)((8 * (lane >> 5)) ^ k_swizzle(m & 15));
}

// The same for a tile whose two 16-key sub-tiles are runs of rows `stride` bytes apart, from uniform byte
// offsets base[h] into K: the address of a load is a scalar base plus a lane-constant offset, so a tile
// costs few vector instructions.  The caller knows that all 32 rows lie in the layout.
__device__ inline void dma_krun(const uint16_t* k, const uint64_t (&base)[2], uint32_t stride, uint32_t dst) {
  // the lane offsets are formed again for each tile, from the lane index up: kept across the loop they
  // cost spills, and a reload waits for every load in flight
  int lane;
  asm volatile(
      "v_mbcnt_lo_u32_b32 %0, -1, 0\n"
      "v_mbcnt_hi_u32_b32 %0, -1, %0"
      : "=&v"(lane));
  const uint32_t voff_row = (uint32_t)(4 * (lane >> 4)) * stride;
  const uint32_t voff_chunk = 16u * (uint32_t)((lane & 15) ^ k_swizzle(4 * (lane >> 4)));
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t voff = voff_row + (voff_chunk ^ (32u * (uint32_t)i));
#pragma unroll
    for (int h = 0; h < 2; ++h)
      dma16_hidden(reinterpret_cast<const uint16_t*>(reinterpret_cast<const uint8_t*>(k) + base[h] + (uint64_t)((uint32_t)i * stride)),
                voff, dst + (4 * h + i) * 1024);
  }
}

// Row offsets of a paged tile's lane rows from the slot table (loads and their wait in one statement).
__device__ inline void read_krows(u32x4 (&r)[2], uint32_t roff_lds, int slot0, int lane) {
  const uint32_t a = roff_lds + 4 * (slot0 + 4 * (lane >> 4));
  asm volatile(
      "ds_read_b128 %0, %2\n"
      "ds_read_b128 %1, %2 offset:64\n"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(r[0]), "=&v"(r[1])
      : "v"(a));
}

// Sums of 16 values over the 32 lanes of each half: value i ends in lanes 2i and 2i + 1 of the half
// (half_sum_index).  Each step halves the values a lane carries and doubles the lanes summed: step 1 pairs value
// i with value i + 8 over lanes 16 apart (one permlane16_swap serves both), the others exchange within a row of
// 16, the last one over the two lanes that keep the sum.
__device__ inline float half_sums(const float (&v)[16], int lane) {
  float a[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 8]), false, false);
    a[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);      // even rows: value i, odd rows: value i + 8
  }
  const bool b8 = lane & 8, b4 = lane & 4, b2 = lane & 2;
  float c[4], d[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {      // lanes l and l ^ 8 (a rotation by 8 of the row)
    const float keep = b8 ? a[i + 4] : a[i], give = b8 ? a[i] : a[i + 4];
    c[i] = keep + __builtin_amdgcn_update_dpp(0.0f, give, 0x128, 0xF, 0xF, false);   // row_ror:8
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {      // the mirrored half row holds lane l ^ 7: bit 2 differs
    const float keep = b4 ? c[i + 2] : c[i], give = b4 ? c[i] : c[i + 2];
    d[i] = keep + __builtin_amdgcn_update_dpp(0.0f, give, 0x141, 0xF, 0xF, false);   // row_half_mirror
  }
  const float keep = b2 ? d[1] : d[0], give = b2 ? d[0] : d[1];
  float e = keep + __builtin_amdgcn_update_dpp(0.0f, give, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
  e += __builtin_amdgcn_update_dpp(0.0f, e, 0xB1, 0xF, 0xF, false);                  // quad_perm [1,0,3,2]
  return e;
}
__device__ inline int half_sum_index(int lane) {
  return (lane & 31) >> 1;
}

// One pass over the causal key range of (sequence, KV head, row block of 32*RT rows, split).  Each wave
// streams every kWaves-th 32-key tile through a kRing-deep ring of LDS slots.
//   PASS 1: per observation row, running max and sum of exp of the scaled logits;
//   PASS 2: every key's column sum of the rows' normalised weights (complete within the row
//           block: one plain store per key).
// Per 32 x 32 scores a wave needs 8 products (32 cycles each) and 48 vector instructions (16 of them
// exponentials at 8 cycles): the two units have like work, so the tile loop is pipelined by row tile,
// products of one beside the exponentials of the one before.  What bounds it: the chain of the two at two
// waves per SIMD (over the kernel matrix units 27-30% and vector units 45-48% busy), and for 128 rows at
// 16K x 8 the K stream, which pass 1 reads from HBM (54-59 us where the caches hold none of it).
// Measured, 16K keys, passes 1 and 2: 8 sequences, 128 rows 58 + 51 -> 46 + 44.5 us; one sequence, 1,024
// rows (8 blocks, K from the caches) 57.5 + 50.5 -> 43.5 + 43 us; at 4K, 128 workgroups 14.4 + 12.4 ->
// 10.6 + 8.3 us.  Before: 16x16x32 products with all of a tile's products ahead of its exponentials, row
// maxima for every tile, and the rows read by every wave from memory.
template <int RT, bool PAGED, int PASS>
__global__ __launch_bounds__(kThreads) void score_kernel(SelectParams p) {
  __shared__ ScoreSmem<RT, PAGED> sm;
  constexpr int kRows = 32 * RT;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lg = lane >> 4, lr = lane & 31, hf = lane >> 5;
  const int bid = xcd_remap(blockIdx.x + fetch_select_args(p), gridDim.x);
  const int rb = bid % p.n_rb;
  const int rest = bid / p.n_rb;
  const int split = rest % p.nsplit;
  const int pair = rest / p.nsplit;
  const int g = pair % p.Hkv, s = pair / p.Hkv;
  const int L = seq_len(p.kv, s);
  if (p.budget >= L) return;               // whole cache kept: nothing to score
  const int k0 = split * p.kps;
  int k1 = k0 + p.kps;
  if (k1 > L) k1 = L;
  const int64_t stat_base = (((int64_t)pair * p.n_rb + rb) * p.nsplit) * kStatRows * 2;
  if (PASS == 2 && k1 <= k0) return;       // a split past this sequence's end: no key to score

  const int ntiles = k1 > k0 ? (k1 - k0 + kTile - 1) / kTile : 0;
  // pages holding whole 16-key sub-tiles (page_size a multiple of 16, host-checked): a table of page
  // offsets, one entry per page; k / page_size is computed as (k / 16) / (page_size / 16), exact for
  // keys below 2^26 (host-checked); k0 is a multiple of kWaves * kTile
  const bool page_arith = PAGED && p.page_arith != 0;
  const int psub = PAGED ? p.kv.page_size >> 4 : 1;
  const float inv_psub = __builtin_amdgcn_rcpf((float)psub);
  const int page0 = page_arith ? div_small(k0 >> 4, psub, inv_psub) : 0;
  const uint32_t ring_lds = lds_addr(sm.ring[wave][0]);
  const uint32_t roff_lds = lds_addr(sm.roff);
  const uint64_t row0 = PAGED ? 0 : (uint64_t)((int64_t)s * p.kv.stride_seq + (int64_t)g * p.kv.stride_head);
  const uint32_t base16 = (uint32_t)(row0 >> 3), tok16 = (uint32_t)(p.kv.stride_tok >> 3);
  const bool runs = p.kv.stride_tok <= (1 << 26);          // a run's lane offsets fit 32 bits
  // pass 2 takes its tiles last first: pass 1 read them first to last, so the most recent (still in
  // the memory-side cache) are read before the lines pass 1 read first are replaced
  auto real = [&](int it) { return PASS == 2 ? ntiles - 1 - it : it; };
  auto issue = [&](int tile, int slot) {
    const uint32_t dst = ring_lds + slot * kTileBytes;
    u32x4 r[2];
    if (tile >= ntiles) {
      r[0] = r[1] = u32x4{0u, 0u, 0u, 0u};   // padding: row 0, a safe, cache-resident address
    } else {
      const int tb = k0 + kTile * real(tile);
      if constexpr (PAGED) {
        if (page_arith) {
          // sub-tile h (keys tb+16h .. +15) lies in one page: its offset + (key mod page_size) rows
          uint32_t a[2], w[2], b[2];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int t = tb + 16 * h;
            const int pi = div_small(t >> 4, psub, inv_psub);
            a[h] = roff_lds + 4 * (uint32_t)(t < k1 ? pi - page0 : 0);   // past the split: entry 0, masked
            w[h] = (uint32_t)(t - pi * p.kv.page_size);
          }
          asm volatile(
              "ds_read_b32 %0, %2\n"
              "ds_read_b32 %1, %3\n"
              "s_waitcnt lgkmcnt(0)"
              : "=&v"(b[0]), "=&v"(b[1])
              : "v"(a[0]), "v"(a[1]));
          if (runs) {
            uint64_t base[2];
#pragma unroll
            for (int h = 0; h < 2; ++h)
              base[h] = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(b[h]) +
                         (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(w[h]) * tok16) << 4;
            dma_krun(p.kv.k, base, tok16 << 4, dst);
            return;
          }
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i) r[h][i] = b[h] + (w[h] + (uint32_t)(4 * lg + i)) * tok16;
        } else {
          read_krows(r, roff_lds, kTile * real(tile), lane);
        }
      } else {
        if (runs && tb + kTile <= k1) {        // whole tiles lie in the cache
          uint64_t base[2];
#pragma unroll
          for (int h = 0; h < 2; ++h) base[h] = (row0 + (uint64_t)(tb + 16 * h) * (uint64_t)p.kv.stride_tok) << 1;
          dma_krun(p.kv.k, base, tok16 << 4, dst);
          return;
        }
        const uint32_t r0 = base16 + (uint32_t)(tb + 4 * lg) * tok16;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int i = 0; i < 4; ++i) r[h][i] = r0 + (uint32_t)(16 * h + i) * tok16;
      }
    }
    dma_ktile(p.kv.k, r, p.max_roff, dst, lane);
  };

  // a contiguous cache's first tile needs only the length: it loads beside the rows
  if (!PAGED && wave < ntiles) issue(wave, 0);

  // observation rows n = rb*kRows + 32*t + lane%32 -> (window row i, head h).  All waves need them all: each
  // brings its 4*RT rows to LDS whole (its second tile slot), chunks swizzled as a K tile's.  Read straight
  // from memory, every wave touched a line per lane and load, 4 lines a row each, and the row loads alone
  // took several microseconds of the CU's address path.
  {
    const uint32_t dst = lds_addr(sm.ring[wave][1]);
#pragma unroll
    for (int q = 0; q < RT; ++q) {
      const int r = 4 * RT * wave + 4 * q + lg;
      const int n = rb * kRows + r < p.R ? rb * kRows + r : p.R - 1;     // rows past R are dropped when read
      const int i = n / p.G, h = g * p.G + n - i * p.G;
      dma16_hidden(p.q_win + (((int64_t)s * p.W + i) * p.Hq + h) * kD + 8 * ((lane & 15) ^ k_swizzle(r & 15)), dst + q * 1024);
    }
  }
  int rowpos[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int n = rb * kRows + 32 * t + lr;
    rowpos[t] = n < p.R ? L - p.W + n / p.G : -1;   // padded rows see no key
  }

  if (page_arith) {
    // entry j: offset (16-byte units) of page page0 + j for head g, 0 for a page outside the pool (its
    // keys read pool rows and score as whatever those hold); all page-table loads issued first
    constexpr int kPer = (kSlotCap + kThreads - 1) / kThreads;
    const int npg = k1 > k0 ? div_small((k1 - 1) >> 4, psub, inv_psub) - page0 + 1 : 0;
    const int32_t* prow = p.kv.page_table + (int64_t)s * p.kv.max_pages_per_seq + page0;
    int pg[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int j = tid + k * kThreads;
      pg[k] = j < npg ? prow[j] : -1;
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int j = tid + k * kThreads;
      if (j < npg)
        sm.roff[j] = (unsigned)pg[k] < (unsigned)p.kv.num_pages
                         ? (int)(((int64_t)pg[k] * p.kv.stride_page + (int64_t)g * p.kv.stride_head) >> 3)
                         : 0;
    }
  } else if constexpr (PAGED) {
    // slot table of this split: all page-table loads issued before any result is used; padding
    // slots (past the split) hold row 0, a safe, cache-resident address
    constexpr int kPer = (kSlotCap + kThreads - 1) / kThreads;
    int pg[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int t = k0 + tid + k * kThreads;
      pg[k] = t < k1 ? p.kv.page_table[(int64_t)s * p.kv.max_pages_per_seq + t / p.kv.page_size] : -1;
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int i = tid + k * kThreads;
      if (i < kSlotCap) {
        const int t = k0 + i;
        int64_t o = 0;
        if ((unsigned)pg[k] < (unsigned)p.kv.num_pages)
          o = (int64_t)pg[k] * p.kv.stride_page + (int64_t)g * p.kv.stride_head +
              (int64_t)(t % p.kv.page_size) * p.kv.stride_tok;
        sm.roff[i] = (int)(o >> 3);
      }
    }
  }

  // lse of each row (pass 2): the caller's, or merged from the pass-1 statistics.  Padded rows get
  // +inf, so their weights are exactly zero even where no mask is applied.
  // pass 1 per row: reference mu (log2 units) and this lane's sum rl of exp2 relative to it
  float rm[RT], rl[RT], lse2[RT];
  if constexpr (PASS == 2) {
    if (tid < kRows) {
      const int n = rb * kRows + tid;
      float v = INFINITY;
      if (n < p.R) {
        if (p.lse_win) {
          const int i = n / p.G, h = g * p.G + n % p.G;
          v = p.lse_win[((int64_t)s * p.W + i) * p.Hq + h] * kLog2e;
        } else {
          // the splits merge in order; a batch of records is loaded before the first is used
          constexpr int kBatch = 8;
          float m = -INFINITY, l = 0.f;
          const float2* st = reinterpret_cast<const float2*>(p.stats + stat_base) + tid;
          for (int sp0 = 0; sp0 < p.nsplit; sp0 += kBatch) {
            float2 x[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) x[u] = st[(int64_t)(sp0 + u < p.nsplit ? sp0 + u : sp0) * kStatRows];
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
              if (sp0 + u < p.nsplit) merge_ml(m, l, x[u].x, x[u].y);
          }
          v = l > 0.f ? m + __log2f(l) : INFINITY;   // empty row contributes nothing
        }
      }
      sm.lse2[tid] = v;
    }
  } else {
#pragma unroll
    for (int t = 0; t < RT; ++t) { rm[t] = kNoRef; rl[t] = 0.f; }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's rows (and first tile) are in LDS
  __syncthreads();
  // lane half hf holds the head dimension's half hf, in 8 steps of 8 (the order of a contraction does not
  // matter)
  bf16x8 qop[RT][8];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int r = 32 * t + lr, w = r / (4 * RT), rw = r - w * (4 * RT);
    const bool valid = rb * kRows + r < p.R;
    const uint8_t* row = sm.ring[w][1] + 256 * rw;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const u32x4 x = *reinterpret_cast<const u32x4*>(row + 16 * ((8 * hf + j) ^ k_swizzle(r & 15)));
      qop[t][j] = as_bf16x8(valid ? x : u32x4{0u, 0u, 0u, 0u});
    }
  }
  if constexpr (PASS == 2) {
#pragma unroll
    for (int t = 0; t < RT; ++t) lse2[t] = sm.lse2[32 * t + lr];
  }
  __syncthreads();                         // every wave has the rows: the second slots take tiles

  // tiles whose keys all lie inside the split and at or before the block's earliest row position
  // need no mask
  const int minpos = L - p.W + (rb * kRows) / p.G;
  int first_dirty;
  {
    const int c1 = minpos - k0 - (kTile - 1);
    const int fd1 = c1 < 0 ? 0 : c1 / kTile + 1;
    const int fd2 = (k1 - k0) / kTile;
    first_dirty = fd1 < fd2 ? fd1 : fd2;
  }

  float* raw_part = p.raw_part + ((int64_t)pair * p.n_rb + rb) * p.max_L;

  bf16x8 kt[8];                            // the tile's keys: row lane%32, half hf of the head dimension
  // scores of the tile against row tile t
  auto products = [&](f32x16& acc, int t) {
    f32x16 a;
#pragma unroll
    for (int i = 0; i < 16; ++i) a[i] = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kt[j], qop[t][j], a, 0, 0, 0);
    acc = a;
  };
  // Causal and split mask.  Only tiles that can hold a masked key call it: a mask behind a runtime flag
  // was if-converted, and every tile paid it.  `tb`: the tile's first key.
  auto mask = [&](f32x16& acc, int t, int tb) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int key = tb + 8 * (i >> 2) + 4 * hf + (i & 3);
      if (!(key < k1 && key <= rowpos[t])) acc[i] = -INFINITY;
    }
  };
  // Pass 1: this lane's 16 weights of row tile t, relative to the row's reference, join its sum.  The
  // reference is raised when they sum to more than kRaiseSum (an overflow included): the maximum over the
  // row's keys of the tile becomes the reference, and the weights are formed again.  No maximum is taken
  // in the common case, and rows start at a reference below every logit, so their first key raises it.
  auto pass1_sum = [&](const f32x16& acc, int t) {
    auto weights = [&]() {
      float x[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = __builtin_amdgcn_exp2f(fmaf(acc[i], p.scale_log2, -rm[t]));
#pragma unroll
      for (int i = 4; i < 16; ++i) x[i & 3] += __builtin_amdgcn_exp2f(fmaf(acc[i], p.scale_log2, -rm[t]));
      return (x[0] + x[1]) + (x[2] + x[3]);
    };
    float w = weights();
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(w > kRaiseSum) != 0, 0)) {
      float m = acc[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) m = fmaxf(m, acc[i]);
      m = max_xor32(m) * p.scale_log2;     // both halves of the row; scale > 0: the max commutes with it
      if (m > rm[t]) {
        rl[t] *= __builtin_amdgcn_exp2f(rm[t] - m);
        rm[t] = m;
      }
      w = weights();
    }
    rl[t] += w;
  };
  // Pass 2: every key's column sum of the rows' normalised weights; after the last row tile the 32 lanes
  // of a half reduce their 16 keys' sums and each key's lanes store it.
  float col[16];
  auto pass2_sum = [&](const f32x16& acc, int t) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float w = __builtin_amdgcn_exp2f(fmaf(acc[i], p.scale_log2, -lse2[t]));
      col[i] = t == 0 ? w : col[i] + w;
    }
  };
  const int my = half_sum_index(lane);
  const int my_key = 8 * (my >> 2) + 4 * hf + (my & 3);
  auto pass2_store = [&](int tb, bool checked) {
    const float v = half_sums(col, lane);
    const int key = tb + my_key;
    if (!checked || key < k1) raw_part[key] = v;     // two lanes hold each key's sum, with equal bits
  };

  if (wave < ntiles) {
    if (PAGED) issue(wave, 0);
    issue(wave + kWaves, 1);
    int j = 0;
    const int steps = (ntiles - wave + kWaves - 1) / kWaves;   // this wave's tiles: wave + kWaves*j, j < steps
    const uint32_t koff = k_lane_off(lane);
    // The tile of step j: its keys from LDS (read_tile), then its slot refilled (refill, once the keys
    // have arrived in registers).  Returns the tile's first key.
    auto read_tile = [&]() -> int {
      // the tile about to be read was issued (kRing-1) tiles before the newest
      static_assert(kRing == 2, "the wait below assumes one tile (8 loads) issued after the one read");
      asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
      const uint8_t* slot = sm.ring[wave][0] + (j % kRing) * kTileBytes;
#pragma unroll
      for (int c = 0; c < 8; ++c) kt[c] = *reinterpret_cast<const bf16x8*>(slot + (koff ^ (16u * (uint32_t)c)));
      return k0 + kTile * real(wave + kWaves * j);
    };
    auto refill = [&]() {
      asm volatile("" : "+v"(kt[0]), "+v"(kt[1]), "+v"(kt[2]), "+v"(kt[3]), "+v"(kt[4]), "+v"(kt[5]), "+v"(kt[6]), "+v"(kt[7]) :: "memory");
      issue(wave + kWaves * (j + kRing), j % kRing);
    };
    // Tiles that hold a masked key, one step after the other.
    auto run_dirty = [&](int end) {
      for (; j < end; ++j) {
        const int tb = read_tile();
        refill();
#pragma unroll
        for (int t = 0; t < RT; ++t) {
          f32x16 acc;
          products(acc, t);
          mask(acc, t, tb);
          if constexpr (PASS == 1) pass1_sum(acc, t);
          else pass2_sum(acc, t);
        }
        if constexpr (PASS == 2) pass2_store(tb, true);
      }
    };
    // Mask-free tiles, pipelined: the products of a row tile (or of the next tile's first) beside the
    // exponentials and sums of the one before.
    auto sum = [&](const f32x16& acc, int t) {
      if constexpr (PASS == 1) pass1_sum(acc, t);
      else pass2_sum(acc, t);
    };
    auto run_clean = [&](int end) {
      if (j >= end) return;
      f32x16 acc[2];
      int tb = read_tile();
      products(acc[0], 0);
      refill();
      // tile of step j, its row tile 0's scores in acc[par]; true after the last
      auto tile = [&](auto par_tag) -> bool {
        constexpr int par = decltype(par_tag)::value;
#pragma unroll
        for (int t = 1; t < RT; ++t) {
          products(acc[(par + t) & 1], t);
          sum(acc[(par + t - 1) & 1], t - 1);
          interleave_mfma_valu<8, 6>();
        }
        const int tb0 = tb;
        ++j;
        if (j >= end) {
          sum(acc[(par + RT - 1) & 1], RT - 1);
          if constexpr (PASS == 2) pass2_store(tb0, false);
          return true;
        }
        tb = read_tile();
        products(acc[(par + RT) & 1], 0);
        sum(acc[(par + RT - 1) & 1], RT - 1);
        interleave_mfma_valu<8, 6>();
        if constexpr (PASS == 2) {
          // the reduction after the sums: beside them its temporaries exceeded the registers
          __builtin_amdgcn_sched_barrier(0);
          pass2_store(tb0, false);
        }
        refill();
        return false;
      };
      for (;;) {
        if (tile(std::integral_constant<int, 0>{})) break;
        if (RT % 2 == 1 && tile(std::integral_constant<int, 1>{})) break;
      }
    };
    // a wave's tiles increase in pass 1, so its mask-free ones come first; in pass 2 they come last
    if constexpr (PASS == 1) {
      const int c = first_dirty - wave + kWaves - 1;             // c / kWaves steps lie below first_dirty
      run_clean(c <= 0 ? 0 : (c / kWaves < steps ? c / kWaves : steps));
      run_dirty(steps);
    } else {
      const int c = ntiles - first_dirty - wave + kWaves - 1;    // c / kWaves steps lie at or past it
      run_dirty(c <= 0 ? 0 : (c / kWaves < steps ? c / kWaves : steps));
      run_clean(steps);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // padding loads land before the block ends
  }

  if constexpr (PASS == 1) {
    // merge the 2 lane halves, then the waves, and publish per-row (max, sum) of this split
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      // no visible key: the empty (max, sum).  A logit of +inf leaves NaN in one half's sum and 0 in the other's
      // (they share the reference): under a maximum of +inf the NaN comes through every merge, and the row gives
      // no key a weight
      if (!(rl[t] > 0.f)) rm[t] = rl[t] == 0.f ? -INFINITY : INFINITY;
      const float m2 = shfl_xor_f(rm[t], 32), l2 = shfl_xor_f(rl[t], 32);
      merge_ml(rm[t], rl[t], m2, l2);
      if (hf == 0) {
        sm.m[wave][32 * t + lr] = rm[t];
        sm.l[wave][32 * t + lr] = rl[t];
      }
    }
    __syncthreads();
    if (tid < kRows) {
      float m = sm.m[0][tid], l = sm.l[0][tid];
      for (int w = 1; w < kWaves; ++w) merge_ml(m, l, sm.m[w][tid], sm.l[w][tid]);
      float* st = p.stats + stat_base + ((int64_t)split * kStatRows + tid) * 2;
      st[0] = m;
      st[1] = l;
    }
  }
}

// ---- top-B -------------------------------------------------------------------

// Inclusive prefix sum over the 64 lanes of a wave with DPP moves (no LDS round trips): shifts by
// 1, 2, 4 and 8 lanes within each row of 16 (lanes without a source add 0), then rows 1 and 3 add
// lane 15 of the row below and rows 2 and 3 add lane 31.
__device__ inline uint32_t wave_inclusive_scan(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);   // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);   // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);   // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);   // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);   // row_bcast:15
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);   // row_bcast:31
  return v;
}

// Exclusive prefix sum of x over the workgroup's threads in thread order; total = the sum of all.
// Every wave scans the wave totals itself, so one barrier separates the two levels; the last one
// lets the next call reuse wsum.
__device__ inline uint32_t block_exclusive_scan(uint32_t x, uint32_t* wsum, uint32_t& total) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int kW = kTopkThreads / kWave;
  const uint32_t v = wave_inclusive_scan(x);
  if (lane == kWave - 1) wsum[wave] = v;
  __syncthreads();
  const uint32_t ws = wave_inclusive_scan(lane < kW ? wsum[lane] : 0u);
  const uint32_t below = wave > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)ws, wave - 1) : 0u;
  total = (uint32_t)__builtin_amdgcn_readlane((int)ws, kW - 1);
  __syncthreads();
  return below + v - x;
}

// Add one to bin `d` of a histogram held in `stride` copies (bin d's copy c at d*stride + c; this
// lane adds to copy `copy`).  When every active lane of the wave holds the same digit one lane adds
// the count to copy 0.  Otherwise each lane adds one: an LDS atomic serialises the lanes that meet
// on one word, and the copies spread lanes with equal digits over `stride` words.
__device__ inline void hist_add(uint32_t* hist, uint32_t d, uint32_t stride, uint32_t copy) {
  const uint64_t active = __builtin_amdgcn_read_exec();
  const uint32_t d0 = __builtin_amdgcn_readfirstlane(d);
  const uint64_t same = __builtin_amdgcn_ballot_w64(d == d0);
  if (same == active) {
    if ((uint32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(active >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)active, 0u)) == 0u)
      atomicAdd(&hist[d0 * stride], (uint32_t)__builtin_popcountll(active));
  } else {
    atomicAdd(&hist[d * stride + copy], 1u);
  }
}

template <int V>
struct IntTag { static constexpr int value = V; };

// Code size matters here: every wave runs each phase once, so a fully unrolled kernel is bound
// by instruction fetch (75 KB of straight-line code measured 39 us).  Only the pooling keeps its
// candidates in registers; it stores them in LDS and every later phase is a short loop over them.
// One workgroup runs the whole (sequence, KV head), so the phases are bound by the CU's own LDS and
// VALU throughput: candidate c belongs to thread c % kTopkThreads (slot e = c / kTopkThreads), so
// a wave's lanes hold consecutive candidates: pooling reads consecutive LDS words (no bank
// conflicts), the keys sit at keys[c], and the ordered compaction ranks candidates by ballots.
__global__ __launch_bounds__(kTopkThreads) void topk_kernel(SelectParams p) {
  constexpr int kTopkWaves = kTopkThreads / kWave;
  constexpr int kPad = 4;                              // -1 words on either side of the staged range
  constexpr int kCells = kMaxPerThread * kTopkWaves;   // (slot, wave) cells of the compaction
  static_assert(2 * kCells <= kHistWords, "compaction counts live in the histogram's space");
  __shared__ float raw_lds[BD_SELECT_MAX_PREFIX + 2 * kPad];   // the pooled range, staged once; then the keys
  __shared__ __align__(16) uint32_t hist[kHistWords];
  __shared__ uint32_t wsum[kTopkWaves];
  __shared__ uint32_t s_digit, s_krem;
  uint32_t* keys = reinterpret_cast<uint32_t*>(raw_lds);
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int pair = blockIdx.x + fetch_select_args(p);
  const int g = pair % p.Hkv, s = pair / p.Hkv;
  const int L = seq_len(p.kv, s);
  const int B = p.budget, W = p.W, ld = p.ld;
  int32_t* idx_row = p.idx_out + (int64_t)pair * ld;

  if (B >= L) {
    for (int t = tid; t < ld; t += kTopkThreads) idx_row[t] = t < L ? t : -1;
    if (g == 0 && tid == 0) p.nsel_out[s] = L;
    return;
  }
  if (g == 0 && tid == 0) p.nsel_out[s] = ld < L ? ld : L;

  // 1. total raw scores (row blocks summed in order), staged in LDS over the prefix [0, N) at
  // raw_lds[kPad + t] and exported when the caller asked for them; each batch of loads is issued
  // before any is summed
  const int N = L - W, K = p.keep, rad = p.pool_kernel / 2;
  float* raw = p.raw ? p.raw + (int64_t)pair * p.max_L : nullptr;
  const float* part = p.raw_part + (int64_t)pair * p.n_rb * p.max_L;
  constexpr int kStageBatch = 16, kStageRows = 2;
  for (int c0 = 0; c0 < L; c0 += kStageBatch * kTopkThreads) {
    float v[kStageBatch];
#pragma unroll
    for (int e = 0; e < kStageBatch; ++e) {
      const int t = c0 + tid + e * kTopkThreads;
      v[e] = t < L ? part[t] : 0.f;
    }
    // the other row blocks, in order, kStageRows of them loaded at a time: one at a time, each cost a
    // memory round trip (8 blocks of 16K scores: 49 us for the kernel, 23 us with two at a time; four gain nothing more)
    for (int r0 = 1; r0 < p.n_rb; r0 += kStageRows) {
      float y[kStageRows][kStageBatch];
#pragma unroll
      for (int u = 0; u < kStageRows; ++u)
#pragma unroll
        for (int e = 0; e < kStageBatch; ++e) {
          const int t = c0 + tid + e * kTopkThreads;
          y[u][e] = r0 + u < p.n_rb && t < L ? part[(int64_t)(r0 + u) * p.max_L + t] : 0.f;
        }
#pragma unroll
      for (int u = 0; u < kStageRows; ++u)
#pragma unroll
        for (int e = 0; e < kStageBatch; ++e) v[e] += y[u][e];
    }
#pragma unroll
    for (int e = 0; e < kStageBatch; ++e) {
      const int t = c0 + tid + e * kTopkThreads;
      if (t < N) raw_lds[kPad + t] = v[e];
      if (raw && t < L) raw[t] = v[e];
    }
  }
  if (tid < kPad) { raw_lds[tid] = -1.f; raw_lds[kPad + N + tid] = -1.f; }
  __syncthreads();

  // 2. the candidates: prefix positions [0, N) with max-pooled scores (token level), or the chunks
  // of s positions of the prefix with their scores' sums (TopKChunks, chunk c covering
  // [c*s, min((c+1)*s, N)), summed left to right in fp32).  The top KE of the M candidates are
  // kept.  Scores are >= 0, so their float bits order like their values.
  const int chunk = p.chunk;
  const int M = chunk > 0 ? (N + chunk - 1) / chunk : N;
  int KE = chunk > 0 ? K / chunk : K;
  if (KE > M) KE = M;
  const int E = (M + kTopkThreads - 1) / kTopkThreads;   // slots in use
  const float* rl = raw_lds + kPad;
  uint32_t key[kMaxPerThread];
  if (chunk > 0) {
#pragma unroll
    for (int e = 0; e < kMaxPerThread; ++e) {
      const int c = e * kTopkThreads + tid;
      float sum = 0.f;
      if (e < E && c < M) {
        const int b = c * chunk, n = N - b < chunk ? N - b : chunk;
        for (int j = 0; j < n; ++j) sum += rl[b + j];
      }
      key[e] = e < E && c < M ? __float_as_uint(sum) : 0u;
    }
  } else if (rad <= kPad - 1) {
    // radius <= 3: the -1 words around the range stand in for positions outside it (every
    // pooled score is >= 0), so no bounds checks.  Groups of 8 slots, all reads of a group issued
    // together; a slot past E reads words inside the array and is masked.
    auto pool = [&](auto rtag) {
      constexpr int R = decltype(rtag)::value;
#pragma unroll
      for (int e0 = 0; e0 < kMaxPerThread; e0 += 8) {
        if (e0 < E) {
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int e = e0 + j, c = e * kTopkThreads + tid;
            float m = rl[c];
#pragma unroll
            for (int d = 1; d <= R; ++d) m = fmaxf(m, fmaxf(rl[c - d], rl[c + d]));
            key[e] = e < E && c < N ? __float_as_uint(m) : 0u;
          }
        } else {
#pragma unroll
          for (int j = 0; j < 8; ++j) key[e0 + j] = 0u;
        }
      }
    };
    if (rad == 3) pool(IntTag<3>{});
    else if (rad == 2) pool(IntTag<2>{});
    else if (rad == 1) pool(IntTag<1>{});
    else pool(IntTag<0>{});
  } else {
    auto raw_at = [&](int t) { return t >= 0 && t < N ? rl[t] : -1.f; };
    float m[kMaxPerThread];
#pragma unroll
    for (int e = 0; e < kMaxPerThread; ++e) m[e] = -1.f;
    for (int d = -rad; d <= rad; ++d) {
#pragma unroll
      for (int e = 0; e < kMaxPerThread; ++e)
        if (e < E) m[e] = fmaxf(m[e], raw_at(e * kTopkThreads + tid + d));
    }
#pragma unroll
    for (int e = 0; e < kMaxPerThread; ++e)
      key[e] = e < E && e * kTopkThreads + tid < N ? __float_as_uint(m[e]) : 0u;
  }
  __syncthreads();                            // every raw value read: the LDS now holds the keys
#pragma unroll
  for (int e = 0; e < kMaxPerThread; ++e)
    if (e < E) keys[e * kTopkThreads + tid] = key[e];
  __syncthreads();
  // Keys in batches of kBatch slots, every read issued before the first is used (an LDS atomic or a
  // ballot between a read and the next would otherwise wait for the LDS round trip each slot).
  // Slots past E read slot E-1 again: the caller's c < M test rejects them.
  constexpr int kBatch = 8;
  auto load_keys = [&](uint32_t (&k)[kBatch], int e0) {
#pragma unroll
    for (int j = 0; j < kBatch; ++j) k[j] = keys[(e0 + j < E ? e0 + j : E - 1) * kTopkThreads + tid];
  };

  // 3. radix select of the KE-th largest key over digits of 8, 11 and 12 bits: the exponent, then
  // the mantissa's top 11 and low 12 bits (the sign bit is always clear); krem = how many keys
  // equal to it are taken.  Most scores share a few exponents and their neighbours share leading
  // mantissa bits, so lane l adds to copy l % 16 (exponent) or l % 2 (top mantissa bits) of the
  // histogram: with one copy of a 12-bit first digit about 18 lanes of a wave met on one word and
  // the serialised atomics took 5 us of the kernel.
  uint32_t prefix = 0, pmask = 0, krem = (uint32_t)KE;
  if (KE > 0) {
    for (int pass = 0; pass < kDigits; ++pass) {
      const int bits = digit_bits(pass), shift = digit_shift(pass);
      const uint32_t ncopy = (uint32_t)digit_copies(pass);
      const uint32_t copy = (uint32_t)lane & (ncopy - 1u);
      const uint32_t nb = 1u << bits, dm = nb - 1;
      for (int i = tid; i < (int)(nb * ncopy); i += kTopkThreads) hist[i] = 0;
      __syncthreads();
      for (int e0 = 0; e0 < E; e0 += kBatch) {
        uint32_t k[kBatch];
        load_keys(k, e0);
#pragma unroll
        for (int j = 0; j < kBatch; ++j)
          if ((e0 + j) * kTopkThreads + tid < M && (k[j] & pmask) == prefix)
            hist_add(hist, (k[j] >> shift) & dm, ncopy, copy);
      }
      __syncthreads();
      // thread tid owns digits nb-1 - (per*tid + q): a block scan counts the keys above them
      constexpr int kMaxPer = kHistWords / kTopkThreads;
      const int per = (int)nb >= kTopkThreads ? (int)nb / kTopkThreads : 1;
      uint32_t h[kMaxPer], c = 0;
#pragma unroll
      for (int q = 0; q < kMaxPer; ++q) {
        const uint32_t x = (uint32_t)(per * tid + q), d = nb - 1 - x;
        h[q] = 0;
        if (q < per && x < nb) {
          if (ncopy >= 4) {
            const uint4* w = reinterpret_cast<const uint4*>(hist + d * ncopy);
            for (uint32_t i = 0; i < ncopy / 4; ++i) { const uint4 v = w[i]; h[q] += v.x + v.y + v.z + v.w; }
          } else if (ncopy == 2) {
            const uint2 v = *reinterpret_cast<const uint2*>(hist + d * 2);
            h[q] = v.x + v.y;
          } else {
            h[q] = hist[d];
          }
        }
        c += h[q];
      }
      uint32_t tot;
      uint32_t a = block_exclusive_scan(c, wsum, tot);
#pragma unroll
      for (int q = 0; q < kMaxPer; ++q) {
        if (q < per && a < krem && krem <= a + h[q]) { s_digit = nb - 1 - (uint32_t)(per * tid + q); s_krem = krem - a; }
        a += h[q];
      }
      __syncthreads();
      prefix |= s_digit << shift;
      pmask |= dm << shift;
      krem = s_krem;
      __syncthreads();
    }
  }

  // 4. ordered compaction: all candidates above the threshold, the first krem equal to it, in
  // ascending order.  Cell (e, wave) holds candidates e*kTopkThreads + 64*wave + [0, 64): ballots
  // count each cell's keys above and equal to the threshold, two scans over the cells in candidate
  // order give each cell its first equal key's rank and its first output slot, and a lane adds the
  // ballot's lanes below it.  A candidate contributes its positions (one, or its chunk's: every
  // chunk but the last has s of them, so a taken candidate's first slot is its rank times s).
  uint32_t* c_eq = hist;                      // per cell: equal keys, then equal keys before it
  uint32_t* c_gt = hist + kCells;             // per cell: keys above, then output slots before it
  const uint64_t below = (1ull << lane) - 1ull;
  const bool any = KE > 0;
  for (int e0 = 0; e0 < E; e0 += kBatch) {
    uint32_t k[kBatch];
    load_keys(k, e0);
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int e = e0 + j, c = e * kTopkThreads + tid;
      const uint64_t beq = __builtin_amdgcn_ballot_w64(any && c < M && k[j] == prefix);
      const uint64_t bgt = __builtin_amdgcn_ballot_w64(any && c < M && k[j] > prefix);
      if (lane == 0 && e < E) {
        c_eq[e * kTopkWaves + wave] = (uint32_t)__builtin_popcountll(beq);
        c_gt[e * kTopkWaves + wave] = (uint32_t)__builtin_popcountll(bgt);
      }
    }
  }
  __syncthreads();
  const int ncell = E * kTopkWaves;
  const uint32_t n_eq = tid < ncell ? c_eq[tid] : 0u, n_gt = tid < ncell ? c_gt[tid] : 0u;
  // One scan of both counts packed as equal << 16 | above (each sum is at most 32768).  The equal
  // keys are taken in candidate order until krem of them are, so min(krem, equal keys before) of
  // them lie in earlier cells.
  uint32_t tot;
  const uint32_t before = block_exclusive_scan(n_eq << 16 | n_gt, wsum, tot);
  const uint32_t eq_before = before >> 16, take_before = (before & 0xFFFFu) + min(krem, eq_before);
  const int taken = (int)((tot & 0xFFFFu) + min(krem, tot >> 16));   // candidates kept
  // Prefix positions kept: unit per taken candidate, less the missing positions of a short last
  // chunk when it is taken (all other equal keys precede it, so an equal last key is taken only
  // when every equal key is).  The window and the unused slots are written first.
  const int unit = chunk > 0 ? chunk : 1;
  int kept = taken * unit;
  if (chunk > 0 && M > 0) {
    const uint32_t kl = keys[M - 1];
    if (any && (kl > prefix || (kl == prefix && krem == tot >> 16))) kept -= unit - (N - (M - 1) * chunk);
  }
  if (kept > K) kept = K;
  for (int i = tid; i < W; i += kTopkThreads) idx_row[kept + i] = N + i;
  for (int i = kept + W + tid; i < ld; i += kTopkThreads) idx_row[i] = -1;   // unused slots
  if (tid < ncell) { c_eq[tid] = eq_before; c_gt[tid] = take_before; }
  __syncthreads();
  for (int e0 = 0; e0 < E; e0 += kBatch) {
    uint32_t k[kBatch], eqb[kBatch], tkb[kBatch];
    load_keys(k, e0);
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int cell = (e0 + j < E ? e0 + j : E - 1) * kTopkWaves + wave;
      eqb[j] = c_eq[cell];
      tkb[j] = c_gt[cell];
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int c = (e0 + j) * kTopkThreads + tid;
      const bool isq = any && c < M && k[j] == prefix;
      const uint64_t beq = __builtin_amdgcn_ballot_w64(isq);
      const bool take = (any && c < M && k[j] > prefix) ||
                        (isq && eqb[j] + (uint32_t)__builtin_popcountll(beq & below) < krem);
      const uint64_t bt = __builtin_amdgcn_ballot_w64(take);
      if (take) {
        const int off = ((int)tkb[j] + __builtin_popcountll(bt & below)) * unit;
        if (chunk == 0) {
          if (off < K) idx_row[off] = c;      // guard: never write past the K prefix slots
        } else {
          const int b = c * chunk, n = N - b < chunk ? N - b : chunk;
          for (int i = 0; i < n; ++i)
            if (off + i < K) idx_row[off + i] = b + i;
        }
      }
    }
  }
}

template <int RT, bool PAGED>
hipError_t launch_scores(const SelectParams& p, int nblocks, hipStream_t stream) {
  if (!p.lse_win) {
    hipLaunchKernelGGL((score_kernel<RT, PAGED, 1>), dim3(nblocks), dim3(kThreads), 0, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((score_kernel<RT, PAGED, 2>), dim3(nblocks), dim3(kThreads), 0, stream, p);
  return hipGetLastError();
}

// 32-row tiles of a row block: n_rb blocks of at most 128 rows, of equal size
int select_blocks(int R) { return (R + kStatRows - 1) / kStatRows; }
int select_rt(int R) {
  const int n_rb = select_blocks(R);
  return ((R + n_rb - 1) / n_rb + 31) / 32;
}

}  // namespace

SelectPlan plan_select(int S, int Hkv, int Hq, int W, int max_L, bool paged, int page_size) {
  SelectPlan pl;
  const int G = Hq / Hkv;
  const int R = W * G;
  pl.n_rb = select_blocks(R);
  const int64_t units = (int64_t)S * Hkv * pl.n_rb;
  constexpr int64_t kStep = kWaves * kTile;
  // a paged split's table holds kSlotCap entries: one per key, or one per page when pages hold whole
  // 16-key sub-tiles (kps keys span at most kps / page_size + 2 pages); keys below 2^26 keep the
  // kernel's page division exact
  pl.page_arith = paged && page_size > 0 && page_size % 16 == 0 && max_L <= (1 << 26) - 64;
  const int64_t cap = !paged ? INT64_MAX
                             : (pl.page_arith ? ((int64_t)(kSlotCap - 2) * page_size) / kStep * kStep : kMaxPagedKeys);
  // Keys per split.  A CU holds one workgroup, so the launch runs in rounds of kTargetBlocks workgroups and
  // the count that ends first is taken: rounds x (a split's keys + the fixed cost of a workgroup, ~7 us
  // beside 2 us per 256 keys).  Just filling the CUs once, 18 sequences of 20K with 8 KV heads (144 units)
  // took two splits each, 288 workgroups in two rounds, the second nearly empty; with five each (2.8 rounds
  // of a fifth) the two passes take 129 + 141 us there instead of 226 + 210 (the 32x32 row tiles included).
  // Only the largest split counts of 1, 2, ... whole rounds can be best.
  constexpr int64_t kFixedKeys = 768;
  const int64_t whole = max_L > 0 ? (max_L + kStep - 1) / kStep * kStep : kStep;
  int64_t kps = whole, best = INT64_MAX;
  for (int64_t r = 1; r <= 16; ++r) {
    int64_t ns = kTargetBlocks * r / units;
    if (ns < 1) ns = 1;
    int64_t k = (whole / kStep + ns - 1) / ns * kStep;
    if (k > cap) k = cap;
    const int64_t blocks = units * ((whole + k - 1) / k);
    const int64_t cost = (blocks + kTargetBlocks - 1) / kTargetBlocks * (k + kFixedKeys);
    if (cost < best) { best = cost; kps = k; }
  }
  pl.kps = (int)kps;
  pl.nsplit = max_L > 0 ? (int)((max_L + kps - 1) / kps) : 1;
  pl.stats_bytes = align256(sizeof(float) * (size_t)units * pl.nsplit * kStatRows * 2);
  pl.raw_part_bytes = align256(sizeof(float) * (size_t)units * max_L);
  pl.ws_bytes = BD_WS_COUNTER_BYTES + pl.stats_bytes + pl.raw_part_bytes;
  return pl;
}

hipError_t launch_select(const SelectParams& p, bool paged, hipStream_t stream) {
  const int nblocks = p.S * p.Hkv * p.n_rb * p.nsplit;
  hipError_t e = hipSuccess;
  switch (select_rt(p.R)) {
    case 1: e = paged ? launch_scores<1, true>(p, nblocks, stream) : launch_scores<1, false>(p, nblocks, stream); break;
    case 2: e = paged ? launch_scores<2, true>(p, nblocks, stream) : launch_scores<2, false>(p, nblocks, stream); break;
    case 3: e = paged ? launch_scores<3, true>(p, nblocks, stream) : launch_scores<3, false>(p, nblocks, stream); break;
    default: e = paged ? launch_scores<4, true>(p, nblocks, stream) : launch_scores<4, false>(p, nblocks, stream); break;
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(topk_kernel, dim3(p.S * p.Hkv), dim3(kTopkThreads), 0, stream, p);
  return hipGetLastError();
}

}  // namespace bd
