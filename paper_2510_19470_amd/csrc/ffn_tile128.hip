// Grouped bf16 expert GEMMs in tiles of 128 token rows x 128 weight rows, for layers whose 256 x 256
// tiles (ffn_mfma.hip) are about two rounds on the chip or less.  (Paper Sec. 2.1, 3.1: as there.)
//
// Such launches are bound by the time of one tile, whatever it holds, by compute units without one and
// by the partial sums of the K-split that fills them.  A quarter of the tile divides the work finer,
// and two blocks of 256 threads on a compute unit cover each other's start, waits and epilogue.  What it
// costs is half as much work per byte copied into LDS: 32 KB per 2.1e6 operations, at the copy path's
// 15 TB/s about 1000 TFLOP/s, which is why full chips keep the larger tile.
//
// 4 wavefronts (2 along rows x 2 along columns), wavefront tile 64 x 64 = 2 x 2 accumulators of
// v_mfma_f32_32x32x16_bf16; k-steps of 64 through two LDS stages of 32 KB.  A step: wait for its copies,
// read all 16 fragments, issue the copies of the step after the next into the same stage, 16 MFMAs.
// (Three stages where at most 64 rows need 24 KB a step: no difference.)
// 32-row blocks that hold no rows are neither copied nor multiplied.
// No schedule launch: every block counts the tiles from the counts (one scan over the experts) and finds
// its own by a search.  A contraction is cut into parts only where there are tiles for at most half of
// the resident blocks; the blocks add the parts themselves (join_parts).
#include <algorithm>

#include "ffn_tile.h"

namespace {

constexpr int TM = 128;          // token rows per tile
constexpr int TN = 128;          // weight rows per tile (gate/up: 64 of each matrix)
constexpr int NT = 256;          // threads
constexpr int OPERAND = TM * BK * 2;      // bytes of an operand's part of a stage
constexpr int STAGE = 2 * OPERAND;
constexpr int SPLIT_MAX = 8;     // parts of a contraction at most
constexpr int SPLIT_STEPS = 4;   // k-steps of a part at least
constexpr int ORDER_GROUP_M = 8; // row blocks per group of the tile order

struct TileArgs {
  GemmArgs g;
  const int32_t *counts, *offsets;
  const void* const* present;    // [E] experts with weights
  const void* const* b0;         // [E] weight-role operand
  const void* const* b1;         // [E] gate/up: W3; k-major: the second segment's (may be nullptr)
  int E, S;
  TileSched* status;             // n_mtiles for the kernels after this one: 0 if counts do not fit
  bool offered;                  // dH: status is the larger tiles' schedule, and says whose turn it is
  bool again;                    // forward: the pass reads the weights again
};

// Row blocks of all experts, counted by every block for itself: start[e] is the first one of expert e.
// Everything that a tile needs to know of its expert is loaded at once here (a block's start is a chain of
// cold loads otherwise, 1 to 2 us each).
struct TileMap {
  int32_t start[MOE_MAX_EXPERTS + 1];
  int32_t wave_sum[NT / 64], wave_used[NT / 64];
  int32_t rows[MOE_MAX_EXPERTS], row0[MOE_MAX_EXPERTS];
  const void *b0[MOE_MAX_EXPERTS], *b1[MOE_MAX_EXPERTS];
};
// Called by all threads; returns the number of row blocks (0 when a segment of a present expert does not
// lie inside the S rows of the buffers, or they are more than S rows can have) and the experts that have any.
__device__ __forceinline__ int count_tiles(const TileArgs& p, TileMap& m, int& used) {
  static_assert(NT == MOE_MAX_EXPERTS, "one expert per thread");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int mine = 0;
  bool bad = false;
  if (tid < p.E) {
    const void* w = p.present[tid];
    const int n = p.counts[tid], o = p.offsets[tid];
    const void* b0 = p.b0[tid];
    const void* b1 = p.b1 != nullptr ? p.b1[tid] : b0;
    if (w != nullptr) {
      bad = n < 0 || o < 0 || (long)o + n > (long)p.S;
      mine = bad ? 0 : (n + TM - 1) / TM;
    }
    m.rows[tid] = n;
    m.row0[tid] = o;
    m.b0[tid] = b0;
    m.b1[tid] = b1;
  }
  int incl = mine;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int v = __shfl_up(incl, off, 64);
    if (lane >= off) incl += v;
  }
  const int some = __popcll(__ballot(mine > 0));
  if (lane == 63) m.wave_sum[wave] = incl, m.wave_used[wave] = some;
  const int any_bad = __syncthreads_or(bad);
  for (int w = 0; w < wave; ++w) incl += m.wave_sum[w];
  m.start[tid + 1] = incl;
  if (tid == 0) m.start[0] = 0;
  __syncthreads();
  used = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) used += __builtin_amdgcn_readfirstlane(m.wave_used[w]);
  const int total = __builtin_amdgcn_readfirstlane(m.start[MOE_MAX_EXPERTS]);
  return any_bad || total > p.S / TM + p.E ? 0 : total;   // (segments that overlap)
}

// Parts of every contraction of a launch of `tiles` tiles on `slots` resident blocks, two on a compute unit: the
// number that is done first by its k-steps and the levels of neighbours that add their sums (join_parts), 3.9 steps each.
// Where there are units with two blocks, a step is 2.3 times as long if every tile has weights of its own, which one
// block on every unit streams as fast as they come, and 1.8 times if tiles share them (one_block: experts have
// one row block, or three in two of them at most).  From 482 GEMMs of 2 to 256 tiles, 8 to 256 steps, 5 to 1000 rows
// per expert, forward and backward, weights from HBM, with every number of parts; from the fastest one, mean and
// most: one row block 0.2 us, 5 us (1.8: 0.6, 14 us); more of them 0.3, 9 us (2.3: 2.1, 60 us or 24 %); as many parts as
// there are blocks for 2.8 us, 29 %.  Both GEMMs, us, 1, 2, 3, 4 ... parts of the second: one row block: 12 tiles of 46
// steps 55, 41, 38, 36, 37, 35, 34, 35; 48 of 64: 67, 50, 46, 44, 45, 49; 128 of 16: 42, 42, 45, 47; 240 of 112: 163, 174; more: 96
// of 128: 141, 98, 88, 86, 85; 216 of 94: 206, 181; 192 of 256: 310, 250.
__host__ __device__ inline int join_levels(int parts) { return parts > 4 ? 3 : parts > 2 ? 2 : parts - 1; }
__host__ __device__ inline int parts_of(int tiles, int slots, int kt, bool one_block) {
  auto best = [&](int most, float two) {
    const int one_each = slots / 2 > SPLIT_MAX ? slots / 2 : SPLIT_MAX;
    int parts = 1;
    float least = (float)kt;
    for (int n = 2; n <= most && tiles * n <= slots && kt / n >= SPLIT_STEPS; ++n) {
      const float t = (float)((kt + n - 1) / n) * (tiles * n <= one_each ? 1.f : two) + 3.9f * join_levels(n);
      if (t < least) least = t, parts = n;
    }
    return parts;
  };
  return best(best(SPLIT_MAX, 1.f), one_block ? 2.3f : 1.8f);   // no more than of one tile alone: the workspace is sized for those
}

// ---- Contractions that are cut into parts.  The blocks add the parts of a tile themselves, as a tree over
// neighbours (0 + 1) + (2 + 3) ...: of two neighbours the one that is done first publishes its sum and ends, the
// other adds it to its own registers and goes on to the next level.  Nobody waits for anybody, so the blocks
// need not be resident together, and the result does not depend on who comes first (a + b is b + a).
// The sums and the counters are written and read with device-scope relaxed atomics, which go past the L2 of an
// XCD to what all XCDs share; a sum is complete there (vmcnt 0 in every wavefront, then the barrier) before its
// counter says so.
constexpr int JOIN_COUNTERS = SPLIT_MAX;   // of a tile: 4 + 2 + 1 pairs; zero between launches

typedef unsigned long long join_word;
__device__ __forceinline__ int join_get(int32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Called by all threads of a block, each with its own 64 accumulators.  slots: one partial tile for every part;
// n_act: 32-row blocks of this wavefront that hold rows (the same in every part); flag: JOIN_COUNTERS integers of
// LDS.  True: the accumulators hold the whole sum.
__device__ __forceinline__ bool join_parts(f32x16 (&acc)[2][2], float* slots, int32_t* counters, int part, int parts,
                                           int n_act, int32_t* flag) {
  const int tid = threadIdx.x;
  int node = part, width = parts, first = 0;
  for (int level = 0; width > 1; ++level) {
    if ((node ^ 1) < width) {
      int32_t* count = counters + first + (node >> 1);
      if (tid == 0) flag[2 * level] = join_get(count);
      __syncthreads();
      if (__builtin_amdgcn_readfirstlane(flag[2 * level]) == 0) {   // the neighbour is not there yet: publish
        join_word* mine = reinterpret_cast<join_word*>(slots + (size_t)(node << level) * (TM * TN)) + tid;
#pragma unroll
        for (int i = 0; i < 2; ++i)
          if (i < n_act)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
              for (int q = 0; q < 8; ++q) {
                const float2 v = make_float2(acc[j][i][2 * q], acc[j][i][2 * q + 1]);
                __hip_atomic_store(mine + ((i * 2 + j) * 8 + q) * NT, __builtin_bit_cast(join_word, v),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0)
          flag[2 * level + 1] = __hip_atomic_fetch_add(count, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(flag[2 * level + 1]) == 0) return false;   // the neighbour goes on with it
      }
      if (tid == 0) __hip_atomic_store(count, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      join_word* theirs = reinterpret_cast<join_word*>(slots + (size_t)((node ^ 1) << level) * (TM * TN)) + tid;
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (i < n_act) {
          join_word v[2][8];
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 8; ++q)
              v[j][q] = __hip_atomic_load(theirs + ((i * 2 + j) * 8 + q) * NT, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 8; ++q) {
              const float2 t = __builtin_bit_cast(float2, v[j][q]);
              acc[j][i][2 * q] += t.x;
              acc[j][i][2 * q + 1] += t.y;
            }
        }
    }
    first += (width + 1) >> 1;
    node >>= 1;
    width = (width + 1) >> 1;
  }
  return true;
}

// One tile, or one part of its contraction (all fields wave-uniform).
struct Unit128 {
  int valid, expert, row0, rows, nblk;
  int kstart, KT;          // first k-step and their number
  int tile, part, parts;   // index in the order; parts > 1: this is one of them
  int once;                // the expert's only row block: nobody else reads these weights
};

// Tile L of the order: expert by expert; inside an expert in groups of 8 row blocks; inside a group
// column block by column block, the group's row blocks in a row (they share a weight panel).
__device__ __forceinline__ Unit128 find_tile(const TileArgs& p, const TileMap& m, int L) {
  Unit128 u;
  const int nt = p.g.n_tiles_n;
  int lo = 0, hi = p.E;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (m.start[mid] * nt <= L) lo = mid; else hi = mid;
  }
  lo = __builtin_amdgcn_readfirstlane(lo);
  const int first = __builtin_amdgcn_readfirstlane(m.start[lo]);
  const int me = __builtin_amdgcn_readfirstlane(m.start[lo + 1]) - first;
  const int rel = L - first * nt, mg = rel / (ORDER_GROUP_M * nt), r2 = rel % (ORDER_GROUP_M * nt);
  const int gm = min(ORDER_GROUP_M, me - mg * ORDER_GROUP_M);
  const int mb = mg * ORDER_GROUP_M + r2 % gm;
  u.valid = 1;
  u.expert = lo;
  u.nblk = r2 / gm;
  u.row0 = __builtin_amdgcn_readfirstlane(m.row0[lo]) + mb * TM;
  u.rows = min(TM, __builtin_amdgcn_readfirstlane(m.rows[lo]) - mb * TM);
  u.kstart = 0;
  u.KT = p.g.kt;
  u.tile = L;
  u.part = 0;
  u.parts = 1;
  u.once = me == 1;
  return u;
}

// MODE_UP .. MODE_DH1, BKM, and what happens at sizes that the tile does not divide: as
// ffn_mfma_kernel's (here always its RAG form).
template <int MODE, bool BKM>
__global__ __launch_bounds__(NT, 2) void ffn_tile128_kernel(const TileArgs p) {
  __shared__ uint4 lds[2 * STAGE / 16];
  __shared__ TileMap map;
  __shared__ int32_t join_flag[JOIN_COUNTERS];
  const GemmArgs& g = p.g;
  // (dH, whose epilogue is long, is not cut: 1 % slower where it need not be.  Gate/up, 3 experts of 2048 x 2048, 100
  // tokens: pass 51.7 -> 46.2 us)
  constexpr bool CUT = MODE != MODE_DH && MODE != MODE_DH1;
  if ((MODE == MODE_DH || MODE == MODE_DH1) && p.offered && p.status->dh_small == 0) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  int used;
  const int blocks128 = count_tiles(p, map, used), total = blocks128 * g.n_tiles_n;
  const int split = CUT ? parts_of(total, gridDim.x, g.kt, 2 * blocks128 < 3 * used) : 1;
  if (blockIdx.x == 0 && threadIdx.x == 0 && !p.offered) p.status->n_mtiles = total;
  const int units = total * split;
  // The idx-th unit of this block: rounds of gridDim.x units, a round in 8 chunks of consecutive ones
  // for the XCDs (blocks with index = x mod 8 are on XCD x), the last round in 8 equal chunks as well.
  auto fetch = [&](int idx) -> Unit128 {
    Unit128 u;
    u.valid = 0;
    const int G = (int)gridDim.x, x = blockIdx.x & 7, slot = (int)(blockIdx.x >> 3);
    const int full = units / G, last = units - full * G, per_last = (last + 7) >> 3;
    int U;
    if (idx < full) U = idx * G + x * (G >> 3) + slot;
    else if (idx == full && slot < per_last && x * per_last + slot < last) U = full * G + x * per_last + slot;
    else return u;
    u = find_tile(p, map, U / split);
    if (split > 1) {
      const int part = U % split, base = g.kt / split, rem = g.kt % split;
      u.kstart = part * base + min(part, rem);
      u.KT = base + (part < rem ? 1 : 0);
      u.part = part;
      u.parts = split;
    }
    return u;
  };

  // ---- copies.  Row-major operand: instruction c (0..15) fills rows 8c + (lane >> 3), 8 chunk slots
  // each, slot s of row r holds chunk s ^ swz(r); k-major: k-rows 4c + (lane >> 4), 16 slots each, s ^
  // tr_swz(r).  Wavefront w issues c = w + 4i: i is the 32-row block of the tokens.
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)lds;
  const uint32_t a_pitch = g.lda * 2, b_pitch = BKM ? g.ldb * 2 : g.K * 2;
  const int lc = (lane & 7) ^ swz(8 * wave + (lane >> 3));   // the lane's chunk of a row-major step
  uint32_t a_off[4], b_off[4];
  const char *a_base, *b_base0, *b_base1;
  bool once;
  auto open = [&](const Unit128& u) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = 8 * (wave + 4 * i) + (lane >> 3);
      a_off[i] = (uint32_t)min(r, u.rows - 1) * a_pitch + lc * 16;
      if (BKM) {
        const int kr = 4 * (wave + 4 * i) + (lane >> 4);
        b_off[i] = (uint32_t)kr * b_pitch + min((lane & 15) ^ tr_swz(kr), (g.N - u.nblk * TN) / 8 - 1) * 16;
      } else if (MODE == MODE_UP) {   // i = 0, 1: rows of W1; 2, 3: the same rows of W3
        b_off[i] = (uint32_t)min(r & 63, g.N - 1 - u.nblk * 64) * b_pitch + lc * 16;
      } else {
        b_off[i] = (uint32_t)min(r, g.N - 1 - u.nblk * TN) * b_pitch + lc * 16;
      }
    }
    a_base = uniform_ptr(g.A + (size_t)u.row0 * g.lda);
    const size_t ofs = BKM ? (size_t)u.nblk * (TN * 2)
                           : (size_t)u.nblk * (MODE == MODE_UP ? 64 : TN) * b_pitch;
    b_base0 = uniform_ptr((const char*)map.b0[u.expert] + ofs);
    b_base1 = uniform_ptr((const char*)map.b1[u.expert] + ofs);
    once = u.once && (BKM || (!p.again && (((uintptr_t)b_base0 | (uintptr_t)b_base1 | b_pitch) & 127) == 0));
  };
  // copies of step t into stage t & 1: weight rows, then the token rows' na blocks
  auto issue = [&](const Unit128& u, int na, int t) {
    const int kg = u.kstart + t, kk = kg < g.kseg ? kg : kg - g.kseg;   // step inside its segment
    const int kv = g.kseg_len - kk * BK;                                // k of the step that exist
    const uint32_t dst = lds0 + (t & 1) * STAGE + wave * 1024;
    const char* a = a_base + (kg < g.kseg ? 0 : (size_t)g.kseg_len * 2) + kk * (BK * 2);
    const char* b[2];   // weight rows of copies 0, 1 and 2, 3
    if (BKM) b[0] = b[1] = (kg < g.kseg ? b_base0 : b_base1) + (size_t)kk * BK * b_pitch;
    else b[0] = b_base0 + kk * (BK * 2), b[1] = (MODE == MODE_UP ? b_base1 : b_base0) + kk * (BK * 2);
    if (kv < BK) {   // the step ends inside the segment: zeros for the rest
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (i < na) dma16v(lc < kv >> 3 ? a + a_off[i] : g.zero, dst + OPERAND + i * 4096);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        dma16v((BKM ? 4 * (wave + 4 * i) + (lane >> 4) < kv : lc < kv >> 3) ? b[i >> 1] + b_off[i] : g.zero,
               dst + i * 4096);
      return;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i < na) dma16(a_off[i], a, dst + OPERAND + i * 4096);
    // Weights that one tile alone reads are copied past the last-level cache, where they would displace
    // activations and weights that are read again.  64 tokens, 8 experts of 4096 x 14336: pass 518 -> 465 us (gate/up
    // 5.8 -> 6.5 TB/s); two-matrix training, 64 rows per expert of 1024 x 4096: 225 -> 200.  Rows in pieces of 128 bytes only
    // where those are lines (177 tokens, 1880 x 3928: 243 -> 283; 2858 tokens, 1528 x 2592: 156 -> 173; k-major ones in pieces of
    // 256 anywhere: backward, 584 tokens, 1888 x 2256: 176 -> 156), and not where the pass itself
    // reads them again (chunks of a pipeline: 2048 tokens in four, 12 of 64 experts of 2048 x 1408: 271 -> 310).  It pays on
    // layers that fit the cache as well, as long as other layers run in between (four in turn, 151 MB of weights:
    // 50 -> 45, 208 MB: 59 -> 55); one that runs alone again and again loses (101 MB: 28 -> 31, 151: 37 to 40 -> 44,
    // 208: 43 -> 58, 302: 65 -> 67).  With two row blocks the second one finds the weights in L2 less often: 250
    // rows per expert, 1160 x 2888: 117 -> 133.
    if (once) {
#pragma unroll
      for (int i = 0; i < 4; ++i) dma16_once(b_off[i], b[i >> 1], dst + i * 4096);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) dma16(b_off[i], b[i >> 1], dst + i * 4096);
    }
  };

  // ---- fragment reads
  const int fr_row = lane & 31, fr_half = lane >> 5, fr_swz = swz(fr_row);
  uint32_t tr_adr[2];   // k-major: LDS byte address of the lane's 4 columns, k-rows 0..3 of a slice
  {
    const int g16 = lane >> 4, j4 = (lane & 15) >> 2, q4 = lane & 3, row = 8 * (g16 >> 1) + j4;
#pragma unroll
    for (int j = 0; j < 2; ++j)
      tr_adr[j] = lds0 + row * 256 + (q4 & 1) * 8 +
                  ((((j * 64 + wn * 32 + (g16 & 1) * 16) / 8 + (q4 >> 1)) ^ tr_swz(row)) << 4);
  }

  Unit128 cur = fetch(0);
  if (!cur.valid) return;
  auto blocks = [](const Unit128& u) { return (u.rows + 31) >> 5; };   // 32-row blocks that hold rows
  int na = blocks(cur);
  auto start = [&](const Unit128& u, int blocks) {
    open(u);
    issue(u, blocks, 0);
    if (u.KT > 1) issue(u, blocks, 1);
  };
  start(cur, na);
  f32x16 acc[2][2];
  for (int idx = 0;; ++idx) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.f;
    const int mine = na - 2 * wm;   // of them this wavefront's
    for (int t = 0; t < cur.KT; ++t) {
      // step t has landed (the 4 + na copies of step t + 1, issued last, may be in flight)
      if (t + 1 == cur.KT) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      else if (na == 4) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
      else if (na == 3) asm volatile("s_waitcnt vmcnt(7)" ::: "memory");
      else if (na == 2) asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(5)" ::: "memory");
      asm volatile("s_barrier" ::: "memory");
      const uint4* Bs = lds + (t & 1) * (STAGE / 16);
      const uint4* As = Bs + OPERAND / 16;
      bf16x8 xa[2][4], wb[2][4];
      if (mine > 0) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            if (BKM) {
              const uint32_t a0 = tr_adr[j] + (t & 1) * STAGE + kk * 4096;
              const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)a0);
              const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)(a0 + 4 * 256));
              const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
              wb[j][kk] = __builtin_bit_cast(bf16x8, v);
            } else {
              wb[j][kk] = __builtin_bit_cast(bf16x8, Bs[(j * 64 + wn * 32 + fr_row) * 8 + ((kk * 2 + fr_half) ^ fr_swz)]);
            }
          }
#pragma unroll
          for (int i = 0; i < 2; ++i)
            if (i < mine)
              xa[i][kk] = __builtin_bit_cast(bf16x8, As[(wm * 64 + i * 32 + fr_row) * 8 + ((kk * 2 + fr_half) ^ fr_swz)]);
        }
      }
      // everybody's reads are done: the stage is free
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      if (t + 2 < cur.KT) issue(cur, na, t + 2);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (i < mine) {
#pragma unroll
          for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int j = 0; j < 2; ++j)
              acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wb[j][kk], xa[i][kk], acc[j][i], 0, 0, 0);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
    // the next unit's first steps fly under this one's epilogue (nobody reads either stage any more)
    const Unit128 nxt = fetch(idx + 1);
    const int na_n = blocks(nxt);
    if (nxt.valid) start(nxt, na_n);
    if (!CUT || cur.parts == 1 ||
        join_parts(acc, g.split_ws + (size_t)cur.tile * cur.parts * (TM * TN), g.joined + cur.tile * JOIN_COUNTERS,
                          cur.part, cur.parts, mine, join_flag))
      tile_epilogue<MODE, true, 2>(g, acc, cur.row0, cur.rows, cur.nblk, wm, wn, lane);
    if (!nxt.valid) break;
    cur = nxt;
    na = na_n;
  }
}

// A GEMM: A [rows, lda], contraction of `segs` segments of `seg_len`, N output columns in blocks of bn
// (ldb: row length of a k-major weight-role operand, else 0).
TileArgs tile_args(const moe_ctx* c, const int32_t* counts, const int32_t* offsets, const void* A, int lda,
                   int bn, int seg_len, int segs, int ldb, int N, void* C, int w0, int w1) {
  TileArgs a{};
  a.g.A = (const uint16_t*)A;
  a.g.lda = lda;
  a.g.n_tiles_n = ceil_div(N, bn);
  a.g.K = seg_len * segs;
  a.g.N = N;
  a.g.C = (uint16_t*)C;
  a.g.ldb = ldb;
  a.g.kseg = ceil_div(seg_len, BK);
  a.g.kt = segs * a.g.kseg;
  a.g.kseg_len = seg_len;
  a.g.zero = (const char*)c->d_zero;
  a.g.split_ws = c->d_split_ws;
  a.g.joined = c->d_joined;
  a.counts = counts;
  a.offsets = offsets;
  a.present = c->d_wtab;
  a.b0 = c->d_wtab + w0 * MOE_MAX_EXPERTS;
  a.b1 = w1 >= 0 ? c->d_wtab + w1 * MOE_MAX_EXPERTS : nullptr;
  a.E = c->cfg.E;
  a.S = c->S_call;
  a.status = c->d_sched[1];
  a.again = c->weights_again;
  return a;
}

int slots_of(int n_cu) { return std::max(8, (2 * n_cu / 8) * 8); }
int slots(const moe_ctx* c) { return slots_of(c->n_cu); }

// Floats of the partial tiles of a context with S rows: as many as there are resident blocks at most, fewer
// where there cannot be as many parts (dX of the gated expert has the longest contraction).
size_t split_floats(int S, int E, int d, int f, int n_cu) {
  const long long blocks = (long long)S / TM + E;
  auto tiles = [&](int kt, int cols) {
    const int most = parts_of(1, SPLIT_MAX, kt, true);
    return most == 1 ? 0 : std::min<long long>(slots_of(n_cu), blocks * cols * most);
  };
  return (size_t)std::max(tiles(2 * ceil_div(f, BK), ceil_div(d, TN)) /* dX */,
                          tiles(ceil_div(d, BK), ceil_div(f, 64)) /* gate/up */) * (TM * TN);
}

template <int MODE, bool BKM>
void launch(const moe_ctx* c, const TileArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((ffn_tile128_kernel<MODE, BKM>), dim3(slots(c)), dim3(NT), 0, s, a);
}

}  // namespace

// (two parts at least, on at most `slots` blocks)
size_t ffn_join_counters(const moe_ctx* c) { return (size_t)slots(c) / 2 * JOIN_COUNTERS; }

size_t ffn_tile128_split_floats(const moe_ctx* c) {
  return split_floats(c->S_max, c->cfg.E, c->cfg.d, c->cfg.f, c->n_cu);
}

int launch_ffn_tile128(moe_ctx* c, bool gated, const int32_t* counts, const int32_t* offsets,
                       const void* x_packed, void* y_packed, void* G, void* U, hipStream_t s) {
  const int d = c->cfg.d, f = c->cfg.f;
  prof_mark(c, 0, s);
  prof_mark(c, 1, s);   // no schedule launch
  TileArgs up = tile_args(c, counts, offsets, x_packed, d, gated ? 64 : TN, d, 1, 0, f, c->d_H, 0, gated ? 1 : -1);
  up.g.Gs = (uint16_t*)G;
  up.g.Us = (uint16_t*)U;
  if (gated) launch<MODE_UP, false>(c, up, s);
  else launch<MODE_UP1, false>(c, up, s);
  prof_mark(c, 2, s);
  launch<MODE_DOWN, false>(c, tile_args(c, counts, offsets, c->d_H, f, TN, f, 1, 0, d, y_packed, 2, -1), s);
  prof_mark(c, 3, s);
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_EHIP;
}

// The two halves of the data gradients (the weight gradients come between them, see
// launch_ffn_bwd_mfma): dH = dY W2 with the activation's derivative, and dX.
int launch_ffn_tile128_dh(moe_ctx* c, bool gated, const void* dy, const void* G, const void* U,
                          const int32_t* counts, const int32_t* offsets, bool offered, hipStream_t s) {
  const int d = c->cfg.d, f = c->cfg.f;
  TileArgs dh = tile_args(c, counts, offsets, dy, d, TN, d, 1, f, f, c->d_dGU, 2, -1);
  dh.offered = offered;
  dh.g.C2 = (uint16_t*)c->d_H;
  dh.g.Gs = (uint16_t*)const_cast<void*>(G);
  dh.g.Us = (uint16_t*)const_cast<void*>(U);
  if (gated) launch<MODE_DH, true>(c, dh, s);
  else launch<MODE_DH1, true>(c, dh, s);
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_EHIP;
}

int launch_ffn_tile128_dx(moe_ctx* c, bool gated, const int32_t* counts, const int32_t* offsets, void* dxp,
                          hipStream_t s) {
  const int d = c->cfg.d, f = c->cfg.f, segs = gated ? 2 : 1;
  launch<MODE_DOWN, true>(c, tile_args(c, counts, offsets, c->d_dGU, segs * f, TN, f, segs, d, d, dxp, 0,
                                       gated ? 1 : -1), s);
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_EHIP;
}

// One round of 128-row tiles in dH, with `rows` rows on each of `experts` experts.
static bool dh_one_round(int experts, long long rows, int f, int slots) {
  return experts > 0 && experts * ((rows + TM - 1) / TM) * ceil_div(f, TN) <= slots;
}

// Time in us of a GEMM's launch with `rows` rows on each of `experts` experts and weights of `mb` MB: a
// constant, and the rounds of tiles, or the weights from HBM where those take longer; contractions are cut as the
// kernels cut them.  A k-step of a round costs more the more of the chip has tiles, the more rows these hold and,
// in the larger tiles, where the sizes are not multiples of theirs.  (Constants: least squares of the logarithms over
// 331 calls of 1 to 8400 tokens, forward and backward, evenly routed and with all tokens on the same experts,
// weights that are not in the last-level cache; three of them, at which the choice had been wrong, counted 20 times.
// Either side is within 13 % of what was measured in the mean square, their ratio within 8 %; on 110 other calls
// 15 % and 9 %.)
static double us_256(int experts, int rows, int N, int bn, int K, int kt, bool down, bool bwd, double mb, int n_cu) {
  const int blocks = ceil_div(rows, 256), tiles = experts * blocks * ceil_div(N, bn), tail = tiles % n_cu;
  const int split = down ? split_parts(tail, n_cu, kt) : 1;
  const double full = 1.102 * rows / (256.0 * blocks) + (K % 128 != 0 || N % bn != 0 ? 0.234 : 0);
  const double loop = tiles / n_cu * (kt * (0.729 + full) + 8.01) +
                      (tail > 0 ? (double)kt / split * (0.729 + full * tail * split / n_cu) + 8.01 : 0);
  return 6.3 /* half of the schedule in it */ + (split > 1 ? 8.73 : 0) + std::max(loop, mb / (bwd ? 5.59 : 4.87));
}
static double us_128(int experts, int rows, int N, int bn, int kt, bool cut, double mb, int n_cu) {
  const int blocks = ceil_div(rows, TM), tiles = experts * blocks * ceil_div(N, bn), slots = 2 * n_cu;
  const int split = cut ? parts_of(tiles, slots, kt, blocks == 1) : 1, units = tiles * split, tail = units % slots;
  const double steps = (double)kt / split, full = 0.78 * rows / ((double)TM * blocks);
  const double loop = units / slots * (steps * (0.577 + full) + 3.74) +
                      (tail > 0 ? steps * (0.577 + full * tail / slots) + 3.74 : 0);
  return 2.12 + 3.77 * join_levels(split) + std::max(loop, mb / 5.56);
}
// Both GEMMs of a call, larger and smaller tiles.  (dH: with its epilogue; beside the larger tiles it is offered to the
// smaller ones, see ffn_tile128_dh_offered, and taken by the rounds of both as in mfma_sched_kernel.)
static void tile_us(int experts, int rows, int d, int f, bool gated, bool backward, int n_cu, double& large,
                    double& small) {
  const int bn = gated && !backward ? 128 : 256;   // columns of the larger tiles, first GEMM
  const int segs = gated && backward ? 2 : 1;
  const double mb = 2e-6 * experts * d * f, mb1 = bn == 128 ? 2 * mb : mb, mb2 = segs * mb;
  large = us_256(experts, rows, f, bn, d, k_steps(d, 1), false, backward, mb1, n_cu) + (backward ? 21.5 : 0);
  small = us_128(experts, rows, f, bn / 2, ceil_div(d, BK), !backward, mb1, n_cu) + (backward ? 7.5 : 0);
  if (backward && dh_one_round(experts, rows, f, 2 * n_cu)) {
    const int rounds = ceil_div(experts * ceil_div(rows, 256) * ceil_div(f, 256), n_cu);
    large = (2 < 3 * rounds ? small : large) + 6.93;
  }
  large += us_256(experts, rows, d, 256, f, k_steps(f, segs), true, backward, mb2, n_cu);
  small += us_128(experts, rows, d, TN, segs * ceil_div(f, BK), true, mb2, n_cu);
}

// The smaller tiles are taken where by this estimate they are the faster ones for an even routing, and all
// tokens on the same experts (more rows on fewer experts: more and fuller tiles) cost them no more than twice
// what they gain there.  Besides, they are held to calls whose first GEMM has at most two rounds of larger tiles with
// any routing or, forward, at most one row block per expert; backward, one round with an even routing.  Of 287
// measured calls that these lines admit the choice is the slower one by more than 3 % in 21 with an even routing (by 1 %
// in the mean), 1 % in the mean with popularity falling off as rank^-1.2 or all tokens on the same experts.  Both GEMMs
// with sums and schedule, larger tiles (backward: dH by turn) -> smaller ones, us: even routing; rank^-1.2; all
// tokens on the same experts (T, d, f, E, k, resident):
//   forward: 1999, 1160, 2888, 16, 2, 6: 101 -> 85; 153 -> 153; 155 -> 153
//            two-matrix 1024, 1024, 4096, 32, 2, 8: 63 -> 44; 78 -> 64; 84 -> 66
//            64, 4096, 14336, 8, 2, 8: 532 -> 451; 530 -> 459; 168 -> 135
//            751, 664, 384, 64, 3, 11: 45 -> 22; 52 -> 27; 49 -> 26
//            7513, 1536, 1536, 32, 1, 9, two-matrix: 80 -> 50; 86 -> 99; 86 -> 101
//            275, 4096, 4480, 8, 3, 8: 247 -> 204; 253 -> 244; 146 -> 188
//   backward: 2000, 768, 1024, 16, 4, 6: 64 -> 52; 84 -> 69; 92 -> 76
//            1999, 1160, 2888, 16, 2, 6: 112 -> 101; 162 -> 183; 168 -> 187
//            338, 3840, 3712, 64, 1, 16: 234 -> 209; 256 -> 251; 111 -> 104
//   left to the larger ones, forward: 953, 4096, 1024, 64, 8, 12: 114 -> 89; 169 -> 196; 180 -> 241
//            2615, 3840, 768, 64, 3, 22: 139 -> 131; 183 -> 203; 149 -> 192
//            1422, 1816, 2672, 8, 3, 3: 95 -> 100; 170 -> 156; 191 -> 222
//            two-matrix 1000, 3072, 3072, 64, 6, 10: 125 -> 91; 164 -> 239; 265 -> 304
//   backward: 2999, 3328, 1280, 64, 8, 8: 128 -> 140; 421 -> 463; 602 -> 837
//            996, 2304, 1664, 64, 8, 8: 94 -> 83; 146 -> 162; 235 -> 286
//            two-matrix 2166, 1792, 1408, 32, 4, 16: 106 -> 107; 125 -> 135; 119 -> 132
bool ffn_tile128_rule(int T, int d, int f, int E, int k, int n_res, bool gated, bool backward, int n_cu) {
  if (n_res == 0) return false;
  const int cols = ceil_div(f, gated && !backward ? 128 : 256);
  if (((long long)T * std::min(k, n_res) / 256 + n_res) * cols > 2 * n_cu && (backward || T > TM)) return false;
  const int rows = (int)(((long long)T * k + E - 1) / E);
  if (backward && (long long)n_res * ceil_div(rows, 256) * cols > n_cu) return false;
  double large, small, large_hot, small_hot;
  tile_us(n_res, rows, d, f, gated, backward, n_cu, large, small);
  tile_us(std::min(k, n_res), T, d, f, gated, backward, n_cu, large_hot, small_hot);
  return small < large && small_hot - large_hot <= 2 * (large - small);
}

// dH where the larger tiles take the call: its long epilogue (five arrays of S x f) runs under another block's main
// loop in the smaller ones, so that these serve one round faster (kernel, larger -> smaller, us: 6 experts of 2048 x
// 2048, 250 rows: 69 -> 38, 512 rows: 76 -> 54; 768 rows, where they are two rounds and the larger ones one: 73 -> 92).
// How many rounds either takes shows on the device: where an even routing makes it one of the smaller tiles, both
// kernels are launched, and the schedule says which of them works (dh_small); the other one ends at once (3 us).
// Training step, us: 4096 tokens, 2048 x 2048, 6 of 32 experts: 512 -> 498; 1536 x 2048: 390 -> 373; 2048 x 1408, 12 of 64
// with popularity rank^-1.2, where the larger tiles would begin a third round: 1404 -> 1385; 1024 x 2048, rank^-0.6,
// two rounds against one: 427 -> 430.
bool ffn_tile128_dh_offered(const moe_ctx* c) {
  if (c->tile_rows != 0) return c->tile_rows == 256 + TM;
  int n_res = 0;
  for (int e = 0; e < c->cfg.E; ++e) n_res += c->h_wtab[0][e] != nullptr;
  return dh_one_round(n_res, ((long long)c->S_call + c->cfg.E - 1) / c->cfg.E, c->cfg.f, slots(c));
}

bool ffn_tile128_wanted(const moe_ctx* c, bool gated, bool backward) {
  if (c->tile_rows != 0) return c->tile_rows == TM;
  int n_res = 0;
  for (int e = 0; e < c->cfg.E; ++e) n_res += c->h_wtab[0][e] != nullptr;
  return ffn_tile128_rule(c->S_call / c->cfg.k, c->cfg.d, c->cfg.f, c->cfg.E, c->cfg.k, n_res, gated, backward,
                          c->n_cu);
}

// Not part of the interface, for tests: the rule and its estimate; the parts of a launch of `tiles` tiles
// and the workspace for them; and the tiles of one context whatever the rule (0: the rule), of all its products or of the weight
// gradients alone.
extern "C" int moe_internal_ffn_tile128(int32_t T, int32_t d, int32_t f, int32_t E, int32_t k, int32_t n_res,
                                        int32_t gated, int32_t backward, int32_t n_cu) {
  return ffn_tile128_rule(T, d, f, E, k, n_res, gated != 0, backward != 0, n_cu) ? 1 : 0;
}
extern "C" void moe_internal_ffn_tile_us(int32_t experts, int32_t rows, int32_t d, int32_t f, int32_t gated,
                                         int32_t backward, int32_t n_cu, double* us) {
  tile_us(experts, rows, d, f, gated != 0, backward != 0, n_cu, us[0], us[1]);
}
extern "C" int moe_internal_tile128_parts(int32_t tiles, int32_t slots, int32_t kt) {
  return parts_of(tiles, slots, kt, true);
}
extern "C" int moe_internal_tile128_parts_shared(int32_t tiles, int32_t slots, int32_t kt) {
  return parts_of(tiles, slots, kt, false);
}
extern "C" int64_t moe_internal_tile128_split_floats(int32_t S, int32_t E, int32_t d, int32_t f, int32_t n_cu) {
  return (int64_t)split_floats(S, E, d, f, n_cu);
}
extern "C" void moe_internal_ffn_tile_rows(moe_ctx* c, int32_t rows) { c->tile_rows = c->wgrad_rows = rows; }
extern "C" void moe_internal_wgrad_rows(moe_ctx* c, int32_t rows) { c->wgrad_rows = rows; }
