// Grouped SwiGLU expert FFN on the matrix cores (bf16 in, fp32 accumulate) for gfx950.
// (Paper Sec. 2.1: experts are replicated FFNs; Sec. 3.1: computation latency is
// dominated by the expert GEMMs and the experts of one GPU run on their own tokens.)
//
// Two launches walk a device-built tile list (no host sync on the token counts):
//   gate/up : H[r, n] = silu(x_r . W1[e][n,:]) * (x_r . W3[e][n,:])   (SwiGLU fused)
//   down    : Y[r, c] = H[r,:] . W2[e][c,:]
// Every operand is contiguous along the contraction dimension, so each lane feeds the
// MFMA with one 16-byte LDS read per operand fragment.
//
// Tiling: 512 threads = 8 wavefronts (2 along rows x 4 along columns), block tile
// 256 rows x 256 weight rows x 64 (k), wavefront tile 128 x 64 = 4 x 2 MFMA 32x32x16
// accumulators (128 fp32 registers).  For gate/up the 256 weight rows are 128 rows of W1
// and the matching 128 rows of W3, laid out so that a wavefront owns gate and up of the
// same columns and applies silu(g)*u in registers.  The weight rows are the MFMA "A"
// operand and the token rows the "B" operand: a lane then holds 4 consecutive output
// columns of one token row and stores them as one 8-byte write.
// LDS: 2 stages x (32 KB tokens + 32 KB weights) = 128 KB, filled by asynchronous
// global->LDS copies (no registers in between); 16-byte chunks are XOR-swizzled by row so
// that the 16-byte fragment reads of 16 consecutive rows fall on distinct banks.
// Main loop ("ping-pong"): the wavefronts of the upper 128 token rows and those of the
// lower 128 rows alternate between a memory cluster (fragment reads of one 32-row token
// block, two copy instructions) and a compute cluster (8 MFMAs), the second group one
// cluster behind the first, so every SIMD always has one wavefront on the matrix core
// and one on memory.  A token block is refilled as soon as its group has read it, the
// weight rows as soon as both groups have read them (first cluster of a step), each with
// the data of two steps ahead: copies are spread evenly over the step and have more
// than one step to land.
// Tile order: an expert's row blocks in groups of 8; inside a group the tiles that share a
// weight panel (same column block) are consecutive, and the block index is remapped so that
// each of the 8 XCDs (private L2) works on a contiguous range of that order: the 32 tiles an
// XCD has in flight are 8 row blocks x 4 column blocks.
#include <algorithm>

#include "ffn_tile.h"

namespace {

constexpr int BM = MFMA_BM;       // token rows per block tile
constexpr int NT = 512;           // threads
constexpr int STAGE_VEC = 2048;   // uint4 per operand per stage (256 rows x 8 chunks)
constexpr int ORDER_GROUP_M = 8;  // row blocks per group of the tile order

// Most partial tiles there can be with at most `tiles` tiles: parts times tiles of the tail.
size_t split_tiles_max(long long tiles, int n_cu, int kt_down) {
  const int most = split_parts(1, 8, kt_down);   // parts with no limit from the tail
  return most == 1 ? 0 : (size_t)std::min<long long>(n_cu, tiles * most);
}

__global__ __launch_bounds__(256) void mfma_sched_kernel(
    const int32_t* __restrict__ counts, const int32_t* __restrict__ offsets,
    const void* const* __restrict__ present, int E, int S, int max_mtiles, int nt_up, int nt_down,
    int n_cu, int kt_down, int nt_dh128, TileSched* __restrict__ sched, const void* const* __restrict__ up_b0,
    const void* const* __restrict__ up_b1, const void* const* __restrict__ down_b0,
    const void* const* __restrict__ down_b1, TileDesc* __restrict__ order_up,
    TileDesc* __restrict__ order_down) {
  __shared__ int32_t start[MOE_MAX_EXPERTS + 1];
  __shared__ int bad, blocks128;
  const int tid = threadIdx.x;
  if (tid == 0) {
    start[0] = 0;
    bad = 0;
    blocks128 = 0;
  }
  __syncthreads();
  // per-expert tile counts (E <= 256: one expert per thread), then an inclusive scan
  int mine = 0;
  if (tid < E && present[tid] != nullptr) {
    const int n = counts[tid], o = offsets[tid];
    if (n < 0 || o < 0 || (long)o + n > (long)S) bad = 1;  // caller's arrays are inconsistent
    else {
      mine = (n + BM - 1) / BM;
      atomicAdd(&blocks128, (n + 127) / 128);
    }
  }
  start[tid + 1] = mine;
  __syncthreads();
  for (int off = 1; off < 256; off <<= 1) {
    int v = 0;
    if (tid >= off) v = start[tid + 1 - off];
    __syncthreads();
    if (tid >= off) start[tid + 1] += v;
    __syncthreads();
  }
  const int total_m = (bad || start[E] > max_mtiles) ? 0 : start[E];
  if (blockIdx.x == 0 && tid == 0) {
    sched->n_mtiles = total_m;
    // Down GEMM: when the last round of tiles fills at most half of the compute units, its
    // tiles are cut along the contraction into `split` parts (2 .. 8; every part a whole
    // number >= 4 of k-step pairs, the first parts one pair longer when the pairs do not
    // divide evenly; all parts together still one round), summed afterwards.
    const int total = total_m * nt_down;
    const int tail = total % n_cu;
    const int split = split_parts(tail, n_cu, kt_down);
    sched->down_split = split;
    sched->down_split_tiles = split > 1 ? tail : 0;
    sched->down_full = split > 1 ? total - tail : total;
    // dH: a round of 128-row tiles (two blocks on a compute unit) takes 0.6 to 0.7 times as long as one of these.
    // (Segments that overlap may have more row blocks than the smaller tiles' kernel takes.)
    const int small_rounds = (blocks128 * nt_dh128 + 2 * n_cu - 1) / (2 * n_cu);
    const int rounds = (total_m * nt_up + n_cu - 1) / n_cu;
    sched->dh_small = total_m > 0 && nt_dh128 > 0 && blocks128 <= S / 128 + E && 2 * small_rounds < 3 * rounds;
  }
  const int gsz = gridDim.x * blockDim.x;
  const int gid = blockIdx.x * blockDim.x + tid;
  // tile order: expert by expert; inside an expert in groups of 8 row blocks; inside a group
  // column block by column block, the group's row blocks in a row (they share a weight panel)
  for (int pass = 0; pass < 2; ++pass) {
    const int nt = pass == 0 ? nt_up : nt_down;
    TileDesc* order = pass == 0 ? order_up : order_down;
    const int total = total_m * nt;
    for (int L = gid; L < total; L += gsz) {
      int lo = 0, hi = E;
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (start[mid] * nt <= L) lo = mid; else hi = mid;
      }
      const int me = start[lo + 1] - start[lo];
      const int rel = L - start[lo] * nt;
      // groups of up to 8 row blocks: inside a group column block by column block, so that 32
      // consecutive tiles are 8 row blocks x 4 column blocks (12 panels for 32 tiles)
      const int per_group = ORDER_GROUP_M * nt;
      const int mg = rel / per_group, r2 = rel % per_group;
      const int gm = min(ORDER_GROUP_M, me - mg * ORDER_GROUP_M);
      const int n = r2 / gm, m = mg * ORDER_GROUP_M + r2 % gm;
      TileDesc t;
      t.row0 = offsets[lo] + m * BM;
      t.rows = min(BM, counts[lo] - m * BM);
      t.nblk = n;
      t.expert = lo;
      t.b0 = pass == 0 ? up_b0[lo] : down_b0[lo];
      const void* const* tab1 = pass == 0 ? up_b1 : down_b1;
      t.b1 = tab1 != nullptr ? tab1[lo] : nullptr;
      order[L] = t;
    }
  }
}

// One unit of work of a block: a whole tile, or one K-split part of a tile (all fields are
// wave-uniform and live in scalar registers).
struct Unit {
  int valid;
  int row0, rows, nblk;     // tile: first packed row, valid rows, column block
  const char* abase;        // token-role operand: first row of the tile, first k of the range
  const char* bbase0;       // weight-role operand: first row of the column block (gate/up: W1)
  const char* bbase1;       // gate/up: the same rows of W3; else bbase0 + 128 rows
  int KT;                   // k-steps of 64 (even)
  int kstart;               // first k-step of the unit (K-split parts; 0 otherwise)
  int ws_unit;              // >= 0: K-split part, index of its partial tile in the workspace
};

// The idx-th unit of this block.  The hardware deals blocks round-robin to the XCDs: XCD x
// (= blockIdx & 7) holds the blocks x, x + 8, ...  The tile order is walked in rounds of
// gridDim tiles; a round is cut into 8 chunks of consecutive tiles (32 in a full round: 8 row
// blocks x 4 column blocks that share 12 panels), chunk x goes to XCD x, one tile per block:
// at any time an XCD works on one chunk.  The last, partial round is cut into 8 equal chunks as
// well, so that every XCD stays in use.  Going round by round (rather than giving an XCD a
// contiguous eighth of the whole order) spreads the cheap tiles of short row blocks -- which
// come in runs -- over all XCDs.  After its whole tiles a block takes its share of the
// K-split units of the tail (a contiguous range per XCD).  The sequence of a block is dense:
// once a unit is invalid, all later ones are.
template <int MODE, bool BKM, bool RAG>
__device__ __forceinline__ Unit fetch_unit(const GemmArgs& p, int idx) {
  Unit u;
  u.valid = 0;
  u.ws_unit = -1;
  constexpr bool DH = MODE == MODE_DH || MODE == MODE_DH1;
  const int total = DH && p.sched->dh_small ? 0 : p.sched->n_mtiles * p.n_tiles_n;
  const int n_full = MODE == MODE_DOWN ? p.sched->down_full : total;
  const int split = MODE == MODE_DOWN ? p.sched->down_split : 1;
  const int n_units = MODE == MODE_DOWN ? p.sched->down_split_tiles * split : 0;
  const int per_xcd_s = (n_units + 7) >> 3;
  const int x = blockIdx.x & 7, slot = (int)(blockIdx.x >> 3);
  const int G = (int)gridDim.x, gsz = G >> 3;
  const int rfull = n_full / G, m_last = n_full - rfull * G;   // full rounds, tiles of the last one
  const int per_last = (m_last + 7) >> 3;
  const bool in_last = slot < per_last && x * per_last + slot < m_last;
  const int nfu = rfull + (in_last ? 1 : 0);
  const int ns = max(0, min(per_xcd_s, n_units - x * per_xcd_s));
  const int kt_all = RAG ? p.kt : p.K / BK;
  int L, part = 0, kstart = 0;   // kstart: first k-step of a K-split part
  if (idx < nfu) {
    L = idx < rfull ? idx * G + x * gsz + slot : rfull * G + x * per_last + slot;
    u.KT = kt_all;
  } else {
    const int qs = slot + (idx - nfu) * gsz;   // among the XCD's split units
    if (qs >= ns) return u;
    const int su = x * per_xcd_s + qs;
    L = n_full + su / split;
    part = su % split;
    // pairs of k-steps of this part: the first `rem` parts take one pair more
    const int pairs = kt_all / 2, base = pairs / split, rem = pairs % split;
    u.KT = 2 * (base + (part < rem ? 1 : 0));
    kstart = 2 * (part * base + min(part, rem));
    u.ws_unit = su;
  }
  const TileDesc td = p.order[L];
  u.valid = 1;
  u.row0 = td.row0;
  u.rows = td.rows;
  u.nblk = td.nblk;
  u.kstart = kstart;
  const size_t kbeg = RAG ? 0 : (size_t)kstart * (BK * 2);  // bytes into a row (RAG: per copy)
  u.abase = (const char*)p.A + (size_t)td.row0 * p.lda * 2 + kbeg;
  if (BKM) {   // column block of the k-major matrices; the k-step is applied per copy
    u.bbase0 = (const char*)td.b0 + (size_t)td.nblk * 512;
    u.bbase1 = (const char*)td.b1 + (size_t)td.nblk * 512;
  } else if (MODE == MODE_UP) {
    u.bbase0 = (const char*)td.b0 + (size_t)td.nblk * 128 * p.K * 2 + kbeg;
    u.bbase1 = (const char*)td.b1 + (size_t)td.nblk * 128 * p.K * 2 + kbeg;
  } else {
    u.bbase0 = (const char*)td.b0 + (size_t)td.nblk * 256 * p.K * 2 + kbeg;
    u.bbase1 = RAG ? u.bbase0 : u.bbase0 + (size_t)128 * p.K * 2;   // RAG: rows 0..255 in b_off
  }
  return u;
}

// One cluster pair of the main loop: memory cluster of token block I in stage S (fragment
// reads; two copies, base + offset each, into the rows read one cluster ago), then the
// compute cluster.
//
// both: the second 128 columns of the column block hold any (RAG; in gate/up they are W3's rows).  Where a last
// column block has none there, they are not multiplied (training step of 2048 x 1408, dH: 1415 -> 1411 us; leaving out
// their fragment reads as well made two versions of the loop, which spilled).
// na: token blocks of the copies' target that are copied at all (4 unless the target is lean, see
// the kernel).  WAIT: copies that may be outstanding at the end of the memory cluster, or < 0: 3
// where `strict`, else 6.
template <int S, int I, bool BKM, bool RAG, int WAIT>
__device__ __forceinline__ void pp_cluster(f32x16 (&acc)[2][4], bf16x8 (&wb)[2][4],
                                           const uint4* lds, const int (&fr_a)[4],
                                           const int (&fr_b)[2], int fr_half, int fr_swz,
                                           uint32_t offa, const Src& srca, uint32_t offb,
                                           const Src& srcb, uint32_t a_dst, uint32_t b_dst,
                                           int nact, int na, bool both, bool strict, int lc,
                                           int brow, const char* zero) {
  const uint4* As = lds + (2 * S) * STAGE_VEC;
  const uint4* Bs = lds + (2 * S + 1) * STAGE_VEC;
  bf16x8 xa[4];
  if (I == 0) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (BKM) {
          // k-major stage (64 k-rows x 512 bytes): fr_b[j] is the lane's LDS byte address for
          // k-rows 0..3 of its 16-row group; two transpose reads make the 8 k of the fragment
          const uint32_t a0 = (uint32_t)fr_b[j] + (2 * S + 1) * 32768 + kk * 8192;
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)a0);
          const s16x4 hi =
              __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)(a0 + 4 * 512));
          const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
          wb[j][kk] = __builtin_bit_cast(bf16x8, v);
        } else {
          wb[j][kk] = __builtin_bit_cast(bf16x8, Bs[fr_b[j] + ((kk * 2 + fr_half) ^ fr_swz)]);
        }
      }
  }
  // nact (wave-uniform): 32-row blocks of this wavefront's half of the tile that hold rows;
  // the others are neither read nor multiplied (their accumulators stay zero and are not
  // stored), the copies and barriers go on as ever
  const bool act = I < nact;
  if (act) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      xa[kk] = __builtin_bit_cast(bf16x8, As[fr_a[I] + ((kk * 2 + fr_half) ^ fr_swz)]);
  }
  constexpr int blk = (I + 3) & 3;
  constexpr int st = I == 0 ? (S ^ 1) : S;
  if (WAIT == 6 || blk < na) dma_step<RAG>(offa, srca, a_dst + st * 65536 + blk * 4096, 8, lc, zero);
  dma_step<RAG>(offb, srcb, b_dst + st * 65536 + blk * 8192, BKM ? BK : 8,
                BKM ? brow + 16 * blk : lc, zero);
  // My fragment reads are done (the rows may be refilled after the next barrier) and all
  // but my last 6 (3) vector-memory operations have completed: with two copies a cluster (at
  // least one) the data read in cluster n was copied in clusters <= n-4 and every wavefront
  // passes this point in cluster n-1 before anybody reads in cluster n.  (Stores of an epilogue
  // count as well and only make the wait stricter: copies complete in issue order among
  // themselves.)
  if (WAIT == 6) asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)" ::: "memory");
  else if (WAIT == 3 || strict) asm volatile("s_waitcnt vmcnt(3) lgkmcnt(0)" ::: "memory");
  else asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)" ::: "memory");
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_setprio(1);
  if (act && !RAG) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[j][I] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wb[j][kk], xa[kk], acc[j][I], 0, 0, 0);
  } else if (act) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      acc[0][I] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wb[0][kk], xa[kk], acc[0][I], 0, 0, 0);
    if (both)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        acc[1][I] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wb[1][kk], xa[kk], acc[1][I], 0, 0, 0);
  }
  __builtin_amdgcn_s_setprio(0);
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
}

// MODE_UP   : H = silu(A W1^T) * (A W3^T)            (gate/up, SwiGLU fused)
// MODE_UP1  : H = max(A W1^T, 0)                      (first GEMM of the two-matrix expert)
// MODE_DOWN : C = A B^T                               (down projection; also dX = [dG|dU][W1^T|W3^T]^T)
// MODE_DH   : dH = A B^T, then dG = dH*u*silu'(g), dU = dH*silu(g), H = silu(g)*u
// MODE_DH1  : dH = A B^T, then dG = dH where g > 0 (else 0), H = max(g, 0)   (two-matrix expert)
//
// Tiled modes run persistent blocks (one per compute unit) over a static share of the tile
// order, and the copy stream does not stop at a tile boundary: during the last two k-steps
// of a tile the rows that become free are refilled with the first two k-steps of the
// block's next tile, so that only the very first tile of a block pays a load latency.
//
// BKM: the weight-role operand is stored k-major, B[k][n] (the data gradients contract over
// the other index of the weights).  A stage then holds 64 k-rows x 256 columns (512 bytes
// per row, 16-byte chunks XOR-swizzled by tr_swz(row)), copied as it is -- one copy
// instruction fills two k-rows -- and the fragments come out of LDS through the transpose
// read ds_read_b64_tr_b16 (the layout and the lane arithmetic of wgrad_tr.hip).
//
// RAG: sizes that the tile does not divide (multiples of 8, so that every 16-byte chunk exists
// or does not).  The k-steps are rounded up to an even number; the chunks of both operands past
// the end of the contraction come from 16 bytes of zeros, fetched by the per-lane address form
// in the k-steps that need it (a scalar branch: the other steps copy as ever).  Weight rows
// (columns, when k-major) past the end of the matrix repeat the last one and are not stored.
// Measured against the vector-ALU kernels that such sizes used before (bound by LDS reads and
// FMAs, 16-23 TFLOP/s): 1500 rows, d = 1160, f = 2888: gate/up 594 -> 52 us, down 664 -> 47 us;
// 13100 rows, d = 2048, f = 1408: dH 2398 -> 266 us, dX 4954 -> 223 us, weight gradients 6242 ->
// 469 us.  The bound is the tile's again (copies and MFMAs of whole tiles, 9 % of them padding).
template <int MODE, bool BKM = false, bool RAG = false>
__global__ __launch_bounds__(NT) void ffn_mfma_kernel(const GemmArgs p) {
  // stage s: token rows at (2s) * STAGE_VEC, weight rows at (2s+1) * STAGE_VEC
  __shared__ uint4 lds[4 * STAGE_VEC];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = __builtin_amdgcn_readfirstlane(wave >> 2), wn = wave & 3;
  Unit cur;
  // global -> LDS assignment: one copy instruction fills 8 rows (lane>>3) x 8 chunk slots
  // (lane&7); slot c of row r must hold global chunk c ^ swz(r).  Token rows: copy i of a
  // wavefront fills 8 rows of block i of its own group's half; weight rows: copy i fills
  // row block 8i + wave (gate/up: blocks 0..15 are rows of W1, 16..31 the same rows of W3;
  // otherwise bbase1 is bbase0 + 128 rows).  Per-lane byte offsets from the unit's bases:
  uint32_t a_off[4], b_off[4];
  const int a_pitch = p.lda * 2;                                   // bytes per token-role row
  const int b_pitch = p.K * 2;                                     // ... per weight-role row
  auto token_off = [&](int rows, int i) -> uint32_t {
    const int ra = (16 * wm + 4 * i + wn) * 8 + (lane >> 3);
    return (uint32_t)min(ra, rows - 1) * a_pitch + (((lane & 7) ^ swz(ra)) << 4);
  };
  auto weight_off = [&](int nblk, int i) -> uint32_t {
    if (BKM) {   // copy i of the wavefront: k-rows 2c and 2c+1 of the step, c = 8i + wave
      const int r = 2 * (8 * i + wave) + (lane >> 5);
      int ch = (lane & 31) ^ tr_swz(r);
      if (RAG) ch = min(ch, (p.N - nblk * 256) / 8 - 1);
      return (uint32_t)r * (uint32_t)(p.ldb * 2) + (ch << 4);
    }
    const int rb = (8 * i + wave) * 8 + (lane >> 3);
    int row = rb & 127;
    if (RAG) row = MODE == MODE_UP ? min(row, p.N - 1 - nblk * 128) : min(rb, p.N - 1 - nblk * 256);
    return (uint32_t)row * b_pitch + (((lane & 7) ^ swz(rb)) << 4);
  };
  // RAG: the 16-byte chunk of a row-major k-step this lane copies (the same for every i), and
  // the k-row of a k-major one (+ 16 i)
  const int lc = (lane & 7) ^ swz(wn * 8 + (lane >> 3));
  const int brow = 2 * wave + (lane >> 5);
  // weight-role source of k-step `step` of unit u (half: 0 = first, 1 = second 128 rows of the
  // column block when the operand is row-major)
  const size_t bstep = (size_t)BK * p.ldb * 2;
  auto bsrc = [&](const Unit& u, int step, int half) -> Src {
    const int kg = u.kstart + step;
    const int kk = kg < p.kseg ? kg : kg - p.kseg;   // step inside its segment
    const int kv = RAG ? p.kseg_len - kk * BK : BK;  // k of the step that exist (may be <= 0)
    if (BKM) return {(kg < p.kseg ? u.bbase0 : u.bbase1) + (size_t)kk * bstep, kv};
    return {(half ? u.bbase1 : u.bbase0) + (RAG ? kk : step) * 128, kv >> 3};
  };
  auto asrc = [&](const Unit& u, int step) -> Src {
    if (!RAG) return {u.abase + step * 128, 8};
    const int kg = u.kstart + step;
    const int kk = kg < p.kseg ? kg : kg - p.kseg;
    return {u.abase + (kg < p.kseg ? 0 : p.kseg_len * 2) + kk * 128, (p.kseg_len - kk * BK) >> 3};
  };
  cur = fetch_unit<MODE, BKM, RAG>(p, 0);
  if (!cur.valid) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    a_off[i] = token_off(cur.rows, i);
    b_off[i] = weight_off(cur.nblk, i);
  }

  // ---- fragment read offsets (uint4 units inside one operand stage)
  const int fr_row = lane & 31, fr_half = lane >> 5;
  const int fr_swz = swz(fr_row);
  int fr_a[4], fr_b[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) fr_a[i] = (wm * 128 + i * 32 + fr_row) * 8;
#pragma unroll
  for (int j = 0; j < 2; ++j) fr_b[j] = (j * 128 + wn * 32 + fr_row) * 8;
  if (BKM) {
    // transpose reads: groups of 16 lanes; lane (j4 = (lane & 15) >> 2, q4 = lane & 3) of group
    // g16 = lane >> 4 points at k-row 8 * (g16 >> 1) + j4 and the 4 columns 16 * (g16 & 1) +
    // 4 * q4 .. + 3 of the fragment's 32 columns
    const int g16 = lane >> 4, j4 = (lane & 15) >> 2, q4 = lane & 3;
    const uint32_t lb = (uint32_t)(uintptr_t)(lptr_t)lds;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int chunk = (j * 128 + wn * 32 + (g16 & 1) * 16) / 8 + (q4 >> 1);
      const int row = 8 * (g16 >> 1) + j4;
      fr_b[j] = (int)(lb + row * 512 + ((chunk ^ tr_swz(row)) << 4) + (q4 & 1) * 8);
    }
  }

  f32x16 acc[2][4];

  // 32-row blocks of this wavefront's half of the unit that hold rows (wave-uniform).  A unit is
  // lean for a wavefront with none or one: its other token blocks are not copied either, so that the
  // last row block of an expert does not move 32 KB of repeated rows per step beside 32 KB of weights.
  // (Measured on layers that have nothing but such units and take the 128-row tiles now: 16 rows per
  // expert, 4096 x 14336: 592 -> 562 us the pass; 64 rows per expert, 1024 x 4096, training: 269 -> 248, of
  // it the partial sums below half.)
  auto active = [&](const Unit& u) -> int {
    return __builtin_amdgcn_readfirstlane(min(4, max(0, (u.rows - wm * 128 + 31) >> 5)));
  };

  // ---- epilogue of one unit: lane holds, per 32x32 accumulator, token row (lane&31) and
  // the weight rows 8*g + 4*(lane>>5) + {0..3}, g = 0..3
  auto epilogue = [&](const Unit& u) {
    if (MODE == MODE_DOWN && u.ws_unit >= 0) {
      // partial sums of one K-split part, in accumulator order: [unit][j][i][quad][thread]; the
      // 32-row blocks that hold rows
      float4* ws = reinterpret_cast<float4*>(p.split_ws) + (size_t)u.ws_unit * (32 * NT) + tid;
      const int n_act = active(u);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (i < n_act)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            ws[((j * 4 + i) * 4 + q) * NT] = make_float4(acc[j][i][q * 4], acc[j][i][q * 4 + 1],
                                                         acc[j][i][q * 4 + 2], acc[j][i][q * 4 + 3]);
      return;
    }
    tile_epilogue<MODE, RAG, 4>(p, acc, u.row0, u.rows, u.nblk, wm, wn, lane);
  };

  auto zero_acc = [&]() {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.f;
  };

  // Every unit has an even number of k-steps (the steps of a tile are rounded up to one and the
  // K-split keeps its parts even).  KT == 0 cannot come out of the schedule (K >= 8); should it
  // ever, nothing is loaded and zeros are stored.
  if (cur.KT == 0) {
    zero_acc();
    epilogue(cur);
    return;
  }

  const uint32_t lds_base = (uint32_t)(uintptr_t)(lptr_t)lds;
  // wave-uniform LDS byte addresses: + stage * 65536 + block * 4096 (tokens) / 8192 (weights)
  const uint32_t a_dst = __builtin_amdgcn_readfirstlane(lds_base + (16 * wm + wn) * 1024);
  const uint32_t b_dst = __builtin_amdgcn_readfirstlane(lds_base + 32768 + wave * 1024);
  // first unit: both stages in full (stage 0 first), then the second group falls one
  // cluster behind
#pragma unroll
  for (int st = 0; st < 2; ++st)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      dma_step<RAG>(a_off[i], asrc(cur, st), a_dst + st * 65536 + i * 4096, 8, lc, p.zero);
      dma_step<RAG>(b_off[i], bsrc(cur, st, i >= 2), b_dst + st * 65536 + i * 8192, BKM ? BK : 8,
                    BKM ? brow + 16 * i : lc, p.zero);
    }
  // stage 0 has landed (stage 1 is first read four clusters on, after the vmcnt(6) waits)
  asm volatile("s_waitcnt vmcnt(8)\n\ts_barrier" ::: "memory");
  if (wm == 1) asm volatile("s_barrier" ::: "memory");

  bf16x8 wb[2][4];
  for (int idx = 0;; ++idx) {
    const Unit nxt = fetch_unit<MODE, BKM, RAG>(p, idx + 1);
    zero_acc();
    const int KT = cur.KT;
    const int nact = active(cur), nact_n = nxt.valid ? active(nxt) : nact;
    const bool lean = nact <= 1, lean_n = nact_n <= 1;
    const bool both = MODE == MODE_UP || cur.nblk * 256 + 128 < p.N;
    // steady part: steps 0 .. KT-3; what was read one cluster ago is refilled with the data
    // of its next use (token block i-1 and weight row blocks 8(i-1)+wave of this stage with
    // step k+2; at i == 0 block 3 of the other stage with step k+1)
#define PP(S, I, OA, BA, OB, BB, NA, NC, W)                                                      \
  pp_cluster<S, I, BKM, RAG, W>(acc, wb, lds, fr_a, fr_b, fr_half, fr_swz, OA, BA, OB, BB,       \
                                a_dst, b_dst, NA, NC, both, lean || lean_n, lc, brow, p.zero)
#define STEADY(W)                                                                                \
  for (int kt = 0; kt < KT - 2; kt += 2) {                                                       \
    const Src a1 = asrc(cur, kt + 1), a2 = asrc(cur, kt + 2), a3 = asrc(cur, kt + 3);            \
    PP(0, 0, a_off[3], a1, b_off[3], bsrc(cur, kt + 1, 1), nact, nact, W);                       \
    PP(0, 1, a_off[0], a2, b_off[0], bsrc(cur, kt + 2, 0), nact, nact, W);                       \
    PP(0, 2, a_off[1], a2, b_off[1], bsrc(cur, kt + 2, 0), nact, nact, W);                       \
    PP(0, 3, a_off[2], a2, b_off[2], bsrc(cur, kt + 2, 1), nact, nact, W);                       \
    PP(1, 0, a_off[3], a2, b_off[3], bsrc(cur, kt + 2, 1), nact, nact, W);                       \
    PP(1, 1, a_off[0], a3, b_off[0], bsrc(cur, kt + 3, 0), nact, nact, W);                       \
    PP(1, 2, a_off[1], a3, b_off[1], bsrc(cur, kt + 3, 0), nact, nact, W);                       \
    PP(1, 3, a_off[2], a3, b_off[2], bsrc(cur, kt + 3, 1), nact, nact, W);                       \
  }
    if (lean) {
      STEADY(3)
    } else {
      STEADY(6)
    }
    // last two steps: the refills fetch steps 0 and 1 of the next unit (the token offsets
    // are switched block by block, each right after its last use for this unit).  Without a
    // next unit the last step is fetched again (in bounds, never read): at least one copy per
    // cluster, which the vmcnt arithmetic relies on.
    {
      const int nc = lean ? nact : 4, nn = lean_n ? nact_n : 4;   // token blocks of this and the next unit
      const Src last = asrc(cur, KT - 1);
      const Src na = nxt.valid ? asrc(nxt, 0) : last;                 // next unit's step 0
      const Src nb0 = nxt.valid ? bsrc(nxt, 0, 0) : bsrc(cur, KT - 1, 0);
      const Src nb1 = nxt.valid ? bsrc(nxt, 0, 1) : bsrc(cur, KT - 1, 1);
      const Src ma = nxt.valid ? asrc(nxt, 1) : last;                 // ... its step 1
      const Src nc0 = nxt.valid ? bsrc(nxt, 1, 0) : nb0;
      const Src nc1 = nxt.valid ? bsrc(nxt, 1, 1) : nb1;
      // RAG: a last step that only rounds the count up to even holds nothing but zeros
      const int nact1 = RAG && last.nv <= 0 ? 0 : nact;
      PP(0, 0, a_off[3], last, b_off[3], bsrc(cur, KT - 1, 1), nact, nc, -1);
      if (nxt.valid) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          a_off[i] = token_off(nxt.rows, i);
          if (RAG) b_off[i] = weight_off(nxt.nblk, i);
        }
      }
      PP(0, 1, a_off[0], na, b_off[0], nb0, nact, nn, -1);
      PP(0, 2, a_off[1], na, b_off[1], nb0, nact, nn, -1);
      PP(0, 3, a_off[2], na, b_off[2], nb1, nact, nn, -1);
      if (nxt.valid) {
        a_off[3] = token_off(nxt.rows, 3);
        if (RAG) b_off[3] = weight_off(nxt.nblk, 3);
      }
      PP(1, 0, a_off[3], na, b_off[3], nb1, nact1, nn, -1);
      PP(1, 1, a_off[0], ma, b_off[0], nc0, nact1, nn, -1);
      PP(1, 2, a_off[1], ma, b_off[1], nc0, nact1, nn, -1);
      PP(1, 3, a_off[2], ma, b_off[2], nc1, nact1, nn, -1);
#undef STEADY
#undef PP
    }
    epilogue(cur);
    if (!nxt.valid) break;
    cur = nxt;
  }
  if (wm == 0) asm volatile("s_barrier" ::: "memory");  // as many barriers as the other group
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // no copy in flight into LDS at exit
}

// Sums the parts of every K-split tile of the down GEMM in a fixed order (part 0, 1, ...:
// deterministic) and stores the tile like the GEMM's own epilogue.  Eight blocks per split
// tile, one per accumulator (j, i) of the GEMM's wavefront tile; thread and accumulator
// indices mean what they mean in ffn_mfma_kernel.  All parts of a quad are loaded before
// they are added.
__global__ __launch_bounds__(NT) void ffn_split_reduce_kernel(const GemmArgs p) {
  const int n_tiles = p.sched->down_split_tiles;
  const int tile = blockIdx.x >> 3, ji = blockIdx.x & 7;
  if (tile >= n_tiles) return;
  const int split = p.sched->down_split;
  const TileDesc tl = p.order[p.sched->down_full + tile];
  const int j = ji >> 2, i = ji & 3;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 2, wn = wave & 3;
  const int fr_row = lane & 31, fr_half = lane >> 5;
  if (wm * 128 + i * 32 >= tl.rows) return;   // no rows here: nothing was stored
  const float4* ws = reinterpret_cast<const float4*>(p.split_ws) +
                     (size_t)tile * split * (32 * NT) + (size_t)(ji * 4) * NT + tid;
  const int m_local = wm * 128 + i * 32 + fr_row;
  const bool live = m_local < tl.rows;
  const size_t row = (size_t)(tl.row0 + m_local);
  const int col0 = tl.nblk * 256 + j * 128 + wn * 32 + 4 * fr_half;
  // every part of all four quads is requested before anything is added (up to 32 loads of
  // 16 bytes in flight per thread: with one quad at a time the kernel was bound by four
  // memory latencies in a row)
  float4 part[4][8];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int pt = 0; pt < 8; ++pt)
      part[q][pt] = pt < split ? ws[(size_t)pt * (32 * NT) + q * NT] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float4 v = part[q][0];
#pragma unroll
    for (int pt = 1; pt < 8; ++pt) {
      v.x += part[q][pt].x; v.y += part[q][pt].y; v.z += part[q][pt].z; v.w += part[q][pt].w;
    }
    if (live && col0 + 8 * q < p.N)
      *reinterpret_cast<uint2*>(p.C + row * p.N + col0 + 8 * q) =
          make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
  }
}

}  // namespace

// bf16 storage: the tiled kernels take every size the boundary takes (multiples of 8) as long as the
// 32-bit byte offsets inside a tile (255 rows of 2f or of d elements) stay far below their limit; the
// vector-ALU kernels serve longer rows.
bool ffn_mfma_supported(const moe_ctx* c) {
  return c->cfg.dtype == MOE_BF16 && c->cfg.f <= 128 * 4095 && c->cfg.d <= 256 * 4095;
}

size_t ffn_mfma_order_entries(const moe_ctx* c) {
  return (size_t)c->max_mtiles[1] * std::max(ceil_div(c->cfg.f, 128), ceil_div(c->cfg.d, 256));
}

// dX of the gated expert has the longest contraction of the down-type GEMMs.
size_t ffn_mfma_split_tiles(const moe_ctx* c) {
  return split_tiles_max((long long)c->max_mtiles[1] * ceil_div(c->cfg.d, 256), c->n_cu, k_steps(c->cfg.f, 2));
}

// Not part of the interface, for the test of the bound above (needs no GPU): partial tiles of a launch
// of `tiles` tiles, and the most there can be with up to `tiles_max`.
extern "C" void moe_internal_split_tiles(int32_t tiles, int64_t tiles_max, int32_t n_cu, int32_t kt,
                                         int32_t* used, int64_t* most) {
  const int tail = tiles % n_cu, split = split_parts(tail, n_cu, kt);
  *used = split > 1 ? tail * split : 0;
  *most = (int64_t)split_tiles_max(tiles_max, n_cu, kt);
}

static int run_sched(moe_ctx* c, const int32_t* counts, const int32_t* offsets, int nt_a, int nt_b,
                     int kt_b, int nt_dh128, const void* const* up_b0, const void* const* up_b1,
                     const void* const* down_b0, const void* const* down_b1, hipStream_t s) {
  hipLaunchKernelGGL(mfma_sched_kernel, dim3(32), dim3(256), 0, s, counts, offsets,
                     c->d_wtab + 0 * MOE_MAX_EXPERTS, c->cfg.E, c->S_call, c->max_mtiles[1], nt_a,
                     nt_b, c->n_cu, kt_b, nt_dh128, c->d_sched[1], up_b0, up_b1, down_b0, down_b1,
                     c->d_order_up, c->d_order_down);
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_EHIP;
}

// One block per compute unit (a block takes all of a unit's LDS), a multiple of 8 so that
// every XCD gets the same number of blocks.
static int persistent_grid(const moe_ctx* c) { return std::max(8, (c->n_cu / 8) * 8); }

// A GEMM of the tile list `order`: A [rows, lda], contraction of `segs` segments of `seg_len`,
// N output columns in blocks of bn (ldb: row length of a k-major weight-role operand, else 0).
static GemmArgs tiled_args(moe_ctx* c, const void* A, int lda, const TileDesc* order, int bn,
                           int seg_len, int segs, int ldb, int N, void* C) {
  GemmArgs a{};
  a.A = (const uint16_t*)A;
  a.lda = lda;
  a.sched = c->d_sched[1];
  a.order = order;
  a.n_tiles_n = ceil_div(N, bn);
  a.K = seg_len * segs;
  a.N = N;
  a.C = (uint16_t*)C;
  a.ldb = ldb;
  a.kt = k_steps(seg_len, segs);
  a.kseg = segs == 1 ? a.kt : ceil_div(seg_len, BK);
  a.kseg_len = seg_len;
  a.zero = (const char*)c->d_zero;
  return a;
}

// The plain kernel where the tile divides the sizes (an even number of whole k-steps, no segment
// ends inside one, whole column blocks): its copies need neither the per-step test nor the
// column clamp, 10 to 16 registers less.  Anything else takes the RAG kernel.
template <int MODE, bool BKM>
static void launch_gemm(moe_ctx* c, const GemmArgs& a, hipStream_t s) {
  const bool whole = a.K % (2 * BK) == 0 && a.kseg_len % BK == 0 &&
                     a.N % (MODE == MODE_UP ? 128 : 256) == 0;
  if (whole)
    hipLaunchKernelGGL((ffn_mfma_kernel<MODE, BKM, false>), dim3(persistent_grid(c)), dim3(NT), 0, s, a);
  else
    hipLaunchKernelGGL((ffn_mfma_kernel<MODE, BKM, true>), dim3(persistent_grid(c)), dim3(NT), 0, s, a);
}

// Down-type GEMM (plain epilogue) with the K-split tail: the GEMM, then the sum of the parts.
template <bool BKM>
static void launch_down(moe_ctx* c, GemmArgs& a, hipStream_t s) {
  a.split_ws = c->d_split_ws;
  launch_gemm<MODE_DOWN, BKM>(c, a, s);
  hipLaunchKernelGGL(ffn_split_reduce_kernel, dim3((c->n_cu / 2) * 8), dim3(NT), 0, s, a);
}

int launch_ffn_mfma(moe_ctx* c, bool gated, const int32_t* counts, const int32_t* offsets,
                    const void* x_packed, void* y_packed, void* G, void* U, hipStream_t s) {
  const int d = c->cfg.d, f = c->cfg.f;
  const int bn_up = gated ? 128 : 256;
  const void* const* W1 = c->d_wtab + 0 * MOE_MAX_EXPERTS;
  const void* const* W3 = c->d_wtab + 1 * MOE_MAX_EXPERTS;
  const void* const* W2 = c->d_wtab + 2 * MOE_MAX_EXPERTS;
  prof_mark(c, 0, s);
  int st = run_sched(c, counts, offsets, ceil_div(f, bn_up), ceil_div(d, 256), k_steps(f, 1), 0, W1,
                     gated ? W3 : nullptr, W2, nullptr, s);
  if (st != MOE_OK) return st;
  prof_mark(c, 1, s);
  GemmArgs up = tiled_args(c, x_packed, d, c->d_order_up, bn_up, d, 1, 0, f, c->d_H);
  up.Gs = (uint16_t*)G;
  up.Us = (uint16_t*)U;
  if (gated) launch_gemm<MODE_UP, false>(c, up, s);
  else launch_gemm<MODE_UP1, false>(c, up, s);
  prof_mark(c, 2, s);
  GemmArgs dn = tiled_args(c, c->d_H, f, c->d_order_down, 256, f, 1, 0, d, y_packed);
  launch_down<false>(c, dn, s);
  prof_mark(c, 3, s);
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_EHIP;
}

// dy, xp: [S,d]; G, U: [S,f] (forward saves); dxp out.  Workspace (context): d_H [S,f],
// d_dGU [S,2f].  Two-matrix expert (!gated): no U, no W3: d_dGU holds dG [S,f], two weight
// gradients.  The weights are read as they are stored: W2 [d,f] is k-major for dH = dY W2,
// W1 and W3 [f,d] are k-major for dX = dG W1 + dU W3 (one GEMM over the concatenated k).
int launch_ffn_bwd_mfma(moe_ctx* c, bool gated, const void* dy, const void* xp, const void* G,
                        const void* U, const int32_t* counts, const int32_t* offsets, void* dxp,
                        hipStream_t s) {
  const int d = c->cfg.d, f = c->cfg.f;
  const void* const* W1 = c->d_wtab + 0 * MOE_MAX_EXPERTS;
  const void* const* W3 = c->d_wtab + 1 * MOE_MAX_EXPERTS;
  const void* const* W2 = c->d_wtab + 2 * MOE_MAX_EXPERTS;
  const int segs = gated ? 2 : 1;     // dX contracts over dG and dU
  const bool small = ffn_tile128_wanted(c, gated, true);
  int st;
  // dH = dY W2 with the activation's derivative in the epilogue -> [dG|dU], H
  if (small) {
    st = launch_ffn_tile128_dh(c, gated, dy, G, U, counts, offsets, false, s);
    if (st != MOE_OK) return st;
  } else {
    const bool offered = ffn_tile128_dh_offered(c);   // the 128-row tiles' dH as well
    st = run_sched(c, counts, offsets, ceil_div(f, 256), ceil_div(d, 256), k_steps(f, segs),
                   offered ? ceil_div(f, 128) : 0, W2, nullptr, W1, gated ? W3 : nullptr, s);
    if (st == MOE_OK && offered) st = launch_ffn_tile128_dh(c, gated, dy, G, U, counts, offsets, true, s);
    if (st != MOE_OK) return st;
    GemmArgs dh = tiled_args(c, dy, d, c->d_order_up, 256, d, 1, f, f, c->d_dGU);
    dh.C2 = (uint16_t*)c->d_H;
    dh.Gs = (uint16_t*)const_cast<void*>(G);
    dh.Us = (uint16_t*)const_cast<void*>(U);
    if (gated) launch_gemm<MODE_DH, true>(c, dh, s);
    else launch_gemm<MODE_DH1, true>(c, dh, s);
  }
  // weight gradients straight from dY, X, H and [dG|dU] (transpose reads from LDS), right
  // after the kernel that wrote H and [dG|dU]; dX last, so that the caller's next kernel
  // (the backward of dispatch) finds it in the last-level cache
  st = launch_wgrad_tr(c, gated, dy, xp, c->d_H, c->d_dGU, counts, offsets, s);
  if (st != MOE_OK) return st;
  // dX = [dG|dU] [W1; W3]  (one GEMM with contraction length 2f; f without U)
  if (small) return launch_ffn_tile128_dx(c, gated, counts, offsets, dxp, s);
  GemmArgs dx = tiled_args(c, c->d_dGU, segs * f, c->d_order_down, 256, f, segs, d, d, dxp);
  launch_down<true>(c, dx, s);
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_EHIP;
}
