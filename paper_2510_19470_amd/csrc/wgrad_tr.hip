// Weight gradients of the expert FFN on the matrix cores without transposed copies of the
// activations: the chain rule of the expert FFN of Sec. 2.1 taken with respect to its
// weights (the paper itself only notes, in Sec. 6, that the backward pass adds a constant
// all-reduce term to its model).
//
//   dW[e][m, n] = sum over the rows r of expert e of  P[r, m] * Q[r, n]      (fp32 out)
//
// Both operands are stored with the contraction index (the token row) OUTERMOST: an MFMA
// fragment (one output row or column, 8 consecutive k) is a column of 8 rows in memory.  The
// tiles are copied to LDS as they are (16 token rows x 256 columns, 512 bytes per row, direct
// global -> LDS copies) and read with the LDS transpose read of gfx950,
// ds_read_b64_tr_b16: inside a group of 16 lanes, lane s supplies the address of 4 elements
// of row (s >> 2) -- column group (s & 3) -- and lane i receives element (i & 3) of the four
// addresses of lanes (i >> 2) + {0, 4, 8, 12}.  With lane s pointing at row k0 + (s >> 2),
// columns c0 + 4 * (s & 3) .. + 3, lane i ends up with column c0 + i, rows k0 .. k0 + 3: two
// such reads give the 8 consecutive k of one MFMA operand register pair.
//
// Block tile 256 (m) x 256 (n), 8 wavefronts (2 along m x 4 along n), wavefront tile 128 x 64
// = 4 x 2 accumulators of v_mfma_f32_32x32x16_bf16, as in the forward kernels.  The contraction
// runs in slices of 16 token rows through a ring of 8 LDS slots of 16 KB (P 8 KB + Q 8 KB), seven
// slices ahead.  The two groups of four wavefronts (wm) alternate as in the forward kernel: while
// one multiplies a slice (8 MFMAs), the other reads its 12 fragments of the next one and issues two
// copies.  16-byte chunks of a row are XOR-swizzled (tr_swz), which puts the rows x 32 bytes that the
// groups of 16 lanes sharing an LDS cycle read on distinct banks.  Rows past the end of the
// expert's segment are fetched from a row of zeros, so a ragged segment needs no padded copy.
//
// What bounds it.  The P columns are the MFMA "A" operand and the Q columns the "B" operand: a
// lane holds one column of dW, and a store instruction writes two whole 128-byte lines.  (The other
// way round, 16 bytes per lane spread over 32 rows, it writes 32-byte pieces of 32 lines: the same
// loop takes 223 us instead of 204.)  The loop takes about 0.5 us per slice, without copies 0.42 us;
// registers-only MFMAs on random operands take 0.34 us (the clock falls under the power limit).  6190 rows, 6 experts, d = f = 2048: 234 -> 203 us (1.5e11
// flop, 302 MB written); 21000 rows, 12 experts, 2048 x 1408: 515 -> 475; 1500 rows, 6 experts, 1160
// x 2888: 99 -> 91, against the loop of 32-row half-steps with one barrier each.  Within 3 % of it:
// all reads of the next slice between the MFMAs of this one, one barrier a slice (207); 256 x 128
// tiles with two blocks on a compute unit (204 to 209); persistent blocks that copy on across tiles
// (208).
#include <type_traits>

#include "ffn_tile.h"

namespace {

constexpr int NT = 512;
constexpr int HK = 16;                 // token rows per slice
constexpr int SLOTS = 8;
constexpr int TILE_BYTES = HK * 512;   // one operand tile of a slot
constexpr int SLOT_BYTES = 2 * TILE_BYTES;

// few rows per expert (wgrad_few_kernel): tiles of 256 x 128, half-steps of 32 rows, 3 stages of 24 KB
constexpr int F_NT = 256, F_BN = 128, F_HK = 32, F_STAGES = 3;
constexpr int F_P_BYTES = F_HK * 512, F_STAGE_BYTES = F_P_BYTES + F_HK * F_BN * 2;
constexpr int F_COPIES = F_STAGE_BYTES / 1024 / (F_NT / 64);   // per wavefront and half-step

struct WgradArgs {
  struct Job {
    const uint16_t* P;   // [S, p_pitch]; the tile's columns start at p_col0 + 256 * (row block)
    const uint16_t* Q;   // [S, q_pitch]
    const void* const* dWt;   // [E] fp32 outputs [Mo, No]
    int p_pitch, p_col0, q_pitch, Mo, No;
  } job[3];
  int n_jobs, E;
  int n_list;                         // experts that get weight gradients
  uint8_t list[MOE_MAX_EXPERTS];      // ... their ids, ascending
  const int32_t* counts;
  const int32_t* offsets;
  const TileSched* sched;     // of the data-gradient GEMMs of the same call: n_mtiles == 0 when
                              // the caller's counts and offsets do not fit the buffers
  const uint16_t* zero_row;   // 512 bytes of zeros
};

// A wavefront's 128 x 64 of dW from (m0, n0): a lane holds column (lane & 31) of each 32-column block and
// the rows 8g + 4(lane >> 5) + {0..3} of each 32-row block.  The gradients are the call's largest array, and the
// dX GEMM after this launch reads the weights and [dG|dU]: stores past the last-level cache leave those in it
// (training step, us: 6190 rows, 2048 x 2048, 302 MB of gradients: 782 -> 768; two-matrix, 64 rows per expert of
// 1024 x 4096, 268 MB: 197 -> 190; 2048 tokens, 1024 x 1024, 75 MB: 174 -> 171).  With an update of fp32 weights that reads
// them right after it, backward and update, us: 25 MB: 66 -> 66; 50 MB: 83 -> 84; 75 MB: 117 -> 115; 151 MB: 192 -> 186, 317 -> 312;
// 268 MB: 243 -> 238; 302 MB: 523 -> 505; 415 MB: 507 -> 475.  Only where the 32 columns of a store are a 128-byte line:
// pieces of lines lose (1160 x 2888: 291 -> 296; 648 x 1400: 243 -> 248).
template <bool RAG, bool LINES, int NI = 4, int NJ = 2>
__device__ __forceinline__ void store_tile(const f32x16 (&acc)[2][4], float* dW, int m0, int n0, int Mo, int No,
                                           int lane) {
  const int col = lane & 31, half = lane >> 5;
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + i * 32 + 8 * g + 4 * half + r;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int n = n0 + j * 32 + col;
          if (RAG && (m >= Mo || n >= No)) continue;
          if (LINES) __builtin_nontemporal_store(acc[j][i][g * 4 + r], dW + (size_t)m * No + n);
          else dW[(size_t)m * No + n] = acc[j][i][g * 4 + r];
        }
      }
}

// RAG: some last block is not whole (d or f no multiple of 256): columns are clamped and guarded.
// A kernel of its own, so that whole sizes do not pay for the guards of the stores.  LINES: see store_tile
// (a template argument: of two ways to store in one kernel the compiler makes one, the plain one).
template <bool RAG, bool LINES>
__global__ __launch_bounds__(NT) void wgrad_tr_kernel(const WgradArgs p) {
  __shared__ uint4 lds[SLOTS * SLOT_BYTES / 16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;

  // block -> tile.  The tiles are ordered (expert, job, groups of 4 row blocks of dW, column
  // block, row block inside the group): 32 consecutive tiles are a 4 x 8 patch of one matrix,
  // 12 operand panels for 32 tiles.  The hardware deals blocks round-robin to the 8 XCDs, each
  // with an L2 of its own, so XCD x (= blockIdx & 7) takes the chunks of 32 consecutive tiles
  // x, x + 8, ...: the 32 blocks resident on an XCD share their panels in its L2.  (Every job
  // has the same number of tiles per expert.)
  const int tiles = ((p.job[0].Mo + 255) >> 8) * ((p.job[0].No + 255) >> 8);
  const int total = p.n_list * p.n_jobs * tiles;
  const int slot = (int)(blockIdx.x >> 3), xcd = (int)(blockIdx.x & 7);
  const int L = ((slot >> 5) * 8 + xcd) * 32 + (slot & 31);
  if (L >= total) return;
  const int ej = L / tiles, rel = L % tiles;
  const int e = p.list[ej / p.n_jobs];
  const WgradArgs::Job& J = p.job[ej % p.n_jobs];
  const int NoT = (J.No + 255) >> 8, MoT = (J.Mo + 255) >> 8;
  const int mg = rel / (4 * NoT), r2 = rel % (4 * NoT);
  const int gm = min(4, MoT - 4 * mg);
  const int nblk = r2 / gm, mblk = 4 * mg + r2 % gm;
  float* dW = (float*)J.dWt[e];
  if (dW == nullptr) return;   // this gradient is not wanted
  // counts and offsets are the caller's; the schedule kernel of this call has checked them
  // against the buffer size (no tiles at all if any segment does not fit: zeros come out)
  const int n_e = p.sched->n_mtiles > 0 ? p.counts[e] : 0;
  const int row0 = p.offsets[e];
  const int NS = (n_e + HK - 1) / HK;   // slices

  f32x16 acc[2][4];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.f;

  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;

  // ---- copies: wavefront w fills rows 2w (lanes 0-31) and 2w+1 (lanes 32-63) of both operand
  // tiles of a slice, 32 chunk slots each; slot c of row r holds global chunk c ^ tr_swz(r)
  const int c_row = 2 * wave + (lane >> 5);
  const int gch = (lane & 31) ^ tr_swz(c_row);
  // ... held inside the matrix (multiples of 8 columns) in a last block that is not whole: what it
  // repeats is not stored
  const int gp = RAG ? min(gch, (J.Mo - mblk * 256) / 8 - 1) : gch;
  const int gq = RAG ? min(gch, (J.No - nblk * 256) / 8 - 1) : gch;
  const uint32_t p_pitch = J.p_pitch * 2, q_pitch = J.q_pitch * 2;
  const uint32_t p_off = c_row * p_pitch + gp * 16, q_off = c_row * q_pitch + gq * 16;
  const char* p_base = uniform_ptr((const char*)(J.P + J.p_col0 + mblk * 256) + (size_t)row0 * p_pitch);
  const char* q_base = uniform_ptr((const char*)(J.Q + nblk * 256) + (size_t)row0 * q_pitch);
  const uint32_t dst = __builtin_amdgcn_readfirstlane(lds_base + wave * 1024);
  const char* zp = (const char*)p.zero_row;
  int left = n_e;        // rows from the next slice to copy on (negative: all of it are zeros)
  uint32_t cslot = 0;    // byte offset of its slot
  auto issue = [&]() {
    if (left >= HK) {
      dma16(p_off, p_base, dst + cslot);
      dma16(q_off, q_base, dst + cslot + TILE_BYTES);
    } else {
      const bool ok = c_row < left;
      dma16v(ok ? p_base + p_off : zp, dst + cslot);
      dma16v(ok ? q_base + q_off : zp, dst + cslot + TILE_BYTES);
    }
    p_base += HK * p_pitch;
    q_base += HK * q_pitch;
    left -= HK;
    cslot = (cslot + SLOT_BYTES) & (SLOTS * SLOT_BYTES - 1);
  };

  // ---- transpose reads: LDS byte addresses of the lane's 4 columns in slot 0
  const int g16 = lane >> 4, hh = g16 >> 1, cb = g16 & 1;
  const int s16 = lane & 15, j4 = s16 >> 2, q4 = s16 & 3;
  const int rd_row = 8 * hh + j4;                 // and + 4: the swizzle is the same
  const int rd_swz = tr_swz(rd_row);
  const uint32_t rd0 = lds_base + rd_row * 512 + (q4 & 1) * 8;
  auto frag = [&](uint32_t a0) -> bf16x8 {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)a0);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)(a0 + 4 * 512));
    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  };

  // NI x NJ: 32 x 32 blocks of a wavefront.  A last block of rows or columns that holds at most 128 of its 256
  // is shared by all wavefronts (half the MFMAs each) instead of leaving half of them with padding
  // (12 experts of 2048 x 1408, training step: 1429 -> 1411 us).
  auto tile = [&](auto ni, auto nj) {
    constexpr int NI = decltype(ni)::value, NJ = decltype(nj)::value;
    uint32_t x_adr[NI], w_adr[NJ];
#pragma unroll
    for (int i = 0; i < NI; ++i)
      x_adr[i] = rd0 + ((((wm * (32 * NI) + i * 32 + cb * 16) / 8 + (q4 >> 1)) ^ rd_swz) << 4);
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      w_adr[j] = rd0 + TILE_BYTES + ((((wn * (32 * NJ) + j * 32 + cb * 16) / 8 + (q4 >> 1)) ^ rd_swz) << 4);
    if (NS > 0) {
#pragma unroll
      for (int h = 0; h < SLOTS - 1; ++h) issue();
      // slice 0 has landed; then the second group falls one barrier behind
      asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * (SLOTS - 2)) : "memory");
      if (wm == 1) asm volatile("s_barrier" ::: "memory");
      uint32_t sb = 0;
      for (int s = 0; s < NS; ++s) {
        bf16x8 xa[NI], wb[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) wb[j] = frag(w_adr[j] + sb);
#pragma unroll
        for (int i = 0; i < NI; ++i) xa[i] = frag(x_adr[i] + sb);
        // Slice s + 7 goes to the slot of slice s - 1: the other group's reads of it ended before the
        // last barrier, at which every wavefront's reads were done (lgkmcnt below).
        issue();
        sb = (sb + SLOT_BYTES) & (SLOTS * SLOT_BYTES - 1);
        // All but the last 12 copies have landed: those of slices s + 2 .. s + 7.  Every wavefront
        // has passed this point of step s before anybody reads slice s + 1.
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * (SLOTS - 2)) : "memory");
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int i = 0; i < NI; ++i)
            acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xa[i], wb[j], acc[j][i], 0, 0, 0);
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_barrier" ::: "memory");
      }
      if (wm == 0) asm volatile("s_barrier" ::: "memory");   // as many barriers as the other group
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // no copy in flight into LDS at exit
    }
    store_tile<RAG, LINES, NI, NJ>(acc, dW, mblk * 256 + wm * (32 * NI), nblk * 256 + wn * (32 * NJ), J.Mo, J.No, lane);
  };
  typedef std::integral_constant<int, 1> one;
  typedef std::integral_constant<int, 2> two;
  typedef std::integral_constant<int, 4> four;
  if (!RAG) {
    tile(four{}, two{});
  } else {
    const bool few_m = J.Mo - mblk * 256 <= 128, few_n = J.No - nblk * 256 <= 128;
    if (few_m && few_n) tile(two{}, one{});
    else if (few_m) tile(two{}, two{});
    else if (few_n) tile(four{}, one{});
    else tile(four{}, two{});
  }
}

// The same for few rows per expert, where a block's start (its expert, counts and first copies: three cold
// loads in a row) and its stores take longer than its few slices: 256 x 128 tiles of 256 threads, two blocks
// on a compute unit, so that one starts or stores while the other computes; one barrier per half-step.
// 64 rows, 8 experts, 1024 x 4096: 88 -> 77 us (403 MB written); 250 rows, 6 experts, 1160 x 2888: 91 -> 95;
// 1032 rows, 2048 x 2048: 203 -> 204 to 209 (half as much work per byte copied).
template <bool RAG, bool LINES>
__global__ __launch_bounds__(F_NT, 2) void wgrad_few_kernel(const WgradArgs p) {
  __shared__ uint4 lds[F_STAGES * F_STAGE_BYTES / 16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  // block -> tile, ordered as above; the 64 blocks resident on an XCD are a 4 x 16 patch.  (The jobs have
  // different numbers of tiles where a matrix ends inside one.)
  auto tiles_of = [&](const WgradArgs::Job& J) { return ((J.Mo + 255) >> 8) * ((J.No + F_BN - 1) / F_BN); };
  const int slot = (int)(blockIdx.x >> 3), xcd = (int)(blockIdx.x & 7);
  int L = ((slot >> 6) * 8 + xcd) * 64 + (slot & 63);
  const int t0 = tiles_of(p.job[0]), t1 = tiles_of(p.job[1]), per_e = t0 + (p.n_jobs - 1) * t1;
  if (L >= p.n_list * per_e) return;
  const int e = p.list[L / per_e];
  L %= per_e;
  const int ji = L < t0 ? 0 : 1 + (L - t0) / t1;
  if (ji > 0) L = (L - t0) % t1;
  const WgradArgs::Job& J = p.job[ji];
  const int NoT = (J.No + F_BN - 1) / F_BN, MoT = (J.Mo + 255) >> 8;
  const int mg = L / (4 * NoT), r2 = L % (4 * NoT);
  const int gm = min(4, MoT - 4 * mg);
  const int nblk = r2 / gm, mblk = 4 * mg + r2 % gm;
  float* dW = (float*)J.dWt[e];
  if (dW == nullptr) return;   // this gradient is not wanted
  const int n_e = p.sched->n_mtiles > 0 ? p.counts[e] : 0;   // (checked, as above)
  const int row0 = p.offsets[e];
  const int NH = (n_e + F_HK - 1) / F_HK;

  f32x16 acc[2][4];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.f;

  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
  // copies: instruction c of P (0..15) fills rows 2c, 2c + 1, of Q (0..7) rows 4c .. 4c + 3; wavefront w
  // issues c = w, w + 4, ...
  const char* p_col = (const char*)(J.P + J.p_col0 + mblk * 256);
  const char* q_col = (const char*)(J.Q + nblk * F_BN);
  int p_row[4], q_row[2], p_ch[4], q_ch[2];   // row inside the stage, byte offset inside the row
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    p_row[u] = 2 * (wave + 4 * u) + (lane >> 5);
    const int ch = (lane & 31) ^ tr_swz(p_row[u]);
    p_ch[u] = (RAG ? min(ch, (J.Mo - mblk * 256) / 8 - 1) : ch) * 16;
  }
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    q_row[u] = 4 * (wave + 4 * u) + (lane >> 4);
    const int ch = (lane & 15) ^ tr_swz(q_row[u]);
    q_ch[u] = (RAG ? min(ch, (J.No - nblk * F_BN) / 8 - 1) : ch) * 16;
  }
  const uint32_t p_pitch = J.p_pitch * 2, q_pitch = J.q_pitch * 2;
  const char* zp = (const char*)p.zero_row;
  auto issue = [&](int h, uint32_t sb) {   // all copies of half-step h; rows past the segment: zeros
    const uint32_t dp = __builtin_amdgcn_readfirstlane(sb + wave * 1024);
    if ((h + 1) * F_HK <= n_e) {
      const char* pb = uniform_ptr(p_col + (size_t)(row0 + h * F_HK) * p_pitch);
      const char* qb = uniform_ptr(q_col + (size_t)(row0 + h * F_HK) * q_pitch);
#pragma unroll
      for (int u = 0; u < 4; ++u) dma16(p_row[u] * p_pitch + p_ch[u], pb, dp + u * 4096);
#pragma unroll
      for (int u = 0; u < 2; ++u) dma16(q_row[u] * q_pitch + q_ch[u], qb, dp + F_P_BYTES + u * 4096);
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int rg = h * F_HK + p_row[u];
        dma16v(rg < n_e ? p_col + (size_t)(row0 + rg) * p_pitch + p_ch[u] : zp, dp + u * 4096);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int rg = h * F_HK + q_row[u];
        dma16v(rg < n_e ? q_col + (size_t)(row0 + rg) * q_pitch + q_ch[u] : zp, dp + F_P_BYTES + u * 4096);
      }
    }
  };
  const int g16 = lane >> 4, hh = g16 >> 1, cb = g16 & 1;
  const int s16 = lane & 15, j4 = s16 >> 2, q4 = s16 & 3;
  const int rd_row = 8 * hh + j4;                 // + 16 kk + 4 t leaves the swizzle unchanged
  const int rd_swz = tr_swz(rd_row);
  uint32_t x_off[4], w_off[2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    x_off[i] = rd_row * 512 + (q4 & 1) * 8 +
               ((((wm * 128 + i * 32 + cb * 16) / 8 + (q4 >> 1)) ^ rd_swz) << 4);
#pragma unroll
  for (int j = 0; j < 2; ++j)
    w_off[j] = F_P_BYTES + rd_row * (F_BN * 2) + (q4 & 1) * 8 +
               ((((wn * 64 + j * 32 + cb * 16) / 8 + (q4 >> 1)) ^ rd_swz) << 4);
  auto frag = [&](uint32_t a0, int pitch) -> bf16x8 {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)a0);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)(a0 + 4 * pitch));
    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  };
  if (NH > 0) {
    uint32_t sb = lds_base, sb2 = lds_base + 2 * F_STAGE_BYTES;   // stages of half-steps h and h + 2
    issue(0, sb);
    issue(1, sb + F_STAGE_BYTES);
    for (int h = 0; h < NH; ++h) {
      // half-step h has landed (the copies of h + 1 may be in flight) for everybody behind the barrier;
      // everybody has also read half-step h - 1, whose stage takes half-step h + 2
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(F_COPIES) : "memory");
      issue(h + 2, sb2);
      bf16x8 xa[2][4], wb[2][2];
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
        for (int j = 0; j < 2; ++j) wb[kk][j] = frag(sb + w_off[j] + kk * 16 * (F_BN * 2), F_BN * 2);
#pragma unroll
        for (int i = 0; i < 4; ++i) xa[kk][i] = frag(sb + x_off[i] + kk * 16 * 512, 512);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xa[kk][i], wb[kk][j], acc[j][i], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      sb = sb == lds_base + 2 * F_STAGE_BYTES ? lds_base : sb + F_STAGE_BYTES;
      sb2 = sb2 == lds_base + 2 * F_STAGE_BYTES ? lds_base : sb2 + F_STAGE_BYTES;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no copy in flight into LDS at exit
  }
  store_tile<RAG, LINES>(acc, dW, mblk * 256 + wm * 128, nblk * F_BN + wn * 64, J.Mo, J.No, lane);
}

}  // namespace

// dy, xp: [S,d]; H: [S,f]; dGU: [S,gw] (dG | dU, or dG alone for the two-matrix expert).
int launch_wgrad_tr(moe_ctx* c, bool gated, const void* dy, const void* xp, const void* H,
                    const void* dGU, const int32_t* counts, const int32_t* offsets,
                    hipStream_t s) {
  const int d = c->cfg.d, f = c->cfg.f, E = c->cfg.E;
  const int gw = gated ? 2 * f : f;
  WgradArgs a{};
  a.n_jobs = gated ? 3 : 2;
  a.E = E;
  a.counts = counts;
  a.offsets = offsets;
  a.sched = c->d_sched[1];
  for (int e = 0; e < E; ++e)   // host copy of the pointer tables: resident, some dW wanted
    if (c->h_wtab[0][e] != nullptr &&
        (c->h_wtab[3][e] != nullptr || c->h_wtab[4][e] != nullptr || c->h_wtab[5][e] != nullptr))
      a.list[a.n_list++] = (uint8_t)e;
  if (a.n_list == 0) return MOE_OK;
  a.zero_row = (const uint16_t*)c->d_zero;
  const void* const* dW1 = c->d_wtab + 3 * MOE_MAX_EXPERTS;
  const void* const* dW3 = c->d_wtab + 4 * MOE_MAX_EXPERTS;
  const void* const* dW2 = c->d_wtab + 5 * MOE_MAX_EXPERTS;
  // dW2 [d,f] = dY^T H;  dW1 [f,d] = dG^T X;  dW3 [f,d] = dU^T X
  a.job[0] = {(const uint16_t*)dy, (const uint16_t*)H, dW2, d, 0, f, d, f};
  a.job[1] = {(const uint16_t*)dGU, (const uint16_t*)xp, dW1, gw, 0, d, f, d};
  a.job[2] = {(const uint16_t*)dGU, (const uint16_t*)xp, dW3, gw, f, d, f, d};
  // whole lines to store (store_tile), by the sizes and by where the gradients lie
  bool lines = d % 32 == 0 && f % 32 == 0;
  for (int i = 0; i < a.n_list; ++i)
    for (int w = 3; w < 6; ++w) lines &= ((uintptr_t)c->h_wtab[w][a.list[i]] & 127) == 0;
  const bool rag = d % 256 != 0 || f % 256 != 0 || !lines;
  // By the rows per expert of an even routing.  On sizes that are no multiples of 256 the two differ by 2 % up to 128
  // rows and the kernel for few rows loses beyond; with whole lines to store and at least three rounds of the larger
  // tiles (fewer are one round more in the smaller ones) it gains up to 512 and loses 2 % there where popularity falls
  // off as rank^-1.2.  Backward, us, many -> few at 64, 128, 256, 512 rows; even, and rank^-1.2:
  //   2048 x 2048, 6 of 32 experts: 150 -> 145, 173 -> 163, 232 -> 219, 277 -> 267; 214 -> 204, 264 -> 254, 364 -> 356, 645 -> 648
  //   two-matrix 1024 x 4096, 8 of 32: 119 -> 115, 137 -> 129, 189 -> 180, 233 -> 225; 159 -> 150, 205 -> 192, 323 -> 322,
  //   517 -> 530
  //   1160 x 2888, 6 of 16: 161 -> 162, 190 -> 190, 248 -> 252, 304 -> 313; 214 -> 217, 240 -> 243, 301 -> 306, 458 -> 474
  //   2048 x 1408, 12 of 64: 182 -> 180, 206 -> 206, 269 -> 269, 333 -> 336; 263 -> 266, 333 -> 339, 584 -> 607, 1025 -> 1067
  // 2048 x 2048 at 1024 rows, step: 774 -> 772; 288 tiles of 1024 x 1024, 256 rows: 158 -> 161.
  const int tiles256 = a.n_jobs * a.n_list * ((d + 255) / 256) * ((f + 255) / 256);
  const int line = !rag && tiles256 >= 3 * c->n_cu ? 512 : 128;
  const bool few = c->wgrad_rows != 0 ? c->wgrad_rows == 128 : c->S_call <= line * E;
  if (few) {
    auto tiles = [](int m, int n) { return ((m + 255) / 256) * ((n + F_BN - 1) / F_BN); };
    const int total = a.n_list * (tiles(d, f) + (a.n_jobs - 1) * tiles(f, d));
    const dim3 grid((total + 511) / 512 * 512);
    auto kern = !rag ? wgrad_few_kernel<false, true> : lines ? wgrad_few_kernel<true, true> : wgrad_few_kernel<true, false>;
    hipLaunchKernelGGL(kern, grid, dim3(F_NT), 0, s, a);
  } else {
    const dim3 grid((tiles256 + 255) / 256 * 256);
    auto kern = !rag ? wgrad_tr_kernel<false, true> : lines ? wgrad_tr_kernel<true, true> : wgrad_tr_kernel<true, false>;
    hipLaunchKernelGGL(kern, grid, dim3(NT), 0, s, a);
  }
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_EHIP;
}
