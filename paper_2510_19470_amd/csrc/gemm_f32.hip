// Grouped expert FFN for fp32 storage on the matrix cores (v_mfma_f32_16x16x4_f32: full fp32
// multiply-add, 256 flop per clock and compute unit), forward and backward.  (Paper Sec. 2.1:
// experts are FFNs; Sec. 3.1: the experts of a GPU run one after another on their own tokens --
// here every launch covers all of them.)
//
// Block = 256 threads = 4 wavefronts (2 x 2) on a tile of TM token rows x TN output columns;
// weights are the MFMA "A" operand and tokens the "B" operand, so a lane ends up with 4
// consecutive columns of one token (one 16-byte store).  Contraction steps of 32 through two or three
// LDS stages filled by asynchronous copies, one or two steps in flight, one barrier per step.  (Loads
// through registers, three steps ahead: the compiler waited for all of them at the head of every
// step, 15-30 % slower.)  A lane takes 4 consecutive k of its row per fragment (the four MFMAs
// of 16 k use the elements 0..3 of both operands: the order of k inside a group of 16 does not
// matter as long as both agree).  Operands contiguous along k are read 16 bytes at a time,
// operands with k outermost (the backward's weights, the weight gradients) 4 bytes at a time;
// 16-byte chunks are XOR-swizzled so that either read spreads over all 64 banks.
// All sizes are multiples of 8, so a 16-byte piece exists or does not; pieces past the end of the
// contraction come from a page of zeros.
//
// The (expert, row block) of a block comes from the counts inside the kernel (one wavefront scan
// per 64 experts): no schedule launch.  The bound is the MFMA rate for many rows (8192 rows, d =
// 1024, f = 2048: 103-111 of 157 TFLOP/s; the vector-ALU kernels reach 10-12) and the latency of a
// block's start and of its few steps otherwise (1024 rows, d = 512, f = 1024: forward FFN 350 -> 61
// us, backward 659 -> 113 us).
#include <algorithm>

#include "moe_internal.h"
#include "numeric.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int BK = 32;
constexpr int NTHR = 256;

struct Tile {
  int expert, row0, rows;   // rows == 0: nothing to do
};

// The idx-th block of bm rows over all experts with weights (ids ascending).  Called by all lanes
// of a wavefront; the result is wave-uniform.  Nothing at all when a segment of a present expert
// does not lie inside the S rows of the buffers.
__device__ __forceinline__ Tile find_tile(int idx, int bm, const int32_t* __restrict__ counts,
                                          const int32_t* __restrict__ offsets,
                                          const void* const* __restrict__ present, int E, int S) {
  const int lane = threadIdx.x & 63;
  Tile t = {0, 0, 0};
  int before = 0;
  bool bad = false;
  for (int e0 = 0; e0 < E; e0 += 64) {
    const int e = e0 + lane;
    int n = 0, o = 0;
    if (e < E && present[e] != nullptr) {
      n = counts[e];
      o = offsets[e];
    }
    bad |= n < 0 || o < 0 || (long)o + n > (long)S;
    const int mine = (n + bm - 1) / bm;
    int incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int v = __shfl_up(incl, off, 64);
      if (lane >= off) incl += v;
    }
    const int first = before + incl - mine;
    const bool hit = idx >= first && idx < first + mine;
    const unsigned long long m = __ballot(hit);
    if (m != 0) {
      const int l = __ffsll((long long)m) - 1;
      const int blk = idx - __shfl(first, l, 64);
      t.expert = e0 + l;
      t.row0 = __shfl(o, l, 64) + blk * bm;
      t.rows = min(bm, __shfl(n, l, 64) - blk * bm);
    }
    before += __shfl(incl, 63, 64);
  }
  if (__ballot(bad) != 0) t.rows = 0;
  t.expert = __builtin_amdgcn_readfirstlane(t.expert);
  t.row0 = __builtin_amdgcn_readfirstlane(t.row0);
  t.rows = __builtin_amdgcn_readfirstlane(t.rows);
  return t;
}

// 16 bytes per lane global -> LDS, 64-bit address per lane; the wavefront's 1 KB lands at lds_addr
// (wave-uniform, via M0) + lane * 16.  Completion is counted by hand (vmcnt) in Mma::run.
__device__ __forceinline__ void dma16v(const float* src, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds_addr)
               : "memory", "m0");
}

// One operand of a tile: ROWS rows (output columns or tokens) x BK.
template <int ROWS, bool KFAST>
struct Operand {
  static constexpr int FLOATS = ROWS * BK;
  static constexpr int NV = FLOATS / 256 / (NTHR / 64);   // copy instructions per wavefront and step
  uint32_t off[NV];   // the lane's piece of every copy, floats from the tile's (row 0, k = 0)
  int k[NV];          // ... its first k
  // swizzle of the 16-byte chunks: KFAST, 128-byte rows, so that the 16 rows of a fragment read
  // fall on distinct banks; else the 4 k-groups (q) of a read on different quarters of the banks
  __device__ __forceinline__ static int swz(int r) { return ((r >> 1) & 7) ^ ((r & 1) << 2); }
  // ld: floats between rows (KFAST) or between k.  Rows that do not exist read row 0 (their
  // outputs are not stored).
  __device__ __forceinline__ void init(uint32_t ld, int rows) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = wave + i * (NTHR / 64);
      int r;
      if (KFAST) {
        r = 8 * c + (lane >> 3);
        k[i] = ((lane & 7) ^ swz(r)) * 4;
      } else {
        static_assert(KFAST || ROWS == 64 || ROWS == 32, "layouts of a k-outermost operand");
        const int slot = lane / (ROWS / 4), ch = lane % (ROWS / 4);
        if (ROWS == 64) {   // 4 k per copy: those of one q
          k[i] = 4 * c + slot;
          r = (ch ^ ((c & 3) << 2)) * 4;
        } else {            // 8 k per copy: j-th k of q = 2 (c & 1) + {0, 1} in 128-byte slots 2j + {0, 1}
          k[i] = 8 * c + 4 * (slot & 1) + (slot >> 1);
          r = (ch ^ ((c & 1) << 2)) * 4;
        }
      }
      if (r >= rows) r = 0;
      off[i] = KFAST ? r * ld + k[i] : k[i] * ld + r;
    }
  }
  // k-step starting at k0 (base: the tile's (row 0, k0)); what lies past K comes from `zero`
  __device__ __forceinline__ void copy(const float* base, int k0, int K, const float* zero,
                                       uint32_t lds) const {
    const int wave = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < NV; ++i)
      dma16v(k0 + k[i] < K ? base + off[i] : zero,
             __builtin_amdgcn_readfirstlane(lds + (wave + i * (NTHR / 64)) * 1024));
  }
  // k = 16 s + 4 q + {0..3} of row r (q = lane >> 4)
  __device__ __forceinline__ static f32x4 frag(const float* lds, int r, int s, int q) {
    if (KFAST) return *reinterpret_cast<const f32x4*>(lds + r * BK + (((4 * s + q) ^ swz(r)) << 2));
    if (ROWS == 64) {
      const float* p = lds + (16 * s + 4 * q) * 64 + (r ^ (q << 4));
      return f32x4{p[0], p[64], p[128], p[192]};
    }
    const float* p = lds + (2 * s + (q >> 1)) * 256 + (q & 1) * 32 + (r ^ ((q >> 1) << 4));
    return f32x4{p[0], p[64], p[128], p[192]};
  }
};

// All but the last N copies have landed and my LDS reads are done, then a barrier.
template <int N>
__device__ __forceinline__ void wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// acc[b][j][i] += tokens x weights over one segment of length K; b: weight matrix (two for gate
// and up), j / i: 16-column / 16-token block of the wavefront's tile.
template <int TM, int TN, int NB, bool XK, bool WK, int STAGES>
struct Mma {
  static constexpr int MI = TM / 32, NJ = TN / 32;   // 16-blocks per wavefront (2 x 2 wavefronts)
  typedef Operand<TM, XK> X;
  typedef Operand<TN, WK> W;
  static constexpr int STAGE = X::FLOATS + NB * W::FLOATS;
  static constexpr int COPIES = X::NV + NB * W::NV;   // per wavefront and step
  f32x4 acc[NB][NJ][MI];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < MI; ++i) acc[b][j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // x1, w1: the operands of the second segment (segs == 2), same sizes
  __device__ __forceinline__ void run(float* lds, const float* x0, const float* x1, int ldx,
                                      int rows, const float* const (&w0)[NB],
                                      const float* const (&w1)[NB], int ldw, int cols, int K,
                                      int segs, const float* zeros) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 15, q = lane >> 4, wm = wave >> 1, wn = wave & 1;
    const int per = (K + BK - 1) / BK, steps = per * segs;
    if (steps == 0) return;
    X x;
    W w;
    x.init(ldx, rows);
    w.init(ldw, cols);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
    // past the last step the last one is copied again: a fixed number of copies in flight
    auto issue = [&](int h) {
      const int st = min(h, steps - 1);
      const bool second = st >= per;
      const int k0 = (second ? st - per : st) * BK;
      const uint32_t sb = lds0 + (h % STAGES) * (STAGE * 4);
      x.copy((second ? x1 : x0) + (XK ? (size_t)k0 : (size_t)k0 * ldx), k0, K, zeros, sb);
#pragma unroll
      for (int b = 0; b < NB; ++b)
        w.copy((second ? w1[b] : w0[b]) + (WK ? (size_t)k0 : (size_t)k0 * ldw), k0, K, zeros,
               sb + (X::FLOATS + b * W::FLOATS) * 4);
    };
#pragma unroll
    for (int h = 0; h < STAGES - 1; ++h) issue(h);
    for (int st = 0; st < steps; ++st) {
      // step st has landed for this wavefront (the copies of the next STAGES - 2 steps may be in
      // flight) and, behind the barrier, for everybody; everybody has also read step st - 1,
      // whose stage takes step st + STAGES - 1
      wait_barrier<(STAGES - 2) * COPIES>();
      issue(st + STAGES - 1);
      const float* p = lds + (st % STAGES) * STAGE;
#pragma unroll
      for (int s = 0; s < BK / 16; ++s) {
        f32x4 xf[MI], wf[NB][NJ];
#pragma unroll
        for (int i = 0; i < MI; ++i) xf[i] = X::frag(p, wm * (TM / 2) + i * 16 + n, s, q);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            wf[b][j] = W::frag(p + X::FLOATS + b * W::FLOATS, wn * (TN / 2) + j * 16 + n, s, q);
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
          for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
              for (int i = 0; i < MI; ++i)
                acc[b][j][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[b][j][k], xf[i][k], acc[b][j][i], 0, 0, 0);
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no copy in flight into LDS at exit
  }
  // f(j, i, token row inside the tile, first of 4 columns inside the tile)
  template <typename F>
  __device__ __forceinline__ void each(F&& f) const {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 15, q = lane >> 4, wm = wave >> 1, wn = wave & 1;
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int i = 0; i < MI; ++i)
        f(j, i, wm * (TM / 2) + i * 16 + n, wn * (TN / 2) + j * 16 + 4 * q);
  }
};

struct F32Args {
  const float* x;          // token-role operand
  const float* x1;         // ... of the second segment (dX of the gated expert: dU)
  int K, N;                // contraction per segment, output columns
  const void* const* w0;   // [E] weights
  const void* const* w1;   // [E] second matrix (gate/up: W3; dX: W3) or nullptr
  const int32_t* counts;
  const int32_t* offsets;
  const void* const* present;
  int E, S;
  const float* zero;       // 16 bytes of zeros
  float* out;              // UP: H; DOWN, DX: the result; DH: dG
  float* out2;             // DH: dU
  float* out3;             // DH: H
  float* G;                // UP: saved (out, may be nullptr); DH: saved (in)
  float* U;
};

enum { F_UP, F_UP1, F_DOWN, F_DH, F_DX };

template <int MODE, int TM, int TN>
__global__ __launch_bounds__(NTHR) void ffn_f32_kernel(const F32Args p) {
  constexpr bool WK = MODE == F_UP || MODE == F_UP1 || MODE == F_DOWN;   // weights contiguous in k
  constexpr int NB = MODE == F_UP ? 2 : 1;
  // LDS stages, all but one in flight from memory.  64x64 tiles: two, so that five blocks share a compute unit's LDS
  // instead of three (with two weight matrices three instead of two) and cover each other's waits (2048 tokens, d =
  // 1024, f = 2048, 6 of 8 experts, step: 1408 -> 1346 us; forward, 2000 tokens, 1000 x 1800: 391 -> 385).  32x32 tiles
  // have six blocks (four) with three of them (two: 194 -> 196.5, 1024 tokens, 512 x 1024; four: 3-10 % slower).
  constexpr int STAGES = TM == 64 ? 2 : 3;
  typedef Mma<TM, TN, NB, true, WK, STAGES> M;
  __shared__ __align__(16) float lds[STAGES * M::STAGE];
  const Tile tl = find_tile(blockIdx.x, TM, p.counts, p.offsets, p.present, p.E, p.S);
  if (tl.rows == 0) return;
  const int n0 = blockIdx.y * TN, cols = min(TN, p.N - n0);
  const int ldw = WK ? p.K : p.N;
  const size_t wofs = WK ? (size_t)n0 * p.K : n0;
  const bool two = p.w1 != nullptr;
  const float* w0[NB];
  const float* w1[NB];
  w0[0] = w1[0] = (const float*)p.w0[tl.expert] + wofs;
  if (NB == 2) w0[NB - 1] = w1[NB - 1] = (const float*)p.w1[tl.expert] + wofs;
  if (MODE == F_DX && two) w1[0] = (const float*)p.w1[tl.expert] + wofs;
  const size_t xo = (size_t)tl.row0 * p.K;
  M m;
  m.zero();
  m.run(lds, p.x + xo, MODE == F_DX && two ? p.x1 + xo : p.x + xo, p.K, tl.rows, w0, w1, ldw, cols,
        p.K, MODE == F_DX && two ? 2 : 1, p.zero);
  m.each([&](int j, int i, int r, int c) {
    if (r >= tl.rows || c >= cols) return;
    const size_t o = (size_t)(tl.row0 + r) * p.N + n0 + c;
    const f32x4 a = m.acc[0][j][i];
    f32x4* out = reinterpret_cast<f32x4*>(p.out + o);
    if (MODE == F_DOWN || MODE == F_DX) {
      *out = a;
    } else if (MODE == F_UP || MODE == F_UP1) {
      f32x4 h;
      const f32x4 u = m.acc[NB - 1][j][i];
#pragma unroll
      for (int e = 0; e < 4; ++e) h[e] = MODE == F_UP ? a[e] / (1.f + expf(-a[e])) * u[e] : fmaxf(a[e], 0.f);
      *out = h;
      if (p.G != nullptr) {
        *reinterpret_cast<f32x4*>(p.G + o) = a;
        if (MODE == F_UP) *reinterpret_cast<f32x4*>(p.U + o) = u;
      }
    } else {   // F_DH: dG = dH*u*silu'(g), dU = dH*silu(g), H; two-matrix: dG = dH where g > 0
      const f32x4 g = *reinterpret_cast<const f32x4*>(p.G + o);
      f32x4 dg, h;
      if (p.U == nullptr) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          dg[e] = g[e] > 0.f ? a[e] : 0.f;
          h[e] = fmaxf(g[e], 0.f);
        }
      } else {
        const f32x4 u = *reinterpret_cast<const f32x4*>(p.U + o);
        f32x4 du;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float sg = 1.f / (1.f + expf(-g[e]));
          dg[e] = a[e] * u[e] * sg * (1.f + g[e] * (1.f - sg));
          du[e] = a[e] * g[e] * sg;
          h[e] = g[e] * sg * u[e];
        }
        *reinterpret_cast<f32x4*>(p.out2 + o) = du;
      }
      *out = dg;
      *reinterpret_cast<f32x4*>(p.out3 + o) = h;
    }
  });
}

// dW[e] [Mo, No] = P_e^T Q_e over the rows of expert e, up to three of them in one launch
// (blockIdx.z = expert * n_jobs + job; every job has as many 64x64 tiles).
struct DwArgs {
  struct Job {
    const float* P;
    const float* Q;
    const void* const* dWt;
    int Mo, No;
  } job[3];
  int n_jobs, E, S;
  const float* zero;
  const int32_t* counts;
  const int32_t* offsets;
  const void* const* present;
};

template <int STAGES>
__global__ __launch_bounds__(NTHR) void ffn_f32_dw_kernel(const DwArgs p) {
  constexpr int TS = 64;
  typedef Mma<TS, TS, 1, false, false, STAGES> M;
  __shared__ __align__(16) float lds[STAGES * M::STAGE];
  const int e = blockIdx.y / p.n_jobs;
  const DwArgs::Job& J = p.job[blockIdx.y % p.n_jobs];
  float* dW = (float*)J.dWt[e];
  if (dW == nullptr || p.present[e] == nullptr) return;
  const int nt = (J.No + TS - 1) / TS;
  const int m0 = (int)(blockIdx.x / nt) * TS, n0 = (int)(blockIdx.x % nt) * TS;
  // any segment of the call that does not fit the buffers: zeros come out
  const bool ok = find_tile(0, 1 << 30, p.counts, p.offsets, p.present, p.E, p.S).rows > 0;
  const int rows = ok ? p.counts[e] : 0;
  const size_t row0 = ok ? p.offsets[e] : 0;
  M m;
  m.zero();
  const float* q[1] = {J.Q + row0 * J.No + n0};
  m.run(lds, J.P + row0 * J.Mo + m0, nullptr, J.Mo, min(TS, J.Mo - m0), q, q, J.No,
        min(TS, J.No - n0), rows, 1, p.zero);
  m.each([&](int j, int i, int r, int c) {
    if (m0 + r < J.Mo && n0 + c < J.No)
      *reinterpret_cast<f32x4*>(dW + (size_t)(m0 + r) * J.No + n0 + c) = m.acc[0][j][i];
  });
}

int ceil_div(int a, int b) { return (a + b - 1) / b; }

template <int MODE, int TM, int TN>
void launch_tile(const moe_ctx* c, const F32Args& a, hipStream_t s) {
  const dim3 grid(c->S_call / TM + c->cfg.E, ceil_div(a.N, TN));
  hipLaunchKernelGGL((ffn_f32_kernel<MODE, TM, TN>), grid, dim3(NTHR), 0, s, a);
}

// 64x64 tiles from three of them per compute unit on, else 32x32: few large tiles leave units idle or make a round of
// a few; the 32x32 tile reads twice as much from L2 per flop.  64x64 against 32x32, us a GEMM, in the mean over 70 layers
// of 512 to 2048 tokens with an even routing, by the expected number of 64x64 tiles (gate/up, down, dH, dX; three blocks
// of 64x64 fit a unit in gate/up, five in the others):
//   300 to 400: +22, +30, +8, +61; 512 to 640: +18, +7, +7, +6; 640 to 768: +18, +6, +2, -9; 768 to 900: -12, -15, -18, -38;
//   2000 and more: -89, -156, -74, -332.  Popularity as rank^-1 makes more tiles than expected: down and dX gain from 400 on
//   (-20, -58), gate/up and dH from 770.
template <int MODE>
void launch_mode(const moe_ctx* c, const F32Args& a, hipStream_t s) {
  int present = 0;
  for (int e = 0; e < c->cfg.E; ++e) present += c->h_wtab[0][e] != nullptr;
  // rows expected here (the counts stay on the device), every expert's last block half full
  const long rows = (long)c->S_call * present / c->cfg.E;
  const long tiles = (rows / 64 + present / 2 + 1) * (long)ceil_div(a.N, 64);
  if (tiles >= 3L * c->n_cu) launch_tile<MODE, 64, 64>(c, a, s);
  else launch_tile<MODE, 32, 32>(c, a, s);
}

F32Args base_args(const moe_ctx* c, const int32_t* counts, const int32_t* offsets) {
  F32Args a{};
  a.counts = counts;
  a.offsets = offsets;
  a.present = c->d_wtab;
  a.E = c->cfg.E;
  a.S = c->S_call;
  a.zero = (const float*)c->d_zero;
  return a;
}

}  // namespace

int launch_ffn_f32(moe_ctx* c, bool gated, const int32_t* counts, const int32_t* offsets,
                   const void* x_packed, void* y_packed, void* G, void* U, hipStream_t s) {
  const void* const* W1 = c->d_wtab + 0 * MOE_MAX_EXPERTS;
  const void* const* W3 = c->d_wtab + 1 * MOE_MAX_EXPERTS;
  const void* const* W2 = c->d_wtab + 2 * MOE_MAX_EXPERTS;
  prof_mark(c, 0, s);
  prof_mark(c, 1, s);
  F32Args up = base_args(c, counts, offsets);
  up.x = (const float*)x_packed;
  up.K = c->cfg.d;
  up.N = c->cfg.f;
  up.w0 = W1;
  up.w1 = gated ? W3 : nullptr;
  up.out = (float*)c->d_H;
  up.G = (float*)G;
  up.U = (float*)U;
  if (gated) launch_mode<F_UP>(c, up, s);
  else launch_mode<F_UP1>(c, up, s);
  prof_mark(c, 2, s);
  F32Args dn = base_args(c, counts, offsets);
  dn.x = (const float*)c->d_H;
  dn.K = c->cfg.f;
  dn.N = c->cfg.d;
  dn.w0 = W2;
  dn.out = (float*)y_packed;
  launch_mode<F_DOWN>(c, dn, s);
  prof_mark(c, 3, s);
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_EHIP;
}

int launch_ffn_bwd_f32(moe_ctx* c, bool gated, const void* dy, const void* xp, const void* G,
                       const void* U, const int32_t* counts, const int32_t* offsets, void* dxp,
                       void* dG_tmp, void* dU_tmp, void* H_tmp, hipStream_t s) {
  const int d = c->cfg.d, f = c->cfg.f;
  F32Args dh = base_args(c, counts, offsets);
  dh.x = (const float*)dy;
  dh.K = d;
  dh.N = f;
  dh.w0 = c->d_wtab + 2 * MOE_MAX_EXPERTS;   // W2 [d, f]: k outermost
  dh.out = (float*)dG_tmp;
  dh.out2 = (float*)dU_tmp;
  dh.out3 = (float*)H_tmp;
  dh.G = (float*)const_cast<void*>(G);
  dh.U = gated ? (float*)const_cast<void*>(U) : nullptr;
  launch_mode<F_DH>(c, dh, s);
  F32Args dx = base_args(c, counts, offsets);
  dx.x = (const float*)dG_tmp;
  dx.x1 = (const float*)dU_tmp;
  dx.K = f;
  dx.N = d;
  dx.w0 = c->d_wtab + 0 * MOE_MAX_EXPERTS;   // W1, W3 [f, d]: k outermost
  dx.w1 = gated ? c->d_wtab + 1 * MOE_MAX_EXPERTS : nullptr;
  dx.out = (float*)dxp;
  launch_mode<F_DX>(c, dx, s);
  DwArgs a{};
  const void* const* dWt = c->d_wtab + 3 * MOE_MAX_EXPERTS;   // rows dW1, dW3, dW2
  a.job[0] = {(const float*)dy, (const float*)H_tmp, dWt + 2 * MOE_MAX_EXPERTS, d, f};
  a.job[1] = {(const float*)dG_tmp, (const float*)xp, dWt, f, d};
  a.job[2] = {(const float*)dU_tmp, (const float*)xp, dWt + MOE_MAX_EXPERTS, f, d};
  a.n_jobs = gated ? 3 : 2;
  a.E = c->cfg.E;
  a.S = c->S_call;
  a.zero = (const float*)c->d_zero;
  a.counts = counts;
  a.offsets = offsets;
  a.present = c->d_wtab;
  const dim3 grid(ceil_div(d, 64) * ceil_div(f, 64), a.E * a.n_jobs);
  // Two stages where there are two steps or fewer on average: what counts then is blocks that start and store beside
  // each other (step, us: 37 rows per expert 466 -> 450, 12 rows 130 -> 128; 131 rows 327 -> 326, 187 rows 288 -> 289.5,
  // 256 rows 193.7 -> 198.6)
  if (a.S <= 64 * a.E) hipLaunchKernelGGL((ffn_f32_dw_kernel<2>), grid, dim3(NTHR), 0, s, a);
  else hipLaunchKernelGGL((ffn_f32_dw_kernel<3>), grid, dim3(NTHR), 0, s, a);
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_EHIP;
}
