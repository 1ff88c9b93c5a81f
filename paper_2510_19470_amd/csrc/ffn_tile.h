// Shared pieces of the bf16 grouped expert GEMMs on the matrix cores (ffn_mfma.hip: 256-row tiles,
// ffn_tile128.hip: 128-row tiles) and of the weight gradients (wgrad_tr.hip): LDS layouts, copies,
// epilogues.
#pragma once
#include "moe_internal.h"
#include "numeric.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;

constexpr int BK = 64;            // k per stage

// Swizzle of the 16-byte chunks of a row-major stage's rows ...
__device__ __forceinline__ int swz(int row) { return ((row >> 1) & 7) ^ ((row & 1) << 2); }
// ... and of a k-major tile's (rows of a multiple of 256 bytes, transpose reads).  A transpose read
// takes, per group of 16 lanes, 4 rows (row & 3) x 32 bytes; the four groups of a wavefront are (bit 3 of
// the row, the 32-byte column half).  LDS has 64 banks of 4 bytes and serves 32 lanes per cycle: the 16
// chunks of any two groups that can share a cycle must differ modulo 16.  Bits 2-3 of the chunk take
// row & 3, bit 1 takes bit 3 of the row (the column half sits in bit 1 already).
__device__ __forceinline__ int tr_swz(int row) { return ((row & 3) << 2) ^ (((row >> 3) & 1) << 1); }

typedef __attribute__((address_space(3))) void* lptr_t;

// Asynchronous 16 bytes per lane global -> LDS: lane reads base + off (wave-uniform 64-bit
// base in scalar registers, 32-bit per-lane byte offset), the wavefront's 1 KB lands at
// lds_addr (wave-uniform byte address, via M0) + lane * 16.  Written as assembly so that
// the compiler does not serialise later LDS reads behind it; completion is tracked by hand
// (vmcnt) in the main loop.
__device__ __forceinline__ void dma16(uint32_t off, const char* base, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds_addr)
               : "memory", "m0");
}
// The same copy of data that is read once: it does not displace what the last-level cache holds.
__device__ __forceinline__ void dma16_once(uint32_t off, const char* base, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(off), "s"(base), "s"(lds_addr)
               : "memory", "m0");
}
// The same copy with a 64-bit address per lane (k-steps that end inside the operand's rows:
// the lanes past the end read zeros from elsewhere).
__device__ __forceinline__ void dma16v(const char* src, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds_addr)
               : "memory", "m0");
}

// A pointer that is the same in all lanes, in scalar registers.
__device__ __forceinline__ const char* uniform_ptr(const void* q) {
  const uint64_t v = (uint64_t)q;
  return (const char*)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32 |
                       (uint32_t)__builtin_amdgcn_readfirstlane((int)v));
}

// Source of one copy instruction: wave-uniform base and, in RAG kernels, how much of the k-step
// exists (16-byte chunks of a row; k-rows when the operand is k-major).
struct Src {
  const char* base;
  int nv;
};
template <bool RAG>
__device__ __forceinline__ void dma_step(uint32_t off, const Src& src, uint32_t lds_addr, int full,
                                         int idx, const char* zero) {
  if (!RAG || src.nv >= full) dma16(off, src.base, lds_addr);
  else dma16v(idx < src.nv ? src.base + off : zero, lds_addr);
}

// Epilogue stores.  A lane holds, per accumulator, 4 consecutive output columns 8g + 4h + {0..3}
// (h = lane >> 5) of one token row for g = 0..3: 8-byte pieces.  Swapping between the two
// half-wavefronts turns the pieces of g and g+1 into one 16-byte piece per lane -- lanes 0-31
// get columns 8g .. 8g+7, lanes 32-63 columns 8(g+1) .. 8(g+1)+7 of their row -- so that a
// wavefront stores 32 contiguous bytes per row with one instruction instead of 16 with two.
__device__ __forceinline__ uint4 pair16(uint2 a /* piece g */, uint2 b /* piece g+1 */) {
  // v_permlane32_swap: lanes 32-63 of the first operand <-> lanes 0-31 of the second
  const auto x = __builtin_amdgcn_permlane32_swap(a.x, b.x, false, false);
  const auto y = __builtin_amdgcn_permlane32_swap(a.y, b.y, false, false);
  return make_uint4(x[0], y[0], x[1], y[1]);
}
__device__ __forceinline__ uint2 pack4(float a, float b, float c, float d) {
  return make_uint2(pack_bf16x2(a, b), pack_bf16x2(c, d));
}
// The inverse, for epilogue loads: every lane loads the 16 bytes pair16 would store (lanes
// 0-31 columns 8g .. 8g+7, lanes 32-63 columns 8(g+1) .. 8(g+1)+7 of their row); the swaps
// give each lane its own 8-byte pieces of g (a) and g+1 (b).
__device__ __forceinline__ void unpair16(const uint4& v, uint2& a, uint2& b) {
  const auto x = __builtin_amdgcn_permlane32_swap(v.x, v.z, false, false);
  const auto y = __builtin_amdgcn_permlane32_swap(v.y, v.w, false, false);
  a = make_uint2(x[0], y[0]);
  b = make_uint2(x[1], y[1]);
}

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
// k-steps of a contraction of `segs` segments of `len` each in the 256-row tiles (an even number)
inline int k_steps(int len, int segs) { return (segs * ceil_div(len, BK) + 1) & ~1; }
// Parts that a 256-row tile of the down GEMM's tail is cut into (see mfma_sched_kernel).
__host__ __device__ inline int split_parts(int tail, int n_cu, int kt_down) {
  const int pairs = kt_down / 2;
  int split = 1;
  while (tail > 0 && split < 8 && tail * (split + 1) <= n_cu && pairs / (split + 1) >= 4) ++split;
  return split;
}

enum { MODE_UP = 0, MODE_DOWN = 1, MODE_DH = 2, MODE_UP1 = 4, MODE_DH1 = 5 };

struct GemmArgs {
  const uint16_t* A;    // token-role operand: [rows, lda]
  int lda;              // elements per row of A
  const TileSched* sched;
  const TileDesc* order;
  int n_tiles_n;
  int K;                   // contraction length
  int N;                   // elements per output row
  uint16_t* C;             // UP: H; DOWN: Y / dX; DH: [dG|dU] with row pitch 2N
  uint16_t* C2;            // DH: H
  float* split_ws;         // fp32 partial tiles of contractions that are cut
  int32_t* joined;         // ... and the counters of their tiles
  uint16_t* Gs;            // UP: optional save (out); DH: saved G (in)
  uint16_t* Us;
  // k-major weight-role operand (BKM kernels): B[k][n] with ldb elements per k-row; the first
  // kseg k-steps come from the tile's first matrix, the rest from its second one
  int ldb, kseg;
  // RAG kernels: k-steps of a whole tile (even), elements of a contraction segment (kseg steps;
  // only its last step may be partial), 16 bytes of zeros
  int kt, kseg_len;
  const char* zero;
};

// bf16 outputs of a tile.  A wavefront holds 32 NI token rows x 64 weight rows: acc[j][i] is token
// block i and weight rows j HB + 32 wn .. of the tile's 2 HB = 64 NI (MODE_UP: j = 0 gate, j = 1 up).  A
// lane holds, per 32x32 accumulator, token row (lane & 31) and the weight rows 8g + 4(lane >> 5) +
// {0..3}, g = 0..3.
template <int MODE, bool RAG, int NI>
__device__ __forceinline__ void tile_epilogue(const GemmArgs& p, const f32x16 (&acc)[2][NI], int row0,
                                              int rows, int nblk, int wm, int wn, int lane) {
  constexpr int HB = 32 * NI;
  const int fr_row = lane & 31, fr_half = lane >> 5;
  // bf16 outputs: every lane takes part in the half-wavefront swaps, only the stores are
  // predicated on the row being inside the tile; gp = 0, 1 are the column pairs g = (0,1), (2,3)
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int m_local = wm * (32 * NI) + i * 32 + fr_row;
    const bool live = m_local < rows;
    const size_t row = (size_t)(row0 + m_local);
    // MODE_DH, MODE_DH1: the saved G (and U) of the whole row block, 16 bytes per lane at the
    // addresses the outputs are stored to, all requested before the first is used
    uint4 gsv[2][2], usv[2][2];
    if (MODE == MODE_DH || MODE == MODE_DH1) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int gp = 0; gp < 2; ++gp) {
          const size_t col = (size_t)nblk * (2 * HB) + j * HB + wn * 32 + 8 * fr_half + 16 * gp;
          gsv[j][gp] = usv[j][gp] = make_uint4(0, 0, 0, 0);
          if (live && (!RAG || col < (size_t)p.N)) {
            gsv[j][gp] = *reinterpret_cast<const uint4*>(p.Gs + row * p.N + col);
            if (MODE == MODE_DH) usv[j][gp] = *reinterpret_cast<const uint4*>(p.Us + row * p.N + col);
          }
        }
    }
    if (MODE == MODE_UP) {
      const int colb = nblk * HB + wn * 32 + 8 * fr_half;
#pragma unroll
      for (int gp = 0; gp < 2; ++gp) {
        uint2 hp[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const int g = 2 * gp + t;
          float h[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) h[r] = silu_f(acc[0][i][g * 4 + r]) * acc[1][i][g * 4 + r];
          hp[t] = pack4(h[0], h[1], h[2], h[3]);
        }
        const size_t o = row * p.N + colb + 16 * gp;
        const bool put = live && (!RAG || colb + 16 * gp < p.N);
        const uint4 hv = pair16(hp[0], hp[1]);
        if (put) *reinterpret_cast<uint4*>(p.C + o) = hv;
        if (p.Gs != nullptr) {
          const int g = 2 * gp;
          const uint4 gv = pair16(pack4(acc[0][i][g * 4], acc[0][i][g * 4 + 1], acc[0][i][g * 4 + 2], acc[0][i][g * 4 + 3]),
                                  pack4(acc[0][i][g * 4 + 4], acc[0][i][g * 4 + 5], acc[0][i][g * 4 + 6], acc[0][i][g * 4 + 7]));
          const uint4 uv = pair16(pack4(acc[1][i][g * 4], acc[1][i][g * 4 + 1], acc[1][i][g * 4 + 2], acc[1][i][g * 4 + 3]),
                                  pack4(acc[1][i][g * 4 + 4], acc[1][i][g * 4 + 5], acc[1][i][g * 4 + 6], acc[1][i][g * 4 + 7]));
          if (put) {
            *reinterpret_cast<uint4*>(p.Gs + o) = gv;
            *reinterpret_cast<uint4*>(p.Us + o) = uv;
          }
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int colb = nblk * (2 * HB) + j * HB + wn * 32 + 8 * fr_half;
#pragma unroll
        for (int gp = 0; gp < 2; ++gp) {
          const int g0 = 2 * gp;
          const size_t col = colb + 16 * gp;
          const bool put = live && (!RAG || col < (size_t)p.N);
          if (MODE == MODE_DOWN) {
            const uint4 v = pair16(pack4(acc[j][i][g0 * 4], acc[j][i][g0 * 4 + 1], acc[j][i][g0 * 4 + 2], acc[j][i][g0 * 4 + 3]),
                                   pack4(acc[j][i][g0 * 4 + 4], acc[j][i][g0 * 4 + 5], acc[j][i][g0 * 4 + 6], acc[j][i][g0 * 4 + 7]));
            if (put) *reinterpret_cast<uint4*>(p.C + row * p.N + col) = v;
          } else if (MODE == MODE_UP1) {
            float r[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) r[q] = fmaxf(acc[j][i][g0 * 4 + q], 0.f);
            const uint4 v = pair16(pack4(r[0], r[1], r[2], r[3]), pack4(r[4], r[5], r[6], r[7]));
            if (put) *reinterpret_cast<uint4*>(p.C + row * p.N + col) = v;
            if (p.Gs != nullptr) {
              const uint4 gv = pair16(pack4(acc[j][i][g0 * 4], acc[j][i][g0 * 4 + 1], acc[j][i][g0 * 4 + 2], acc[j][i][g0 * 4 + 3]),
                                      pack4(acc[j][i][g0 * 4 + 4], acc[j][i][g0 * 4 + 5], acc[j][i][g0 * 4 + 6], acc[j][i][g0 * 4 + 7]));
              if (put) *reinterpret_cast<uint4*>(p.Gs + row * p.N + col) = gv;
            }
          } else {  // MODE_DH, MODE_DH1
            uint2 dgp[2], dup[2], hhp[2];
            uint2 gqs[2], uqs[2];
            unpair16(gsv[j][gp], gqs[0], gqs[1]);
            unpair16(usv[j][gp], uqs[0], uqs[1]);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
              const int g = g0 + t;
              const uint2 gq = gqs[t], uq = uqs[t];
              const uint32_t gw[2] = {gq.x, gq.y}, uw[2] = {uq.x, uq.y};
              float dg[4], du[4], hh[4];
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const float gv = __uint_as_float((r & 1) ? (gw[r >> 1] & 0xffff0000u) : (gw[r >> 1] << 16));
                const float dh = acc[j][i][g * 4 + r];
                if (MODE == MODE_DH1) {   // two-matrix expert: dG = dH where g > 0, H = max(g, 0)
                  dg[r] = gv > 0.f ? dh : 0.f;
                  du[r] = 0.f;
                  hh[r] = fmaxf(gv, 0.f);
                } else {
                  const float uv = __uint_as_float((r & 1) ? (uw[r >> 1] & 0xffff0000u) : (uw[r >> 1] << 16));
                  const float sg = sigmoid_f(gv);
                  dg[r] = dh * uv * sg * (1.f + gv * (1.f - sg));
                  du[r] = dh * gv * sg;
                  hh[r] = gv * sg * uv;
                }
              }
              dgp[t] = pack4(dg[0], dg[1], dg[2], dg[3]);
              dup[t] = pack4(du[0], du[1], du[2], du[3]);
              hhp[t] = pack4(hh[0], hh[1], hh[2], hh[3]);
            }
            const uint4 dgv = pair16(dgp[0], dgp[1]), hhv = pair16(hhp[0], hhp[1]);
            if (MODE == MODE_DH) {
              const uint4 duv = pair16(dup[0], dup[1]);
              if (put) {
                *reinterpret_cast<uint4*>(p.C + row * (2 * (size_t)p.N) + col) = dgv;
                *reinterpret_cast<uint4*>(p.C + row * (2 * (size_t)p.N) + p.N + col) = duv;
              }
            } else if (put) {
              *reinterpret_cast<uint4*>(p.C + row * p.N + col) = dgv;
            }
            if (put) *reinterpret_cast<uint4*>(p.C2 + row * p.N + col) = hhv;
          }
        }
      }
    }
  }
}

}  // namespace
