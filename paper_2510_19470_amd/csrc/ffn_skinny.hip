// Expert FFN for a handful of rows per expert (generation), bf16 in, fp32 accumulate.
//
// What bounds it is reading every weight of the used experts once.  The 256-row tiles of
// ffn_mfma_kernel serve that badly where few experts are used: one block per 128 to 256 weight
// rows leaves compute units idle and needs a K-split with partial sums through memory, and a
// tile list has to be built first.  Here a block takes 16 weight rows (of W1 and the same ones
// of W3 for gate/up; 32 in small calls), its 8 wavefronts cut the contraction among themselves in units of 64 (one
// 128-byte line per weight row), and nothing is staged: a weight fragment is one 16-byte load per
// lane, used for all of the expert's rows, and the wavefronts' sums meet in LDS (added in
// wavefront order: deterministic).  No schedule launch, no partial sums in memory.  The token rows
// come from L2 once per block, which is what limits the rows: see few_rows.
#include <algorithm>

#include "moe_internal.h"
#include "numeric.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NT = 512;
constexpr int NW = NT / 64;

enum { SK_UP = 0, SK_UP1 = 1, SK_DOWN = 2 };

constexpr int WROWS = 16;    // weight rows (output columns) of a fragment
constexpr int GROUPS = 4;    // groups of 16 token rows that one pass over the weights serves

struct SkinnyArgs {
  const uint16_t* A;              // [S, K] packed rows
  const void* const* B0;          // [E] weight tables: W1 (gate/up), W2 (down)
  const void* const* B1;          // gate/up: W3
  uint16_t *C, *Gs, *Us;          // [S, N]; G and U saves of the backward (or NULL)
  const int32_t *counts, *offsets;
  int K, N, S;
  int n_list;
  uint8_t list[MOE_MAX_EXPERTS];  // experts that are looked at (those without weights are skipped)
};

__device__ __forceinline__ bf16x8 as_frag(const uint4& v) { return __builtin_bit_cast(bf16x8, v); }

// Whole units u, u + NW, ... of one wavefront, UNR of them requested before the first is used, while
// UNR are left.  Fragment of a unit's half h: 16-byte chunk 4h + (lane >> 4) of row (lane & 15), the
// same permutation of k for weights and tokens.
template <int UNR, int NF, int G>
__device__ __forceinline__ void skinny_units(f32x4 (&acc)[NF][G], const uint4* const (&w)[NF],
                                             const uint4* const (&x)[G], int full, int& u) {
  const int q = (threadIdx.x & 63) >> 4;
  for (; u + (UNR - 1) * NW < full; u += UNR * NW) {
    uint4 wv[UNR][2][NF], xv[UNR][2][G];
#pragma unroll
    for (int n = 0; n < UNR; ++n)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int ch = (u + n * NW) * 8 + 4 * h + q;
#pragma unroll
        for (int f = 0; f < NF; ++f) wv[n][h][f] = w[f][ch];
#pragma unroll
        for (int g = 0; g < G; ++g) xv[n][h][g] = x[g][ch];
      }
#pragma unroll
    for (int n = 0; n < UNR; ++n)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
          for (int g = 0; g < G; ++g)
            acc[f][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_frag(wv[n][h][f]), as_frag(xv[n][h][g]),
                                                                acc[f][g], 0, 0, 0);
  }
}

// Sums of one wavefront over its units: acc[f][g] for weight matrix f and token group g.
template <int NF, int G>
__device__ __forceinline__ void skinny_sums(f32x4 (&acc)[NF][G], const uint4* const (&w)[NF],
                                            const uint4* const (&x)[G], int n_chunks, int wave) {
  const int q = (threadIdx.x & 63) >> 4;
  const int full = n_chunks >> 3;   // whole units
  int u = wave;
  // 128 registers in all.  Short rows have fewer than four units for a wavefront; one at a time they
  // waited for memory once each (FFN call, 6 experts of 1024 x 4096: 1 token 22.9 -> 19.2 us, 8 tokens
  // 43.4 -> 40.2; two-matrix, 3072 x 3072, 8 tokens: 80.7 -> 77.2).
  if constexpr (NF + G <= 3) skinny_units<4, NF, G>(acc, w, x, full, u);
  if constexpr (NF + G <= 5) skinny_units<2, NF, G>(acc, w, x, full, u);
  // the units left over, the last of which may hold fewer than 8 chunks (zeros for the rest)
  for (; u * 8 < n_chunks; u += NW)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int ch = u * 8 + 4 * h + q;
      const bool ok = ch < n_chunks;
      uint4 wv[NF], xv[G];
#pragma unroll
      for (int f = 0; f < NF; ++f) wv[f] = ok ? w[f][ch] : make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int g = 0; g < G; ++g) xv[g] = ok ? x[g][ch] : make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int g = 0; g < G; ++g)
          acc[f][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_frag(wv[f]), as_frag(xv[g]), acc[f][g], 0, 0, 0);
    }
}

__device__ __forceinline__ uint2 pack4(const f32x4& v) {
  return make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
}

// One pass over the block's weight rows (WG groups of 16) for `rows` (1 .. 16 G) token rows from packed row `row0`.
template <int MODE, int G, int WG>
__device__ __forceinline__ void skinny_pass(const SkinnyArgs& p, const void* b0, const void* b1,
                                            size_t row0, int rows, f32x4* red) {
  constexpr int NM = MODE == SK_UP ? 2 : 1, NF = NM * WG;   // fragment f: matrix f % NM, row group f / NM
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n0 = blockIdx.x * (WROWS * WG);
  const uint4* w[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const size_t wrow = min(n0 + f / NM * WROWS + (lane & 15), p.N - 1);   // past the matrix: not stored
    w[f] = reinterpret_cast<const uint4*>((const uint16_t*)(f % NM == 0 ? b0 : b1) + wrow * p.K);
  }
  const uint4* x[G];
#pragma unroll
  for (int g = 0; g < G; ++g)
    x[g] = reinterpret_cast<const uint4*>(p.A + (row0 + min(g * 16 + (lane & 15), rows - 1)) * p.K);
  f32x4 acc[NF][G];
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int g = 0; g < G; ++g) acc[f][g] = f32x4{0.f, 0.f, 0.f, 0.f};
  skinny_sums<NF, G>(acc, w, x, p.K >> 3, wave);
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int g = 0; g < G; ++g) red[((wave * NF + f) * G + g) * 64 + lane] = acc[f][g];
  __syncthreads();
  // wavefront g finishes token group g % G of row group g / G: a lane holds token lane & 15, 4 consecutive columns
  if (wave < G * WG) {
    const int tg = wave % G, wg = wave / G;
    f32x4 s[2];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const f32x4* part = red + ((wg * NM + m) * G + tg) * 64 + lane;
      s[m] = part[0];
#pragma unroll
      for (int v = 1; v < NW; ++v) s[m] += part[v * NF * G * 64];
    }
    const int r = tg * 16 + (lane & 15), col = n0 + wg * WROWS + 4 * (lane >> 4);
    if (r < rows && col < p.N) {   // N is a multiple of 8: the four columns exist or do not
      const size_t o = (row0 + r) * p.N + col;
      if (MODE != SK_DOWN && p.Gs != nullptr) {
        *reinterpret_cast<uint2*>(p.Gs + o) = pack4(s[0]);
        if (MODE == SK_UP) *reinterpret_cast<uint2*>(p.Us + o) = pack4(s[1]);
      }
      f32x4 h = s[0];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (MODE == SK_UP) h[i] = silu_f(s[0][i]) * s[1][i];
        if (MODE == SK_UP1) h[i] = fmaxf(s[0][i], 0.f);
      }
      *reinterpret_cast<uint2*>(p.C + o) = pack4(h);
    }
  }
  __syncthreads();   // `red` is free for the next pass
}

// Block (x: 16 WG output columns, y: expert of the list).  128 registers: two blocks per compute
// unit, 16 wavefronts with 4 to 16 KB of weights in flight each.
template <int MODE, int WG>
__global__ __launch_bounds__(NT, 4) void ffn_skinny_kernel(const SkinnyArgs p) {
  __shared__ f32x4 red[NW * (MODE == SK_UP ? 2 : 1) * (WG > 1 ? WG : GROUPS) * 64];
  // counts and offsets are the caller's: nothing is computed unless every segment fits the
  // buffers (the rule of the tile schedule)
  int bad = 0;
  if ((int)threadIdx.x < p.n_list) {
    const int l = p.list[threadIdx.x], n = p.counts[l], o = p.offsets[l];
    bad = p.B0[l] != nullptr && (n < 0 || o < 0 || (long)o + n > (long)p.S);
  }
  const int e = p.list[blockIdx.y];
  const int n_e = p.counts[e], row0 = p.offsets[e];
  const void* b0 = p.B0[e];
  if (__syncthreads_or(bad) || b0 == nullptr) return;
  const void* b1 = MODE == SK_UP ? p.B1[e] : nullptr;
  if (WG > 1) {   // calls of at most 16 tokens: one pass, unless the caller's counts have a token twice
    for (int r = 0; r < n_e; r += 16) skinny_pass<MODE, 1, WG>(p, b0, b1, (size_t)row0 + r, min(16, n_e - r), red);
    return;
  }
  for (int r = 0; r < n_e; r += 16 * GROUPS) {
    const int rows = min(16 * GROUPS, n_e - r);
    const size_t first = (size_t)row0 + r;
    if (rows <= 16) skinny_pass<MODE, 1, 1>(p, b0, b1, first, rows, red);
    else if (rows <= 32) skinny_pass<MODE, 2, 1>(p, b0, b1, first, rows, red);
    else skinny_pass<MODE, GROUPS, 1>(p, b0, b1, first, rows, red);
  }
}

template <int MODE>
int launch(const SkinnyArgs& a, int T, int n_cu, hipStream_t s) {
  // A wavefront has K / 512 units.  Where it can ask for all of them at once (16 registers a unit and row group: four
  // units of one matrix, two of two), a block that takes 32 weight rows has twice as much in flight behind one start
  // (kernel arguments, counts, sums).  16 rows -> 32, both GEMMs, us; one matrix: 2048 x 1408, 12 of 64 experts, T = 8:
  // 57.8 -> 54.4, T = 16: 57.2 -> 53.5; 4096 x 2048, 16 experts, T = 16: 161 -> 152; two-matrix, 2048 x 14336, T = 8: 201 -> 183;
  // two (gate/up): 256 x 6784, 32 of 64, T = 7: 110 -> 83; 512 x 2944, 32 experts, T = 6: 78 -> 68; 768 x 6144, 37 of 64, T = 2: 109 ->
  // 97.  Two units of two matrices lose where blocks are few (1024 x 4096, 6 of 16, T = 8:
  // 40.5 -> 43.0; 32 of 64 experts of 1024 x 6272: 91 -> 85), four more so (2048 x 4096, 16 experts, T = 12: 159 -> 176).  One
  // matrix up to K = 4096: 159 -> 164; one token on 1024 x 4096: 18.2 -> 21.5; two-matrix 3072 x 3072, T = 8: 71 -> 65.  With
  // more token rows there are too few registers.  Blocks that have rows have to be left for every unit twice (11 tokens on 2
  // experts of 512 x 1024: 10.5 -> 11.5; one token, k = 1, 16 experts of 1376 x 1296: 9.6 -> 11.0), unless there are many
  // without (64 experts of 1024 x 1408, 3 tokens: 26 -> 16).
  const int blocks = (a.N + 2 * WROWS - 1) / (2 * WROWS);
  if (T <= 16 && a.K <= (MODE == SK_UP ? 768 : 2048) &&
      (blocks * std::min(a.n_list, a.S) >= 2 * n_cu || blocks * a.n_list >= 8 * n_cu)) {
    const dim3 grid(blocks, a.n_list);
    hipLaunchKernelGGL((ffn_skinny_kernel<MODE, 2>), grid, dim3(NT), 0, s, a);
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_EHIP;
  }
  const dim3 grid((a.N + WROWS - 1) / WROWS, a.n_list);
  hipLaunchKernelGGL((ffn_skinny_kernel<MODE, 1>), grid, dim3(NT), 0, s, a);
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_EHIP;
}

}  // namespace

// Reading the token rows once per 16 weight rows costs more the more rows there are; what the tiles
// cost depends on whether they fill the chip.  FFN call, tiles -> this kernel, us, rows spread evenly:
//   (S/E: rows per expert)
//   fewer gate/up tiles than compute units (d = 1024, f = 4096, 4 experts): S/E = 1: 57.6 -> 28.7, 8: 59.9 -> 33.8, 25: 60.0 -> 44.1, 50: 58.6 -> 59.4;
//   d = 2048, f = 1408, 16 experts: S/E = 6: 107 -> 80, 19: 107 -> 98, 37: 109 -> 124;
//   d = 4096, f = 4096, 4 experts: S/E = 25: 136 -> 131
//   more of them (d = 2048, f = 4096, 16 experts): S/E = 2: 207 -> 163, 8: 218 -> 184, 25: 217 -> 257
//   ... and long rows, which the tiles stream at 4.5 to 5.1 TB/s (d = 4096, f = 14336, 8 experts):
//   S/E = 0.25: 164 -> 150, 4: 564 -> 557, 8: 568 -> 619; d = 4096, f = 2048, 16 experts:
//   S/E = 2: 162 -> 160, 8: 180 -> 188
// The counts stay on the device, and tokens need not fall evenly.  At most T rows go to any expert and
// T * min(k, resident) to all of them; their rows come through L2 d * f / 16 times each (4 bytes: once
// for gate/up, once for down), at about 8 TB/s.  The tiles are slower by their schedule launch and the
// K-split sums, 27 us or more at these sizes.  So the rows are held to 200 MB, and to one pass over the weights.  All
// tokens on the same k experts, tiles -> this kernel, us, on both sides of that
// line: d = f = 3072, two-matrix, k = 6: T = 8: 98 -> 55, 24: 100 -> 79, 48: 99 -> 121; d = 2048,
// f = 1408, k = 6: T = 32: 67 -> 44, 48: 67 -> 57, 96: 66 -> 95; d = 2048, f = 14336, two-matrix, k = 2:
// T = 8: 87 -> 63, 16: 88 -> 70, 32: 88 -> 94; d = 4096, f = 14336, k = 2: T = 4: 161 -> 138,
// 8: 161 -> 147, 16: 162 -> 171; d = 1024, f = 4096, k = 2: T = 64: 48 -> 37, 96: 48 -> 56.  (By S/E
// alone, with up to 256 tokens: T = 200 with popularity falling off as rank^-1.2, 64 experts of
// d = f = 3072, k = 6: 135 -> 352; d = 2048, f = 14336, k = 2: 229 -> 529.)
// (The 256-row tiles, that is.)  The 128-row tiles serve most of these sizes better than the 256-row ones, but
// for them a longer row means more k-steps in a row: where they would take the layer, the rows are held to 48 KB
// per element of d (98 MB up to d = 2048).  128-row tiles -> this kernel, us, all tokens on the same experts |
// on the resident ones evenly | on all evenly:
//   1024 x 4096, E = 16, k = 2, 6 resident: T = 8: 29 -> 20 | 39 -> 40 | 39 -> 40, 32 (67 MB): 29 -> 28 | 40 -> 46 |
//   39 -> 41, 48 (101 MB): 35 -> 36 | 40 -> 50 | 40 -> 42, 64: 35 -> 40 | 41 -> 57 | 40 -> 44; 4 resident,
//   T = 64 (134 MB): 35 -> 42 | 33 -> 41 | 32 -> 30
//   2048 x 1408, E = 64, k = 6, 12 resident: T = 8: 38 -> 36 | 50 -> 54 | 53 -> 53, 16 (69 MB): 37 -> 39 | 50 -> 56 |
//   50 -> 53, 24 (104 MB): 37 -> 49 | 51 -> 64 | 50 -> 58, 32: 37 -> 51 | 51 -> 68 | 50 -> 58
//   two-matrix: 768 x 2048, T = 64: 29 -> 21 | 26 -> 19 | 25 -> 16; 2048 x 14336, T = 8 (117 MB): 58 -> 61 | 166 -> 178;
//   3072 x 3072, k = 6, T = 8 (113 MB): 53 -> 66 | 67 -> 77 | 67 -> 68
// Many weights, which the 128-row tiles copy past the last-level cache and whose parts they join, they read faster now:
// 2048 x 4096, E = 16, k = 2, 16 resident, T = 12: 34 -> 35 | 125 -> 159; 4096 x 2048, T = 16: 34 -> 28 | 134 -> 151; 4096 x 14336,
// E = 8, k = 2, 8 resident: T = 1: 126 -> 135, 4: 130 -> 144 | 438 -> 468.  The line is from before that and has not been moved.
static bool few_rows(long long T, int d, int f, int E, int k, int n_res, bool gated, int n_cu) {
  const int bn = gated ? 128 : 256;
  const bool fills = (long long)n_res * ((f + bn - 1) / bn) >= n_cu;
  const int most = !fills ? 24 : d < 4096 ? 8 : 4;   // rows per expert
  const long long l2_bytes = T * std::min(k, n_res) * d * f / 4;
  if (T > 16 * GROUPS || l2_bytes > 200000000ll || T * k > (long long)most * E) return false;
  return l2_bytes <= 48000ll * std::max(d, 2048) ||
         !ffn_tile128_rule((int)T, d, f, E, k, n_res, gated, false, n_cu);
}

bool ffn_skinny_wanted(const moe_ctx* c, bool gated) {
  if (c->tile_rows != 0) return c->tile_rows == WROWS;
  int n_res = 0;
  for (int e = 0; e < c->cfg.E; ++e) n_res += c->h_wtab[0][e] != nullptr;
  return few_rows(c->S_call / c->cfg.k, c->cfg.d, c->cfg.f, c->cfg.E, c->cfg.k, n_res, gated, c->n_cu);
}

// Not part of the interface: the rule above, for tests (one that needs no GPU, and those that want to
// know that they reach this kernel).
extern "C" int moe_internal_ffn_few_rows(int32_t T, int32_t d, int32_t f, int32_t E, int32_t k, int32_t n_res,
                                         int32_t gated, int32_t n_cu) {
  return few_rows(T, d, f, E, k, n_res, gated != 0, n_cu) ? 1 : 0;
}

int launch_ffn_skinny(moe_ctx* c, bool gated, const int32_t* counts, const int32_t* offsets,
                      const void* x_packed, void* y_packed, void* G, void* U, hipStream_t s) {
  const void* const* W1 = c->d_wtab + 0 * MOE_MAX_EXPERTS;
  const void* const* W3 = c->d_wtab + 1 * MOE_MAX_EXPERTS;
  const void* const* W2 = c->d_wtab + 2 * MOE_MAX_EXPERTS;
  SkinnyArgs a{};
  // Resident experts by the host copy of the pointer tables.  A captured launch is replayed on
  // whatever the device tables hold then: it looks at every expert.
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &cs) != hipSuccess) {
    (void)hipGetLastError();
    cs = hipStreamCaptureStatusActive;
  }
  for (int e = 0; e < c->cfg.E; ++e)
    if (c->h_wtab[0][e] != nullptr || cs != hipStreamCaptureStatusNone) a.list[a.n_list++] = (uint8_t)e;
  prof_mark(c, 0, s);
  prof_mark(c, 1, s);   // no schedule launch
  if (a.n_list > 0) {
    a.counts = counts;
    a.offsets = offsets;
    a.S = c->S_call;
    a.A = (const uint16_t*)x_packed;
    a.B0 = W1;
    a.B1 = W3;
    a.C = (uint16_t*)c->d_H;
    a.Gs = (uint16_t*)G;
    a.Us = (uint16_t*)U;
    a.K = c->cfg.d;
    a.N = c->cfg.f;
    const int st = gated ? launch<SK_UP>(a, c->S_call / c->cfg.k, c->n_cu, s) : launch<SK_UP1>(a, c->S_call / c->cfg.k, c->n_cu, s);
    if (st != MOE_OK) return st;
  }
  prof_mark(c, 2, s);
  if (a.n_list > 0) {
    a.A = (const uint16_t*)c->d_H;
    a.B0 = W2;
    a.B1 = nullptr;
    a.C = (uint16_t*)y_packed;
    a.Gs = a.Us = nullptr;
    a.K = c->cfg.f;
    a.N = c->cfg.d;
    const int st = launch<SK_DOWN>(a, c->S_call / c->cfg.k, c->n_cu, s);
    if (st != MOE_OK) return st;
  }
  prof_mark(c, 3, s);
  return MOE_OK;
}
