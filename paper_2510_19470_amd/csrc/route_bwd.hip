// Backward of the gate (paper Sec. 2.1: the gate network picks K experts per token; the
// layer's output depends on the gate through the K combine weights).  The Top-k choice is
// piecewise constant, so the gradient flows only through the weights of the selected experts:
//   p = softmax of the logits over the selected experts (renormalize) or over all E,
//   dlogits[t,e] = p_e * ( [e selected] dw_e - sum_j dw_j w_j ),   w_j = p[idx_j] = topk_w,
//   dWg = dlogits^T x,  dbias = sum_t dlogits[t],  dx += dlogits Wg.
// Two launches: the logit gradients and the input gradient (one wavefront per token, added to the dx
// the dispatch backward has written) beside the weight gradient as per-chunk partial sums over 128
// tokens, and the fixed-order sum of those over the chunks together with dbias (deterministic, no
// floating-point atomics).  Without renormalising the partial sums are a launch of their own.
#include "moe_internal.h"
#include "numeric.h"
#include <type_traits>

namespace {

constexpr int RB_TOK = 128;   // tokens per partial-sum chunk

typedef float f32x4 __attribute__((ext_vector_type(4)));

// 16 bytes of a row of x; x need only be aligned to its elements.
template <typename T, bool ALIGNED>
__device__ __forceinline__ uint4 load_x(const T* p) {
  if constexpr (ALIGNED) return Vec16<T>::load_raw(p);
  union { T e[Vec16<T>::N]; uint4 q; } u;
#pragma unroll
  for (int i = 0; i < Vec16<T>::N; ++i) u.e[i] = p[i];
  return u.q;
}

struct TokenArgs {
  const float* logits;
  const int32_t* topk_idx;
  const float *topk_w, *dtopk_w;
  int Tn, E, k, renormalize, d;
  const void* Wg;
  float* dlogits;
  void* dx;
};

// One wavefront per token; lane e, e+64, ... own the experts.  dlogits[t] stays in registers for
//   dx[t] += sum_e dlogits[t][e] * Wg[e]   (16 bytes per lane; left out without dx),
// in which only the k selected experts have a non-zero logit gradient when renormalising.  Bound by reading
// and writing dx; the k rows of Wg come from L2, all requested together with the piece of dx (one at a time,
// every term waited for its own: 8192 tokens, d = 2048, E = 32, k = 4, dx in the last-level cache: call without dWg
// 18.0 -> 15.0 us).
template <typename T, int K_MAX>
__device__ __forceinline__ void token_grads(const TokenArgs& p, int block) {
  constexpr int V = Vec16<T>::N;
  constexpr int NE = MOE_MAX_EXPERTS / 64;
  const int E = p.E, k = p.k, d = p.d;
  const int lane = threadIdx.x & 63;
  const int t = block * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (t >= p.Tn) return;
  const T* Wg = static_cast<const T*>(p.Wg);
  int idx[K_MAX];
  float tw[K_MAX], dw[K_MAX];
#pragma unroll
  for (int j = 0; j < K_MAX; ++j) {
    const bool on = j < k;
    idx[j] = on ? p.topk_idx[(size_t)t * k + j] : -1;
    tw[j] = on ? p.topk_w[(size_t)t * k + j] : 0.f;
    dw[j] = on ? p.dtopk_w[(size_t)t * k + j] : 0.f;
  }
  float inner = 0.f;
#pragma unroll
  for (int j = 0; j < K_MAX; ++j)
    if (j < k) inner += dw[j] * tw[j];
  const float* logits = p.logits + (size_t)t * E;
  float mx = -INFINITY, den = 1.f;
  if (!p.renormalize) {   // full softmax of the row
    for (int e = lane; e < E; e += 64) mx = fmaxf(mx, logits[e]);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    float s = 0.f;
    for (int e = lane; e < E; e += 64) s += expf(logits[e] - mx);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    den = s;
  }
  float dl[NE];
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    const int e = lane + 64 * i;
    dl[i] = 0.f;
    if (e >= E) continue;
    float sel_dw = 0.f, w = 0.f;
    bool selected = false;
#pragma unroll
    for (int j = 0; j < K_MAX; ++j)
      if (idx[j] == e) {
        selected = true;
        sel_dw = dw[j];
        w = tw[j];
      }
    float pe;
    if (p.renormalize) pe = selected ? w : 0.f;
    else pe = expf(logits[e] - mx) / den;
    dl[i] = pe * ((selected ? sel_dw : 0.f) - inner);
    p.dlogits[(size_t)t * E + e] = dl[i];
  }
  if (p.dx == nullptr) return;
  T* dx = static_cast<T*>(p.dx) + (size_t)t * d;
  auto of_expert = [&](int e) {   // dlogits[t][e], e wave-uniform
    float v = dl[0];
#pragma unroll
    for (int i = 1; i < NE; ++i) v = (e >> 6) == i ? dl[i] : v;
    return __shfl(v, e & 63, 64);
  };
  // every lane takes part in every exchange: columns past the row are not loaded or stored
  if (p.renormalize) {
    float g[K_MAX];
    const T* row[K_MAX];
    bool ok[K_MAX];
#pragma unroll
    for (int j = 0; j < K_MAX; ++j) {
      ok[j] = (unsigned)idx[j] < (unsigned)E;   // the routing is the caller's: stay inside Wg
      const int e = __builtin_amdgcn_readfirstlane(ok[j] ? idx[j] : 0);
      g[j] = of_expert(e);
      row[j] = Wg + (size_t)e * d;
    }
#pragma unroll(K_MAX <= 4 ? 2 : 1)
    for (int c = lane * V; c < d; c += 64 * V) {
      float acc[V];
      const uint4 own = Vec16<T>::load_raw(dx + c);
      uint4 raw[K_MAX];
#pragma unroll
      for (int j = 0; j < K_MAX; ++j) raw[j] = Vec16<T>::load_raw(row[j] + c);
      Vec16<T>::unpack(own, acc);
#pragma unroll
      for (int j = 0; j < K_MAX; ++j) {
        float w[V];
        Vec16<T>::unpack(raw[j], w);
#pragma unroll
        for (int i = 0; i < V; ++i) acc[i] = ok[j] ? fmaf(g[j], w[i], acc[i]) : acc[i];
      }
      Vec16<T>::store(dx + c, acc);
    }
    return;
  }
  for (int c0 = 0; c0 < d; c0 += 64 * V) {
    const int c = c0 + lane * V;
    const bool in = c < d;
    float acc[V] = {};
    if (in) Vec16<T>::load(dx + c, acc);
#pragma unroll 4
    for (int e = 0; e < E; ++e) {
      const float g = of_expert(e);
      float w[V] = {};
      if (in) Vec16<T>::load(Wg + (size_t)e * d + c, w);
#pragma unroll
      for (int i = 0; i < V; ++i) acc[i] = fmaf(g, w[i], acc[i]);
    }
    if (in) Vec16<T>::store(dx + c, acc);
  }
}

// partial[chunk][e][c] = sum over the chunk's 128 tokens of dlogits[t][e] * x[t][c], on the matrix
// cores in fp32 (v_mfma_f32_16x16x4_f32; bf16 x is widened, nothing is rounded).  A block takes 16
// experts and 16 * V columns (V elements are 16 bytes), each of its wavefronts 32 of the tokens:
// lane (m, q) loads columns V*m .. V*m+V-1 of token 4s + q, element j of it is the operand of tile
// j, which so holds columns V*n + j, and a lane ends up with V consecutive columns of 4 experts;
// the wavefronts' sums meet in LDS.  What bounds it is the wait for memory, so a wavefront asks for
// everything at once and its blocks are many.  A thread per column on the vector units -> this, as a
// launch of its own: 29 -> 20 us (8192 tokens, d = 2048, 32 experts), 22 -> 5.7 us (1024 tokens, d = 1024);
// with one wavefront for all 128 tokens 28 and 21 us.
struct DwgArgs {
  const void* x;
  int n_cb, n_eg, n_tiles;   // column blocks, groups of 16 experts, chunks * n_cb
  float* partial;
};
template <typename T>
union DwgShared {
  float4 red[2][16][4 * Vec16<T>::N];
  float dl[RB_TOK][17];   // logit gradients of the chunk and the expert group
};
// OWN: the logit gradients are made here (renormalising: they depend on the token's k experts alone), so
// that the launch need not wait for those of the token blocks.
template <typename T, bool ALIGNED, bool OWN>
__device__ __forceinline__ void dwg_partial(const TokenArgs& t, const DwgArgs& p, DwgShared<T>& lds, int block) {
  constexpr int V = Vec16<T>::N;
  constexpr int STEPS = RB_TOK / 16;   // of 4 tokens, per wavefront
  const int Tn = t.Tn, d = t.d, E = t.E, n_cb = p.n_cb, n_eg = p.n_eg;
  const int lane = threadIdx.x & 63, m = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // the expert groups of one tile (chunk, columns) are blocks of the same XCD: x comes from memory once
  const int e0 = block / 8 % n_eg * 16;
  const int tile = block / (8 * n_eg) * 8 + block % 8;
  if (tile >= p.n_tiles) return;
  const int chunk = tile / n_cb, c0 = tile % n_cb * 16 * V, col = c0 + m * V;
  const int t0 = chunk * RB_TOK + wave * 4 * STEPS + q;
  // lanes past the columns or the experts repeat the first one: their sums are not stored
  const T* xp = static_cast<const T*>(p.x) + (col < d ? col : 0);
  const float* dp = t.dlogits + (e0 + m < E ? e0 + m : 0);
  uint4 xq[STEPS];
  float a[STEPS];
#pragma unroll
  for (int u = 0; u < STEPS; ++u) {   // tokens past the end: the last one, with zeros below
    const size_t row = min(t0 + 4 * u, Tn - 1);
    xq[u] = load_x<T, ALIGNED>(xp + row * d);
    if (!OWN) a[u] = dp[row * E];
  }
  if (OWN) {
    if (threadIdx.x < RB_TOK) {
      float* row = lds.dl[threadIdx.x];
      const size_t s0 = (size_t)min(chunk * RB_TOK + (int)threadIdx.x, Tn - 1) * t.k;
      float inner = 0.f;
      for (int j = 0; j < t.k; ++j) inner += t.dtopk_w[s0 + j] * t.topk_w[s0 + j];
      const float none = 0.f * (0.f - inner);   // of experts not selected: as in dlogits, where a NaN shows for all
#pragma unroll
      for (int i = 0; i < 16; ++i) row[i] = none;
      for (int j = 0; j < t.k; ++j) {
        const int e = t.topk_idx[s0 + j] - e0;
        if ((unsigned)e < 16u) row[e] = t.topk_w[s0 + j] * (t.dtopk_w[s0 + j] - inner);
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < STEPS; ++u) a[u] = lds.dl[wave * 4 * STEPS + q + 4 * u][m];
    __syncthreads();   // the sums take the same place
  }
  f32x4 acc[V];
#pragma unroll
  for (int j = 0; j < V; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < STEPS; ++u) {
    const bool ok = t0 + 4 * u < Tn;
    float v[V];
    Vec16<T>::unpack(ok ? xq[u] : make_uint4(0, 0, 0, 0), v);
    const float au = ok ? a[u] : 0.f;
#pragma unroll
    for (int j = 0; j < V; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(au, v[j], acc[j], 0, 0, 0);
  }
  // (0 + 2) + (1 + 3): half the LDS of all four at once, and twice the blocks on a compute unit
  auto each = [&](auto f) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < V; j += 4) f(lds.red[wave & 1][4 * q + i][(m * V + j) / 4], i, j);
  };
  if (wave >= 2)
    each([&](float4& r, int i, int j) { r = make_float4(acc[j][i], acc[j + 1][i], acc[j + 2][i], acc[j + 3][i]); });
  __syncthreads();
  if (wave < 2)
    each([&](float4& r, int i, int j) {
      r = make_float4(acc[j][i] + r.x, acc[j + 1][i] + r.y, acc[j + 2][i] + r.z, acc[j + 3][i] + r.w);
    });
  __syncthreads();
  for (int i = threadIdx.x; i < 16 * 4 * V; i += 256) {   // 16 bytes a thread and step
    const int r = i / (4 * V), c4 = i % (4 * V);
    float4 s = lds.red[0][r][c4];
    const float4 o = lds.red[1][r][c4];
    s.x += o.x; s.y += o.y; s.z += o.z; s.w += o.w;
    if (e0 + r < E && c0 + 4 * c4 < d)
      *reinterpret_cast<float4*>(p.partial + ((size_t)chunk * E + e0 + r) * d + c0 + 4 * c4) = s;
  }
}

// Both in one launch where neither needs the other (renormalising): the first n_dwg blocks make partial sums,
// the others serve tokens.  Training step, two launches -> one: 1024 tokens, d = 1024, E = 32: 189 -> 185 us; fp32,
// 1024 tokens, d = 512, E = 8: 197 -> 192; 8192 tokens, d = 2048: 768 -> 766; 8192 tokens, d = 1024, k = 8: 567 ->
// 562: with many tokens the fp32 products of the partial sums (7 us at d = 2048) and 100 MB of memory share the time.
// (Token blocks first, or both in turn: no difference.)  Without renormalising the partial sums take the logit
// gradients from the launch before (n_dwg = 0 there).
template <typename T, int K_MAX, bool ALIGNED>
__global__ __launch_bounds__(256) void route_bwd_token_kernel(const TokenArgs t, const DwgArgs p, int n_dwg) {
  __shared__ DwgShared<T> lds;
  if ((int)blockIdx.x < n_dwg) dwg_partial<T, ALIGNED, true>(t, p, lds, (int)blockIdx.x);
  else token_grads<T, K_MAX>(t, (int)blockIdx.x - n_dwg);
}
template <typename T, bool ALIGNED>
__global__ __launch_bounds__(256) void route_bwd_dwg_partial_kernel(const TokenArgs t, const DwgArgs p) {
  __shared__ DwgShared<T> lds;
  dwg_partial<T, ALIGNED, false>(t, p, lds, (int)blockIdx.x);
}

// Blocks 0 .. n_bias-1: dbias[e] = sum_t dlogits[t][e], a fixed reduction tree per expert.  The
// others: dWg[e][c] = sum over the chunks in ascending order.  Both with 8 loads in flight, added
// in order; one launch, since neither fills the chip.
__global__ __launch_bounds__(256) void route_bwd_finish_kernel(
    const float* __restrict__ partial, int n_chunks, size_t ed, float* __restrict__ dWg,
    const float* __restrict__ dlogits, int T, int E, int n_bias, float* __restrict__ dbias) {
  if ((int)blockIdx.x < n_bias) {
    __shared__ float red[256];
    const int e = blockIdx.x;
    float s = 0.f;
    int t = threadIdx.x;
    for (; t + 7 * 256 < T; t += 8 * 256) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = dlogits[(size_t)(t + u * 256) * E + e];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; t < T; t += 256) s += dlogits[(size_t)t * E + e];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int off = 128; off >= 1; off >>= 1) {
      if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
      __syncthreads();
    }
    if (threadIdx.x == 0) dbias[e] = red[0];
    return;
  }
  const size_t i = (blockIdx.x - (size_t)n_bias) * blockDim.x + threadIdx.x;
  if (i >= ed) return;
  float s = 0.f;
  int ch = 0;
  for (; ch + 8 <= n_chunks; ch += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = partial[(size_t)(ch + u) * ed + i];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
  for (; ch < n_chunks; ++ch) s += partial[(size_t)ch * ed + i];
  dWg[i] = s;
}

// T == 0: the sums are empty.  (A fill kernel rather than a memset call, so that the launch
// can be part of a captured graph.)
__global__ void route_bwd_zero_kernel(float* __restrict__ p, size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x)
    p[i] = 0.f;
}

template <typename T, int K_MAX, bool ALIGNED>
void launch_parts_as(const TokenArgs& t, const DwgArgs& w, int n_dwg, hipStream_t s) {
  const int n_tok = (t.Tn + 3) / 4, first = t.renormalize ? n_dwg : 0;
  hipLaunchKernelGGL((route_bwd_token_kernel<T, K_MAX, ALIGNED>), dim3(first + n_tok), dim3(256), 0, s, t, w, first);
  if (n_dwg > first)
    hipLaunchKernelGGL((route_bwd_dwg_partial_kernel<T, ALIGNED>), dim3(n_dwg), dim3(256), 0, s, t, w);
}
template <typename T>
void launch_parts(const TokenArgs& t, const DwgArgs& w, int n_dwg, bool aligned, hipStream_t s) {
  auto run = [&](auto al) {
    constexpr bool AL = decltype(al)::value;
    if (t.k <= 2) launch_parts_as<T, 2, AL>(t, w, n_dwg, s);
    else if (t.k <= 4) launch_parts_as<T, 4, AL>(t, w, n_dwg, s);
    else if (t.k <= 8) launch_parts_as<T, 8, AL>(t, w, n_dwg, s);
    else launch_parts_as<T, MOE_MAX_TOPK, AL>(t, w, n_dwg, s);
  };
  if (aligned) run(std::true_type{});
  else run(std::false_type{});
}

}  // namespace

size_t route_bwd_workspace_floats(const moe_ctx* c) {
  const size_t chunks = ((size_t)c->cfg.T_max + RB_TOK - 1) / RB_TOK;
  return chunks * (size_t)c->cfg.E * c->cfg.d;
}

int launch_route_bwd(moe_ctx* c, const void* x, const void* Wg, const float* logits,
                     const int32_t* topk_idx, const float* topk_w, const float* dtopk_w, int T,
                     float* dlogits, float* dWg, float* dbias, void* dx, hipStream_t s) {
  const int E = c->cfg.E, d = c->cfg.d, k = c->cfg.k, rn = c->cfg.renormalize;
  if (T == 0) {
    if (dWg != nullptr)
      hipLaunchKernelGGL(route_bwd_zero_kernel, dim3(256), dim3(256), 0, s, dWg, (size_t)E * d);
    if (dbias != nullptr)
      hipLaunchKernelGGL(route_bwd_zero_kernel, dim3(1), dim3(256), 0, s, dbias, (size_t)E);
    if (hipGetLastError() != hipSuccess) return MOE_EHIP;
    return MOE_OK;
  }
  const int chunks = (T + RB_TOK - 1) / RB_TOK;
  const int cols = 16 * (16 / (int)c->elem), n_cb = (d + cols - 1) / cols, n_eg = (E + 15) / 16;
  const TokenArgs t = {logits, topk_idx, topk_w, dtopk_w, T, E, k, rn, d, Wg, dlogits, dx};
  const DwgArgs w = {x, n_cb, n_eg, chunks * n_cb, c->d_rbwd_ws};
  const int n_dwg = dWg != nullptr ? (w.n_tiles + 7) / 8 * 8 * n_eg : 0;
  const bool al = ((uintptr_t)x & 15) == 0;
  if (c->cfg.dtype == MOE_BF16) launch_parts<uint16_t>(t, w, n_dwg, al, s);
  else launch_parts<float>(t, w, n_dwg, al, s);
  const size_t ed = dWg != nullptr ? (size_t)E * d : 0;
  const int n_bias = dbias != nullptr ? E : 0;
  if (ed > 0 || n_bias > 0)
    hipLaunchKernelGGL(route_bwd_finish_kernel, dim3((unsigned)(n_bias + (ed + 255) / 256)), dim3(256), 0,
                       s, c->d_rbwd_ws, chunks, ed, dWg, dlogits, T, E, n_bias, dbias);
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_EHIP;
}
