// Backward of the gate (paper Sec. 2.1: the gate network picks K experts per token; the
// layer's output depends on the gate through the K combine weights).  The Top-k choice is
// piecewise constant, so the gradient flows only through the weights of the selected experts:
//   p = softmax of the logits over the selected experts (renormalize) or over all E,
//   dlogits[t,e] = p_e * ( [e selected] dw_e - sum_j dw_j w_j ),   w_j = p[idx_j] = topk_w,
//   dWg = dlogits^T x,  dbias = sum_t dlogits[t],  dx += dlogits Wg.
// Three launches: the logit gradients and the input gradient (one wavefront per token, added to the dx
// the dispatch backward has written), the weight gradient as per-chunk partial sums over 128 tokens,
// and the fixed-order sum of those over the chunks together with dbias (deterministic, no
// floating-point atomics).  Where the weights are renormalised, small calls make the first two one.
#include "moe_internal.h"
#include "numeric.h"

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

// One wavefront per token; lane e, e+64, ... own the experts (NE: how many a lane has, at most).  dlogits[t]
// stays in registers for
//   dx[t] += sum_e dlogits[t][e] * Wg[e]   (16 bytes per lane; left out without dx),
// in which only the k selected experts have a non-zero logit gradient when renormalising.  Bound by reading
// and writing dx, with the full softmax by reading all of Wg from L2.  Four rows of Wg are requested together
// (one at a time, every term waited for its own), two pieces of them where there are more terms than that, and the
// first piece of dx before anything else; 6 to 8 wavefronts per SIMD cover the rest of the wait.  Call, us, a term at
// a time -> this: 8192 tokens, d = 2048, E = 32, k = 4: 47 -> 44; 4096 tokens, d = 2048, E = 64, k = 12: 51 -> 40; full
// softmax: 8192 x 2048, E = 32: 108 -> 77; 4096 x 2048, E = 64: 155 -> 73; 8192 x 2048, E = 256: 709 -> 459.
template <typename T, int NE, int P>
__device__ __forceinline__ void token_grads(const TokenArgs& p, int block) {
  constexpr int V = Vec16<T>::N;
  constexpr int TERMS = 4;
  const int E = p.E, k = p.k, d = p.d;
  const int lane = threadIdx.x & 63;
  const int t = block * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (t >= p.Tn) return;
  const T* Wg = static_cast<const T*>(p.Wg);
  T* dx = static_cast<T*>(p.dx) + (size_t)t * d;
  uint4 own[P];   // of dx, requested first: nothing has to be known for it
  auto load_own = [&](int c) {
#pragma unroll
    for (int q = 0; q < P; ++q)
      if (c + q * 64 * V < d) own[q] = Vec16<T>::load_raw(dx + c + q * 64 * V);
  };
  if (p.dx != nullptr) load_own(lane * V);
  // lane j < k: selected expert j
  static_assert(MOE_MAX_TOPK <= 64, "a lane per selected expert");
  const size_t sel = (size_t)t * k + min(lane, k - 1);
  const int idx = p.topk_idx[sel];
  const float tw = p.topk_w[sel], dw = p.dtopk_w[sel];
  auto of_lane = [](float v, int j) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), j)); };
  float inner = 0.f;
  for (int j = 0; j < k; ++j) inner += of_lane(dw, j) * of_lane(tw, j);
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
  float dl[NE];   // of experts lane, lane + 64, ...
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    const int e = lane + 64 * i;
    float sel_dw = 0.f, w = 0.f;
    bool selected = false;
    for (int j = 0; j < k; ++j)
      if (__builtin_amdgcn_readlane(idx, j) == e) {
        selected = true;
        sel_dw = of_lane(dw, j);
        w = of_lane(tw, j);
      }
    dl[i] = 0.f;
    if (e < E) {
      float pe;
      if (p.renormalize) pe = selected ? w : 0.f;
      else pe = expf(logits[e] - mx) / den;
      dl[i] = pe * ((selected ? sel_dw : 0.f) - inner);
      p.dlogits[(size_t)t * E + e] = dl[i];
    }
  }
  if (p.dx == nullptr) return;
  const int n_terms = p.renormalize ? k : E;
  // (wave-uniform loops: a lane past the row's columns neither loads nor stores, but the others read its dl)
  for (int c0 = 0; c0 < d; c0 += P * 64 * V) {
    const int c = c0 + lane * V;
    float acc[P][V];
    for (int j0 = 0; j0 < n_terms; j0 += TERMS) {
      uint4 raw[TERMS][P];
      int e[TERMS];
#pragma unroll
      for (int u = 0; u < TERMS; ++u) {
        e[u] = -1;
        if (j0 + u < n_terms) e[u] = p.renormalize ? __builtin_amdgcn_readlane(idx, j0 + u) : j0 + u;
        if ((unsigned)e[u] >= (unsigned)E) continue;   // the routing is the caller's: stay inside Wg
#pragma unroll
        for (int q = 0; q < P; ++q)
          if (c + q * 64 * V < d) raw[u][q] = Vec16<T>::load_raw(Wg + (size_t)e[u] * d + c + q * 64 * V);
      }
      if (j0 == 0) {
#pragma unroll
        for (int q = 0; q < P; ++q) Vec16<T>::unpack(own[q], acc[q]);
        load_own(c + P * 64 * V);
      }
#pragma unroll
      for (int u = 0; u < TERMS; ++u) {
        if ((unsigned)e[u] >= (unsigned)E) continue;
        float v = dl[0];
#pragma unroll
        for (int i = 1; i < NE; ++i) v = (e[u] >> 6) == i ? dl[i] : v;
        const float g = of_lane(v, e[u] & 63);
#pragma unroll
        for (int q = 0; q < P; ++q) {
          float w[V];
          Vec16<T>::unpack(raw[u][q], w);
#pragma unroll
          for (int i = 0; i < V; ++i) acc[q][i] = fmaf(g, w[i], acc[q][i]);
        }
      }
    }
#pragma unroll
    for (int q = 0; q < P; ++q)
      if (c + q * 64 * V < d) Vec16<T>::store(dx + c + q * 64 * V, acc[q]);
  }
}

// The same for renormalised weights of up to K_MAX experts, beside blocks that leave it half as many wavefronts
// (route_bwd_joint_kernel): what a wavefront needs is in registers and requested without a branch between, two
// pieces of the row at a time where they fit.
template <typename T, int K_MAX>
__device__ __forceinline__ void token_grads_selected(const TokenArgs& p, int block) {
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
  float dl[NE];   // of experts lane, lane + 64, ...
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    const int e = lane + 64 * i;
    dl[i] = 0.f;
    if (e >= E) continue;
    float sel_dw = 0.f, w = 0.f;
#pragma unroll
    for (int j = 0; j < K_MAX; ++j)
      if (idx[j] == e) {
        sel_dw = dw[j];
        w = tw[j];
      }
    dl[i] = w * (sel_dw - inner);
    p.dlogits[(size_t)t * E + e] = dl[i];
  }
  if (p.dx == nullptr) return;
  T* dx = static_cast<T*>(p.dx) + (size_t)t * d;
  float g[K_MAX];
  const T* row[K_MAX];
  bool ok[K_MAX];
#pragma unroll
  for (int j = 0; j < K_MAX; ++j) {
    ok[j] = (unsigned)idx[j] < (unsigned)E;   // the routing is the caller's: stay inside Wg
    const int e = __builtin_amdgcn_readfirstlane(ok[j] ? idx[j] : 0);
    float v = dl[0];
#pragma unroll
    for (int i = 1; i < NE; ++i) v = (e >> 6) == i ? dl[i] : v;
    g[j] = __shfl(v, e & 63, 64);   // (every lane takes part)
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

template <typename T, int NE, int P>
__global__ __launch_bounds__(256) void route_bwd_token_kernel(const TokenArgs t) {
  token_grads<T, NE, P>(t, (int)blockIdx.x);
}
template <typename T, bool ALIGNED>
__global__ __launch_bounds__(256) void route_bwd_dwg_partial_kernel(const TokenArgs t, const DwgArgs p) {
  __shared__ DwgShared<T> lds;
  dwg_partial<T, ALIGNED, false>(t, p, lds, (int)blockIdx.x);
}
// Both in one launch (renormalising, where neither needs the other): the first n_dwg blocks make partial sums,
// the others serve tokens.
template <typename T, int K_MAX, bool ALIGNED>
__global__ __launch_bounds__(256) void route_bwd_joint_kernel(const TokenArgs t, const DwgArgs p, int n_dwg) {
  __shared__ DwgShared<T> lds;
  const int block = (int)blockIdx.x - n_dwg;
  if (block < 0) dwg_partial<T, ALIGNED, true>(t, p, lds, (int)blockIdx.x);
  else token_grads_selected<T, K_MAX>(t, block);
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

template <typename T, bool ALIGNED>
void launch_parts(const TokenArgs& t, const DwgArgs& w, int n_dwg, bool joint, hipStream_t s) {
  const int n_tok = (t.Tn + 3) / 4;
  if (joint) {
    auto kern = t.k <= 2   ? route_bwd_joint_kernel<T, 2, ALIGNED>
                : t.k <= 4 ? route_bwd_joint_kernel<T, 4, ALIGNED>
                : t.k <= 8 ? route_bwd_joint_kernel<T, 8, ALIGNED>
                           : route_bwd_joint_kernel<T, MOE_MAX_TOPK, ALIGNED>;
    hipLaunchKernelGGL(kern, dim3(n_dwg + n_tok), dim3(256), 0, s, t, w, n_dwg);
    return;
  }
  constexpr int MANY = MOE_MAX_EXPERTS / 64;
  const bool two = t.d > 64 * Vec16<T>::N && (!t.renormalize || t.k > 4);   // pieces of a row at a time
  auto token = t.E <= 64 ? (two ? route_bwd_token_kernel<T, 1, 2> : route_bwd_token_kernel<T, 1, 1>)
                         : (two ? route_bwd_token_kernel<T, MANY, 2> : route_bwd_token_kernel<T, MANY, 1>);
  hipLaunchKernelGGL(token, dim3(n_tok), dim3(256), 0, s, t);
  if (n_dwg > 0)
    hipLaunchKernelGGL((route_bwd_dwg_partial_kernel<T, ALIGNED>), dim3(n_dwg), dim3(256), 0, s, t, w);
}

// One launch or two where one is possible.  One saves 2 to 3 us of start and gap, but its token blocks get half as
// many wavefronts, and its weight-gradient blocks make the logit gradients again, once per 16 experts and 128 (64)
// columns.  Call, us, two launches -> one (n_dwg: blocks of the weight gradient):
//   512 blocks or less: 1024 tokens, d = 1024, E = 32, k = 2: 11.9 -> 9.8; 2048, 2048, 32, 4: 18.0 -> 15.2; 8192, 1024, 8,
//   2: 22.0 -> 19.2; 2048, 1024, 64, 8: 16.9 -> 15.6
//   768: 2048, 1536, 64, 8: 21.5 -> 20.1; 3072, 1024, 64, 8: 20.5 -> 21.3; 1024: 2048, 2048, 64, 6: 23.7 -> 22.1, k = 8: 24.7 ->
//   25.3; 4096, 2048, 32, 4: 24.9 -> 26.2; 1536: 3072, 2048, 64, 6: 28.4 -> 30.1, k = 8: 29.6 -> 33.7; few tokens: 700, 4096,
//   128, 6: 32.7 -> 27.1
//   2048: 8192, 2048, 32, 4: 44.4 -> 48.5; 4096, 2048, 64, 6: 38.2 -> 45.0; 8192: 8192, 4096, 64, 7: 117 -> 153
//   more than eight selected experts (three wavefronts per SIMD): 1024, 4096, 32, 12: 25.5 -> 22.5; 4096, 136, 32, 12: 15.4 ->
//   15.2; 8192, 512, 16, 9: 21.1 -> 25
bool joint_wanted(int T, int n_dwg, int k, int n_cu) {
  if (k > 8) return n_dwg <= 2 * n_cu && T <= 16 * n_cu;
  return n_dwg <= (k > 6 ? 3 : T > 4 * n_cu ? 5 : 8) * n_cu;
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
  const bool joint = rn && n_dwg > 0 && (c->gate_joint != 0 ? c->gate_joint == 1 : joint_wanted(T, n_dwg, k, c->n_cu));
  if (c->cfg.dtype == MOE_BF16) (al ? launch_parts<uint16_t, true> : launch_parts<uint16_t, false>)(t, w, n_dwg, joint, s);
  else (al ? launch_parts<float, true> : launch_parts<float, false>)(t, w, n_dwg, joint, s);
  const size_t ed = dWg != nullptr ? (size_t)E * d : 0;
  const int n_bias = dbias != nullptr ? E : 0;
  if (ed > 0 || n_bias > 0)
    hipLaunchKernelGGL(route_bwd_finish_kernel, dim3((unsigned)(n_bias + (ed + 255) / 256)), dim3(256), 0,
                       s, c->d_rbwd_ws, chunks, ed, dWg, dlogits, T, E, n_bias, dbias);
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_EHIP;
}

// Not part of the interface, for tests: one launch (1) or two (2) for the logit and the weight gradients (0: the rule).
extern "C" void moe_internal_gate_joint(moe_ctx* c, int32_t joint) { c->gate_joint = joint; }
