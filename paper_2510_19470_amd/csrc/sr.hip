// Shared/residual expert compression (paper Sec. 4.2 "SR-Based Expert Compression",
// Fig. "SRexpert"(b); compression ratio: Sec. 5.4).
//
//   encode: residual = expert - shared expert (float32); keep the k entries of largest
//           magnitude (equal magnitudes: lower index first) as a value-index list in
//           ascending index order, values rounded to the storage type;
//   decode: expert' = shared + scattered residual, one pass.
//
// The selection is exact.  The magnitude of a float32 is monotone in its low 31 bits (the key).
// Expert and shared are streamed ONCE, because a sample tells beforehand where the k-th largest
// key will be found:
//   1. sample: histogram of the top 12 key bits of about 512 K elements (128-byte pieces spread
//      over the matrix);
//   2. compact: the one pass over both matrices.  Every block takes from the sample's histogram
//      the highest bin b_lo whose count of keys at or above it exceeds the expected share of k by
//      a margin.  Every element whose top bits reach b_lo (k of them and a few per cent more) is
//      appended, as (residual bits, index), to a list in the workspace: one contiguous run per
//      chunk of 8192 elements, in index order inside the run, in a region of the list that the
//      block owns.  The same pass makes the histogram of 13 leading bits of the listed keys: 512
//      bins counted from b_lo (16 binades), since the k-th largest lies just above it;
//   3. fine: every block derives from it the bin of the k-th largest key; the listed keys of that
//      bin (4 % of the list) are counted by their upper 9 and by all 18 remaining bits;
//   4. count: every block derives the threshold from those, then counts the keys above and equal
//      to it, per chunk;
//   5. emit: a block sums the counts of the chunks before its own (the keys taken before chunk c
//      are G + min(E, wanted), G above and E equal) and writes the value-index list.
// Every step derives what it needs from the histogram of the step before, redundantly in every
// block and while its first loads are in flight: that takes 2-3 us, where a one-block launch in
// between (8 us) or the last block to finish (10 us: its atomics are returned one after another)
// leave the rest of the part idle.
// Steps 3 to 5 read the list only (11 MB at n = 14336 x 4096, k = n / 50).
// When the sample promised too much (fewer than k keys listed), a block's runs do not fit its
// region (the list has room for n/6 entries, every block for its share of the chunks: many equal
// magnitudes, k a larger fraction of n, or large residuals in a few chunks only) or
// the k-th largest lies beyond the 512 bins, step 3 says so in `mode`, and the matrices are streamed
// again instead of the list: step 3 makes a histogram of the 12 leading key bits of all elements,
// step 4 counts those of the bin it gives by their 19 remaining bits, step 5 counts per chunk and the
// last launch (which otherwise only clears the histograms) emits.
// The output never depends on the sample; it is deterministic (integer atomics only).
//
// What bounds it, n = 14336 x 4096 bf16: the pass over both matrices (235 MB).  Encode 157 -> 95 us
// against the version that streamed both matrices twice (histogram, then list) and picked bins in
// one-block launches (matrices not in the last-level cache); of it the pass takes 58 us (4.1 TB/s; 51 us
// with the expert past the cache, see sr_once), the five short launches 4.6-12 us each.  Half of the pass is
// vector instructions (selecting the residual by a tree of moves instead of one comparison per word
// made it 80 us, reading it again from memory 64; two chunks ahead instead of one: no faster).  Decode
// 60 -> 46 us (5.1 TB/s): the shared expert is requested before the search, 1 KB per load instruction,
// and the LDS of a block went from 40 to 17 KB.
#include "moe_internal.h"
#include "numeric.h"

#include <algorithm>
#include <type_traits>

namespace {

constexpr int SR_THREADS = 512;
constexpr int SR_WAVES = SR_THREADS / 64;
constexpr int SR_PER_THREAD = 16;
constexpr int SR_CHUNK = SR_THREADS * SR_PER_THREAD;  // 8192 elements
constexpr int SR_BINS = 4096;
constexpr uint32_t SR_INF_BIN = 0x7f800000u >> 19;   // leading 12 key bits of infinity
constexpr int SR_REPL = 4;    // copies of a global histogram (fewer same-address atomics)
constexpr int64_t SR_SAMPLE = 1 << 19;
constexpr int SR_COARSE = 1024, SR_FINE = 1 << 19;  // upper 10 and all of 19 low key bits (18 of
                                                    // them in mode 0: the lower half is used)

struct SrState {            // device-side selection state, at the front of the workspace
  uint32_t b_lo;            // listed: keys with (key >> 19) >= b_lo
  uint32_t bin;             // leading key bits of the k-th largest: key >> 18 (mode 1: key >> 19)
  int32_t k_rem;            // keys still to take among those that share them
  int32_t mode;             // 0: the list serves; 1: the later launches stream the matrices
  uint32_t thr;             // threshold key, and how many of the keys equal to it are taken
  int32_t need_eq;
  int32_t overflow;         // a block of the compact pass ran out of room
  int32_t pad;
};
constexpr int SR_STATE_INTS = 8;
static_assert(sizeof(SrState) == SR_STATE_INTS * 4, "the state has its place in the workspace");
// histograms, zero between calls: of the sample and of all elements (SR_REPL copies each), of the
// list (copies of 512 bins), then coarse and fine
enum { H_SAMPLE, H_ALL, H_COUNT };
constexpr int SR_HIST = SR_REPL * SR_BINS;
constexpr int SR_LIST_BINS = 512, H_LIST_AT = H_COUNT * SR_HIST;
constexpr int SR_HIST_INTS = H_LIST_AT + SR_REPL * SR_LIST_BINS + SR_COARSE + SR_FINE;

// capacity of the candidate list, in entries of 8 bytes
inline int64_t sr_list_cap(int64_t n) { return std::max<int64_t>(n / 6, 65536); }

// Chunks and list entries of the blocks of the compact pass.  Chunks are dealt in turn, so that some
// blocks take one more than the others; their regions are larger by a chunk's share.  (Equal regions:
// 512 blocks on 520 chunks, k = n / 12, sent every call to the streaming launches, 54 -> 41 us;
// fp32 77 -> 60 us.)
struct SrDeal {
  int64_t q, r, share;   // block b takes q chunks, one more if b < r; list entries per chunk
  __host__ __device__ int64_t chunks(int64_t b) const { return q + (b < r ? 1 : 0); }
  __host__ __device__ int64_t first(int64_t b) const { return (b * q + (b < r ? b : r)) * share; }
};

// The bin b with  above(b) < want <= above(b) + count(b)  (above: keys in higher bins) of a
// histogram that an earlier launch made in SR_REPL copies; every thread of the block gets it.
// False when fewer than `want` keys were counted.
__device__ __forceinline__ bool pick_bin(const int32_t* __restrict__ hist, int64_t want, int* bin,
                                         int32_t* above_out) {
  __shared__ int32_t wtot[SR_WAVES];
  __shared__ int32_t s_bin, s_above;
  constexpr int PER = SR_BINS / SR_THREADS;   // 8 consecutive bins per thread
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int4 q[SR_REPL][2];
#pragma unroll
  for (int r = 0; r < SR_REPL; ++r)
#pragma unroll
    for (int j = 0; j < 2; ++j)
      q[r][j] = *reinterpret_cast<const int4*>(hist + r * SR_BINS + tid * PER + 4 * j);
  int32_t c[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) c[j] = 0;
#pragma unroll
  for (int r = 0; r < SR_REPL; ++r)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      c[4 * j] += q[r][j].x; c[4 * j + 1] += q[r][j].y; c[4 * j + 2] += q[r][j].z; c[4 * j + 3] += q[r][j].w;
    }
  int sum = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) sum += c[j];
  int incl = sum;   // lane l: the sum of lanes l .. 63
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int t = __shfl_down(incl, off, 64);
    if (lane + off < 64) incl += t;
  }
  if (lane == 0) wtot[wave] = incl;
  if (tid == 0) s_bin = -1;
  __syncthreads();
  int above = incl - sum;
#pragma unroll
  for (int w = 0; w < SR_WAVES; ++w) above += w > wave ? wtot[w] : 0;
#pragma unroll
  for (int j = PER - 1; j >= 0; --j) {
    if (above < want && want <= above + c[j]) {   // at most one bin of the block
      s_bin = tid * PER + j;
      s_above = above;
    }
    above += c[j];
  }
  __syncthreads();
  *bin = s_bin;
  *above_out = s_above;
  return s_bin >= 0;
}

// The same when every thread holds one bin.  -1: fewer than `want` keys.
__device__ __forceinline__ int pick_512(int32_t mine, int32_t want, int32_t* above_out) {
  static_assert(SR_THREADS == 512, "a bin per thread");
  __shared__ int32_t wtot[SR_WAVES];
  __shared__ int32_t s_bin, s_above;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int incl = mine;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int t = __shfl_down(incl, off, 64);
    if (lane + off < 64) incl += t;
  }
  __syncthreads();   // the results of an earlier call have been read
  if (lane == 0) wtot[wave] = incl;
  if (tid == 0) { s_bin = -1; s_above = 0; }
  __syncthreads();
  int above = incl - mine;
#pragma unroll
  for (int w = 0; w < SR_WAVES; ++w) above += w > wave ? wtot[w] : 0;
  if (above < want && want <= above + mine) {
    s_bin = tid;
    s_above = above;
  }
  __syncthreads();
  *above_out = s_above;
  return s_bin;
}

// 16 elements per thread of one chunk in NV vectors of 16 bytes: vector v holds the elements
// v * 512 * V + tid * V .. + V - 1 of the chunk, so that every load instruction of a wavefront
// covers 1 KB without gaps.
template <typename T>
struct SrLane {
  static constexpr int V = 16 / (int)sizeof(T);
  static constexpr int NV = SR_PER_THREAD / V;
  uint4 w[NV], s[NV];
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  __device__ __forceinline__ static int64_t first(int64_t c, int v) {
    return c * SR_CHUNK + v * (SR_THREADS * V) + (int)threadIdx.x * V;
  }
  // ONCE: past the last-level cache (see sr_once)
  template <bool ONCE = false>
  __device__ __forceinline__ static uint4 load_vec(const T* __restrict__ p, int64_t i, int64_t n) {
    if (i + V <= n) {
      const u32x4* q = reinterpret_cast<const u32x4*>(p + i);
      const u32x4 r = ONCE ? __builtin_nontemporal_load(q) : *q;
      return make_uint4(r.x, r.y, r.z, r.w);
    }
    T e[V];   // the end of the array
#pragma unroll
    for (int j = 0; j < V; ++j) e[j] = i + j < n ? p[i + j] : T(0);
    uint4 q;
    __builtin_memcpy(&q, e, 16);
    return q;
  }
  template <bool ONCE = false>   // of W
  __device__ __forceinline__ void load(const T* __restrict__ W, const T* __restrict__ S, int64_t c,
                                       int64_t n) {
#pragma unroll
    for (int v = 0; v < NV; ++v) w[v] = load_vec<ONCE>(W, first(c, v), n);
#pragma unroll
    for (int v = 0; v < NV; ++v) s[v] = load_vec(S, first(c, v), n);
  }
  __device__ __forceinline__ void residual(int v, float (&r)[V]) const {
    float a[V], b[V];
    Vec16<T>::unpack(w[v], a);
    Vec16<T>::unpack(s[v], b);
#pragma unroll
    for (int e = 0; e < V; ++e) r[e] = a[e] - b[e];
  }
  // element j = v * V + e, j known at run time only: selected from the registers
  __device__ __forceinline__ float residual_of(int j) const {
    constexpr int PER = 4 / (int)sizeof(T);   // elements per 32-bit word
    uint32_t a = 0, b = 0;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const uint32_t wv[4] = {w[v].x, w[v].y, w[v].z, w[v].w}, sv[4] = {s[v].x, s[v].y, s[v].z, s[v].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool hit = j / PER == v * 4 + i;
        a = hit ? wv[i] : a;
        b = hit ? sv[i] : b;
      }
    }
    if (PER == 2) {   // bf16: the high or the low half
      a = (j & 1) ? a & 0xffff0000u : a << 16;
      b = (j & 1) ? b & 0xffff0000u : b << 16;
    }
    return __uint_as_float(a) - __uint_as_float(b);
  }
};
__device__ __forceinline__ uint32_t key_of(float r) { return __float_as_uint(r) & 0x7fffffffu; }

// Inclusive prefix sum over the wavefront, with data-parallel moves instead of LDS permutes (the pass 59.3 ->
// 57.9 us): inside rows of 16 lanes, then a row's last lane to the rows after it.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t add_moved(uint32_t v) {
  return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
  v = add_moved<0x111, 0xf>(v);   // row_shr 1, 2, 4, 8
  v = add_moved<0x112, 0xf>(v);
  v = add_moved<0x114, 0xf>(v);
  v = add_moved<0x118, 0xf>(v);
  v = add_moved<0x142, 0xa>(v);   // row_bcast 15 into rows 1 and 3
  return add_moved<0x143, 0xc>(v);   // row_bcast 31 into rows 2 and 3
}
__device__ __forceinline__ unsigned long long wave_scan(unsigned long long v) {   // halves never carry
  return (unsigned long long)wave_scan((uint32_t)(v >> 32)) << 32 | wave_scan((uint32_t)v);
}

// Per-vector counts of a thread packed into one integer (16 bits each, a vector has at most 4096
// elements in the block): exclusive prefix over the block and total of all of them in one scan.
// `slot` alternates between two LDS rows, so that one barrier per scan is enough.
template <int NV>
struct BlockScan {
  typedef typename std::conditional<NV == 2, uint32_t, unsigned long long>::type word;
  static_assert(NV == 2 || NV == 4, "16 bits per vector");
  word before, total;
  __device__ __forceinline__ void run(word mine, word (*wsum)[SR_WAVES], int slot) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const word incl = wave_scan(mine);
    if (lane == 63) wsum[slot][wave] = incl;
    __syncthreads();
    before = incl - mine;
    total = 0;
#pragma unroll
    for (int w = 0; w < SR_WAVES; ++w) {
      const word t = wsum[slot][w];
      before += w < wave ? t : 0;
      total += t;
    }
  }
  __device__ __forceinline__ static int part(word p, int v) { return (int)((p >> (16 * v)) & 0xffff); }
};

// LDS histogram -> one of its global copies.
__device__ __forceinline__ void flush_hist(const int32_t* h, int nb, int32_t* hist,
                                           int pitch = SR_BINS) {
  int32_t* mine = hist + ((int)blockIdx.x % SR_REPL) * pitch;
  for (int i = threadIdx.x; i < nb; i += SR_THREADS)
    if (h[i] != 0) atomicAdd(&mine[i], h[i]);
}

// ---- step 1.  Segment i of the sample is 128 bytes: eight lanes, 16 bytes each.
template <typename T>
__global__ __launch_bounds__(SR_THREADS) void sr_sample_kernel(const T* __restrict__ W,
                                                               const T* __restrict__ S,
                                                               int64_t rate, int64_t n_sample,
                                                               int32_t* __restrict__ hist) {
  __shared__ int32_t h[SR_BINS];
  constexpr int V = 16 / (int)sizeof(T), SEG = 8 * V;
  for (int i = threadIdx.x; i < SR_BINS; i += SR_THREADS) h[i] = 0;
  __syncthreads();
  const int64_t gid = (int64_t)blockIdx.x * SR_THREADS + threadIdx.x;
  for (int64_t i = gid >> 3; i < n_sample; i += (int64_t)gridDim.x * (SR_THREADS / 8)) {
    const int64_t seg = i * rate + (uint32_t)(i * 2654435761u >> 7) % (uint32_t)rate;
    const int64_t e0 = seg * SEG + (gid & 7) * V;
    float a[V], b[V];
    Vec16<T>::load(W + e0, a);
    Vec16<T>::load(S + e0, b);
#pragma unroll
    for (int e = 0; e < V; ++e) atomicAdd(&h[key_of(a[e] - b[e]) >> 19], 1);
  }
  __syncthreads();
  flush_hist(h, SR_BINS, hist);
}

// The bin b_lo of the sample's histogram: the expected number of sampled keys among the k largest,
// 6 % (a bin is 6 % wide: what a matrix that is not the same everywhere may be off by) and eight
// standard deviations more.  Everything was sampled when rate == 1.
__device__ __forceinline__ uint32_t pick_b_lo(const int32_t* __restrict__ hist, int64_t n, int64_t k,
                                              int64_t rate, int64_t sampled) {
  const double share = (double)k * (double)sampled / (double)n;
  const int64_t want = rate == 1 ? k : (int64_t)(1.06 * share + 8.0 * sqrt(share) + 8.0);
  int bin;
  int32_t above;
  // at most the bin of infinity: the bins above it hold NaN keys only, and a NaN is no bound that a
  // finite residual could be compared with
  return pick_bin(hist, want, &bin, &above) ? min((uint32_t)bin, SR_INF_BIN) : 0u;
}

// ---- step 2.
template <typename T, bool ONCE>
__global__ __launch_bounds__(SR_THREADS) void sr_compact_kernel(
    const T* __restrict__ W, const T* __restrict__ S, int64_t n, int64_t k, int64_t rate,
    int64_t n_sample, SrState* __restrict__ st, int32_t* __restrict__ hists, SrDeal deal,
    uint2* __restrict__ list, int32_t* __restrict__ run_start, int32_t* __restrict__ run_cnt) {
  typedef SrLane<T> Lane;
  constexpr int V = Lane::V, NV = Lane::NV;
  typedef BlockScan<NV> Scan;
  __shared__ int32_t h[SR_LIST_BINS];
  __shared__ typename Scan::word wsum[2][SR_WAVES];
  const int64_t n_chunks = (n + SR_CHUNK - 1) / SR_CHUNK;
  Lane cur;
  if ((int64_t)blockIdx.x < n_chunks) cur.template load<ONCE>(W, S, blockIdx.x, n);
  static_assert(SR_LIST_BINS == SR_THREADS, "a bin per thread");
  h[threadIdx.x] = 0;
  const uint32_t b_lo = pick_b_lo(hists + H_SAMPLE * SR_HIST, n, k, rate, n_sample * (8 * V));
  if (blockIdx.x == 0 && threadIdx.x == 0) st->b_lo = b_lo;
  const float least = __uint_as_float(b_lo << 19);   // magnitudes below it are not listed (a NaN is)
  // the list has fewer than 2^31 / 6 entries
  const int region = (int)deal.first(blockIdx.x), room = (int)(deal.chunks(blockIdx.x) * deal.share);
  int used = 0;   // entries of this block's region in use (the same in every thread)
  int slot = 0;
  for (int64_t c = blockIdx.x; c < n_chunks; c += gridDim.x) {
    Lane nxt = cur;
    if (c + gridDim.x < n_chunks) nxt.template load<ONCE>(W, S, c + gridDim.x, n);   // in flight meanwhile
    uint32_t sel = 0;   // bit j = v * V + e
    typename Scan::word mine = 0;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      float r[V];
      cur.residual(v, r);
      uint32_t m = 0;
#pragma unroll
      for (int e = V - 1; e >= 0; --e) m = (m << 1) | (fabsf(r[e]) < least ? 0u : 1u);
      if ((c + 1) * SR_CHUNK > n)   // the last chunk
        m &= (1u << (int)max((int64_t)0, min((int64_t)V, n - Lane::first(c, v)))) - 1u;
      sel |= m << (v * V);
      mine += (typename Scan::word)__popc(m) << (16 * v);
    }
    Scan sc;
    sc.run(mine, wsum, slot);
    slot ^= 1;
    int total = 0, first[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      first[v] = total + Scan::part(sc.before, v);
      total += Scan::part(sc.total, v);
    }
    const bool fits = used + total <= room;
    const int run0 = region + used;
    if (threadIdx.x == 0) {
      run_start[c] = fits ? run0 : 0;
      run_cnt[c] = fits ? total : 0;
      if (!fits) st->overflow = 1;
    }
    // few of the 16 elements are listed: a loop over the set bits (two or three rounds for a
    // wavefront) instead of 16 divergent blocks
    for (uint32_t rest = sel; rest != 0; rest &= rest - 1) {
      const int j = __ffs(rest) - 1, v = j / V;
      const float r = cur.residual_of(j);
      atomicAdd(&h[min((key_of(r) >> 18) - (b_lo << 1), (uint32_t)SR_LIST_BINS - 1)], 1);
      int f = first[0];
#pragma unroll
      for (int u = 1; u < NV; ++u) f = v == u ? first[u] : f;
      const int rank = __popc(sel & ((1u << j) - 1u) & (((1u << V) - 1u) << (v * V)));
      if (fits)
        list[run0 + f + rank] = make_uint2(__float_as_uint(r), (uint32_t)(Lane::first(c, v) + j % V));
    }
    if (fits) used += total;
    cur = nxt;
  }
  __syncthreads();
  flush_hist(h, SR_LIST_BINS, hists + H_LIST_AT, SR_LIST_BINS);
}

// mode 1: f(residual, index) for every element of the matrices, chunks dealt to the blocks.
template <typename T, typename F>
__device__ __forceinline__ void each_element(const T* __restrict__ W, const T* __restrict__ S,
                                             int64_t n, F&& f) {
  typedef SrLane<T> Lane;
  const int64_t n_chunks = (n + SR_CHUNK - 1) / SR_CHUNK;
  for (int64_t c = blockIdx.x; c < n_chunks; c += gridDim.x) {
    Lane L;
    L.load(W, S, c, n);
#pragma unroll
    for (int v = 0; v < Lane::NV; ++v) {
      float r[Lane::V];
      L.residual(v, r);
#pragma unroll
      for (int e = 0; e < Lane::V; ++e)
        if (Lane::first(c, v) + e < n) f(r[e]);
    }
  }
}

// Counts of the low key bits, in LDS first: few distinct keys may be hit very often (differences of
// bf16 values have few mantissa bits, a quantised residual has few values at all; 15 000 global
// atomics on a few addresses took 130 us).  A table of 2048 (low bits, count) slots, addressed by
// a hash; a key that finds its slot taken by another one goes to global memory directly.
struct LowCounter {
  static constexpr int SLOTS = SR_BINS / 2;
  int32_t* tag;
  int32_t* num;
  int32_t* coarse;
  int32_t* fine;
  __device__ __forceinline__ LowCounter(int32_t* lds, int32_t* c, int32_t* f)
      : tag(lds), num(lds + SLOTS), coarse(c), fine(f) {
    for (int i = threadIdx.x; i < SLOTS; i += SR_THREADS) {
      tag[i] = -1;
      num[i] = 0;
    }
    __syncthreads();
  }
  __device__ __forceinline__ void add(int low) {
    const int slot = (int)((uint32_t)low * 2654435761u >> 21);
    const int old = atomicCAS(&tag[slot], -1, low);
    if (old == -1 || old == low) {
      atomicAdd(&num[slot], 1);
    } else {
      atomicAdd(&coarse[low >> 9], 1);
      atomicAdd(&fine[low], 1);
    }
  }
  __device__ __forceinline__ void flush() {
    __syncthreads();
    for (int i = threadIdx.x; i < SLOTS; i += SR_THREADS)
      if (num[i] != 0) {
        atomicAdd(&coarse[tag[i] >> 9], num[i]);
        atomicAdd(&fine[tag[i]], num[i]);
      }
  }
};

// The threshold key from the counts of the low bits (an earlier launch made them): `bin` holds the
// bits above them; *need_eq = keys equal to it that are taken.
__device__ __forceinline__ uint32_t pick_threshold(const int32_t* __restrict__ coarse,
                                                   const int32_t* __restrict__ fine, int mode,
                                                   uint32_t bin, int32_t want, int32_t* need_eq) {
  const int tid = threadIdx.x;
  const int2 c = reinterpret_cast<const int2*>(coarse)[tid];
  int32_t a;
  int hi = 2 * max(0, pick_512(c.x + c.y, want, &a));
  const int32_t upper = coarse[hi + 1];
  if (want - a <= upper) {
    ++hi;
  } else {
    a += upper;
  }
  want -= a;
  const int lo = max(0, pick_512(fine[hi * 512 + tid], want, &a));
  *need_eq = want - a;
  return (bin << (mode == 0 ? 18 : 19)) | (uint32_t)(hi * 512 + lo);
}

// f(lane's entry, whether it exists) for the entries of a run in order, 64 at a time; 256 are
// requested together (a run holds about 8192 k / n of them).
template <typename F>
__device__ __forceinline__ void each_entry(const uint2* __restrict__ run, int cnt, F&& f) {
  const int lane = threadIdx.x & 63;
  for (int i0 = 0; i0 < cnt; i0 += 256) {
    uint2 en[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) en[u] = run[min(i0 + u * 64 + lane, cnt - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i0 + u * 64 < cnt) f(en[u], i0 + u * 64 + lane < cnt);
  }
}

// Chunks of the list dealt to the wavefronts of the launch.
template <typename F>
__device__ __forceinline__ void each_run(int64_t n_chunks, F&& f) {
  const int wave = threadIdx.x >> 6;
  for (int64_t c = (int64_t)blockIdx.x * SR_WAVES + wave; c < n_chunks;
       c += (int64_t)gridDim.x * SR_WAVES)
    f(c);
}

// ---- step 3.
template <typename T>
__global__ __launch_bounds__(SR_THREADS) void sr_fine_kernel(
    const T* __restrict__ W, const T* __restrict__ S, int64_t n, int64_t k,
    SrState* __restrict__ st, int32_t* __restrict__ hists, int32_t* __restrict__ coarse,
    int32_t* __restrict__ fine, const uint2* __restrict__ list,
    const int32_t* __restrict__ run_start, const int32_t* __restrict__ run_cnt) {
  __shared__ int32_t h[SR_BINS];
  int32_t listed = 0, above;
#pragma unroll
  for (int r = 0; r < SR_REPL; ++r) listed += hists[H_LIST_AT + r * SR_LIST_BINS + threadIdx.x];
  const int rel = pick_512(listed, (int32_t)k, &above);
  const int mode = rel >= 0 && rel < SR_LIST_BINS - 1 && st->overflow == 0 ? 0 : 1;
  const uint32_t bin = (uint32_t)rel + (st->b_lo << 1);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->mode = mode;
    st->bin = bin;
    st->k_rem = (int32_t)k - above;
  }
  if (mode != 0) {
    for (int i = threadIdx.x; i < SR_BINS; i += SR_THREADS) h[i] = 0;
    __syncthreads();
    each_element(W, S, n, [&](float r) { atomicAdd(&h[key_of(r) >> 19], 1); });
    __syncthreads();
    flush_hist(h, SR_BINS, hists + H_ALL * SR_HIST);
    return;
  }
  LowCounter low(h, coarse, fine);
  each_run((n + SR_CHUNK - 1) / SR_CHUNK, [&](int64_t c) {
    each_entry(list + run_start[c], run_cnt[c], [&](const uint2& en, bool valid) {
      const uint32_t key = en.x & 0x7fffffffu;
      if (valid && (key >> 18) == bin) low.add((int)(key & 0x3ffffu));
    });
  });
  low.flush();
}

// ---- step 4.  cnt[c] = keys of chunk c above the threshold, keys equal to it.
template <typename T>
__global__ __launch_bounds__(SR_THREADS) void sr_count_kernel(
    const T* __restrict__ W, const T* __restrict__ S, int64_t n, int64_t k,
    SrState* __restrict__ st, const int32_t* __restrict__ hists, int32_t* __restrict__ coarse,
    int32_t* __restrict__ fine, int2* __restrict__ cnt_out, const uint2* __restrict__ list,
    const int32_t* __restrict__ run_start, const int32_t* __restrict__ run_cnt) {
  if (st->mode != 0) {
    __shared__ int32_t h[SR_BINS];
    int bin;
    int32_t above;
    pick_bin(hists + H_ALL * SR_HIST, k, &bin, &above);   // k <= n: always found
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      st->bin = (uint32_t)bin;
      st->k_rem = (int32_t)k - above;
    }
    LowCounter low(h, coarse, fine);
    each_element(W, S, n, [&](float r) {
      if ((key_of(r) >> 19) == (uint32_t)bin) low.add((int)(key_of(r) & 0x7ffffu));
    });
    low.flush();
    return;
  }
  const int lane = threadIdx.x & 63;
  int32_t need_eq;
  const uint32_t thr = pick_threshold(coarse, fine, 0, st->bin, st->k_rem, &need_eq);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->thr = thr;
    st->need_eq = need_eq;
  }
  each_run((n + SR_CHUNK - 1) / SR_CHUNK, [&](int64_t c) {
    int gt = 0, eq = 0;
    each_entry(list + run_start[c], run_cnt[c], [&](const uint2& en, bool valid) {
      const uint32_t key = en.x & 0x7fffffffu;
      gt += valid && key > thr;
      eq += valid && key == thr;
    });
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      gt += __shfl_xor(gt, off, 64);
      eq += __shfl_xor(eq, off, 64);
    }
    if (lane == 0) cnt_out[c] = make_int2(gt, eq);
  });
}

// Keys above / equal to the threshold in the chunks before the block's first one, and before each
// of its `m` chunks c0 .. (in LDS: start[j]); called by the whole block, m <= SR_EMIT_MAX.
constexpr int SR_EMIT_MAX = 512;
__device__ __forceinline__ void emit_starts(const int2* __restrict__ cnt, int64_t c0, int m,
                                            int2* start) {
  __shared__ int2 wred[SR_WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int gt = 0, eq = 0;
  int64_t i = tid;
  for (; i + 7 * SR_THREADS < c0; i += 8 * SR_THREADS) {   // 8 loads in flight
    int2 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = cnt[i + u * SR_THREADS];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      gt += v[u].x;
      eq += v[u].y;
    }
  }
  for (; i < c0; i += SR_THREADS) {
    const int2 v = cnt[i];
    gt += v.x;
    eq += v.y;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    gt += __shfl_xor(gt, off, 64);
    eq += __shfl_xor(eq, off, 64);
  }
  if (lane == 0) wred[wave] = make_int2(gt, eq);
  __syncthreads();
  int2 base = make_int2(0, 0);
#pragma unroll
  for (int w = 0; w < SR_WAVES; ++w) {
    base.x += wred[w].x;
    base.y += wred[w].y;
  }
  if (wave == 0) {   // exclusive prefix over the block's own chunks
    for (int j0 = 0; j0 < m; j0 += 64) {
      const int2 v = j0 + lane < m ? cnt[c0 + j0 + lane] : make_int2(0, 0);
      int2 incl = v;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const int tx = __shfl_up(incl.x, off, 64), ty = __shfl_up(incl.y, off, 64);
        if (lane >= off) { incl.x += tx; incl.y += ty; }
      }
      if (j0 + lane < m) start[j0 + lane] = make_int2(base.x + incl.x - v.x, base.y + incl.y - v.y);
      base.x += __shfl(incl.x, 63, 64);
      base.y += __shfl(incl.y, 63, 64);
    }
  }
  __syncthreads();
}

// mode 1: counts of a chunk from the matrices (a block per chunk).
template <typename T>
__device__ __forceinline__ void count_chunks(const T* __restrict__ W, const T* __restrict__ S,
                                             int64_t n, uint32_t thr, int2* __restrict__ cnt_out) {
  typedef SrLane<T> Lane;
  __shared__ int2 red[SR_WAVES];
  const int64_t n_chunks = (n + SR_CHUNK - 1) / SR_CHUNK;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int64_t c = blockIdx.x; c < n_chunks; c += gridDim.x) {
    Lane L;
    L.load(W, S, c, n);
    int gt = 0, eq = 0;
#pragma unroll
    for (int v = 0; v < Lane::NV; ++v) {
      float r[Lane::V];
      L.residual(v, r);
#pragma unroll
      for (int e = 0; e < Lane::V; ++e)
        if (Lane::first(c, v) + e < n) {
          gt += key_of(r[e]) > thr;
          eq += key_of(r[e]) == thr;
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      gt += __shfl_xor(gt, off, 64);
      eq += __shfl_xor(eq, off, 64);
    }
    if (lane == 0) red[wave] = make_int2(gt, eq);
    __syncthreads();
    if (threadIdx.x == 0) {
      int2 t = make_int2(0, 0);
      for (int w = 0; w < SR_WAVES; ++w) {
        t.x += red[w].x;
        t.y += red[w].y;
      }
      cnt_out[c] = t;
    }
    __syncthreads();
  }
}

// ---- step 5.  Block b writes the entries of the chunks [b * per, (b + 1) * per).
template <typename T>
__global__ __launch_bounds__(SR_THREADS) void sr_emit_kernel(
    const T* __restrict__ W, const T* __restrict__ S, int64_t n, SrState* __restrict__ st,
    const int32_t* __restrict__ coarse, const int32_t* __restrict__ fine, int2* __restrict__ cnt,
    int per, int64_t k, T* __restrict__ values, int32_t* __restrict__ indices,
    const uint2* __restrict__ list, const int32_t* __restrict__ run_start,
    const int32_t* __restrict__ run_cnt) {
  if (st->mode != 0) {
    int32_t need_eq;
    const uint32_t thr = pick_threshold(coarse, fine, 1, st->bin, st->k_rem, &need_eq);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      st->thr = thr;
      st->need_eq = need_eq;
    }
    count_chunks(W, S, n, thr, cnt);
    return;
  }
  __shared__ int2 start[SR_EMIT_MAX];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t n_chunks = (n + SR_CHUNK - 1) / SR_CHUNK;
  const int64_t c0 = (int64_t)blockIdx.x * per;
  if (c0 >= n_chunks) return;
  const int m = (int)min((int64_t)per, n_chunks - c0);
  emit_starts(cnt, c0, m, start);
  const uint32_t thr = st->thr;
  const int32_t need_eq = st->need_eq;
  const unsigned long long below = (1ull << lane) - 1ull;
  for (int j = wave; j < m; j += SR_WAVES) {
    int eq_rank = start[j].y;
    int64_t pos = (int64_t)start[j].x + min(eq_rank, need_eq);
    // ranks by ballot: lane order = index order
    each_entry(list + run_start[c0 + j], run_cnt[c0 + j], [&](const uint2& en, bool valid) {
      const uint32_t key = en.x & 0x7fffffffu;
      const bool iseq = valid && key == thr;
      const unsigned long long eqm = __ballot(iseq);
      const bool sel = valid && (key > thr || (iseq && eq_rank + __popcll(eqm & below) < need_eq));
      const unsigned long long sm = __ballot(sel);
      const int64_t p = pos + __popcll(sm & below);
      if (sel && p < k) {   // p < k always holds when the counts are consistent
        values[p] = from_f32<T>(__uint_as_float(en.x));
        indices[p] = (int32_t)en.y;
      }
      eq_rank += __popcll(eqm);
      pos += __popcll(sm);
    });
  }
}

// mode 1: the value-index list from the matrices (a block per chunk of its range).  Both modes:
// clears the histograms and the overflow flag for the next call.
template <typename T>
__global__ __launch_bounds__(SR_THREADS) void sr_emit_stream_kernel(
    const T* __restrict__ W, const T* __restrict__ S, int64_t n, SrState* __restrict__ st,
    int32_t* __restrict__ hists, const int2* __restrict__ cnt_in, int per, int64_t k,
    T* __restrict__ values, int32_t* __restrict__ indices) {
  typedef SrLane<T> Lane;
  constexpr int V = Lane::V, NV = Lane::NV;
  typedef BlockScan<NV> Scan;
  __shared__ int2 start[SR_EMIT_MAX];
  __shared__ typename Scan::word wsum[2][SR_WAVES];
  static_assert(SR_HIST_INTS % 4 == 0, "cleared 16 bytes at a time");
  for (int i = blockIdx.x * SR_THREADS + threadIdx.x; i < SR_HIST_INTS / 4; i += gridDim.x * SR_THREADS)
    reinterpret_cast<int4*>(hists)[i] = make_int4(0, 0, 0, 0);
  if (blockIdx.x == 0 && threadIdx.x == 0) st->overflow = 0;
  if (st->mode == 0) return;
  const int64_t n_chunks = (n + SR_CHUNK - 1) / SR_CHUNK;
  const int64_t c0 = (int64_t)blockIdx.x * per;
  if (c0 >= n_chunks) return;
  const int m = (int)min((int64_t)per, n_chunks - c0);
  emit_starts(cnt_in, c0, m, start);
  const uint32_t thr = st->thr;
  const int32_t need_eq = st->need_eq;
  for (int j = 0; j < m; ++j) {
    const int64_t c = c0 + j;
    Lane L;
    L.load(W, S, c, n);
    typename Scan::word mine = 0;
    uint32_t eqm[NV], sel[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      float r[V];
      L.residual(v, r);
      eqm[v] = sel[v] = 0;
#pragma unroll
      for (int e = 0; e < V; ++e)
        if (Lane::first(c, v) + e < n) {
          if (key_of(r[e]) == thr) eqm[v] |= 1u << e;
          if (key_of(r[e]) > thr) sel[v] |= 1u << e;
        }
      mine += (typename Scan::word)__popc(eqm[v]) << (16 * v);
    }
    Scan sc;
    sc.run(mine, wsum, 0);
    int rank = start[j].y;   // of the thread's first equal key of vector v
    mine = 0;
    int ahead = 0;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      int q = rank + ahead + Scan::part(sc.before, v);
#pragma unroll
      for (int e = 0; e < V; ++e)
        if ((eqm[v] >> e) & 1u) {
          if (q < need_eq) sel[v] |= 1u << e;
          ++q;
        }
      ahead += Scan::part(sc.total, v);
      mine += (typename Scan::word)__popc(sel[v]) << (16 * v);
    }
    sc.run(mine, wsum, 1);
    int64_t pos = (int64_t)start[j].x + min(start[j].y, need_eq);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      int64_t p = pos + Scan::part(sc.before, v);
      float r[V];
      L.residual(v, r);
#pragma unroll
      for (int e = 0; e < V; ++e)
        if ((sel[v] >> e) & 1u) {
          if (p < k) {   // always true when the counts are consistent
            values[p] = from_f32<T>(r[e]);
            indices[p] = (int32_t)(Lane::first(c, v) + e);
          }
          ++p;
        }
      pos += Scan::part(sc.total, v);
    }
    __syncthreads();
  }
}

// Decode: out = shared, plus the residual where the list has an entry.  A block takes one chunk:
// it requests its piece of the shared expert first, finds the chunk's contiguous piece of the
// ascending list with a 64-wide search while those loads are in flight, puts the values into LDS
// with a bit per element (untouched elements keep the shared expert's exact bits), and writes.
template <typename T, bool ONCE>
__global__ __launch_bounds__(SR_THREADS) void sr_decode_kernel(
    const T* __restrict__ S, const T* __restrict__ values, const int32_t* __restrict__ indices,
    int64_t n, int64_t k, T* __restrict__ out) {
  typedef SrLane<T> Lane;
  constexpr int V = Lane::V, NV = Lane::NV;
  __shared__ T res[SR_CHUNK];
  __shared__ uint32_t has[SR_CHUNK / 32];
  __shared__ int64_t range[2];
  const int64_t c = blockIdx.x, start = c * SR_CHUNK, end = min(n, start + SR_CHUNK);
  uint4 q[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) q[v] = Lane::load_vec(S, Lane::first(c, v), n);
  if (threadIdx.x < 128) {   // lower_bound of start (wavefront 0) / end (wavefront 1), 64 probes
                             // per round (4 rounds for a million entries)
    const int lane = threadIdx.x & 63;
    const int64_t target = threadIdx.x < 64 ? start : end;
    int64_t lo = 0, hi = k;
    while (hi > lo) {
      const int64_t stride = (hi - lo + 63) / 64;
      const int64_t pos = lo + lane * stride;
      const bool below = pos < hi && (int64_t)indices[pos] < target;
      const int m = __popcll(__ballot(below));   // probes 0..m-1 are below the target
      if (m == 0) {
        hi = lo;
      } else {
        hi = min(hi, lo + m * stride);           // probe m (if any) is not below
        lo = lo + (m - 1) * stride + 1;
      }
    }
    if (lane == 0) range[threadIdx.x >> 6] = lo;
  } else if (threadIdx.x < 128 + SR_CHUNK / 32) {
    has[threadIdx.x - 128] = 0;
  }
  __syncthreads();
  for (int64_t e = range[0] + threadIdx.x; e < range[1]; e += SR_THREADS) {
    const int64_t i = (int64_t)indices[e] - start;
    if (i >= 0 && i < SR_CHUNK) {   // the list is the caller's: stay inside the chunk
      res[i] = values[e];
      atomicOr(&has[i >> 5], 1u << (i & 31));
    }
  }
  __syncthreads();
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int l0 = v * (SR_THREADS * V) + (int)threadIdx.x * V;
    const uint32_t bits = (has[l0 >> 5] >> (l0 & 31)) & ((1u << V) - 1u);
    T o[V];
    __builtin_memcpy(o, &q[v], 16);
    if (bits != 0) {
#pragma unroll
      for (int e = 0; e < V; ++e)
        if ((bits >> e) & 1u) o[e] = from_f32<T>(to_f32(o[e]) + to_f32(res[l0 + e]));
    }
    const int64_t i0 = start + l0;
    if (i0 + V <= n) {
      typename Lane::u32x4 r;
      __builtin_memcpy(&r, o, 16);
      if (ONCE) __builtin_nontemporal_store(r, reinterpret_cast<typename Lane::u32x4*>(out + i0));
      else *reinterpret_cast<typename Lane::u32x4*>(out + i0) = r;
    } else {
#pragma unroll
      for (int e = 0; e < V; ++e)
        if (i0 + e < n) out[i0 + e] = o[e];
    }
  }
}

// From two matrices of 32 MB on, the expert's is read past the last-level cache (256 MB) and the rebuilt one written
// past it; the shared one, which the next expert's encode or decode reads again, is not.  Plain -> all three past the
// cache -> this, us:
//   one of eight experts encoded in a row, 42, 64, 117 MB a matrix: 47.0, 58.0, 77.5 -> 47.7, 59.2, 81.1 -> 46.1, 56.7, 76.0;
//   fp32, 235 MB: 195 -> 182 -> 173
//   decoded in a row, 42, 64, 117 MB: 24.4, 33.3, 55.3 -> 21.2, 28.9, 49.4 -> 20.3, 28.7, 49.3
//   an expert's three matrices decoded and the expert computed for 8 tokens, 34, 42, 67, 117 MB: 87, 112, 156, 261 -> 84, 111,
//   151, 244 -> 83, 109, 152, 245; four experts decoded, then computed: 92, 118, 161, 257 -> 80, 111, 151, 243 -> 84, 109, 148,
//   245.  (Where nothing but a copy of it follows a decode, 42 to 64 MB lose 1 %.)
//   17 MB, plain -> past the cache, three matrices in turn, which it holds: 41.7 -> 42.0
bool sr_once(int64_t n, size_t elem) { return 2 * n * (int64_t)elem >= (int64_t)64 << 20; }

// blocks of the launches that deal chunks out: two per compute unit
int64_t sr_list_blocks(int64_t n_chunks, int n_cu) { return std::min<int64_t>(n_chunks, 2 * (int64_t)n_cu); }
SrDeal sr_deal(int64_t n_chunks, int64_t blocks, int64_t n) {
  return {n_chunks / blocks, n_chunks % blocks, sr_list_cap(n) / n_chunks};
}

// A new workspace: state and histograms are zero on entry of every encode (its last launch leaves them
// so).  The rest is written before it is read.
__global__ __launch_bounds__(SR_THREADS) void sr_clear_kernel(int4* __restrict__ ws) {
  static_assert((SR_STATE_INTS + SR_HIST_INTS) % 4 == 0, "cleared 16 bytes at a time");
  const int i = blockIdx.x * SR_THREADS + threadIdx.x;
  if (i < (SR_STATE_INTS + SR_HIST_INTS) / 4) ws[i] = make_int4(0, 0, 0, 0);
}

template <typename T>
int encode_t(moe_ctx* c, const T* W, const T* S, int64_t n, int64_t k, T* values, int32_t* indices,
             hipStream_t s) {
  const int64_t n_chunks = (n + SR_CHUNK - 1) / SR_CHUNK;
  const int64_t nc2 = (n_chunks + 3) & ~(int64_t)3;   // keeps the arrays 16-byte aligned
  SrState* st = reinterpret_cast<SrState*>(c->d_sr_ws);
  int32_t* hists = c->d_sr_ws + SR_STATE_INTS;   // zero on entry: at allocation, and by the last launch
  int32_t* coarse = hists + H_LIST_AT + SR_REPL * SR_LIST_BINS;
  int32_t* fine = coarse + SR_COARSE;
  int2* cnt = reinterpret_cast<int2*>(fine + SR_FINE);
  int32_t* run_start = reinterpret_cast<int32_t*>(cnt + nc2);
  int32_t* run_cnt = run_start + nc2;
  uint2* list = reinterpret_cast<uint2*>(run_cnt + nc2);
  const int cu = c->n_cu;
  const int64_t seg = 128 / (int64_t)sizeof(T), n_seg = n / seg;
  const int64_t rate = std::max<int64_t>(1, n / SR_SAMPLE), n_sample = n_seg / rate;
  auto grid = [&](int64_t work, int most) { return dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>(work, most))); };
  const dim3 g_sample = grid((n_sample * 8 + SR_THREADS - 1) / SR_THREADS, cu / 2);
  const dim3 g_list((unsigned)sr_list_blocks(n_chunks, cu));
  const SrDeal deal = sr_deal(n_chunks, g_list.x, n);
  // chunks per block of the emit steps: four blocks per compute unit, at most SR_EMIT_MAX chunks each
  const int per = (int)std::max<int64_t>(1, std::min<int64_t>(SR_EMIT_MAX, (n_chunks + cu * 4 - 1) / (cu * 4)));
  const dim3 g_emit((unsigned)((n_chunks + per - 1) / per));
#define SR_LAUNCH_AS(kern, g, ...) hipLaunchKernelGGL(kern, g, dim3(SR_THREADS), 0, s, __VA_ARGS__)
#define SR_LAUNCH(kern, g, ...) SR_LAUNCH_AS((kern<T>), g, __VA_ARGS__)
  SR_LAUNCH(sr_sample_kernel, g_sample, W, S, rate, n_sample, hists + H_SAMPLE * SR_HIST);
  SR_LAUNCH_AS((sr_once(n, sizeof(T)) ? sr_compact_kernel<T, true> : sr_compact_kernel<T, false>), g_list, W, S, n, k,
               rate, n_sample, st, hists, deal, list, run_start, run_cnt);
  SR_LAUNCH(sr_fine_kernel, g_list, W, S, n, k, st, hists, coarse, fine, list, run_start, run_cnt);
  SR_LAUNCH(sr_count_kernel, g_list, W, S, n, k, st, hists, coarse, fine, cnt, list, run_start, run_cnt);
  SR_LAUNCH(sr_emit_kernel, g_emit, W, S, n, st, coarse, fine, cnt, per, k, values, indices, list,
            run_start, run_cnt);
  SR_LAUNCH(sr_emit_stream_kernel, g_emit, W, S, n, st, hists, cnt, per, k, values, indices);
#undef SR_LAUNCH
#undef SR_LAUNCH_AS
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_EHIP;
}

template <typename T>
int decode_t(const T* S, const T* values, const int32_t* indices, int64_t n, int64_t k, T* out, hipStream_t s) {
  const dim3 grid((unsigned)((n + SR_CHUNK - 1) / SR_CHUNK));
  auto kern = sr_once(n, sizeof(T)) ? sr_decode_kernel<T, true> : sr_decode_kernel<T, false>;
  hipLaunchKernelGGL(kern, grid, dim3(SR_THREADS), 0, s, S, values, indices, n, k, out);
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_EHIP;
}

}  // namespace

// Not part of the interface: the list region of one block of an encode of n elements on n_cu compute
// units (*chunks, *first, *entries); returns the number of blocks and the list's room in *cap.  For the
// test of the rule, which needs no GPU.
extern "C" int moe_internal_sr_region(int64_t n, int32_t n_cu, int32_t block, int64_t* chunks, int64_t* first,
                                      int64_t* entries, int64_t* cap) {
  const int64_t n_chunks = (n + SR_CHUNK - 1) / SR_CHUNK;
  const int64_t blocks = sr_list_blocks(n_chunks, n_cu);
  const SrDeal deal = sr_deal(n_chunks, blocks, n);
  *chunks = deal.chunks(block);
  *first = deal.first(block);
  *entries = deal.chunks(block) * deal.share;
  *cap = sr_list_cap(n);
  return (int)blocks;
}

size_t sr_workspace_ints(int64_t n) {
  const int64_t n_chunks = (n + SR_CHUNK - 1) / SR_CHUNK;
  const int64_t nc2 = (n_chunks + 3) & ~(int64_t)3;
  // state, histograms, four integers per chunk, the candidate list (8 bytes per entry)
  return (size_t)(SR_STATE_INTS + SR_HIST_INTS + 4 * nc2 + 2 * sr_list_cap(n));
}

int launch_sr_clear(int32_t* ws, hipStream_t s) {
  const dim3 grid(((SR_STATE_INTS + SR_HIST_INTS) / 4 + SR_THREADS - 1) / SR_THREADS);
  hipLaunchKernelGGL(sr_clear_kernel, grid, dim3(SR_THREADS), 0, s, reinterpret_cast<int4*>(ws));
  return hipGetLastError() == hipSuccess ? MOE_OK : MOE_EHIP;
}

int launch_sr_encode(moe_ctx* c, const void* W, const void* S, int64_t n, int64_t k, void* values,
                     int32_t* indices, hipStream_t s) {
  if (c->cfg.dtype == MOE_BF16)
    return encode_t<uint16_t>(c, (const uint16_t*)W, (const uint16_t*)S, n, k, (uint16_t*)values,
                              indices, s);
  return encode_t<float>(c, (const float*)W, (const float*)S, n, k, (float*)values, indices, s);
}

int launch_sr_decode(moe_ctx* c, const void* S, const void* values, const int32_t* indices,
                     int64_t n, int64_t k, void* out, hipStream_t s) {
  if (c->cfg.dtype == MOE_BF16)
    return decode_t<uint16_t>((const uint16_t*)S, (const uint16_t*)values, indices, n, k, (uint16_t*)out, s);
  return decode_t<float>((const float*)S, (const float*)values, indices, n, k, (float*)out, s);
}
