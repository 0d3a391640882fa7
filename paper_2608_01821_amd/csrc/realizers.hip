// Pruning and merging evidence realizers (Sec. 4.3, "Compatible evidence
// realizers": pruning varies the retention ratio, merging the aggregation
// strength; the allocation policy is unchanged).  The paper gives neither
// criterion; the readings implemented here:
//   prune  token saliency = float64 L1 norm; per crop, level l keeps the n_l
//          most salient tokens (nested over levels), one member each;
//   merge  single linkage over the crop's 4-neighbour grid graph, edges
//          weighted by float64 cosine similarity, partition snapshotted when
//          n_l groups remain.
// n_l is the pooling pyramid's per-crop count, so every level costs the
// same as under pooling, and the levels go through the same CSR index maps.
//
// Three stages, each a kernel: keys (HBM-bound pass over v: one wavefront
// per token or grid edge, float64 accumulation), decisions (one 1024-thread
// workgroup per crop, everything in LDS: the keys are sorted; prune keeps a
// prefix; merge finds the minimum spanning tree of the ranked edges and takes
// components of its first edges, see merge_maps_kernel), and the level rows
// of every level in one launch (CSR means, float64 sums in member order,
// rounded once).

#include <mutex>
#include <string>

#include "common.h"

namespace davet {
namespace {

constexpr int RZ_NT = 1024;                                   // decision block
constexpr int RZ_MAXN = DAVET_MAX_REALIZER_GRID * DAVET_MAX_REALIZER_GRID;
constexpr int RZ_MAXE =
    2 * DAVET_MAX_REALIZER_GRID * (DAVET_MAX_REALIZER_GRID - 1);
constexpr int RZ_PER = RZ_MAXN / RZ_NT;                       // tokens/thread
static_assert(RZ_PER * RZ_NT == RZ_MAXN, "scan covers the largest crop");

struct LvlCnt { int n[DAVET_MAX_LEVELS]; };                   // per crop
struct MapPtrs {
  int32_t* offs[DAVET_MAX_LEVELS];
  int32_t* mem[DAVET_MAX_LEVELS];
};

// Eight consecutive features of one token as float64 (16-byte loads).
template <typename Fmt>
__device__ __forceinline__ void load8d(const typename Fmt::st* p, double* x) {
  if constexpr (sizeof(typename Fmt::st) == 2) {
    const u32x4 w = *reinterpret_cast<const u32x4*>(p);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      x[2 * q] = (double)Fmt::load((uint16_t)(w[q] & 0xffffu));
      x[2 * q + 1] = (double)Fmt::load((uint16_t)(w[q] >> 16));
    }
  } else {
    const float4 a = *reinterpret_cast<const float4*>(p);
    const float4 b = *reinterpret_cast<const float4*>(p + 4);
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
    x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
  }
}

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Ordered code of a key: larger key -> larger code; NaN as -inf, -0 as +0.
__device__ __forceinline__ uint64_t key_code(double x) {
  if (x != x) x = -__builtin_huge_val();
  if (x == 0.0) x = 0.0;
  const uint64_t b = (uint64_t)__double_as_longlong(x);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
// key a (index ia) is taken before key b (index ib)
__device__ __forceinline__ int before(uint64_t a, int ia, uint64_t b, int ib) {
  return (a > b || (a == b && ia < ib)) ? 1 : 0;
}

// Exclusive prefix sum of one int per thread over the block, in thread
// order; *total receives the block sum.  sh holds RZ_NT / 64 + 1 ints.
__device__ int block_scan_excl(int x, int* sh, int* total) {
  constexpr int NW = RZ_NT / 64;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int inc = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(inc, o, 64);
    if (lane >= o) inc += y;
  }
  if (lane == 63) sh[w] = inc;
  __syncthreads();
  if (threadIdx.x == 0) {
    int acc = 0;
    for (int i = 0; i < NW; ++i) {
      const int t = sh[i];
      sh[i] = acc;
      acc += t;
    }
    sh[NW] = acc;
  }
  __syncthreads();
  const int r = sh[w] + inc - x;
  *total = sh[NW];
  __syncthreads();
  return r;
}

// Bitonic sort of S * RZ_NT elements by the whole block, in registers: element
// q * RZ_NT + tid is slot q of thread tid.  A partner at distance j < 64 is a
// lane of the same wave (shuffles), at 64 <= j < RZ_NT a thread of another
// wave (through LDS, two barriers: 10 of the 55 stages of 1024 elements), at
// j >= RZ_NT another slot.  E: element type with shuffle(j), put(i) / get(i)
// (LDS exchange) and before(other), a strict order.  A sort with the elements
// in LDS spent 0.36 us on each stage, mostly LDS latency.  Only the first n
// elements matter, the others order after them and start behind them: the
// network ends with the power of two that covers n.
template <int S, typename E>
__device__ __forceinline__ void bitonic_sort(E (&x)[S], int n) {
  const int tid = threadIdx.x;
  // slot q against partner p: keeps the earlier element if `first`
  auto keep = [](E& mine, const E& other, bool first) {
    if (first != mine.before(other)) mine = other;
  };
  for (int k = 2; k < 2 * n && k <= S * RZ_NT; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      if (j >= RZ_NT) {
#pragma unroll
        for (int dj = S / 2; dj > 0; dj >>= 1) {
          if (j != dj * RZ_NT) continue;
#pragma unroll
          for (int q = 0; q < S; ++q) {
            if (q & dj) continue;
            const bool asc = ((q * RZ_NT + tid) & k) == 0;
            const E lo = x[q], hi = x[q | dj];
            keep(x[q], hi, asc);
            keep(x[q | dj], lo, !asc);
          }
        }
      } else if (j >= 64) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < S; ++q) x[q].put(q * RZ_NT + tid);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < S; ++q) {
          const int i = q * RZ_NT + tid;
          keep(x[q], x[q].get(i ^ j), ((i & j) == 0) == ((i & k) == 0));
        }
      } else {
#pragma unroll
        for (int q = 0; q < S; ++q) {
          const int i = q * RZ_NT + tid;
          keep(x[q], x[q].shuffle(j), ((i & j) == 0) == ((i & k) == 0));
        }
      }
    }
  }
  __syncthreads();
}

// A key of the crop: its code and index (padding: code 0, below the code of
// any key, and an index past the last).
struct KeyElem {
  uint64_t code;
  int id;
  uint64_t* lds_code;
  uint16_t* lds_id;
  __device__ __forceinline__ bool before(const KeyElem& o) const {
    return code > o.code || (code == o.code && id < o.id);
  }
  __device__ __forceinline__ KeyElem shuffle(int j) const {
    KeyElem e = *this;
    e.code = ((uint64_t)__shfl_xor((uint32_t)(code >> 32), j, 64) << 32) |
             __shfl_xor((uint32_t)code, j, 64);
    e.id = __shfl_xor(id, j, 64);
    return e;
  }
  __device__ __forceinline__ void put(int i) const {
    lds_code[i] = code;
    lds_id[i] = (uint16_t)id;
  }
  __device__ __forceinline__ KeyElem get(int i) const {
    KeyElem e = *this;
    e.code = lds_code[i];
    e.id = lds_id[i];
    return e;
  }
};

// A number (ascending).
struct U32Elem {
  uint32_t v;
  uint32_t* lds;
  __device__ __forceinline__ bool before(const U32Elem& o) const { return v < o.v; }
  __device__ __forceinline__ U32Elem shuffle(int j) const {
    return U32Elem{__shfl_xor(v, j, 64), lds};
  }
  __device__ __forceinline__ void put(int i) const { lds[i] = v; }
  __device__ __forceinline__ U32Elem get(int i) const { return U32Elem{lds[i], lds}; }
};

// Sorts the n <= S * RZ_NT keys of a crop: order[r] = index of the key taken
// r-th.  code and order hold S * RZ_NT entries.
template <int S>
__device__ __forceinline__ void sort_keys_s(const double* __restrict__ keys,
                                            int n, uint64_t* code,
                                            uint16_t* order) {
  KeyElem x[S];
#pragma unroll
  for (int q = 0; q < S; ++q) {
    const int i = q * RZ_NT + threadIdx.x;
    x[q] = KeyElem{i < n ? key_code(keys[i]) : 0ull, i, code, order};
  }
  bitonic_sort<S>(x, n);
#pragma unroll
  for (int q = 0; q < S; ++q) order[q * RZ_NT + threadIdx.x] = (uint16_t)x[q].id;
  __syncthreads();
}

// The same for n <= RZ_NT / 4 keys: four lanes count the keys taken before
// each one.  Eight 12 x 12 crops pruned to one level take 13.4 us so, 15.3 by
// the network's 36 stages, 19.7 by all 55.
__device__ __forceinline__ void rank_keys(const double* __restrict__ keys, int n,
                                          uint64_t* code, uint16_t* order) {
  if ((int)threadIdx.x < n) code[threadIdx.x] = key_code(keys[threadIdx.x]);
  __syncthreads();
  const int i = threadIdx.x >> 2, part = threadIdx.x & 3;
  int r = 0;
  if (i < n) {
    const uint64_t mine = code[i];
    for (int j = part; j < n; j += 4) r += before(code[j], j, mine, i);
  }
  r += __shfl_xor(r, 1, 64);
  r += __shfl_xor(r, 2, 64);
  if (i < n && part == 0) order[r] = (uint16_t)i;
  __syncthreads();
}

template <int MAX_S>
__device__ __forceinline__ void sort_keys(const double* __restrict__ keys, int n,
                                          uint64_t* code, uint16_t* order) {
  if (n <= RZ_NT / 4) rank_keys(keys, n, code, order);
  else if (n <= RZ_NT) sort_keys_s<1>(keys, n, code, order);
  else if (n <= 2 * RZ_NT) sort_keys_s<2>(keys, n, code, order);
  else if (MAX_S == 4 || n <= 4 * RZ_NT) sort_keys_s<4>(keys, n, code, order);
  else sort_keys_s<MAX_S>(keys, n, code, order);
}

// out[i] = the i-th smallest of the n <= S * RZ_NT values of x (padding:
// 0xffffffff), in LDS of S * RZ_NT entries; x is read first.
template <int S>
__device__ __forceinline__ void sort_u32(uint32_t* x, int n) {
  U32Elem e[S];
#pragma unroll
  for (int q = 0; q < S; ++q) e[q] = U32Elem{x[q * RZ_NT + threadIdx.x], x};
  bitonic_sort<S>(e, n);
#pragma unroll
  for (int q = 0; q < S; ++q) x[q * RZ_NT + threadIdx.x] = e[q].v;
  __syncthreads();
}

// ------------------------------------------------------------------ keys --

// L1 norm of every token: one wavefront per token.
template <typename Fmt>
__global__ void __launch_bounds__(256)
prune_keys_kernel(const typename Fmt::st* __restrict__ v, int n_tok, int d,
                  double* __restrict__ keys) {
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (t >= n_tok) return;
  const typename Fmt::st* row = v + (size_t)t * d;
  double acc = 0.0;
  for (int e0 = lane * 8; e0 < d; e0 += 512) {
    double x[8];
    load8d<Fmt>(row + e0, x);
#pragma unroll
    for (int k = 0; k < 8; ++k) acc += fabs(x[k]);
  }
  acc = wave_sum_f64(acc);
  if (lane == 0) keys[t] = acc;
}

__device__ __forceinline__ void edge_ends(int e, int G, int& a, int& b) {
  const int H = G * (G - 1);
  if (e < H) {
    a = (e / (G - 1)) * G + e % (G - 1);
    b = a + 1;
  } else {
    a = e - H;
    b = a + G;
  }
}

// Cosine similarity of every grid edge: one wavefront per edge.
template <typename Fmt>
__global__ void __launch_bounds__(256)
merge_keys_kernel(const typename Fmt::st* __restrict__ v, int n_crops, int G,
                  int d, double* __restrict__ keys) {
  const int E = 2 * G * (G - 1);
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (t >= n_crops * E) return;
  const int c = t / E;
  int a, b;
  edge_ends(t - c * E, G, a, b);
  const typename Fmt::st* ra = v + ((size_t)c * G * G + a) * d;
  const typename Fmt::st* rb = v + ((size_t)c * G * G + b) * d;
  double dot = 0.0, na = 0.0, nb = 0.0;
  for (int e0 = lane * 8; e0 < d; e0 += 512) {
    double x[8], y[8];
    load8d<Fmt>(ra + e0, x);
    load8d<Fmt>(rb + e0, y);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      dot += x[k] * y[k];
      na += x[k] * x[k];
      nb += y[k] * y[k];
    }
  }
  dot = wave_sum_f64(dot);
  na = wave_sum_f64(na);
  nb = wave_sum_f64(nb);
  if (lane == 0) keys[t] = (na == 0.0 || nb == 0.0) ? 0.0 : dot / sqrt(na * nb);
}

// ------------------------------------------------------------- decisions --

// Writes the identity map of the finest level (one crop per block).
__device__ void identity_map(const MapPtrs& mp, int K, int n_crops, int N) {
  const int c = blockIdx.x;
  for (int i = threadIdx.x; i < N; i += RZ_NT) {
    const int g = c * N + i;
    if (mp.mem[K - 1]) mp.mem[K - 1][g] = g;
    if (mp.offs[K - 1]) mp.offs[K - 1][g] = g;
  }
  if (c == 0 && threadIdx.x == 0 && mp.offs[K - 1])
    mp.offs[K - 1][n_crops * N] = n_crops * N;
}

// Prune: sort the crop's tokens by key, then per level keep the tokens ranked
// below n_l, compacted in index order by a block scan.  Latency-bound, one
// workgroup per crop, mostly the sort: 15 us for five 27 x 27 crops (29 while
// each thread ranked its token against all others).
__global__ void __launch_bounds__(RZ_NT)
prune_maps_kernel(const double* __restrict__ keys, int n_crops, int G, int K,
                  LvlCnt cnt, MapPtrs mp) {
  __shared__ uint64_t code[RZ_MAXN];
  __shared__ uint16_t order[RZ_MAXN];
  __shared__ uint16_t rank[RZ_MAXN];
  __shared__ int sh[RZ_NT / 64 + 1];
  const int N = G * G, c = blockIdx.x, tid = threadIdx.x;
  sort_keys<4>(keys + (size_t)c * N, N, code, order);
  for (int r = tid; r < N; r += RZ_NT) rank[order[r]] = (uint16_t)r;
  __syncthreads();
  for (int l = 0; l < K - 1; ++l) {
    const int n = cnt.n[l];
    int kept[RZ_PER], local = 0;
#pragma unroll
    for (int q = 0; q < RZ_PER; ++q) {
      const int i = tid * RZ_PER + q;
      kept[q] = (i < N && rank[i] < n) ? 1 : 0;
      local += kept[q];
    }
    int total;
    int pos = block_scan_excl(local, sh, &total);
#pragma unroll
    for (int q = 0; q < RZ_PER; ++q) {
      if (!kept[q]) continue;
      const int slot = c * n + pos;
      if (mp.mem[l]) mp.mem[l][slot] = c * N + tid * RZ_PER + q;
      if (mp.offs[l]) mp.offs[l][slot] = slot;
      ++pos;
    }
    if (c == 0 && tid == 0 && mp.offs[l]) mp.offs[l][n_crops * n] = n_crops * n;
  }
  identity_map(mp, K, n_crops, N);
}

// parent[] becomes root[] (every chain of the forest shortcut): pointer
// doubling, in place; a thread may read an entry another has already
// shortened, which is an ancestor all the same.
__device__ __forceinline__ void flatten(int* parent, int N) {
  bool more = true;
  while (__syncthreads_or(more)) {
    more = false;
    for (int i = threadIdx.x; i < N; i += RZ_NT) {
      const int p = parent[i], q = parent[p];
      if (p != q) {
        parent[i] = q;
        more = true;
      }
    }
  }
}

// Merge.  Taking the edges in key order and joining groups (Kruskal) keeps
// exactly the edges of the minimum spanning tree of the ranks, which the
// strict order makes unique, and after N - n joins n groups are left: the
// components of the tree's first N - n edges in rank order.  So the block
// sorts the edges, finds the tree by Boruvka rounds (every component takes
// its lowest-ranked outgoing edge: LDS atomic minima, at most log2 N rounds),
// numbers the tree's edges by rank with a prefix sum, and per level joins the
// ends of the first N - n_l of them (the larger label joins the smaller, so
// a label ends as its group's smallest member), counts group sizes, scans
// sizes and roots in index order (member start and group index) and lists the
// members by a sort of (label, token).  Latency-bound, one workgroup per
// crop: 80 us for four 27 x 27 crops (457 with the joins in a single lane).
__global__ void __launch_bounds__(RZ_NT)
merge_maps_kernel(const double* __restrict__ keys, int n_crops, int G, int K,
                  LvlCnt cnt, MapPtrs mp) {
  constexpr int P_E = 2 * RZ_MAXN;                 // >= RZ_MAXE, power of two
  static_assert(P_E >= RZ_MAXE && RZ_MAXE % 2 == 0, "edge arrays");
  // code: the sort's keys, afterwards the rounds' minima and the member sort
  __shared__ uint64_t code[P_E];
  __shared__ uint16_t order[P_E];      // edges by rank
  __shared__ uint16_t tree[P_E];       // per rank: in the tree; then its number
  __shared__ int parent[RZ_MAXN];
  __shared__ int label[RZ_MAXN];
  __shared__ int sh[RZ_NT / 64 + 1];
  const int N = G * G, E = 2 * G * (G - 1), c = blockIdx.x, tid = threadIdx.x;
  sort_keys<8>(keys + (size_t)c * E, E, code, order);
  uint32_t* best = reinterpret_cast<uint32_t*>(code);       // [N]
  uint32_t* msort = best + RZ_MAXN;                         // [RZ_MAXN]
  uint32_t* ends = msort + RZ_MAXN;                         // [P_E] by rank
  constexpr uint32_t NONE = 0xffffffffu;
  for (int r = tid; r < E; r += RZ_NT) {
    int a, b;
    edge_ends(order[r], G, a, b);
    ends[r] = (uint32_t)a | ((uint32_t)b << 16);
    tree[r] = 0;
  }
  for (int i = tid; i < N; i += RZ_NT) {
    label[i] = i;
    best[i] = NONE;
  }
  __syncthreads();
  // ---- the spanning tree
  for (;;) {
    bool open = false;
    for (int r = tid; r < E; r += RZ_NT) {
      const uint32_t ab = ends[r];
      const int la = label[ab & 0xffffu], lb = label[ab >> 16];
      if (la != lb) {
        atomicMin(&best[la], (uint32_t)r);
        atomicMin(&best[lb], (uint32_t)r);
        open = true;
      }
    }
    // every round joins every remaining group to another: at most 12 rounds
    if (!__syncthreads_or(open)) break;
    for (int i = tid; i < N; i += RZ_NT) {
      int p = i;
      if (label[i] == i && best[i] != NONE) {
        const uint32_t r = best[i];
        const uint32_t ab = ends[r];
        const int la = label[ab & 0xffffu], lb = label[ab >> 16];
        p = la == i ? lb : la;
        // two groups that took the same edge: the smaller stays the root
        if (best[p] == r && i < p) p = i;
        tree[r] = 1;
      }
      parent[i] = p;
    }
    flatten(parent, N);
    for (int i = tid; i < N; i += RZ_NT) {
      label[i] = parent[label[i]];
      best[i] = NONE;
    }
    __syncthreads();
  }
  // ---- number the tree's edges by rank (0, 1, ...; others 0xffff)
  {
    constexpr int PER = P_E / RZ_NT;
    uint16_t in[PER];
    int local = 0, total;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int r = tid * PER + q;
      in[q] = r < E ? tree[r] : 0;
      local += in[q];
    }
    int k = block_scan_excl(local, sh, &total);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int r = tid * PER + q;
      if (r < E) tree[r] = in[q] ? (uint16_t)k++ : (uint16_t)0xffff;
    }
  }
  for (int i = tid; i < N; i += RZ_NT) label[i] = i;
  __syncthreads();
  for (int l = K - 2; l >= 0; --l) {
    const int n = cnt.n[l];
    // ---- join the ends of the first N - n tree edges
    for (;;) {
      bool open = false;
      for (int r = tid; r < E; r += RZ_NT) {
        if ((int)tree[r] >= N - n) continue;
        const uint32_t ab = ends[r];
        const int la = label[ab & 0xffffu], lb = label[ab >> 16];
        if (la != lb) {
          // roots only: label[] is flat here, and a root joins a smaller one
          atomicMin(&label[max(la, lb)], min(la, lb));
          open = true;
        }
      }
      if (!__syncthreads_or(open)) break;
      flatten(label, N);
    }
    // ---- sizes, member starts, group indices
    int* aux = parent;
    for (int i = tid; i < N; i += RZ_NT) aux[i] = 0;
    for (int i = tid; i < RZ_MAXN; i += RZ_NT)
      msort[i] = i < N ? ((uint32_t)label[i] << 13) | (uint32_t)i : NONE;
    __syncthreads();
    for (int i = tid; i < N; i += RZ_NT) atomicAdd(&aux[label[i]], 1);
    __syncthreads();
    int sz[RZ_PER], rt[RZ_PER], lsz = 0, lrt = 0;
#pragma unroll
    for (int q = 0; q < RZ_PER; ++q) {
      const int i = tid * RZ_PER + q;
      sz[q] = i < N ? aux[i] : 0;
      rt[q] = (i < N && label[i] == i) ? 1 : 0;
      lsz += sz[q];
      lrt += rt[q];
    }
    int total;
    int start = block_scan_excl(lsz, sh, &total);
    int g = block_scan_excl(lrt, sh, &total);
#pragma unroll
    for (int q = 0; q < RZ_PER; ++q) {
      if (rt[q]) {
        // g < n always (exactly n roots remain); the test keeps a broken
        // invariant from writing past the level's offsets
        if (mp.offs[l] && g < n) mp.offs[l][c * n + g] = c * N + start;
        ++g;
      }
      start += sz[q];
    }
    // ---- members: groups by label (their smallest member), tokens ascending
    if (mp.mem[l]) {
      if (N <= RZ_NT) sort_u32<1>(msort, N);
      else if (N <= 2 * RZ_NT) sort_u32<2>(msort, N);
      else sort_u32<4>(msort, N);
      for (int i = tid; i < N; i += RZ_NT)
        mp.mem[l][c * N + i] = c * N + (int)(msort[i] & 0x1fffu);
    }
    if (c == 0 && tid == 0 && mp.offs[l]) mp.offs[l][n_crops * n] = n_crops * N;
    __syncthreads();
  }
  identity_map(mp, K, n_crops, N);
}

// ----------------------------------------------------------------- levels --

// Level rows of every level below the finest, one launch for all levels
// (block x: a token of level 0, then of level 1, ...: the coarsest level's
// groups are the largest and start first).
struct CsrLevels {
  const int32_t* offs[DAVET_MAX_LEVELS];
  const int32_t* mem[DAVET_MAX_LEVELS];
  void* out[DAVET_MAX_LEVELS];
  int n[DAVET_MAX_LEVELS];
};

// Prune: token t is row mem[t] of v (16 bytes a thread; rows are a multiple of
// 16 bytes), as the mean of that one row: 0 + x, so that -0 comes out as +0.
template <typename Fmt>
__global__ void __launch_bounds__(256)
copy_rows_kernel(const typename Fmt::st* __restrict__ v, CsrLevels lv, int d) {
  constexpr int VEC = 16 / (int)sizeof(typename Fmt::st);
  int l = 0, t = blockIdx.x;
  while (t >= lv.n[l]) t -= lv.n[l++];
  const int e0 = (blockIdx.y * 256 + threadIdx.x) * VEC;
  if (e0 >= d) return;
  u32x4 w = *reinterpret_cast<const u32x4*>(v + (size_t)lv.mem[l][t] * d + e0);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if constexpr (VEC == 8)
      w[q] = (uint32_t)Fmt::store(0.f + Fmt::load((uint16_t)(w[q] & 0xffffu))) |
             (uint32_t)Fmt::store(0.f + Fmt::load((uint16_t)(w[q] >> 16))) << 16;
    else
      w[q] = __float_as_uint(0.f + __uint_as_float(w[q]));
  }
  *reinterpret_cast<u32x4*>(reinterpret_cast<typename Fmt::st*>(lv.out[l]) +
                            (size_t)t * d + e0) = w;
}

// Merge: token t = float64 sum of rows mem[offs[t] .. offs[t+1]) of v in that
// order, divided by the member count, rounded once.  The largest merged
// groups hold most of a crop, so the time is their chain of member rows: a
// block owns 512 features of a token, stages the member ids in LDS and keeps
// up to 2 x BATCH rows in flight.
//
// fp16 (EXACT): a finite fp16 value is a multiple of 2^-24 below 2^16, so a
// float64 sum of up to 4096 of them is exact in any order; the block's four
// waves take every fourth member of all 512 features (16-byte loads) and add
// their sums in LDS.  bf16 and fp32 sums depend on the order, so there every
// thread adds all members of its 2 features one after another.
// Four 27 x 27 fp16 crops, both levels: 30 us (329 with all members in one
// chain of 8 rows in flight, ids loaded with each batch, a launch per level).
// The whole build of four crops, then and now: fp16 809 and 120 us, bf16 811 and
// 145, fp32 649 and 188.
constexpr int CSR_IDS = 512;                       // member ids staged at once
static_assert(RZ_MAXN <= 4096, "exact fp16 sums");

template <typename Fmt>
__global__ void __launch_bounds__(256)
pool_csr_kernel(const typename Fmt::st* __restrict__ v, CsrLevels lv, int d) {
  using T = typename Fmt::st;
  constexpr bool EXACT = Fmt::dtype == DAVET_F16;
  constexpr int VEC = EXACT ? 8 : 2;               // features per thread
  constexpr int STEP = EXACT ? 4 : 1;              // waves per feature
  constexpr int BATCH = EXACT ? 8 : 32;
  constexpr int W = VEC * (int)sizeof(T) / 4;      // 32-bit words per row piece
  typedef uint32_t words __attribute__((ext_vector_type(W),
                                        aligned(W >= 4 ? 16 : W * 4)));
  __shared__ int32_t ids[CSR_IDS];
  __shared__ double part[EXACT ? 3 : 1][EXACT ? VEC : 1][64];
  int l = 0, t = blockIdx.x;
  while (t >= lv.n[l]) t -= lv.n[l++];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int e0 = blockIdx.y * 512 + (EXACT ? lane : threadIdx.x) * VEC;
  const bool live = e0 < d;                        // d is a multiple of 8
  const T* src = v + (live ? e0 : 0);
  const int32_t* mem = lv.mem[l];
  const int b = lv.offs[l][t], e = lv.offs[l][t + 1];
  double acc[VEC];
#pragma unroll
  for (int k = 0; k < VEC; ++k) acc[k] = 0.0;
  for (int c0 = b; c0 < e; c0 += CSR_IDS) {
    const int nc = min(CSR_IDS, e - c0);
    if (c0 != b) __syncthreads();
    for (int i = threadIdx.x; i < nc; i += 256) ids[i] = mem[c0 + i];
    __syncthreads();
    const int first = EXACT ? wave : 0;
    words cur[BATCH], nxt[BATCH];
    // members i0, i0 + STEP, ... of the staged ones (the last one repeated)
    auto load = [&](int i0, words (&r)[BATCH]) {
#pragma unroll
      for (int k = 0; k < BATCH; ++k)
        r[k] = *reinterpret_cast<const words*>(
            src + (size_t)ids[min(i0 + k * STEP, nc - 1)] * d);
    };
    if (first < nc) load(first, cur);
    for (int i0 = first; i0 < nc; i0 += BATCH * STEP) {
      if (i0 + BATCH * STEP < nc) load(i0 + BATCH * STEP, nxt);
#pragma unroll
      for (int k = 0; k < BATCH; ++k) {
        if (i0 + k * STEP < nc) {
#pragma unroll
          for (int q = 0; q < W; ++q) {
            if constexpr (sizeof(T) == 2) {
              acc[2 * q] += (double)Fmt::load((uint16_t)(cur[k][q] & 0xffffu));
              acc[2 * q + 1] += (double)Fmt::load((uint16_t)(cur[k][q] >> 16));
            } else {
              acc[q] += (double)__uint_as_float(cur[k][q]);
            }
          }
        }
      }
#pragma unroll
      for (int k = 0; k < BATCH; ++k) cur[k] = nxt[k];
    }
  }
  if constexpr (EXACT) {
    if (e - b > 1) {                               // the same for the block
      if (wave > 0)
#pragma unroll
        for (int k = 0; k < VEC; ++k) part[wave - 1][k][lane] = acc[k];
      __syncthreads();
      if (wave == 0)
#pragma unroll
        for (int w = 0; w < 3; ++w)
#pragma unroll
          for (int k = 0; k < VEC; ++k) acc[k] += part[w][k][lane];
    }
    if (wave > 0) return;
  }
  if (!live) return;
  const double cnt = (double)(e - b);
  words w;
#pragma unroll
  for (int q = 0; q < W; ++q) {
    if constexpr (sizeof(T) == 2)
      w[q] = (uint32_t)Fmt::from_f64(acc[2 * q] / cnt) |
             ((uint32_t)Fmt::from_f64(acc[2 * q + 1] / cnt) << 16);
    else
      w[q] = __float_as_uint((float)(acc[q] / cnt));
  }
  *reinterpret_cast<words*>(reinterpret_cast<T*>(lv.out[l]) + (size_t)t * d + e0) = w;
}

// ------------------------------------------------------------------ host --

bool is_realizer(const davet_view_geom& g) {
  return g.realizer == DAVET_REALIZER_PRUNE || g.realizer == DAVET_REALIZER_MERGE;
}

int key_count(const davet_view_geom& g) {
  if (g.realizer == DAVET_REALIZER_PRUNE) return g.n_crops * g.grid * g.grid;
  if (g.realizer == DAVET_REALIZER_MERGE)
    return g.n_crops * 2 * g.grid * (g.grid - 1);
  return 0;
}

LvlCnt level_counts(const davet_view_geom& g) {
  LvlCnt lc{};
  for (int l = 0; l < g.K; ++l) {
    const int f = 1 << (g.K - 1 - l);
    const int W = (g.grid + f - 1) / f;
    lc.n[l] = W * W;
  }
  return lc;
}

int check_realizer(const davet_view_geom* g, const void* v, const char* who) {
  int rc = check_view_geom(g, who);
  if (rc) return rc;
  DAVET_CHECK_ARG(is_realizer(*g), DAVET_EINVAL,
                  std::string(who) + ": the geometry's realizer is pooling, "
                  "which has no keys");
  DAVET_CHECK_ARG(g->d >= 8 && g->d % 8 == 0, DAVET_ESHAPE,
                  std::string(who) + ": d must be a positive multiple of 8");
  DAVET_CHECK_ARG(g->dtype == DAVET_F32 || g->dtype == DAVET_BF16 ||
                      g->dtype == DAVET_F16, DAVET_EDTYPE,
                  std::string(who) + ": dtype must be DAVET_F32, BF16 or F16");
  DAVET_CHECK_ARG(v == nullptr || ((uintptr_t)v & 15) == 0, DAVET_EINVAL,
                  std::string(who) + ": v must be 16-byte aligned");
  return DAVET_OK;
}

template <typename Fmt>
void launch_keys_t(const davet_view_geom& g, const void* v, double* keys,
                   hipStream_t s) {
  const auto* vv = reinterpret_cast<const typename Fmt::st*>(v);
  const int n = key_count(g);
  if (n == 0) return;
  if (g.realizer == DAVET_REALIZER_PRUNE)
    hipLaunchKernelGGL(prune_keys_kernel<Fmt>, dim3((n + 3) / 4), dim3(256), 0,
                       s, vv, n, g.d, keys);
  else
    hipLaunchKernelGGL(merge_keys_kernel<Fmt>, dim3((n + 3) / 4), dim3(256), 0,
                       s, vv, g.n_crops, g.grid, g.d, keys);
}

int launch_keys(const davet_view_geom& g, const void* v, double* keys,
                hipStream_t s) {
  ProfScope ps(KC_REALIZER_KEYS, s);
  if (g.dtype == DAVET_BF16) launch_keys_t<BF16S>(g, v, keys, s);
  else if (g.dtype == DAVET_F16) launch_keys_t<F16S>(g, v, keys, s);
  else launch_keys_t<F32S>(g, v, keys, s);
  DAVET_HIP(hipGetLastError());
  return DAVET_OK;
}

int launch_maps(const davet_view_geom& g, const double* keys, const MapPtrs& mp,
                hipStream_t s) {
  bool any = false;
  for (int l = 0; l < g.K; ++l) any = any || mp.offs[l] || mp.mem[l];
  if (!any) return DAVET_OK;
  ProfScope ps(KC_REALIZER_MAPS, s);
  const LvlCnt lc = level_counts(g);
  if (g.realizer == DAVET_REALIZER_PRUNE)
    hipLaunchKernelGGL(prune_maps_kernel, dim3(g.n_crops), dim3(RZ_NT), 0, s,
                       keys, g.n_crops, g.grid, g.K, lc, mp);
  else
    hipLaunchKernelGGL(merge_maps_kernel, dim3(g.n_crops), dim3(RZ_NT), 0, s,
                       keys, g.n_crops, g.grid, g.K, lc, mp);
  DAVET_HIP(hipGetLastError());
  return DAVET_OK;
}

template <typename Fmt>
void launch_level_rows_t(const davet_view_geom& g, const void* v,
                         const CsrLevels& lv, int n_tok, hipStream_t s) {
  const auto* vv = reinterpret_cast<const typename Fmt::st*>(v);
  const int copied = 4096 / (int)sizeof(typename Fmt::st);   // features a block
  if (g.realizer == DAVET_REALIZER_PRUNE)
    hipLaunchKernelGGL(copy_rows_kernel<Fmt>,
                       dim3(n_tok, (g.d + copied - 1) / copied), dim3(256), 0,
                       s, vv, lv, g.d);
  else
    hipLaunchKernelGGL(pool_csr_kernel<Fmt>, dim3(n_tok, (g.d + 511) / 512),
                       dim3(256), 0, s, vv, lv, g.d);
}

// Scratch layout: keys, then (offsets, members) of each level < K-1, each
// region 256-byte aligned.
struct RzLayout {
  size_t keys = 0, offs[DAVET_MAX_LEVELS] = {}, mem[DAVET_MAX_LEVELS] = {};
  size_t total = 0;
};

RzLayout rz_layout(const davet_view_geom& g) {
  RzLayout L;
  size_t o = 0;
  L.keys = o;
  o += align_up((size_t)key_count(g) * 8, 256);
  const LvlCnt lc = level_counts(g);
  for (int l = 0; l + 1 < g.K; ++l) {
    const size_t n = (size_t)g.n_crops * lc.n[l];
    const size_t m = g.realizer == DAVET_REALIZER_PRUNE
                         ? n : (size_t)g.n_crops * g.grid * g.grid;
    L.offs[l] = o;
    o += align_up((n + 1) * 4, 256);
    L.mem[l] = o;
    o += align_up(m * 4, 256);
  }
  L.total = o;
  return L;
}

}  // namespace

size_t realizer_scratch_bytes(const davet_view_geom& g) {
  return is_realizer(g) ? rz_layout(g).total : 0;
}

int build_views_realizer(const davet_view_geom& g, const void* v,
                         void* const* levels, int32_t* const* offs,
                         int32_t* const* mem, void* scratch,
                         size_t scratch_bytes, hipStream_t s) {
  const RzLayout L = rz_layout(g);
  DAVET_CHECK_ARG(scratch != nullptr && scratch_bytes >= L.total, DAVET_ENOMEM,
                  "davet_build_views: scratch smaller than "
                  "davet_views_scratch_bytes");
  DAVET_CHECK_ARG(((uintptr_t)scratch & 255) == 0, DAVET_EINVAL,
                  "davet_build_views: scratch must be 256-byte aligned");
  char* sc = static_cast<char*>(scratch);
  double* keys = reinterpret_cast<double*>(sc + L.keys);
  MapPtrs mp{};
  for (int l = 0; l < g.K; ++l) {
    const bool own = l + 1 < g.K;
    mp.offs[l] = offs && offs[l] ? offs[l]
                 : own ? reinterpret_cast<int32_t*>(sc + L.offs[l]) : nullptr;
    mp.mem[l] = mem && mem[l] ? mem[l]
                : own ? reinterpret_cast<int32_t*>(sc + L.mem[l]) : nullptr;
  }
  int rc = launch_keys(g, v, keys, s);
  if (rc) return rc;
  rc = launch_maps(g, keys, mp, s);
  if (rc) return rc;
  const LvlCnt lc = level_counts(g);
  ProfScope ps(KC_VIEWS, s);
  CsrLevels lv{};
  int n_tok = 0;
  for (int l = 0; l + 1 < g.K; ++l) {
    lv.offs[l] = mp.offs[l];
    lv.mem[l] = mp.mem[l];
    lv.out[l] = levels[l];
    lv.n[l] = g.n_crops * lc.n[l];
    n_tok += lv.n[l];
  }
  if (n_tok == 0) return DAVET_OK;               // K = 1
  if (g.dtype == DAVET_BF16) launch_level_rows_t<BF16S>(g, v, lv, n_tok, s);
  else if (g.dtype == DAVET_F16) launch_level_rows_t<F16S>(g, v, lv, n_tok, s);
  else launch_level_rows_t<F32S>(g, v, lv, n_tok, s);
  DAVET_HIP(hipGetLastError());
  return DAVET_OK;
}

}  // namespace davet

extern "C" int davet_realizer_key_count(const davet_view_geom* g,
                                        int32_t* n_keys) {
  using namespace davet;
  DAVET_CHECK_ARG(g && n_keys, DAVET_EINVAL,
                  "davet_realizer_key_count: null argument");
  int rc = check_view_geom(g, "davet_realizer_key_count");
  if (rc) return rc;
  *n_keys = key_count(*g);
  return DAVET_OK;
}

extern "C" int davet_realizer_keys(const davet_view_geom* g, const void* v,
                                   double* keys, hipStream_t stream) {
  using namespace davet;
  DAVET_CHECK_ARG(g && v && keys, DAVET_EINVAL,
                  "davet_realizer_keys: null argument");
  int rc = check_realizer(g, v, "davet_realizer_keys");
  if (rc) return rc;
  DAVET_CHECK_ARG(((uintptr_t)keys & 7) == 0, DAVET_EINVAL,
                  "davet_realizer_keys: keys must be 8-byte aligned");
  return launch_keys(*g, v, keys, stream);
}

extern "C" int davet_realizer_maps(const davet_view_geom* g,
                                   const double* keys,
                                   int32_t* const* idx_offsets,
                                   int32_t* const* idx_members,
                                   hipStream_t stream) {
  using namespace davet;
  DAVET_CHECK_ARG(g, DAVET_EINVAL, "davet_realizer_maps: null geometry");
  int rc = check_realizer(g, nullptr, "davet_realizer_maps");
  if (rc) return rc;
  DAVET_CHECK_ARG(keys != nullptr || key_count(*g) == 0, DAVET_EINVAL,
                  "davet_realizer_maps: null keys");
  DAVET_CHECK_ARG(((uintptr_t)keys & 7) == 0, DAVET_EINVAL,
                  "davet_realizer_maps: keys must be 8-byte aligned");
  MapPtrs mp{};
  for (int l = 0; l < g->K; ++l) {
    mp.offs[l] = idx_offsets ? idx_offsets[l] : nullptr;
    mp.mem[l] = idx_members ? idx_members[l] : nullptr;
  }
  return launch_maps(*g, keys, mp, stream);
}

// ---------------------------------------------------------------------------
// davet_build_views_static: davet_build_views with the realizers' scratch
// (keys and the index maps of the pooled levels) in a file-scope device
// array instead of caller memory, for callers that cannot allocate.  Host
// code never passes the array's name to a kernel (in host code it is only a
// stand-in for the symbol): the device address is resolved once per device
// with hipGetSymbolAddress and kept.  Every call on a device shares that
// device's array; the keys and maps are written in full before they are
// read, so nothing needs clearing, and calls that overlap on one device race.

static __device__ __align__(256) char scratch[DAVET_STATIC_SCRATCH_BYTES];

namespace davet {
namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxDevices] = {};

// Device address of `scratch` on the current device (resolved on the first
// call on that device).
int static_scratch(void** out) {
  int dev = -1;
  DAVET_HIP(hipGetDevice(&dev));
  DAVET_CHECK_ARG(dev >= 0 && dev < kMaxDevices, DAVET_EHIP,
                  "davet_build_views_static: device index out of range");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* p = nullptr;
    DAVET_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    DAVET_CHECK_ARG(p != nullptr && ((uintptr_t)p & 255) == 0, DAVET_EHIP,
                    "davet_build_views_static: scratch address unusable");
    g_scratch_dev[dev] = p;
  }
  *out = g_scratch_dev[dev];
  return DAVET_OK;
}

}  // namespace
}  // namespace davet

extern "C" int davet_build_views_static(const davet_view_geom* g,
                                        const void* v, void* const* levels,
                                        int32_t* const* idx_offsets,
                                        int32_t* const* idx_members,
                                        hipStream_t stream) {
  using namespace davet;
  DAVET_CHECK_ARG(g, DAVET_EINVAL, "davet_build_views_static: null geometry");
  int rc = check_view_geom(g, "davet_build_views_static");
  if (rc) return rc;
  const size_t need = realizer_scratch_bytes(*g);
  DAVET_CHECK_ARG(need <= DAVET_STATIC_SCRATCH_BYTES, DAVET_ENOMEM,
                  "davet_build_views_static: the geometry needs " +
                      std::to_string(need) + " bytes of scratch, more than "
                      "the static maximum of " +
                      std::to_string((size_t)DAVET_STATIC_SCRATCH_BYTES) +
                      " (use davet_build_views with caller scratch)");
  void* sc = nullptr;
  if (need) {
    rc = static_scratch(&sc);
    if (rc) return rc;
  }
  return davet_build_views(g, v, levels, idx_offsets, idx_members, sc,
                           need ? (size_t)DAVET_STATIC_SCRATCH_BYTES : 0,
                           stream);
}
