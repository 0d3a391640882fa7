// float32 GEMMs of the fp32 configuration: C[M,N] = A[M,K] * B[N,K]^T on the
// fp32 matrix cores (v_mfma_f32_16x16x4_f32: full fp32 products and sums).
//
// A wavefront owns MI x NP pairs of 16 x 16 blocks and reads its operands
// straight from global memory into matrix-core lanes, 16 K values at a time:
// lane l holds row (or column) l % 16 and, in one 16-byte load, K values
// 16 kb + 4 (l / 16) .. +3, which feed four matrix ops (A and B use the same
// order of K, so the sum covers every k once).  No LDS staging: the sizes of
// this path are bound by latency, not by bytes (a 192 x 768 x 256 product is
// 1 us of matrix work), and its operands sit in L2.
//
// The two column blocks of a pair are what the epilogue needs side by side:
// gate and up of the same columns (EPI_SWIGLU), dims i and i + D/2 of a head
// (EPI_ROPE), or simply neighbouring columns.
//
// The RMSNorm in front of a projection is fused (NORM): A is then the
// residual row x, each element is multiplied by the norm's gain on its way
// in, the squares are summed alongside, and the finished sums are scaled by
// 1 / sqrt(mean(x^2) + eps) of their row.
//
// Two launch shapes.  Products of fewer than 256 workgroups of 128 rows x 4 pairs
// (128 x 128 outputs, 128 x 64 of gate and up): 16 rows x 1 pair per workgroup, K
// split over its four wavefronts and summed in LDS, so that the chip fills and
// each chain of dependent loads is a quarter as long.  Larger ones: 2 x 2
// wavefronts of 64 rows x 2 pairs, 16 flops per operand byte instead of 5.
// Measured on MI355X, a whole step (these products and the attention) against
// 64 x 64 tiles on the vector ALUs with separate norm, rope and gather
// launches and one attention thread per query: d = 256, 192 rows, two layers
// 1162 -> 95 us; d = 512, 564 rows 2733 -> 284; d = 2048, 964 rows 13.4 ->
// 3.5 ms.

#include "common.h"

namespace davet {
namespace {

// How a wave finds its operands and what it does with the result.
struct F32Args {
  const float* A;
  const float* B;
  const float* B2;              // EPI_SWIGLU: up weights
  float* C;
  int M, N, K, ldc;
  const int32_t* list;          // GATHER: list[0] live rows, packed positions
  const float* gain;            // NORM (null: ones)
  float eps;
  const int32_t* pos;           // EPI_ROPE: rotary position of each row
  const float2* cs;             // ... and the cos/sin table
  int half, rope_cols;          // ... head_dim / 2, rotated columns
};

constexpr int EPI_ROPE = 3;

// packed row of masked position number j
__device__ __forceinline__ int gather_row(const SeqPack& sp, const int32_t* list,
                                          int j) {
  const int g = list[1 + j];
  const int s = g / sp.L, i = g % sp.L;
  return sp.row0[s] + sp.nview[s] + sp.plen[s] + i;
}

// K values k .. k+3 of a row (zeros past the end); VEC: rows are 16-byte
// aligned (K % 4 == 0), so the four are all inside or all outside
template <bool VEC>
__device__ __forceinline__ f32x4 load4(const float* row, int k, int K) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if constexpr (VEC) {
    if (k < K) v = *reinterpret_cast<const f32x4*>(row + k);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (k + e < K) v[e] = row[k + e];
  }
  return v;
}

template <int EPI, bool NORM, bool GATHER, bool VEC, int MI, int NP, int WK>
__global__ void __launch_bounds__(256)
gemm_f32_kernel(F32Args a, SeqPack sp) {
  static_assert(WK == 1 || WK == 4, "one wave per tile, or four along K");
  constexpr int WM = WK == 4 ? 1 : 2, WN = WK == 4 ? 1 : 2;   // wave grid
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int wk = WK == 4 ? wave : 0;
  const int wm = WK == 4 ? 0 : wave >> 1, wn = WK == 4 ? 0 : wave & 1;
  const int m_live = GATHER ? a.list[0] : a.M;
  const int m0 = (blockIdx.y * WM + wm) * 16 * MI;
  if ((int)blockIdx.y * WM * 16 * MI >= m_live) return;
  const int p0 = (blockIdx.x * WN + wn) * NP;      // first column pair

  // first columns of the two blocks of pair p: as rows of B (and B2)
  const int hp = EPI == EPI_ROPE ? a.half / 16 : 1;       // pairs per head
  auto col1 = [&](int p) {
    if constexpr (EPI == EPI_ROPE) return (p / hp) * 2 * a.half + (p % hp) * 16;
    else if constexpr (EPI == EPI_SWIGLU) return p * 16;
    else return p * 32;
  };
  auto col2 = [&](int p) {
    if constexpr (EPI == EPI_ROPE) return col1(p) + a.half;
    else if constexpr (EPI == EPI_SWIGLU) return p * 16;
    else return p * 32 + 16;
  };

  const float* ar[MI];
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    int r = min(m0 + i * 16 + l16, m_live - 1);
    if constexpr (GATHER) r = gather_row(sp, a.list, r);
    ar[i] = a.A + (size_t)r * a.K;
  }
  const float* br[NP][2];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    br[p][0] = a.B + (size_t)min(col1(p0 + p) + l16, a.N - 1) * a.K;
    br[p][1] = (EPI == EPI_SWIGLU ? a.B2 : a.B) +
               (size_t)min(col2(p0 + p) + l16, a.N - 1) * a.K;
  }

  f32x4 acc[MI][NP][2];
  // sums of squares, and what their additions rounded off (Kahan): in a plain
  // chain of K / 4 additions rows of equal magnitude lost 1e-5 at K = 8192,
  // more than all the rest of the path
  float ss[MI], lost[MI];
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    ss[i] = lost[i] = 0.f;
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int h = 0; h < 2; ++h) acc[i][p][h] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const int nkb = (a.K + 15) / 16;
#pragma unroll 4
  for (int kb = wk; kb < nkb; kb += WK) {
    const int k = kb * 16 + g * 4;
    f32x4 av[MI], bv[NP][2];
#pragma unroll
    for (int i = 0; i < MI; ++i) av[i] = load4<VEC>(ar[i], k, a.K);
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int h = 0; h < 2; ++h) bv[p][h] = load4<VEC>(br[p][h], k, a.K);
    if constexpr (NORM) {
      f32x4 gv = {1.f, 1.f, 1.f, 1.f};
      if (a.gain) gv = load4<VEC>(a.gain, k, a.K);
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const f32x4 x = av[i];
        const float y =
            (x[0] * x[0] + x[1] * x[1]) + (x[2] * x[2] + x[3] * x[3]) - lost[i];
        const float sum = ss[i] + y;
        lost[i] = (sum - ss[i]) - y;
        ss[i] = sum;
        av[i] = x * gv;
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
          for (int h = 0; h < 2; ++h)
            acc[i][p][h] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                av[i][e], bv[p][h][e], acc[i][p][h], 0, 0, 0);
  }
  // sum of squares of row l % 16 of each block, over the lanes' K values
  if constexpr (NORM) {
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      // a sum that overflowed ends as NaN (inf - inf); where a value itself was
      // not finite the products are not either
      if (ss[i] != ss[i]) ss[i] = INFINITY;
      ss[i] += __shfl_xor(ss[i], 16, 64);
      ss[i] += __shfl_xor(ss[i], 32, 64);
    }
  }
  auto finish = [&](int row, int p, float x, float y, float sq) {
    if (row >= m_live) return;
    if constexpr (NORM) {
      const float rstd = 1.0f / sqrtf(sq / (float)a.K + a.eps);
      x *= rstd;
      y *= rstd;
    }
    const int c1 = col1(p) + l16, c2 = col2(p) + l16;
    float* c = a.C + (size_t)row * a.ldc;
    if constexpr (EPI == EPI_SWIGLU) {
      if (c1 < a.N) c[c1] = x / (1.0f + expf(-x)) * y;
    } else if constexpr (EPI == EPI_ROPE) {
      if (c1 >= a.N) return;
      if (c1 < a.rope_cols) {
        const float2 t = a.cs[(size_t)a.pos[row] * a.half + (p % hp) * 16 + l16];
        c[c1] = x * t.x - y * t.y;
        c[c2] = y * t.x + x * t.y;
      } else {
        c[c1] = x;
        c[c2] = y;
      }
    } else if constexpr (EPI == EPI_ADD_F32) {
      if (c1 < a.N) c[c1] += x;
      if (c2 < a.N) c[c2] += y;
    } else {
      if (c1 < a.N) c[c1] = x;
      if (c2 < a.N) c[c2] = y;
    }
  };

  // accumulator element r of lane l: row 4 (l / 16) + r, column l % 16
  if constexpr (WK == 1) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float sq = NORM ? __shfl(ss[i], g * 4 + r, 64) : 0.f;
#pragma unroll
        for (int p = 0; p < NP; ++p)
          finish(m0 + i * 16 + g * 4 + r, p0 + p, acc[i][p][0][r],
                 acc[i][p][1][r], sq);
      }
  } else {
    // the four waves' partial sums meet in LDS; wave w finishes element w
    __shared__ float red[WK][MI * NP * 2][4][64];
    __shared__ float rss[WK][MI * 16];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            red[wk][(i * NP + p) * 2 + h][r][lane] = acc[i][p][h][r];
    if constexpr (NORM) {
      if (g == 0)
#pragma unroll
        for (int i = 0; i < MI; ++i) rss[wk][i * 16 + l16] = ss[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int lr = i * 16 + g * 4 + wave;
      float sq = 0.f;
      if constexpr (NORM)
#pragma unroll
        for (int w = 0; w < WK; ++w) sq += rss[w][lr];
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        float x = 0.f, y = 0.f;
#pragma unroll
        for (int w = 0; w < WK; ++w) {
          x += red[w][(i * NP + p) * 2][wave][lane];
          y += red[w][(i * NP + p) * 2 + 1][wave][lane];
        }
        finish(m0 + lr, p0 + p, x, y, sq);
      }
    }
  }
}

template <int EPI, bool NORM, bool GATHER>
int launch(const F32Args& a, const SeqPack& sp, int cls, hipStream_t s) {
  if (a.M <= 0) return DAVET_OK;
  ProfScope ps(cls, s);
  const int pairs = EPI == EPI_SWIGLU ? (a.N + 15) / 16 : (a.N + 31) / 32;
  // 128 x (4 pairs) tiles once they fill the 256 CUs (below that most CUs
  // would idle through K steps of 2048 matrix-core cycles), else 16 x 1 pair
  // with K split over the workgroup
  const bool big = (int64_t)((a.M + 127) / 128) * ((pairs + 3) / 4) >= 256;
  const dim3 grid = big ? dim3((pairs + 3) / 4, (a.M + 127) / 128)
                        : dim3(pairs, (a.M + 15) / 16);
#define GO(V)                                                                 \
  do {                                                                        \
    if (big)                                                                  \
      hipLaunchKernelGGL((gemm_f32_kernel<EPI, NORM, GATHER, V, 4, 2, 1>),    \
                         grid, dim3(256), 0, s, a, sp);                       \
    else                                                                      \
      hipLaunchKernelGGL((gemm_f32_kernel<EPI, NORM, GATHER, V, 1, 1, 4>),    \
                         grid, dim3(256), 0, s, a, sp);                       \
  } while (0)
  if (a.K % 4 == 0) {
    GO(true);
  } else if constexpr (!NORM) {
    GO(false);
  } else {
    // the normed products contract over d, a multiple of 64
    return set_error(DAVET_ESHAPE, "gemm_f32: a normed product needs K % 4 == 0");
  }
#undef GO
  DAVET_HIP(hipGetLastError());
  return DAVET_OK;
}

}  // namespace

// QKV projection of the normed residual rows, rotary embedding on the query
// and key columns.
int launch_f32_qkv(const float* X, const float* gain, float eps, const float* W,
                   float* QKV, int rows, int d, int head_dim,
                   const int32_t* pos, const float* cs, const SeqPack& sp,
                   hipStream_t s) {
  F32Args a{X, W, nullptr, QKV, rows, 3 * d, d, 3 * d, nullptr, gain, eps,
            pos, reinterpret_cast<const float2*>(cs), head_dim / 2, 2 * d};
  return launch<EPI_ROPE, true, false>(a, sp, KC_GEMM_F32, s);
}

// H = silu(norm(X) Wg^T) * (norm(X) Wu^T)
int launch_f32_swiglu(const float* X, const float* gain, float eps,
                      const float* Wg, const float* Wu, float* H, int rows,
                      int d, int ffn, const SeqPack& sp, hipStream_t s) {
  F32Args a{X, Wg, Wu, H, rows, ffn, d, ffn, nullptr, gain, eps,
            nullptr, nullptr, 0, 0};
  return launch<EPI_SWIGLU, true, false>(a, sp, KC_GEMM_F32, s);
}

// X += A W^T
int launch_f32_add(const float* A, const float* W, float* X, int rows, int d,
                   int K, const SeqPack& sp, hipStream_t s) {
  F32Args a{A, W, nullptr, X, rows, d, K, d, nullptr, nullptr, 0.f,
            nullptr, nullptr, 0, 0};
  return launch<EPI_ADD_F32, false, false>(a, sp, KC_GEMM_F32, s);
}

// logits[j] = norm(X[masked position j]) W^T for the list[0] live positions
int launch_f32_head(const float* X, const int32_t* list, const float* gain,
                    float eps, const float* W, float* logits, int max_rows,
                    int vocab, int d, const SeqPack& sp, hipStream_t s) {
  F32Args a{X, W, nullptr, logits, max_rows, vocab, d, vocab, list, gain, eps,
            nullptr, nullptr, 0, 0};
  return launch<EPI_STORE, true, true>(a, sp, KC_HEAD, s);
}

}  // namespace davet
