// 16-bit (fp16 or bf16) matrix-core GEMMs of the denoiser: C[M,N] = A[M,K] B[N,K]^T
// with both operands K-contiguous (activations row-major, weights [out, in]).
//
// CDNA4 design.  A workgroup of 4, 8 or 16 wavefronts (a WM x WN grid, WN = 2
// or 4) owns a BM x BN tile; each wavefront accumulates (BM/WM) x (BN/WN)
// with v_mfma_f32_16x16x32 ops (fp32 accumulators).  K moves in slabs of BK (32
// or 64) through a STAGES-deep ring of LDS stages filled by direct
// global->LDS loads (global_load_lds_dwordx4: no VGPR staging), so up to
// STAGES - 1 slabs are in flight while one feeds the matrix cores; one
// barrier per slab.  Each LDS row holds BK 16-bit values in 16-byte chunks;
// chunk c of row r sits in slot c ^ ((r / rows-per-256-bytes) % chunks),
// which spreads the 16-byte fragment reads of 16 consecutive rows over
// distinct bank groups.  Workgroup ids are remapped so each XCD (ids
// congruent mod 8) walks a contiguous run of tiles, in bands of row tiles, M
// fastest: a weight tile is fetched into one XCD's L2 and reused by the band.
// Long products and the large vocabulary head run a kernel of their own
// (gemm16_phased_kernel).  The variants
// (tile, slab depth, ring depth, waves) and the plan that picks one per
// product shape are listed after the kernel.
//
// Split-K: with few output tiles (short sequences) the K range is cut into
// ksplit parts whose fp32 partial tiles land in a workspace; a row kernel
// sums them in a fixed order (deterministic) and applies the epilogue.
//
// Epilogues, fused:
//   EPI_STORE    16-bit C = acc, with the rotary embedding applied in fp32 to
//                the query/key columns (a lane owns dims i and i+64 of a head)
//   EPI_ADD_F32  fp32 C += acc (residual stream)
//   EPI_SWIGLU   B holds gate rows, B2 up rows; gate and up of one output
//                column sit in the same lane: 16-bit C = silu(gate) * up
//   EPI_HEAD     vocabulary slab reduction per row: (max, first argmax,
//                sum exp(l - max)) with [MASK] excluded
//   EPI_PARTIAL  fp32 partial tile of one K split

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.h"

namespace davet {
namespace {

constexpr int BK_MIN = 32;   // K must be a multiple of this

constexpr int EPI_HEAD = 3;

// Kernel variants: tile BM x BN, K slab BK (64-byte or 128-byte LDS rows),
// STAGES-deep LDS ring, WAVES wavefronts in a (WAVES / WN) x WN grid (WN = 2
// or 4 wave columns); IGLP >= 0 asks the compiler's scheduler for its
// matrix-op interleaving strategy of that number (__builtin_amdgcn_iglp_opt)
// on the slab body; SG = 1 gives it an explicit order instead (schedule
// groups: the first 32-deep step's fragment reads, then the second step's
// reads one per matrix op of the first step, then the remaining matrix ops).
template <int BM_, int BN_, int BK_, int STAGES_, int WAVES_, int IGLP_ = -1,
          int WN_ = 2, int SG_ = 0>
struct Var {
  static constexpr int BM = BM_, BN = BN_, BK = BK_, STAGES = STAGES_,
                       WAVES = WAVES_, IGLP = IGLP_, WN = WN_, SG = SG_;
  static constexpr int LDS = STAGES * (BM + BN) * BK * 2;
  // workgroups per CU the register budget must allow (LDS is 160 KB per CU)
  static constexpr int MINB = LDS <= 80 * 1024 ? (LDS <= 53 * 1024 ? 3 : 2) : 1;
};
constexpr int EPI_PARTIAL = 4;

struct EpiArgs {
  void* C;
  int ldc;
  // rotary embedding (EPI_STORE): columns < rope_cols are rotated
  const int32_t* pos;
  const float2* cs;
  int rope_cols;
  // vocabulary head
  const int32_t* list;
  int vocab, mask_id, n_slabs;
  float* pmax;
  float* psum;
  int32_t* parg;
  float* logits_out;
  // split-K partials: part[ks][row][col], row stride part_ld
  float* part;
  int part_ld;
  int dual;              // B/B2 gate/up weights (SwiGLU), also for partials
  int ffn;
  // B is a tiled vocabulary head of 128 x 64 blocks (davet_pack_head), BN a
  // multiple of 128, BK 32 or 64: slab step kt reads BK columns of each of
  // its BN / 128 blocks in chunk kt * BK / 64, from column kt * BK % 64
  int b_tiled;
  // non-finite 16-bit values stored by EPI_STORE / EPI_SWIGLU (may be null)
  int32_t* overflow;
  int m_band;            // row tiles per band of the tile order
};

__device__ __forceinline__ int remap_xcd(int bid, int nwg) {
  const int full = nwg & ~7;
  if (bid >= full) return bid;
  const int per = full >> 3;
  return (bid & 7) * per + (bid >> 3);
}

// Order of the tiles: bands of m_band row tiles; in a band row tiles fastest,
// then K splits, then columns.
__device__ __forceinline__ void locate_tile(int tile, int n_mtiles,
                                            int n_ntiles, int ksplit,
                                            int m_band, int& mb, int& ks,
                                            int& nb) {
  const int per_band = m_band * ksplit * n_ntiles;
  const int band = tile / per_band;
  const int in_band = tile - band * per_band;
  const int rows = min(m_band, n_mtiles - band * m_band);
  mb = band * m_band + in_band % rows;
  const int rest = in_band / rows;
  ks = rest % ksplit;
  nb = rest / ksplit;
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// s_waitcnt vmcnt(n) for a wave-uniform n in [LO, HI] known only at run time
// (the count is an instruction immediate): a binary tree of scalar branches.
template <int LO, int HI>
__device__ __forceinline__ void wait_vmcnt_rt(int n) {
  if constexpr (LO == HI) {
    wait_vmcnt<LO>();
  } else {
    constexpr int MID = (LO + HI) / 2;
    if (n <= MID) wait_vmcnt_rt<LO, MID>(n);
    else wait_vmcnt_rt<MID + 1, HI>(n);
  }
}

// Workgroup barrier without the memory fence __syncthreads() carries: the
// fence would wait for every outstanding global->LDS load (vmcnt(0)) and
// drain the pipeline.  Each wave has already waited for the slab it needs;
// the empty asm statements keep the compiler from moving LDS accesses across.
__device__ __forceinline__ void barrier_nofence() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

typedef __attribute__((address_space(3))) void* lds_ptr_t;

__device__ __forceinline__ void dma16(const void* g, void* lds) {
  __builtin_amdgcn_global_load_lds(g, (lds_ptr_t)lds, 16, 0, 0);
}

// The same from a wave-uniform address, with `left` bytes behind it (lanes
// past them read zeros), and a 32-bit offset per lane.
__device__ __forceinline__ void dma16_from(const char* from, uint32_t left,
                                           uint32_t off, void* lds) {
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>(from), 0, left, 0x00027000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr_t)lds, 16, off, 0, 0, 0);
}

// Byte offset of chunk c (16 B) of row r inside a stage of BK-wide rows.
// Slot = c ^ f(r) with f chosen so 16 consecutive rows at the same chunk fall
// in 16 distinct 16-byte bank groups of a 256-byte bank line.
template <int BK>
__device__ __forceinline__ int swz(int r, int c) {
  constexpr int CPR = BK / 8;                 // 16-byte chunks per row
  constexpr int RPL = 16 / CPR;               // rows per 256-byte bank line
  return r * (BK * 2) + ((c ^ ((r / RPL) % CPR)) << 4);
}

template <typename Fmt, typename V, int EPI>
__global__ void __launch_bounds__(64 * V::WAVES, V::MINB)
gemm16_kernel(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B,
              const uint16_t* __restrict__ B2, int M, int N, int K,
              int n_mtiles, int n_ntiles, int ksplit, EpiArgs ep) {
  using v8 = typename Fmt::v8;
  constexpr int BM = V::BM, BN = V::BN, BK = V::BK, STAGES = V::STAGES;
  constexpr int WAVES = V::WAVES;
  constexpr int WN = V::WN;              // wave grid WM x WN
  constexpr int WM = WAVES / WN;
  constexpr int WROWS = BM / WM;         // rows per wave
  constexpr int TM = WROWS / 32;         // 32-row sub-tiles per wave
  constexpr int TN = BN / 64;            // 64-column groups of the tile
  constexpr int CW = 64 / WN;            // a wave's columns in each group
  constexpr int QC = CW / 16;            // ... as 16-column blocks
  constexpr int NQ = 2 * QC;             // 16 x 16 accumulators per 32-row
                                         // sub-tile and column group
  static_assert(WN == 2 || WN == 4, "two or four wave columns");
  static_assert(EPI != EPI_HEAD || WN == 2, "the head reduction pairs two wave columns");
  constexpr int CPR = BK / 8;            // 16-byte chunks per LDS row
  constexpr int RPI = 64 / CPR;          // rows per load instruction
  constexpr int AI = BM / (RPI * WAVES); // A load instructions per wave/stage
  constexpr int BI = BN / (RPI * WAVES); // B load instructions per wave/stage
  static_assert(AI >= 1 && BI >= 1 && TM >= 1, "tile too small for the waves");
  constexpr int LPT = AI + BI;
  constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2;
  constexpr int S_BYTES = A_BYTES + B_BYTES;
  __shared__ __attribute__((aligned(1024))) char smem[STAGES * S_BYTES];

  const int nwg = gridDim.x;
  const int tile = remap_xcd(blockIdx.x, nwg);
  int mb, ks, nb;
  locate_tile(tile, n_mtiles, n_ntiles, ksplit, ep.m_band, mb, ks, nb);
  int m_live = M;
  if constexpr (EPI == EPI_HEAD) m_live = ep.list[0];
  const int n0 = nb * BN;
  // M tiles mb, mb + n_mtiles, ... (one tile unless the grid is narrower
  // than the rows: the vocabulary head sizes it for the live rows)
  for (int mt = mb; mt * BM < m_live; mt += n_mtiles) {
  const int m0 = mt * BM;
  if (mt != mb) __syncthreads();      // LDS of the previous tile retired
  const int nk_all = K / BK;
  const int chunk = (nk_all + ksplit - 1) / ksplit;
  const int kt0 = ks * chunk;
  const int nk = min(nk_all, kt0 + chunk) - kt0;

  const int t = threadIdx.x;
  const int lane = t & 63;
  // wave-uniform values live in scalar registers (branches on them are
  // scalar, not exec-masked)
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int l32 = lane & 31, hh = lane >> 5;
  const int l16 = lane & 15, k4 = lane >> 4;
  const bool dual = (EPI == EPI_SWIGLU) || (EPI == EPI_PARTIAL && ep.dual);

  // ---- per-lane sources of this wave's load instructions (fixed over K)
  const uint16_t* a_src[AI];
  const uint16_t* b_src[BI];
#pragma unroll
  for (int q = 0; q < AI; ++q) {
    const int r = (wave * AI + q) * RPI + lane / CPR;
    const int c = (lane % CPR) ^ ((r / (16 / CPR)) % CPR);
    const int gm = min(m0 + r, m_live - 1);
    a_src[q] = A + (size_t)gm * K + (size_t)kt0 * BK + c * 8;
  }
#pragma unroll
  for (int q = 0; q < BI; ++q) {
    const int r = (wave * BI + q) * RPI + lane / CPR;
    const int c = (lane % CPR) ^ ((r / (16 / CPR)) % CPR);
    const uint16_t* base = B;
    int gn;
    if (dual) {
      const int half = BN / 2;
      base = r < half ? B : B2;
      gn = nb * half + (r < half ? r : r - half);
    } else {
      gn = min(n0 + r, N - 1);
    }
    if (ep.b_tiled)
      b_src[q] = B + ((size_t)min(nb * (BN / 128) + (r >> 7), (N - 1) >> 7) * 128 +
                      (r & 127)) * 64 + c * 8;
    else
      b_src[q] = base + (size_t)gn * K + (size_t)kt0 * BK + c * 8;
  }
  const size_t b_kstride =
      ep.b_tiled ? (size_t)((N + 127) / 128) * 128 * 64 : (size_t)BK;

  // A load instructions of this wave holding at least one live row: rows
  // past the last live one are not fetched (their LDS rows feed only output
  // rows that are never stored).  The count is wave-uniform, so the per-slab
  // load count LPT_live of each wave is too.
  const int na = __builtin_amdgcn_readfirstlane(
      max(0, min(AI, (m_live - m0 - wave * AI * RPI + RPI - 1) / RPI)));
  const int lpt_live = na + BI;
  auto issue = [&](int stage, int kt) {
    char* sa = smem + stage * S_BYTES;
    char* sb = sa + A_BYTES;
#pragma unroll
    for (int q = 0; q < AI; ++q)
      if (q < na) dma16(a_src[q] + (size_t)kt * BK, sa + (wave * AI + q) * 1024);
    const int kel = (kt0 + kt) * BK;       // first K element of the slab
    const size_t boff = ep.b_tiled ? (size_t)(kel >> 6) * b_kstride + (kel & 63)
                                   : (size_t)kt * b_kstride;
#pragma unroll
    for (int q = 0; q < BI; ++q)
      dma16(b_src[q] + boff, sb + (wave * BI + q) * 1024);
  };

  // acc[i][j][q]: the 16 x 16 block (q / QC, q % QC) of the wave's
  // 32 x CW block (i, j), one v_mfma_f32_16x16x32 accumulator each
  f32x4 acc[TM][TN][NQ];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][j][q][e] = 0.f;

  // 32-row sub-tiles of this wave holding live rows: always a prefix, NL of
  // them.  The K loop is instantiated per NL, so its body has no branch
  // between the LDS fragment reads and the matrix ops.
  const int nl = max(0, min(TM, (m_live - m0 - wm * WROWS + 31) / 32));

#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s)
    if (s < nk) issue(s, s);

  auto k_loop = [&](auto nl_c) {
    constexpr int NL = decltype(nl_c)::value;
    for (int it = 0; it < nk; ++it) {
      // slab `it` must have landed; later slabs may still be in flight
      const int ahead = min(STAGES - 2, nk - 1 - it);
      static_assert((STAGES - 2) * LPT <= 63, "vmcnt range");
      wait_vmcnt_rt<0, (STAGES - 2) * LPT>(ahead * lpt_live);
      barrier_nofence();        // slab visible to all waves; slab it-1 retired
      if (it + STAGES - 1 < nk) issue((it + STAGES - 1) % STAGES, it + STAGES - 1);
      if constexpr (NL > 0) {
        const char* sa = smem + (it % STAGES) * S_BYTES;
        const char* sb = sa + A_BYTES;
        // 32-deep K steps of 16 x 16 x 32 matrix ops: lane l supplies row
        // (or column) l % 16 of a 16-row fragment and k = 8 (l / 16) .. +7,
        // i.e. 16-byte chunk 4 kk + l / 16 of that LDS row
        if constexpr (V::IGLP >= 0) __builtin_amdgcn_iglp_opt(V::IGLP);
#pragma unroll
        for (int kk = 0; kk < BK / 32; ++kk) {
          const int c = kk * 4 + k4;
          v8 af[NL][2], bfr[TN][QC];
#pragma unroll
          for (int i = 0; i < NL; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const int r = wm * WROWS + i * 32 + h * 16 + l16;
              af[i][h] = *reinterpret_cast<const v8*>(sa + swz<BK>(r, c));
            }
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int h = 0; h < QC; ++h) {
              const int r = j * 64 + wn * CW + h * 16 + l16;
              bfr[j][h] = *reinterpret_cast<const v8*>(sb + swz<BK>(r, c));
            }
#pragma unroll
          for (int i = 0; i < NL; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
              for (int q = 0; q < NQ; ++q)
                acc[i][j][q] = Fmt::mfma16(af[i][q / QC], bfr[j][q % QC],
                                           acc[i][j][q]);
        }
        if constexpr (V::SG == 1) {
          static_assert(BK == 64 && V::IGLP < 0, "two 32-deep steps, no strategy");
          constexpr int DS_READ = 0x100, MATRIX = 0x008;   // group masks
          constexpr int R = NL * 2 + TN * QC;   // fragment reads per step
          constexpr int MO = NL * TN * NQ;      // matrix ops per step
          static_assert(MO >= R, "a read per matrix op");
          __builtin_amdgcn_sched_group_barrier(DS_READ, R, 0);
#pragma unroll
          for (int r = 0; r < R; ++r) {
            __builtin_amdgcn_sched_group_barrier(DS_READ, 1, 0);
            __builtin_amdgcn_sched_group_barrier(MATRIX, 1, 0);
          }
          __builtin_amdgcn_sched_group_barrier(MATRIX, 2 * MO - R, 0);
        }
      }
    }
  };
  static_assert(TM <= 4, "live-prefix dispatch covers up to 4 sub-tiles");
  switch (nl) {
    case 0: k_loop(std::integral_constant<int, 0>{}); break;
    case 1: k_loop(std::integral_constant<int, 1>{}); break;
    case 2: k_loop(std::integral_constant<int, (TM >= 2 ? 2 : TM)>{}); break;
    case 3: k_loop(std::integral_constant<int, (TM >= 3 ? 3 : TM)>{}); break;
    default: k_loop(std::integral_constant<int, TM>{}); break;
  }

  // ---------------------------------------------------------------- epilogue
  // acc[i][j][q][u]: row = wm*WROWS + i*32 + (q/QC)*16 + (lane/16)*4 + u,
  //                  col = j*64 + wn*CW + (q%QC)*16 + lane%16   (tile-local)
  // so a lane's column in each 64-column group j is wn*CW + (q%QC)*16 + l16
  int nf = 0;     // non-finite 16-bit values stored by this lane
  const int rrow = k4 * 4;
  if constexpr (EPI == EPI_STORE) {
    uint16_t* C = reinterpret_cast<uint16_t*>(ep.C);
    const bool rope = ep.pos && n0 < ep.rope_cols;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int row = m0 + wm * WROWS + i * 32 + (q / QC) * 16 + rrow + u;
          if (row >= M) continue;
          const int cl = wn * CW + (q % QC) * 16 + l16;
          uint16_t* crow = C + (size_t)row * ep.ldc + n0 + cl;
          if (rope) {
            // j even / j+1: dims cl and cl+64 of the head starting at n0 + j*64
            const float2 c = ep.cs[(size_t)ep.pos[row] * 64 + cl];
#pragma unroll
            for (int j = 0; j < TN; j += 2) {
              const float x = acc[i][j][q][u], y = acc[i][j + 1][q][u];
              const uint16_t a = Fmt::store(x * c.x - y * c.y);
              const uint16_t b = Fmt::store(y * c.x + x * c.y);
              nf += Fmt::nonfinite(a) + Fmt::nonfinite(b);
              crow[j * 64] = a;
              crow[(j + 1) * 64] = b;
            }
          } else {
#pragma unroll
            for (int j = 0; j < TN; ++j) {
              const uint16_t a = Fmt::store(acc[i][j][q][u]);
              nf += Fmt::nonfinite(a);
              crow[j * 64] = a;
            }
          }
        }
  } else if constexpr (EPI == EPI_ADD_F32) {
    float* C = reinterpret_cast<float*>(ep.C);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int row = m0 + wm * WROWS + i * 32 + (q / QC) * 16 + rrow + u;
          if (row >= M) continue;
          float* crow = C + (size_t)row * ep.ldc + n0 + wn * CW + (q % QC) * 16 + l16;
#pragma unroll
          for (int j = 0; j < TN; ++j) crow[j * 64] += acc[i][j][q][u];
        }
  } else if constexpr (EPI == EPI_SWIGLU) {
    uint16_t* C = reinterpret_cast<uint16_t*>(ep.C);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int row = m0 + wm * WROWS + i * 32 + (q / QC) * 16 + rrow + u;
          if (row >= M) continue;
          uint16_t* crow = C + (size_t)row * ep.ldc + nb * (BN / 2) + wn * CW +
                           (q % QC) * 16 + l16;
#pragma unroll
          for (int j = 0; j < TN / 2; ++j) {
            const float g = acc[i][j][q][u], up = acc[i][j + TN / 2][q][u];
            const uint16_t h = Fmt::store(g / (1.0f + __expf(-g)) * up);
            nf += Fmt::nonfinite(h);
            crow[j * 64] = h;
          }
        }
  } else if constexpr (EPI == EPI_PARTIAL) {
    float* P = ep.part + (size_t)ks * M * ep.part_ld;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int row = m0 + wm * WROWS + i * 32 + (q / QC) * 16 + rrow + u;
          if (row >= M) continue;
          float* prow = P + (size_t)row * ep.part_ld;
          const int cl = wn * CW + (q % QC) * 16 + l16;
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            int col;
            if (ep.dual) {       // gate half -> [0, F), up half -> [F, 2F)
              const int jj = j % (TN / 2);
              col = (j < TN / 2 ? 0 : ep.ffn) + nb * (BN / 2) + jj * 64 + cl;
            } else {
              col = n0 + j * 64 + cl;
            }
            prow[col] = acc[i][j][q][u];
          }
        }
  } else {   // EPI_HEAD
    __shared__ float red_m[2][BM];
    __shared__ float red_s[2][BM];
    __shared__ int red_a[2][BM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int qr = 0; qr < 2; ++qr) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int lrow = wm * WROWS + i * 32 + qr * 16 + rrow + u;
          const int row = m0 + lrow;
          float m = -INFINITY, s = 0.f;
          int a = 0x7fffffff;
          // this lane's columns of the row, ascending: j*64 + wn*32 +
          // qc*16 + l16 for j, then qc
#pragma unroll
          for (int j = 0; j < TN; ++j) {
#pragma unroll
            for (int qc = 0; qc < 2; ++qc) {
              const int col = n0 + j * 64 + wn * 32 + qc * 16 + l16;
              float v = acc[i][j][qr * 2 + qc][u];
              if (ep.logits_out && row < m_live && col < ep.vocab)
                ep.logits_out[(size_t)ep.list[1 + row] * ep.vocab + col] = v;
              if (col == ep.mask_id || col >= ep.vocab) v = -INFINITY;
              if (v > m) {              // columns ascend: keeps the first
                s = s * __expf(m - v) + 1.0f;
                m = v; a = col;
              } else if (v != -INFINITY) {
                s += __expf(v - m);
              }
            }
          }
          // the 16 lanes holding this row (same lane / 16)
#pragma unroll
          for (int o = 1; o < 16; o <<= 1) {
            const float m2 = __shfl_xor(m, o, 64);
            const float s2 = __shfl_xor(s, o, 64);
            const int a2 = __shfl_xor(a, o, 64);
            const float mm = fmaxf(m, m2);
            float ns = 0.f;
            if (m != -INFINITY) ns += s * __expf(m - mm);
            if (m2 != -INFINITY) ns += s2 * __expf(m2 - mm);
            const int na = (m2 > m || (m2 == m && a2 < a)) ? a2 : a;
            m = mm; s = ns; a = na;
          }
          if (l16 == 0) {
            red_m[wn][lrow] = m;
            red_s[wn][lrow] = s;
            red_a[wn][lrow] = a;
          }
        }
      }
    }
    __syncthreads();
    for (int r = t; r < BM; r += 64 * WAVES) {
      const int row = m0 + r;
      if (row >= m_live) continue;
      const float m1 = red_m[0][r], m2 = red_m[1][r];
      const float mm = fmaxf(m1, m2);
      float s = 0.f;
      if (m1 != -INFINITY) s += red_s[0][r] * __expf(m1 - mm);
      if (m2 != -INFINITY) s += red_s[1][r] * __expf(m2 - mm);
      const int a1 = red_a[0][r], a2 = red_a[1][r];
      const int a = (m2 > m1 || (m2 == m1 && a2 < a1)) ? a2 : a1;
      const size_t o = (size_t)row * ep.n_slabs + nb;
      ep.pmax[o] = mm;
      ep.psum[o] = s;
      ep.parg[o] = a;
    }
  }
  if (nf && ep.overflow) atomicAdd(ep.overflow, nf);
  }  // M tiles
}

// Row tiles per band of the tile order.  An XCD works on 32 consecutive tiles
// at a time: in bands of 8 that is 8 row tiles x 4 columns, 12 operand tiles
// through its L2 instead of 33; up to 16 row tiles one band is as fast.
int m_band(int mt) { return mt > 16 ? 8 : mt; }

template <typename Fmt, typename V, int EPI>
int launch_tiles(const uint16_t* A, const uint16_t* B, const uint16_t* B2,
                 int M, int N, int K, int ksplit, EpiArgs ep,
                 hipStream_t s, int max_mtiles = 1 << 30) {
  const int mt = std::min((M + V::BM - 1) / V::BM, max_mtiles);
  const int nt = (N + V::BN - 1) / V::BN;
  const int nwg = mt * nt * ksplit;
  ep.m_band = m_band(mt);
  hipLaunchKernelGGL((gemm16_kernel<Fmt, V, EPI>), dim3(nwg),
                     dim3(64 * V::WAVES), 0, s, A, B, B2, M, N, K, mt, nt,
                     ksplit, ep);
  DAVET_HIP(hipGetLastError());
  return DAVET_OK;
}

// Joins another part (m2, s2, a2) into a row's (max, sum exp, first argmax).
__device__ __forceinline__ void head_join(float& m, float& s, int& a, float m2,
                                          float s2, int a2) {
  const float mm = fmaxf(m, m2);
  float ns = 0.f;
  if (m != -INFINITY) ns += s * __expf(m - mm);
  if (m2 != -INFINITY) ns += s2 * __expf(m2 - mm);
  a = (m2 > m || (m2 == m && a2 < a)) ? a2 : a;
  m = mm;
  s = ns;
}
template <int X>
__device__ __forceinline__ void head_join_lanes(float& m, float& s, int& a) {
  const float m2 = __shfl_xor(m, X, 64), s2 = __shfl_xor(s, X, 64);
  const int a2 = __shfl_xor(a, X, 64);
  head_join(m, s, a, m2, s2, a2);
}
// The 256 x 256 tile of 8 wavefronts in a 2 x 4 grid, a wave accumulating
// 128 x 64, K in slabs of 64.  A slab is worked off in two phases, a 64 x 64
// half of the wave's block each (32 matrix ops); a phase is a read section
// (LDS fragments, global->LDS loads of a later slab) and a matrix section,
// each closed by a barrier.  The waves of row 1 run one section behind those
// of row 0, and a SIMD holds one of each, so that one wave's reads always sit
// under the other's matrix ops.
//
// LDS: two slabs, each four 128-row half tiles (A0, A1, B0, B1) of 16 KB:
// half h of A holds rows h*64 .. +63 of both wave rows, half h of B the
// 16-column blocks 2h, 2h+1 of the four wave columns.  Phase 0 reads A0, B0
// and B1, phase 1 A1.  A read section ends with its fragments in registers, so
// from the next phase on both wave rows may load over what it read: slab
// t+2's A0, B0, B1 in phase 1 of slab t, its A1 in phase 0 of slab t+1, three
// phases before their first use.  What the next phase reads has landed once at
// most the eight youngest loads are outstanding.
//
// What bounds it: the part's power-limited clock and the hand-over between
// sections.  Gate/up of d = 4096, ffn = 12288 at 8000 rows, cold weights: the
// 16-wave tile 1284 us, this one 1260 (1.28 PFLOP/s; matrix pipes busy 68 %
// against 63 %); down 697 -> 671; at 3092 rows 538 -> 528 and 298 -> 290.
// Four phases of 16 matrix ops were 3 % slower; fragments read a phase ahead
// with two barriers a slab were as fast as the 16-wave tile; all loads of one
// tile's addresses (no cache misses) gain 3 %.
//
// The matrix ops take the weights as their first operand, so a lane holds four
// consecutive columns of one row per accumulator and stores (and, for the
// residual, loads) them as one vector.  Column block j of wave column wn is
// placed where the epilogue wants it (block_col).
template <int EPI>
__device__ __forceinline__ int block_col(int wn, int j, bool dual) {
  if (dual) return (j >> 1) * 128 + wn * 32 + (j & 1) * 16;  // gate | up
  if (EPI == EPI_STORE)          // dims i and i + 64 of a head in one lane
    return (wn >> 1) * 128 + (j >> 1) * 64 + (wn & 1) * 32 + (j & 1) * 16;
  return wn * 64 + j * 16;
}

template <typename Fmt, int EPI>
__global__ void __launch_bounds__(512, 1)
gemm16_phased_kernel(const uint16_t* __restrict__ A,
                     const uint16_t* __restrict__ B,
                     const uint16_t* __restrict__ B2, int M, int N, int K,
                     int n_mtiles, int n_ntiles, int ksplit, EpiArgs ep) {
  using v8 = typename Fmt::v8;
  constexpr int HALF = 128 * 64 * 2;           // bytes of a half tile
  constexpr int SLAB = 4 * HALF;
  enum { A0 = 0, A1 = 1, B0 = 2, B1 = 3 };
  __shared__ __attribute__((aligned(1024))) char smem[2 * SLAB];

  int mb, ks, nb;
  locate_tile(remap_xcd(blockIdx.x, gridDim.x), n_mtiles, n_ntiles, ksplit,
              ep.m_band, mb, ks, nb);
  int m_live = M;
  if constexpr (EPI == EPI_HEAD) m_live = ep.list[0];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const int l16 = lane & 15, k4 = lane >> 4;
  const bool dual = (EPI == EPI_SWIGLU) || (EPI == EPI_PARTIAL && ep.dual);
  const bool tiled = EPI == EPI_HEAD && ep.b_tiled;
  const int nk_all = K / 64;
  const int chunk = (nk_all + ksplit - 1) / ksplit;
  const int kt0 = ks * chunk;
  const int nk = min(nk_all, kt0 + chunk) - kt0;

  // row tiles mb, mb + n_mtiles, ... (one, unless the head's grid is narrower
  // than its live rows)
  for (int mt = mb; mt * 256 < m_live; mt += n_mtiles) {
  const int m0 = mt * 256;
  if (mt != mb) __syncthreads();      // LDS of the previous tile retired

  // The two loads of a half bring rows (wave * 2 + q) * 8 + lane / 8 of it,
  // 16-byte chunk swizzled.  A lane's byte offsets are the same for both
  // halves of an operand; rows of A past the last live one lie past the
  // buffer's end and read as zeros.
  uint32_t off_a[2], off_b[2];
  const int b_block = min(nb * 2, (N - 1) >> 7);      // tiled head: 128 rows
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int r = (wave * 2 + q) * 8 + (lane >> 3);
    const uint32_t c = ((lane & 7) ^ ((r >> 1) & 7)) * 16;
    off_a[q] = (uint32_t)((r >> 6) * 128 + (r & 63)) * (uint32_t)(K * 2) + c;
    const int col = block_col<EPI>(r >> 5, (r >> 4) & 1, dual) + (r & 15);
    if (tiled)
      off_b[q] = (uint32_t)((min(nb * 2 + (col >> 7), (N - 1) >> 7) - b_block) *
                                128 + (col & 127)) * 128 + c;
    else
      off_b[q] = (uint32_t)col * (uint32_t)(K * 2) + c;
  }
  const char* base_a = reinterpret_cast<const char*>(A + (size_t)m0 * K + (size_t)kt0 * 64);
  const uint32_t size_a =
      (uint32_t)min(256, m_live - m0) * (uint32_t)(K * 2) - (uint32_t)kt0 * 128;
  const char *base_b, *base_b1;
  if (tiled) {
    base_b = reinterpret_cast<const char*>(B + (size_t)b_block * 128 * 64);
    base_b1 = base_b + 32 * 128;
  } else {
    const size_t at = (size_t)nb * (dual ? 128 : 256) * K + (size_t)kt0 * 64;
    base_b = reinterpret_cast<const char*>(B + at);
    base_b1 = dual ? reinterpret_cast<const char*>(B2 + at)
                   : base_b + (size_t)(EPI == EPI_STORE ? 64 : 32) * K * 2;
  }
  // bytes to the next 64 K columns: a tiled head (never split) steps over all
  // its blocks
  const size_t b_step = tiled ? (size_t)((N + 127) / 128) * 128 * 64 * 2 : 128;
  auto issue = [&](int half, int kt) {
    char* dst = smem + (kt & 1) * SLAB + half * HALF + wave * 2048;
    if (half < 2) {
      const uint32_t skip = (uint32_t)kt * 128 + (half ? (uint32_t)K * 128 : 0u);
      const uint32_t left =
          __builtin_amdgcn_readfirstlane(skip < size_a ? size_a - skip : 0u);
      dma16_from(base_a + skip, left, off_a[0], dst);
      dma16_from(base_a + skip, left, off_a[1], dst + 1024);
    } else {
      const char* from = (half == B0 ? base_b : base_b1) + (size_t)kt * b_step;
      dma16_from(from, 0xffffffffu, off_b[0], dst);
      dma16_from(from, 0xffffffffu, off_b[1], dst + 1024);
    }
  };

  // fragment addresses inside a slab: row wm*64 + i*16 + l16 of a half of A,
  // wn*32 + j*16 + l16 of B; the swizzle depends on l16 alone
  const int sw = (l16 >> 1) & 7;
  const int c0 = (k4 ^ sw) << 4, c1 = ((4 + k4) ^ sw) << 4;
  const int ra = (wm * 64 + l16) * 128, rb = B0 * HALF + (wn * 32 + l16) * 128;
  v8 fa[4][2], fb[4][2];
  // acc[i][j][u]: row wm*128 + i*16 + l16, column block_col(wn, j) + k4*4 + u
  f32x4 acc[8][4];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[i][j][u] = 0.f;
  // wave rows past the last live one are not multiplied
  const bool live0 = m0 + wm * 128 < m_live, live1 = m0 + wm * 128 + 64 < m_live;

  auto section_end = [&] {
    __builtin_amdgcn_sched_barrier(0);
    barrier_nofence();
    __builtin_amdgcn_sched_barrier(0);
  };
  auto read_a = [&](const char* s) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      fa[i][0] = *reinterpret_cast<const v8*>(s + ra + i * 2048 + c0);
      fa[i][1] = *reinterpret_cast<const v8*>(s + ra + i * 2048 + c1);
    }
  };
  auto read_b = [&](const char* s) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const char* r = s + (j >> 1) * HALF + rb + (j & 1) * 2048;
      fb[j][0] = *reinterpret_cast<const v8*>(r + c0);
      fb[j][1] = *reinterpret_cast<const v8*>(r + c1);
    }
  };
  // ends a read section: its fragments are in registers, and of the loads all
  // but the N youngest have landed
  auto read_end = [&](auto n) {
    constexpr int N_ = decltype(n)::value;
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N_) : "memory");
    section_end();
  };
  auto multiply = [&](auto qa, bool live) {
    constexpr int QA = decltype(qa)::value;
    if (live) {
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[QA * 4 + i][j] =
                Fmt::mfma16(fb[j][kk], fa[i][kk], acc[QA * 4 + i][j]);
      __builtin_amdgcn_s_setprio(0);
    }
    section_end();
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I8 = std::integral_constant<int, 8>;
  // LAST = 0: slab kt+2 exists; 1: kt is the last but one; 2: the last
  auto slab = [&](int kt, auto last) {
    constexpr int LAST = decltype(last)::value;
    const char* s = smem + (kt & 1) * SLAB;
    read_b(s);
    read_a(s);
    if constexpr (LAST < 2) {
      issue(A1, kt + 1);
      read_end(I8{});
    } else {
      read_end(I0{});
    }
    multiply(I0{}, live0);

    read_a(s + HALF);
    if constexpr (LAST == 0) {
      issue(A0, kt + 2);
      issue(B0, kt + 2);
      issue(B1, kt + 2);
      read_end(I8{});
    } else {
      read_end(I2{});
    }
    multiply(I1{}, live1);
  };

  issue(A0, 0);
  issue(B0, 0);
  issue(B1, 0);
  issue(A1, 0);
  if (nk > 1) {
    issue(A0, 1);
    issue(B0, 1);
    issue(B1, 1);
    wait_vmcnt<8>();
  } else {
    wait_vmcnt<2>();
  }
  section_end();
  if (wm == 1) section_end();
  for (int kt = 0; kt + 2 < nk; ++kt) slab(kt, I0{});
  if (nk > 1) slab(nk - 2, I1{});
  slab(nk - 1, I2{});
  if (wm == 0) section_end();

  // ---------------------------------------------------------------- epilogue
  int nf = 0;     // non-finite 16-bit values stored by this lane
  auto store4 = [&](uint16_t* C, const uint16_t (&h)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) nf += Fmt::nonfinite(h[u]);
    u32x2 w;
    w[0] = h[0] | (uint32_t)h[1] << 16;
    w[1] = h[2] | (uint32_t)h[3] << 16;
    *reinterpret_cast<u32x2*>(C) = w;
  };
  const int row0 = m0 + wm * 128 + l16;
  if constexpr (EPI == EPI_STORE) {
    uint16_t* C = reinterpret_cast<uint16_t*>(ep.C) + nb * 256;
    const bool rope = ep.pos && nb * 256 + (wn >> 1) * 128 < ep.rope_cols;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int row = row0 + i * 16;
      if (row >= M) continue;
      uint16_t* crow = C + (size_t)row * ep.ldc + k4 * 4;
      const float2* cs = rope ? ep.cs + (size_t)ep.pos[row] * 64 : nullptr;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int col = block_col<EPI>(wn, j, false);
        uint16_t x[4], y[4];
        if (rope) {
          const float4* c4 = reinterpret_cast<const float4*>(cs + (col & 63) + k4 * 4);
          const float4 p = c4[0], q = c4[1];
          const float cc[4] = {p.x, p.z, q.x, q.z}, ss[4] = {p.y, p.w, q.y, q.w};
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float a = acc[i][j][u], b = acc[i][j + 2][u];
            // contracted as in the other tiles' epilogue: the same bits
            x[u] = Fmt::store_fma(a, cc[u], -(b * ss[u]));
            y[u] = Fmt::store_fma(a, ss[u], b * cc[u]);
          }
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            x[u] = Fmt::store(acc[i][j][u]);
            y[u] = Fmt::store(acc[i][j + 2][u]);
          }
        }
        store4(crow + col, x);
        store4(crow + col + 64, y);
      }
    }
  } else if constexpr (EPI == EPI_ADD_F32) {
    float* C = reinterpret_cast<float*>(ep.C) + nb * 256 + wn * 64 + k4 * 4;
    // the residual rows are fetched two blocks of 16 at a time, ahead of the
    // stores (which the compiler cannot move loads across)
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
      f32x4 x[2][4];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int row = min(row0 + (i + h) * 16, M - 1);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          x[h][j] = *reinterpret_cast<const f32x4*>(C + (size_t)row * ep.ldc + j * 16);
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int row = row0 + (i + h) * 16;
        if (row >= M) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          f32x4 v;
#pragma unroll
          for (int u = 0; u < 4; ++u) v[u] = x[h][j][u] + acc[i + h][j][u];
          *reinterpret_cast<f32x4*>(C + (size_t)row * ep.ldc + j * 16) = v;
        }
      }
    }
  } else if constexpr (EPI == EPI_SWIGLU) {
    uint16_t* C = reinterpret_cast<uint16_t*>(ep.C) + nb * 128;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int row = row0 + i * 16;
      if (row >= M) continue;
      uint16_t* crow = C + (size_t)row * ep.ldc + k4 * 4;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        uint16_t h[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float g = acc[i][j][u];
          h[u] = Fmt::store_mul(g / (1.0f + __expf(-g)), acc[i][j + 2][u]);
        }
        store4(crow + block_col<EPI>(wn, j, true), h);
      }
    }
  } else if constexpr (EPI == EPI_PARTIAL) {
    float* P = ep.part + (size_t)ks * M * ep.part_ld + k4 * 4;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int row = row0 + i * 16;
      if (row >= M) continue;
      float* prow = P + (size_t)row * ep.part_ld;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int c = block_col<EPI>(wn, j, dual);
        const int col = dual ? (j < 2 ? 0 : ep.ffn) + nb * 128 + (c & 127)
                             : nb * 256 + c;
        *reinterpret_cast<f32x4*>(prow + col) = acc[i][j];
      }
    }
  } else {   // EPI_HEAD
    // (max, sum exp, first argmax) of each row over the tile's 256 columns:
    // 16 in a lane, then the four lanes of the row, then the four wave columns
    // through the slabs' LDS, which every wave is done with after the barrier
    __syncthreads();
    float* red_m = reinterpret_cast<float*>(smem);      // [4][256] each
    float* red_s = red_m + 1024;
    int* red_a = reinterpret_cast<int*>(red_s + 1024);
    const int col0 = nb * 256 + wn * 64 + k4 * 4;
    const bool vec = (ep.vocab & 3) == 0 && ((uintptr_t)ep.logits_out & 15) == 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int row = row0 + i * 16;
      if (ep.logits_out && row < m_live) {
        float* lrow = ep.logits_out + (size_t)ep.list[1 + row] * ep.vocab;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int col = col0 + j * 16;
          if (vec) {
            if (col < ep.vocab) *reinterpret_cast<f32x4*>(lrow + col) = acc[i][j];
          } else {
#pragma unroll
            for (int u = 0; u < 4; ++u)
              if (col + u < ep.vocab) lrow[col + u] = acc[i][j][u];
          }
        }
      }
      float m = -INFINITY, s = 0.f;
      int a = 0x7fffffff;
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int u = 0; u < 4; ++u) {           // columns ascend: keeps the first
          const int col = col0 + j * 16 + u;
          float v = acc[i][j][u];
          if (col == ep.mask_id || col >= ep.vocab) v = -INFINITY;
          acc[i][j][u] = v;
          if (v > m) { m = v; a = col; }
        }
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (acc[i][j][u] != -INFINITY) s += __expf(acc[i][j][u] - m);
      head_join_lanes<16>(m, s, a);
      head_join_lanes<32>(m, s, a);
      if (k4 == 0) {
        const int o = wn * 256 + wm * 128 + i * 16 + l16;
        red_m[o] = m;
        red_s[o] = s;
        red_a[o] = a;
      }
    }
    __syncthreads();
    if (t < 256 && m0 + t < m_live) {
      float m = red_m[t], s = red_s[t];
      int a = red_a[t];
#pragma unroll
      for (int w = 1; w < 4; ++w)
        head_join(m, s, a, red_m[w * 256 + t], red_s[w * 256 + t], red_a[w * 256 + t]);
      const size_t o = (size_t)(m0 + t) * ep.n_slabs + nb;
      ep.pmax[o] = m;
      ep.psum[o] = s;
      ep.parg[o] = a;
    }
  }
  if (nf && ep.overflow) atomicAdd(ep.overflow, nf);
  }  // row tiles
}

template <typename Fmt, int EPI>
int launch_phased(const uint16_t* A, const uint16_t* B, const uint16_t* B2,
                  int M, int N, int K, int ksplit, EpiArgs ep, hipStream_t s,
                  int max_mtiles = 1 << 30) {
  const int mt = std::min((M + 255) / 256, max_mtiles);
  const int nt = (N + 255) / 256;
  ep.m_band = m_band(mt);
  hipLaunchKernelGGL((gemm16_phased_kernel<Fmt, EPI>), dim3(mt * nt * ksplit),
                     dim3(512), 0, s, A, B, B2, M, N, K, mt, nt, ksplit, ep);
  DAVET_HIP(hipGetLastError());
  return DAVET_OK;
}

// The kernel variants the planner can pick (index = GemmPlan::tile; the
// indices are those of the measurement tables, other tiles measured slower).
// V6 with the scheduler's interleaving strategy 1: measured on MI355X
// (candidates interleaved launch by launch, cold weights) never slower on any
// table entry that uses it, median 5 % faster; the 256 x 256 and 8-wave
// 128 x 128 tiles gain nothing from it.  V14 with explicit schedule groups
// (SG = 1): 4-8 % faster than with strategy 0 on each of nine products at
// 300-2916 rows, on three parts
using V6 = Var<128, 128, 64, 2, 4, 1>; // 64 KB, 2 workgroups per CU
using V8 = Var<256, 256, 64, 2, 8>;    // 128 KB, deep slabs, large M
using V12 = Var<128, 128, 64, 2, 8>;   // 64 KB, 8 wavefronts, 2 WG/CU
// 192-row tiles: fewer padded rows and a fuller last wave of workgroups for
// sequences of ~700-3000 tokens (3 sub-tiles of 32 rows per wave)
using V14 = Var<192, 128, 64, 2, 4, -1, 2, 1>; // 80 KB, 2 workgroups per CU
using V15 = Var<128, 256, 32, 3, 8>;   // 72 KB: tiled vocabulary head
// 16 wavefronts in a 4 x 4 grid (64 x 64 per wave) with the scheduler's
// interleaving strategy 0
using V16 = Var<256, 256, 64, 2, 16, 0, 4>;
constexpr int PHASED = 17;             // gemm16_phased_kernel
// its lanes' offsets into 256 rows of K 16-bit values fit 32 bits
constexpr int PHASED_MAX_K = 1 << 22;
constexpr int ceil_div(int a, int b) { return (a + b - 1) / b; }

int variant_bn(int tile) {
  switch (tile) {
    case 8: case 15: case 16: case PHASED: return 256;
    default: return 128;
  }
}
int variant_bm(int tile) {
  switch (tile) {
    case 14: return 192;
    case 8: case 16: case PHASED: return 256;
    default: return 128;
  }
}
int variant_bk(int tile) {
  return tile == 15 ? 32 : 64;
}
bool variant_known(int tile) {
  return tile == 6 || tile == 8 || tile == 12 || tile == 14 || tile == 16 ||
         tile == PHASED;
}

template <typename Fmt, int EPI>
int launch_shape(const GemmPlan& p, const uint16_t* A, const uint16_t* B,
                 const uint16_t* B2, int M, int N, int K, const EpiArgs& ep,
                 hipStream_t s) {
#define LV(Vn) return launch_tiles<Fmt, Vn, EPI>(A, B, B2, M, N, K, p.ksplit, ep, s)
  switch (p.tile) {
    case 6: LV(V6);
    case 8: LV(V8);
    case 12: LV(V12);
    case 14: LV(V14);
    case 16: LV(V16);
    case PHASED:
      return launch_phased<Fmt, EPI>(A, B, B2, M, N, K, p.ksplit, ep, s);
    default: return set_error(DAVET_EINVAL, "gemm16: unknown tile variant");
  }
#undef LV
}

template <typename Fmt>
int gemm_dispatch(const GemmPlan& p, int epi, const uint16_t* A,
                  const uint16_t* B, const uint16_t* B2, int M, int N, int K,
                  const EpiArgs& ep, hipStream_t s) {
  if (p.ksplit > 1)
    return launch_shape<Fmt, EPI_PARTIAL>(p, A, B, B2, M, N, K, ep, s);
  switch (epi) {
    case EPI_STORE: return launch_shape<Fmt, EPI_STORE>(p, A, B, B2, M, N, K, ep, s);
    case EPI_ADD_F32: return launch_shape<Fmt, EPI_ADD_F32>(p, A, B, B2, M, N, K, ep, s);
    case EPI_SWIGLU: return launch_shape<Fmt, EPI_SWIGLU>(p, A, B, B2, M, N, K, ep, s);
  }
  return set_error(DAVET_EINVAL, "gemm16: unknown epilogue");
}

}  // namespace

// Kernel choice.  For the projections of a d = 4096, ffn = 12288 layer the
// plan is a table measured on MI355X with the weights and activations cold in
// the last-level cache (as inside a denoising step) at 26 token counts: the
// fastest (tile variant, K split) of a sweep over the variants 6, 8, 12, 13,
// 14 and splits {1, 2, 3, 4, 6, 8}, the split-K reduction included (a
// variant replaced the previous choice only when more than 3 % faster); a
// re-sweep on random data with 5-way splits added changed three entries that
// another plan beat by more than 5 % in both of two repetitions (a fourth,
// QKV at 209 rows with 5 splits, measured 1.2 % slower inside the step: its
// larger partials cost the reduction more than the sweep's cold-cache timing
// shows, and was left out).  After the move to 16 x 16 x 32 matrix ops a
// third sweep (variants 4, 6-9 and 12-14, splits 1-6 and 8, the split-K
// reduction or the following norm included) changed thirteen entries whose
// new plan was more than 4 % faster in each of three repetitions.  The
// 4 x 4-wave tile (V16) then replaced an 8 x 2 one wherever it was not slower,
// timed interleaved on every entry: median 5.8 % faster, bit-identical outputs.
// A last interleaved sweep over the current variants (6, 8, 12, 13, 14, 16
// with their scheduling hints, splits 1-6 and 8) moved 21 entries whose new
// plan was at least 3 % faster; a check of gate/up at 330-520 rows on two
// parts then moved three more (192 x 128 at 356, 4 x 4-wave 256 x 256 at 420
// and 480: 12 % and 6 % faster), and one at 150-250 rows (8-wave 128 x 128
// without a K split instead of 256 x 256 with two: 2-14 % faster).
// The phased tile (17) then took the entries where it measured faster (sweep of
// variants 6, 8, 12, 14, 16 and 17, splits 1-6 and 8; 2-9 % each): gate/up from
// 1700 rows except 2600 and at 356-480, down from 2300 rows except 2916 and at
// 1300, QKV at 650-750, 1700-2300, 3300, 12000 and 18020, output at 18020.  Of
// the other tiles' entries that sweep moved QKV at 300 and 356 and output at 889
// (49 us with two splits of V6, 51 with four of V16) and 5000.  Down at 2300
// keeps the three splits it had on an older tile (2171-2445 rows 231-245 us,
// 258-268 on that tile, 261-273 without a split).  The edge ranges below were not
// timed against it.
// Because the number of row tiles and of waves of workgroups changes in
// steps, the best plan is jagged in M; a product of M rows takes the plan of
// the nearest sample point in log M, except in the ranges of kEdge.
constexpr int kPointM[] = {209, 300, 356, 420, 480, 565, 650, 750, 889,
                           960, 1100, 1300, 1500, 1700, 2048, 2300, 2600,
                           2916, 3092, 3300, 3645, 3965, 5000, 8000, 12000,
                           18020};
constexpr int kNP = 26;
struct TableShape { int N, K; GemmPlan plan[kNP]; };
constexpr TableShape kTable[] = {
    // QKV: N = 3d, K = d
    {12288, 4096, {{8, 5}, {14, 2}, {16, 2}, {16, 2}, {16, 2}, {12, 1}, {17, 1}, {17, 1}, {16, 1}, {16, 1}, {16, 1}, {14, 2}, {14, 2}, {17, 1}, {17, 1}, {17, 1}, {16, 1}, {16, 1}, {16, 1}, {17, 1}, {16, 1}, {16, 1}, {16, 1}, {16, 1}, {17, 1}, {17, 1}}},
    // output projection: N = d, K = d
    {4096, 4096, {{6, 8}, {6, 5}, {6, 4}, {6, 4}, {12, 4}, {6, 3}, {6, 2}, {12, 2}, {6, 2}, {6, 2}, {16, 3}, {14, 2}, {14, 2}, {16, 2}, {6, 1}, {14, 1}, {14, 1}, {14, 1}, {16, 1}, {16, 1}, {16, 1}, {16, 1}, {14, 1}, {16, 1}, {16, 1}, {17, 1}}},
    // gate + up: N = 2 ffn, K = d
    {24576, 4096, {{12, 1}, {14, 1}, {17, 1}, {17, 1}, {17, 1}, {12, 1}, {14, 1}, {14, 1}, {14, 1}, {14, 1}, {16, 1}, {14, 1}, {14, 1}, {17, 1}, {17, 1}, {17, 1}, {16, 1}, {17, 1}, {17, 1}, {17, 1}, {17, 1}, {17, 1}, {17, 1}, {17, 1}, {17, 1}, {17, 1}}},
    // down projection: N = d, K = ffn
    {4096, 12288, {{12, 8}, {14, 8}, {16, 8}, {16, 8}, {8, 8}, {16, 5}, {16, 5}, {8, 5}, {16, 4}, {16, 4}, {16, 3}, {17, 2}, {14, 2}, {16, 2}, {16, 2}, {17, 3}, {17, 1}, {14, 1}, {17, 1}, {17, 1}, {17, 1}, {17, 1}, {17, 2}, {17, 1}, {17, 1}, {17, 1}}},
};

// Row counts just past a multiple of a point's tile height, where the point's
// plan would add a nearly empty row tile the point itself does not have: the
// plan measured there instead (each range timed at one row count inside it,
// interleaved against the point's plan: 3-35 % faster; ranges where the next
// point's plan was not faster keep the point's own).
struct EdgeRange { int N, K, lo, hi; GemmPlan plan; };
constexpr EdgeRange kEdge[] = {
    {12288, 4096, 513, 520, {12, 1}},   {12288, 4096, 1537, 1596, {12, 1}},
    {4096, 4096, 513, 520, {6, 3}},     {4096, 4096, 1025, 1027, {16, 3}},
    {4096, 4096, 1537, 1596, {16, 2}},  {4096, 4096, 1793, 1865, {6, 1}},
    {4096, 4096, 2049, 2170, {14, 1}},
    {24576, 4096, 385, 386, {16, 1}},   {24576, 4096, 513, 520, {12, 1}},
    {24576, 4096, 961, 1027, {16, 1}},  {24576, 4096, 1537, 1596, {16, 1}},
    {24576, 4096, 2049, 2170, {14, 1}}, {24576, 4096, 2305, 2445, {16, 1}},
    {4096, 12288, 513, 520, {16, 5}},   {4096, 12288, 769, 816, {16, 4}},
    {4096, 12288, 1025, 1027, {16, 3}}, {4096, 12288, 1537, 1596, {16, 2}},
    {4096, 12288, 2049, 2170, {16, 3}}, {4096, 12288, 4097, 4352, {16, 2}},
};

// Point i serves the rows up to the geometric mean of points i and i+1.
static int point_index(int M) {
  int i = 0;
  while (i + 1 < kNP && (double)M * M > (double)kPointM[i] * kPointM[i + 1]) ++i;
  return i;
}
static int point_top(int i) {            // largest M served by point i
  if (i + 1 >= kNP) return 1 << 30;
  int m = (int)std::sqrt((double)kPointM[i] * kPointM[i + 1]);
  while ((double)(m + 1) * (m + 1) <= (double)kPointM[i] * kPointM[i + 1]) ++m;
  while ((double)m * m > (double)kPointM[i] * kPointM[i + 1]) --m;
  return m;
}

static const TableShape* table_shape(int N, int K) {
  for (const TableShape& t : kTable)
    if (t.N == N && t.K == K) return &t;
  return nullptr;
}

// Other shapes: the (tile, K split) with the least modelled time, in us.
// A product costs a start, a K slab of 64 per slab and round of workgroups
// (less while a tile has its CU to itself), an epilogue per round (the rotary
// store's scattered 2-byte stores cost the older tiles more, four waves most),
// for a split the partials through memory and a second kernel, and never less
// than its weights' stream.  The constants are a fit to 644 products at fifteen
// widths (M 100 - 9000, d 512 - 8192, weights cold; every tile, splits 1 - 6 and
// 8): the plan so chosen is on average 1.5 % slower than the best one measured,
// 0.6 % over the summed times.  Constants fitted to one half of the widths do as
// well on the other (1.6 % and 0.5 %).  With the two 256 x 256 tiles priced
// alike the older one always won: 3.2 % and 4.2 %, although the phased tile takes
// 0.92 - 0.99 of its time at K splits of one.  A rule by row counts alone (128 x
// 128 tiles, K split by powers of two up to 256 tiles for N < 8192, 256 x 256
// tiles past 2-3 thousand rows) was 26 % slower over 140 products.
struct TileCost { int tile; double single, pair, epilogue, rotary; };
constexpr TileCost kTileCost[] = {
    // us a slab alone on a CU and in a pair (0: never two on a CU), us of
    // epilogue, and of rotary store, per round and 256 x 256 elements
    {6, 0.89, 1.00, 3.9, 31.0}, {12, 0.82, 1.04, 3.6, 4.5},
    {14, 1.00, 1.36, 4.8, 35.0}, {16, 1.75, 0, 2.0, 5.2},
    {PHASED, 1.30, 0, 6.5, 0},
};
constexpr size_t GENERIC_PARTIALS = (size_t)512 * 256 * 256 * 4;

static GemmPlan plan_generic(int M, int N, int K, bool rotary) {
  GemmPlan best{12, 1};
  double best_us = 1e30;
  const double stream = 2.0 * N * K / 6.6e6;
  const int slabs = K / 64;
  for (const TileCost& c : kTileCost) {
    const int bm = variant_bm(c.tile), bn = variant_bn(c.tile);
    if (N % bn || (c.tile == PHASED && K > PHASED_MAX_K)) continue;
    const double tiles = (double)ceil_div(M, bm) * (N / bn);
    for (int ks = 1; ks <= 8; ++ks) {
      const int part = ceil_div(slabs, ks);
      const double partials = 4.0 * ks * M * N;
      if (ks == 7) continue;        // the reductions take 2-6 and 8
      if (ks > 1 && (part < 4 || ceil_div(slabs, part) != ks ||
                     partials > (double)GENERIC_PARTIALS))
        continue;
      const double per_cu = std::ceil(tiles * ks / 256);
      const double pairs = c.pair > 0 ? std::floor(per_cu / 2) : 0;
      const double rounds = c.pair > 0 ? std::ceil(per_cu / 2) : per_cu;
      const double mul = part * (pairs * c.pair + (per_cu - 2 * pairs) * c.single);
      const double epi = rounds * bm * bn / 65536 *
                         (c.epilogue + (rotary && ks == 1 ? c.rotary : 0));
      const double us = 4.6 + epi + std::max(mul, stream) +
                        (ks > 1 ? 1.0 + 0.9 * 2 * partials / 5e6 : 0);
      if (us < best_us) {
        best_us = us;
        best = {c.tile, ks};
      }
    }
  }
  return best;
}

GemmPlan plan_gemm16(int M, int N, int K, bool rotary) {
  if (const TableShape* t = table_shape(N, K)) {
    for (const EdgeRange& e : kEdge)
      if (e.N == N && e.K == K && M >= e.lo && M <= e.hi) return e.plan;
    return t->plan[point_index(M)];
  }
  return plan_generic(M, N, K, rotary);
}

// Largest split-K partial buffer (bytes) any M <= max_M needs.  Table shapes:
// within a run of rows that share one plan the size grows with M, so the
// bound is reached at the top of a point's range, of an edge range or of the
// rows below an edge range (or at max_M).  Other shapes: the planner's limit.
size_t gemm16_partial_bound(int max_M, int N, int K) {
  size_t best = 0;
  auto at = [&](int m) {
    if (m < 1) return;
    const GemmPlan p = plan_gemm16(m, N, K, false);
    if (p.ksplit > 1) best = std::max(best, (size_t)p.ksplit * m * N * 4);
  };
  if (table_shape(N, K)) {
    for (int i = 0; i < kNP; ++i) at(std::min(max_M, point_top(i)));
    for (const EdgeRange& e : kEdge)
      if (e.N == N && e.K == K) {
        at(std::min(max_M, e.lo - 1));
        at(std::min(max_M, e.hi));
      }
    at(max_M);
    return best;
  }
  return GENERIC_PARTIALS;
}

int launch_gemm16(int dtype, int epi, const GemmPlan& plan, const uint16_t* A,
                  const uint16_t* B, const uint16_t* B2, void* C, int M, int N,
                  int K, int ldc, const int32_t* pos, const float* cs,
                  int rope_cols, float* partials, size_t partial_cap, int cls,
                  hipStream_t s, int32_t* overflow) {
  if (M <= 0) return DAVET_OK;
  if (plan.ksplit > 1 && (size_t)plan.ksplit * M * N * 4 > partial_cap)
    return set_error(DAVET_ENOMEM, "gemm16: split-K partials exceed the workspace");
  if (!variant_known(plan.tile))
    return set_error(DAVET_EINVAL, "gemm16: unknown tile variant");
  if (N % variant_bn(plan.tile) || K % variant_bk(plan.tile) ||
      (plan.ksplit > 1 && (K / variant_bk(plan.tile)) < plan.ksplit))
    return set_error(DAVET_ESHAPE, "gemm16: N or K not a multiple of the tile");
  if (plan.tile == PHASED &&
      (K > PHASED_MAX_K || ceil_div(K / 64, ceil_div(K / 64, plan.ksplit)) != plan.ksplit))
    return set_error(DAVET_ESHAPE, "gemm16: K out of range or a K split without work");
  if (plan.ksplit > 1 && !partials)
    return set_error(DAVET_EINVAL, "gemm16: split-K needs a partial buffer");
  ProfScope ps(cls, s);
  EpiArgs ep{};
  ep.C = C;
  ep.ldc = ldc;
  ep.pos = pos;
  ep.cs = reinterpret_cast<const float2*>(cs);
  ep.rope_cols = rope_cols;
  ep.part = partials;
  ep.part_ld = N;
  ep.dual = epi == EPI_SWIGLU;
  ep.ffn = N / 2;
  ep.overflow = overflow;
  return dtype == DAVET_F16
             ? gemm_dispatch<F16>(plan, epi, A, B, B2, M, N, K, ep, s)
             : gemm_dispatch<BF16>(plan, epi, A, B, B2, M, N, K, ep, s);
}

// The head kernel a launch runs, for a bound `live` on its live rows.  The
// tiled layout streams 256-column slabs: while at most 128 rows (or an odd
// number of 128-row tiles up to five) are live, 128 x 256 tiles with a
// 32-deep ring (V15: each activation tile re-read for half as many slabs as
// with 128-column slabs, one round of 494 workgroups; measured on MI355X at
// V = 126464, d = 4096: 188 -> 181 us at 2 live rows, 262 -> 232 at 128
// against 128 x 128 tiles); otherwise the head is bound by its matrix work
// and takes the phased 256 x 256 tile, whose cost steps with every 256 rows
// where V15's steps with every 128.  Logits are the same bits whichever runs;
// the slab partials' sums are grouped differently.  The
// row-major layout takes 128 x 128 tiles with 8 wavefronts.
static int head16_variant(int tiled, int live) {
  if (!tiled) return 12;
  const int n128 = (std::max(live, 1) + 127) / 128;
  return (n128 == 1 || (n128 % 2 == 1 && n128 <= 5)) ? 15 : PHASED;
}

int head16_slabs(int vocab, int tiled, int live_bound) {
  const int bn = variant_bn(head16_variant(tiled, live_bound));
  return (vocab + bn - 1) / bn;
}

int launch_head16(int dtype, const uint16_t* Hm, const uint16_t* W,
                  const int32_t* list, int max_rows, int vocab, int d,
                  int mask_id, float* pmax, float* psum, int32_t* parg,
                  float* logits_out, hipStream_t s, int tiled,
                  int live_bound) {
  // Row-major head: 8 wavefronts on the 128 x 128 tile (V12 over V6): the
  // matrix work of a slab is spread over twice the waves, so it hides behind
  // the other workgroup's stream (measured on MI355X: 201 -> 187 us at 2 live
  // rows, 214 -> 192 at 64)
  const int live = live_bound < 0 ? max_rows : std::min(max_rows, live_bound);
  const int variant = head16_variant(tiled, live);
  if (d % BK_MIN) return set_error(DAVET_ESHAPE, "head16: d % 32 != 0");
  ProfScope ps(KC_HEAD, s);
  EpiArgs ep{};
  ep.list = list;
  ep.vocab = vocab;
  ep.mask_id = mask_id;
  ep.n_slabs = head16_slabs(vocab, tiled, live);
  ep.pmax = pmax;
  ep.psum = psum;
  ep.parg = parg;
  ep.logits_out = logits_out;
  ep.b_tiled = tiled;
  if (tiled && d % 64)
    return set_error(DAVET_EINVAL, "head16: the tiled head needs d % 64 == 0");
  // m_slots M slots per vocabulary slab: a workgroup loops over the live row
  // tiles mb, mb + m_slots, ...  m_slots covers live_bound, a bound on the
  // live rows the caller knows on the host (the schedule loop's: at most
  // L - k(t-1) per sequence; a looser bound is still correct), so one slot
  // per live tile streams a slab's weights from HBM once (the tiles of a slab
  // sit on one XCD and share its L2), and late steps with few masked rows
  // launch no idle workgroups.
  const int bm = variant_bm(variant);
  const int m_slots = std::max(1, (live + bm - 1) / bm);
#define HV(Fmt, Vn) return launch_tiles<Fmt, Vn, EPI_HEAD>(Hm, W, nullptr, max_rows, vocab, d, 1, ep, s, m_slots)
#define HEAD_VARIANTS(Fmt)       \
  switch (variant) {             \
    case 12: HV(Fmt, V12);       \
    case PHASED: return launch_phased<Fmt, EPI_HEAD>(Hm, W, nullptr, max_rows, vocab, d, 1, ep, s, m_slots); \
    case 15: HV(Fmt, V15);       \
  }
  if (dtype == DAVET_F16) {
    HEAD_VARIANTS(F16)
  } else {
    HEAD_VARIANTS(BF16)
  }
  return set_error(DAVET_EINVAL, "head16: no such head variant");
#undef HEAD_VARIANTS
#undef HV
}

}  // namespace davet
