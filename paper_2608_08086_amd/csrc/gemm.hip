// Projection GEMMs Y = A W^T of the Archer path with fused epilogues.
//
// bf16 kernel: LDS-tiled MFMA (v_mfma_f32_16x16x32_bf16, fp32 accumulate),
// 256 threads = 4 wave64s in a WGM x WGN grid, double-buffered LDS tiles in
// an XOR-swizzled layout (16-byte chunk c of row r is stored at chunk
// c ^ (r mod chunks-per-row): conflict-free fragment reads, no padding), and a
// one-tile-ahead register prefetch of the global loads.
//
// Split-K.  The K range of a GEMM is cut into S slices, S chosen from (N, K)
// only.  A launch either gives each slice its own workgroup, which writes an
// fp32 partial, and a second kernel sums the partials in slice order and
// applies the epilogue; or runs all slices in one workgroup, accumulating each
// slice from zero and adding the slice sums in the same order.  Both give the
// same bits, so a row's result never depends on how many rows are in the
// launch (CachedForward on its own cache equals FullForward bitwise).
//
// Column pairing (gemm_common.h): tile column r and r + BN/2 are an RoPE or
// SwiGLU pair, and each wave's columns are taken from both halves of the tile
// so that a pair sits in one lane.
//
// Tile order (tile_of in gemm_common.h).  Workgroups are dispatched
// round-robin over the 8 XCDs; each XCD owns every eighth (N tile, slice)
// group (or, for passes with few groups and many M tiles, every second or
// fourth group and a share of the M tiles) and walks blocks of its groups
// times its M tiles, so that the tiles it runs at once share both operands
// through its L2 (with 8 slices each XCD owns one K slice, whose part of A
// stays in its L2).
#include <algorithm>
#include <string>

#include "launch.h"

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

#include "gemm_common.h"


int gemm_grid_size(int n_tiles, int m_tiles, int S) {
  // 8 XCDs times the most workgroups tile_of gives one XCD
  const int groups = n_tiles * S, py = tile_py(groups, m_tiles), px = 8 / py;
  return 8 * ((groups + px - 1) / px) * ((m_tiles + py - 1) / py);
}

#define GEMM_GLOAD(slot, k0)                                                             \
  do {                                                                                   \
    _Pragma("unroll") for (int t = 0; t < NA; ++t)                                       \
      _Pragma("unroll") for (int j = 0; j < A_CH; ++j)                                   \
        RA##slot[t][j] = *(const u32x4*)(Ap[t] + aoffg[j] + (size_t)(k0) * akmul);      \
    _Pragma("unroll") for (int j = 0; j < B_CH; ++j) RB##slot[j] = *(const u32x4*)(bsrc[j] + (size_t)(k0) * wkmul); \
  } while (0)
#define GEMM_SSTORE(slot, buf)                                                           \
  do {                                                                                   \
    _Pragma("unroll") for (int t = 0; t < NA; ++t)                                       \
      _Pragma("unroll") for (int j = 0; j < A_CH; ++j) *(u32x4*)&As[buf][t][aoff[j]] = RA##slot[t][j]; \
    _Pragma("unroll") for (int j = 0; j < B_CH; ++j) *(u32x4*)&Bs[buf][boff[j]] = RB##slot[j]; \
  } while (0)
#define GEMM_COMPUTE(cur)                                                                \
  do {                                                                                   \
    _Pragma("unroll") for (int ks = 0; ks < BK / 32; ++ks) {                             \
      const int ch = ks * 4 + lg;                                                        \
      bf16x8 bfr[CB];                                                                    \
      _Pragma("unroll") for (int cb = 0; cb < CB; ++cb)                                  \
        bfr[cb] = *(const bf16x8*)&Bs[cur][tc[cb] * BK + ((ch ^ (tc[cb] % CPR)) * 8)];  \
      _Pragma("unroll") for (int t = 0; t < NA; ++t) {                                   \
        bf16x8 af[RB];                                                                   \
        _Pragma("unroll") for (int rb = 0; rb < RB; ++rb) {                              \
          const int r_ = wm * WM + rb * 16 + lc;                                         \
          af[rb] = *(const bf16x8*)&As[cur][t][r_ * BK + ((ch ^ (r_ % CPR)) * 8)];       \
        }                                                                                \
        _Pragma("unroll") for (int rb = 0; rb < RB; ++rb)                                \
          _Pragma("unroll") for (int cb = 0; cb < CB; ++cb)                              \
            acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[rb], bfr[cb], acc[rb][cb], 0, 0, 0); \
      }                                                                                  \
    }                                                                                    \
  } while (0)

// ---------------------------------------------------------------------------
// SPLIT: A is the two-term activation (A = hi, A2 = lo); every fragment
// product is issued twice, hi x W and lo x W, into the same accumulator.
// MODE 0: one workgroup covers all of K in one accumulation (ksplit == 1).
// MODE 1: one workgroup covers all ksplit slices, each accumulated from zero
//         and added to the running total in slice order.
// MODE 2: one workgroup per slice, writing an fp32 partial.
template <int BM, int BN, int BK, int WGM, int WGN, int EPI, bool SPLIT, int MODE>
__global__ __launch_bounds__(256, 1) void gemm_bf16_kernel(GemmArgs a) {
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int RB = WM / 16, CB = WN / 16;
  constexpr int CPR = BK / 8;                       // 16-byte chunks per tile row
  constexpr int A_CH = BM * CPR / 256, B_CH = BN * CPR / 256;
  constexpr int NA = SPLIT ? 2 : 1;
  constexpr bool PARTIAL = MODE == 2, FOLD = MODE == 1;
  static_assert(WGM * WGN == 4 && A_CH >= 1 && B_CH >= 1 && CB % 2 == 0 && RB >= 1, "bad tile");
  static_assert(BN % (32 * WGN) == 0, "each wave takes 16-column blocks from both tile halves");
  __shared__ __attribute__((aligned(16))) bf16 As[2][NA][BM * BK];
  __shared__ __attribute__((aligned(16))) bf16 Bs[2][BN * BK];

  const int n_tiles = a.N / BN, m_tiles = (a.M + BM - 1) / BM;
  int tile_n, tile_m, z;
  if (!tile_of(blockIdx.x, n_tiles, m_tiles, PARTIAL ? a.ksplit : 1, &tile_n, &tile_m, &z)) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, lg = lane >> 4, lc = lane & 15;
  const int wm = w / WGN, wn = w % WGN;
  const int m0 = tile_m * BM;
  const int kslice = a.K / a.ksplit;
  const int kbeg = PARTIAL ? z * kslice : 0;
  const int nslices = FOLD ? a.ksplit : 1;
  const int kt_slice = (PARTIAL || FOLD ? kslice : a.K) / BK;   // k tiles per accumulation
  const bf16* Ap[2] = {(const bf16*)a.A, (const bf16*)(SPLIT ? a.A2 : a.A)};
  const int akmul = a.a_tiled ? a.lda : 1, wkmul = a.w_tiled ? a.ldw : 1;

  // rows past M load row M-1 (finite data; those output rows are never stored)
  uint32_t aoffg[A_CH], aoff[A_CH];
#pragma unroll
  for (int j = 0; j < A_CH; ++j) {
    const int c = tid + 256 * j, r = c / CPR, kc = c % CPR;
    const int row = min(m0 + r, a.M - 1);
    // k0 (a multiple of 32) contributes k0 * akmul elements
    aoffg[j] = a.a_tiled ? (uint32_t)((kc / 4) * a.lda * 32 + row * 32 + (kc % 4) * 8) : (uint32_t)row * a.lda + kc * 8;
    aoff[j] = r * BK + ((kc ^ (r % CPR)) * 8);
  }
  const bf16* bsrc[B_CH];
  uint32_t boff[B_CH];
#pragma unroll
  for (int j = 0; j < B_CH; ++j) {
    const int c = tid + 256 * j, r = c / CPR, kc = c % CPR;
    bool second;
    const int wr = brow_index<EPI, BN>(a, tile_n, r, &second);
    bsrc[j] = (const bf16*)(second ? a.W2 : a.W) +
              (a.w_tiled ? (size_t)(kc / 4) * a.ldw * 32 + (size_t)wr * 32 + (kc % 4) * 8 : (size_t)wr * a.ldw + kc * 8);
    boff[j] = r * BK + ((kc ^ (r % CPR)) * 8);
  }
  // tile column of accumulator block cb: blocks 0..CB/2-1 from the first tile
  // half, CB/2..CB-1 the partner columns from the second half
  int tc[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) tc[cb] = (cb / (CB / 2)) * (BN / 2) + wn * (WN / 2) + (cb % (CB / 2)) * 16 + lc;

  u32x4 RA0[NA][A_CH], RB0[B_CH], RA1[NA][A_CH], RB1[B_CH];   // two tiles of prefetch in flight
  f32x4 acc[RB][CB];
  f32x4 tot[FOLD ? RB : 1][FOLD ? CB : 1];
  if constexpr (FOLD) {
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < CB; ++j) tot[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // Pipeline: LDS buffer b holds tile g (b = g & 1), register slot (g + 1) & 1
  // holds tile g + 1 in flight; iteration g issues tile g + 2 into slot g & 1,
  // computes tile g, then moves tile g + 1 from its slot into LDS buffer b ^ 1.
  // Tile indices past the last tile are clamped (a redundant load whose LDS
  // copy is never read).  Tiles per accumulation are even (host-checked), so
  // the parity of g is static in the two unrolled halves.
  const int ntot = nslices * kt_slice;
#define kof(g) (kbeg + min((g), ntot - 1) * BK)
  GEMM_GLOAD(0, kof(0));
  GEMM_GLOAD(1, kof(1));
  GEMM_SSTORE(0, 0);
  __syncthreads();
  for (int sl = 0; sl < nslices; ++sl) {
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < CB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int kt = 0; kt < kt_slice; kt += 2) {
      const int g = sl * kt_slice + kt;             // even
      GEMM_GLOAD(0, kof(g + 2));
      GEMM_COMPUTE(0);
      GEMM_SSTORE(1, 1);
      __syncthreads();
      GEMM_GLOAD(1, kof(g + 3));
      GEMM_COMPUTE(1);
      GEMM_SSTORE(0, 0);
      __syncthreads();
    }
    if constexpr (FOLD) {
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j) tot[i][j] += acc[i][j];
    }
  }

  // accumulator (rb, cb)[i]: row wm*WM + 16*rb + 4*lg + i, tile column tc[cb]
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = m0 + wm * WM + rb * 16 + lg * 4 + i;
      if (row >= a.M) continue;
      if constexpr (PARTIAL) {
        float* pr = a.part + ((size_t)z * a.M + row) * a.N;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) pr[logical_col<EPI, BN>(a, tile_n, tc[cb])] = acc[rb][cb][i];
      } else if constexpr (epi_paired(EPI)) {
#pragma unroll
        for (int cb = 0; cb < CB / 2; ++cb) epi_tile_pair<EPI, bf16, BN>(a, tile_n, tc[cb], row, FOLD ? tot[rb % (FOLD ? RB : 1)][cb % (FOLD ? CB : 1)][i] : acc[rb][cb][i],
                                         FOLD ? tot[rb % (FOLD ? RB : 1)][(cb + CB / 2) % (FOLD ? CB : 1)][i] : acc[rb][cb + CB / 2][i]);
      } else {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          const int col = tile_n * BN + tc[cb];
          const float v = FOLD ? tot[rb % (FOLD ? RB : 1)][cb % (FOLD ? CB : 1)][i] : acc[rb][cb][i];
          if constexpr (EPI == EPI_STORE) epi_store(a, row, col, v);
          else epi_resid(a, row, col, v);
        }
      }
    }
  }
}

// Sum of the S partials in slice order, then the epilogue.  One thread per
// (row, logical pair) for SWIGLU, per (row, column) otherwise.
template <int EPI, class T>
__global__ __launch_bounds__(256) void gemm_reduce_kernel(GemmArgs a) {
  static_assert(EPI != EPI_QKV, "QKV partials are reduced by gemm_reduce_qkv_kernel");
  const int npair = epi_paired(EPI) ? a.N / 2 : a.N;
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long)a.M * npair) return;
  const int row = (int)(idx / npair), p = (int)(idx % npair);
  const size_t plane = (size_t)a.M * a.N;
  const float* pr = a.part + (size_t)row * a.N;
  if constexpr (EPI == EPI_SWIGLU) {
    const int F = a.N / 2;
    float g = pr[p], u = pr[F + p];
    for (int s = 1; s < a.ksplit; ++s) { g += pr[s * plane + p]; u += pr[s * plane + F + p]; }
    epi_swiglu<T>(a, row, p, g, u);
  } else {
    float v = pr[p];
    for (int s = 1; s < a.ksplit; ++s) v += pr[s * plane + p];
    if constexpr (EPI == EPI_STORE) epi_store(a, row, p, v);
    else epi_resid(a, row, p, v);
  }
}

// Split-K reduction of an EPI_RESID GEMM fused with the RMSNorm of the
// updated rows: one block of NORM_THREADS per row; thread t owns the float4
// chunks t, t + NORM_THREADS, ... (KC of them, N <= 4 * KC * NORM_THREADS) as
// in rms_normalize_row, adds the slices in slice order into X (as
// gemm_reduce_kernel does) and normalises the row from the values it keeps in
// registers, with the same expressions in the same order as
// rms_normalize_row (same bits as the stand-alone kernel).
template <class T, int KC>
__global__ __launch_bounds__(NORM_THREADS) void gemm_reduce_resid_norm_kernel(GemmArgs a) {
  constexpr int GRP = KC < 4 ? KC : 4;   // chunks whose slices are requested together
  __shared__ float red[16];
  const int row = blockIdx.x;
  const size_t plane = (size_t)a.M * a.N;
  const float* pr = a.part + (size_t)row * a.N;
  float* xr = a.X + (size_t)row * a.ldx;
  const int step = NORM_THREADS * 4;
  f32x4 xv[KC];
  float4 gv[KC];
#pragma unroll
  for (int k = 0; k < KC; ++k) {
    const int c = threadIdx.x * 4 + k * step;
    if (c < a.N) gv[k] = *(const float4*)(a.ngain + c);
  }
#pragma unroll
  for (int g = 0; g < KC; g += GRP) {
    f32x4 sl[GRP][8];
#pragma unroll
    for (int u = 0; u < GRP; ++u) {
      const int c = threadIdx.x * 4 + (g + u) * step;
      if (c < a.N) {
        xv[g + u] = *(const f32x4*)(xr + c);
#pragma unroll
        for (int s = 0; s < 8; ++s)
          if (s < a.ksplit) sl[u][s] = *(const f32x4*)(pr + s * plane + c);
      }
    }
#pragma unroll
    for (int u = 0; u < GRP; ++u) {
      const int c = threadIdx.x * 4 + (g + u) * step;
      if (c < a.N) {
        f32x4 v = sl[u][0];
#pragma unroll
        for (int s = 1; s < 8; ++s)
          if (s < a.ksplit) v += sl[u][s];
        xv[g + u] += v;
        *(f32x4*)(xr + c) = xv[g + u];
      }
    }
  }
  float ss = 0.f;
#pragma unroll
  for (int k = 0; k < KC; ++k) {
    const int c = threadIdx.x * 4 + k * step;
    if (c < a.N) {
      const f32x4 v = xv[k];
      ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
    }
  }
  ss = block_sum(ss, red);
  const float inv = 1.0f / sqrtf(ss / (float)a.N + a.neps);
#pragma unroll
  for (int k = 0; k < KC; ++k) {
    const int c = threadIdx.x * 4 + k * step;
    if (c < a.N) {
      const f32x4 v = xv[k];
      const float4 g = gv[k];
      const size_t i = act_at(row, c, a.nld, a.ntiled);
      store_act4<T>((T*)a.nout, (T*)a.nout2, i, v.x * inv * g.x, v.y * inv * g.y, v.z * inv * g.z, v.w * inv * g.w);
    }
  }
}

// Split-K reduction of a QKV projection in one launch.  Blocks [0, nvb) sum
// the value heads: 32 rows x hd dimensions of one value head per block
// (float4 loads, slices summed in slice order as in gemm_reduce_kernel),
// staged transposed in LDS and written to V^T with the rows running fastest
// across the threads, so that the 2-byte stores of consecutive rows
// (consecutive K/V destinations within a sequence) coalesce.  The remaining
// blocks sum the q/k column pairs (four consecutive pairs of a head per
// thread, float4 loads) and apply RoPE.
template <class T, int HD>
__global__ __launch_bounds__(256) void gemm_reduce_qkv_kernel(GemmArgs a, int nvb) {
  static_assert(sizeof(T) == 2, "bf16 activations");
  using Q = qkv_t<T>;   // stored q, k, v
  const size_t plane = (size_t)a.M * a.N;
  if ((int)blockIdx.x >= nvb) {
    // four consecutive pairs (j .. j + 3) of one head per thread
    constexpr int Q4 = HD / 8;                    // quads of pairs per head
    const int nquad = (a.hq + a.hkv) * Q4;
    const long idx = (long)(blockIdx.x - nvb) * blockDim.x + threadIdx.x;
    if (idx >= (long)a.M * nquad) return;
    const int row = (int)(idx / nquad), q = (int)(idx % nquad);
    const float* pr = a.part + (size_t)row * a.N;
    const int head = q / Q4, j = (q % Q4) * 4;
    const int c1 = head * HD + j, c2 = c1 + HD / 2;
    f32x4 v1 = *(const f32x4*)(pr + c1), v2 = *(const f32x4*)(pr + c2);
    for (int s = 1; s < a.ksplit; ++s) {
      v1 += *(const f32x4*)(pr + s * plane + c1);
      v2 += *(const f32x4*)(pr + s * plane + c2);
    }
    // RoPE of the four pairs with epi_qkv's expressions, one 8-byte store per half
    const int dst = a.row_dst[row];
    const float2* cs = a.rope + (size_t)a.row_pos[row] * (HD / 2) + j;
    Q* p;
    if (head < a.hq) p = (Q*)a.Qb + ((size_t)head * a.ldq + row) * HD;
    else if (dst_is_fresh(dst)) p = (Q*)a.Kf + ((size_t)(head - a.hq) * a.ldfresh + dst) * HD;
    else p = (Q*)a.Kc + ((size_t)(head - a.hq) * a.ldcache + dst_cache_row(dst)) * HD;
    f16x4 o1, o2;
    rope_rotate4(v1, v2, cs, &o1, &o2);
    *(f16x4*)(p + j) = o1;
    *(f16x4*)(p + j + HD / 2) = o2;
    return;
  }
  constexpr int RT = 32, TPR = HD / 4, RG = 256 / TPR, RPT = RT / RG;
  static_assert(RPT >= 1 && RT % RG == 0, "row tiling");
  __shared__ Q tile[HD][RT + 2];
  const int mb = (a.M + RT - 1) / RT;
  const int vh = blockIdx.x / mb, r0 = (blockIdx.x % mb) * RT;
  const int d4 = (threadIdx.x % TPR) * 4, rg = threadIdx.x / TPR;
  const float* pr = a.part + (size_t)(a.hq + a.hkv + vh) * HD + d4;
  // every slice of this thread's rows is requested before any is summed
  f32x4 v[RPT];
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int row = min(r0 + rg + k * RG, a.M - 1);
    v[k] = *(const f32x4*)(pr + (size_t)row * a.N);
  }
  for (int s = 1; s < a.ksplit; ++s) {
    f32x4 t[RPT];
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int row = min(r0 + rg + k * RG, a.M - 1);
      t[k] = *(const f32x4*)(pr + s * plane + (size_t)row * a.N);
    }
#pragma unroll
    for (int k = 0; k < RPT; ++k) v[k] += t[k];
  }
#pragma unroll
  for (int k = 0; k < RPT; ++k)
#pragma unroll
    for (int e = 0; e < 4; ++e) tile[d4 + e][rg + k * RG] = from_f32<Q>(v[k][e]);
  __syncthreads();
  for (int i = threadIdx.x; i < RT * HD; i += blockDim.x) {
    const int dd = i / RT, rr = i % RT, row = r0 + rr;
    if (row < a.M) {
      const int dst = a.row_dst[row];
      Q* vt;
      int ld, col;
      if (dst_is_fresh(dst)) { vt = (Q*)a.Vtf; ld = a.ldfresh; col = dst; }
      else { vt = (Q*)a.Vtc; ld = a.ldcache; col = dst_cache_row(dst); }
      vt[((size_t)vh * HD + dd) * ld + col] = tile[dd][rr];
    }
  }
}

template <int EPI>
static void reduce_epi(const GemmArgs& a, hipStream_t st) {
  if constexpr (EPI == EPI_RESID) {
    if (a.ngain) {
      if (a.nf16) {
        if (a.N <= 8 * NORM_THREADS) gemm_reduce_resid_norm_kernel<f16, 2><<<a.M, NORM_THREADS, 0, st>>>(a);
        else gemm_reduce_resid_norm_kernel<f16, 4><<<a.M, NORM_THREADS, 0, st>>>(a);
      } else {
        if (a.N <= 8 * NORM_THREADS) gemm_reduce_resid_norm_kernel<bf16, 2><<<a.M, NORM_THREADS, 0, st>>>(a);
        else gemm_reduce_resid_norm_kernel<bf16, 4><<<a.M, NORM_THREADS, 0, st>>>(a);
      }
      return;
    }
  }
  if constexpr (EPI == EPI_QKV) {
    const int nvb = (a.M + 31) / 32 * a.hkv;
    const long nqk = (long)a.M * (a.hq + a.hkv) * a.hd / 8;
    const unsigned grid = (unsigned)(nvb + (nqk + 255) / 256);
    if (a.hd == 128) gemm_reduce_qkv_kernel<bf16, 128><<<grid, 256, 0, st>>>(a, nvb);
    else gemm_reduce_qkv_kernel<bf16, 64><<<grid, 256, 0, st>>>(a, nvb);
  } else {
    const int npair = epi_paired(EPI) ? a.N / 2 : a.N;
    const long total = (long)a.M * npair;
    gemm_reduce_kernel<EPI, bf16><<<(unsigned)((total + 255) / 256), 256, 0, st>>>(a);
  }
}

void launch_gemm_reduce(int epi, const GemmArgs& a, hipStream_t st) {
  switch (epi) {
    case EPI_STORE: reduce_epi<EPI_STORE>(a, st); break;
    case EPI_RESID: reduce_epi<EPI_RESID>(a, st); break;
    case EPI_SWIGLU: reduce_epi<EPI_SWIGLU>(a, st); break;
    default: reduce_epi<EPI_QKV>(a, st); break;
  }
}

// ---------------------------------------------------------------------------
namespace {

template <int BM, int BN, int BK, int WGM, int WGN, int EPI, int MODE>
void run_mode(const GemmArgs& a, int grid, hipStream_t st) {
  if (a.A2) gemm_bf16_kernel<BM, BN, BK, WGM, WGN, EPI, true, MODE><<<grid, 256, 0, st>>>(a);
  else gemm_bf16_kernel<BM, BN, BK, WGM, WGN, EPI, false, MODE><<<grid, 256, 0, st>>>(a);
}

template <int BM, int BN, int BK, int WGM, int WGN, int EPI>
void run_cfg(const GemmArgs& a, bool partial, hipStream_t st) {
  const int n_tiles = a.N / BN, m_tiles = (a.M + BM - 1) / BM;
  const int grid = gemm_grid_size(n_tiles, m_tiles, partial ? a.ksplit : 1);
  if (partial) {
    run_mode<BM, BN, BK, WGM, WGN, EPI, 2>(a, grid, st);
    launch_gemm_reduce(EPI, a, st);
  } else if (a.ksplit > 1) {
    run_mode<BM, BN, BK, WGM, WGN, EPI, 1>(a, grid, st);
  } else {
    run_mode<BM, BN, BK, WGM, WGN, EPI, 0>(a, grid, st);
  }
}

template <int EPI>
void run_epi(int cfg, const GemmArgs& a, bool partial, hipStream_t st) {
  switch (cfg) {
    case 0: run_cfg<128, 128, 64, 2, 2, EPI>(a, partial, st); break;
    case 1: run_cfg<256, 128, 32, 2, 2, EPI>(a, partial, st); break;
    case 2: run_cfg<128, 64, 64, 4, 1, EPI>(a, partial, st); break;
    case 3: run_cfg<256, 64, 64, 4, 1, EPI>(a, partial, st); break;
    case 4: run_cfg<64, 128, 64, 1, 4, EPI>(a, partial, st); break;
    case 5: run_cfg<64, 128, 32, 1, 4, EPI>(a, partial, st); break;
    default: run_cfg<128, 64, 32, 4, 1, EPI>(a, partial, st); break;
  }
}

const int kCfgBN[GEMM_NCFG] = {128, 128, 64, 64, 128, 128, 64};
const int kCfgBK[GEMM_NCFG] = {64, 32, 64, 64, 64, 32, 32};
const int kCfgBM[GEMM_NCFG] = {128, 256, 128, 256, 64, 64, 128};

}  // namespace

int gemm_ksplit(int N, int K, int rows) {
  // One slice when the smallest launch has enough 128-row tiles to fill the
  // GPU on its own (rows >= 2048: at least 16 row tiles); otherwise enough
  // slices that a 256-row launch of 128 x 128 tiles fills the 256 CUs,
  // within the K granularity.  The count is fixed per context (rows is the
  // context's response-row capacity), never per launch, so every pass of a
  // context sums every output in the same order.
  // A 256-row launch that already has three quarters of a round of 128 x 128
  // tiles (N >= 12288) also takes one slice: measured on the LLaDA-8B QKV
  // projection with 128 x 128 tiles, one slice is as fast as two at 256 rows
  // (64 x 192 tiles then gain another 5 us) and needs no partial planes or
  // reduction in a refresh pass.
  if (rows >= 2048) return 1;
  const int tiles = 2 * std::max(N / 128, 1);
  if (tiles >= 192) return 1;
  int S = 1;
  while (S < 8 && tiles * S < 256 && K % (2 * S * 64) == 0) S *= 2;
  return S;
}

// One workgroup per slice with a separate reduction: measured on the LLaDA-8B
// projections at 256 .. 4352 rows, at least as fast as folding the slices into
// one workgroup wherever the partial buffer holds the rows.
static bool use_partials(const GemmArgs& a) { return a.ksplit > 1 && a.part && a.M <= a.part_rows; }

// Time in us of a grid of a configuration's tiles over k of a K dimension: per
// round of 256 workgroups (one per CU) a part that grows with k and TILE_US of
// filling and draining.  Two-term bf16 and single-term fp16 launches; 0: not a
// configuration of the kind.  Fitted to the LLaDA-8B and Dream-7B projections at 64
// to 2048 rows and to the ragged batch's 4096- and 24853-row passes; of 28 launches
// of other shapes (65 to 4300 rows, N 2048 to 30000, K 1024 to 16000) the tile with the
// least time was also the fastest in 22, five lost 3 to 9 % and one 17.  Two
// workgroups of the 64-row tiles share a CU: further rounds cost less than the
// first, and only one fill and drain shows (LLaDA-8B QKV in 64 x 192 tiles: 50 us
// for 1 round, 124 for 3, 311 for 8; O at 1024 rows in 4 slices: 64 x 128 tiles
// 84 us, 128 x 128 91).  A partly filled last round of 128 x 256 tiles is faster than
// a full one (down of the Dream-7B shape, K 18944: 140 workgroups 326 us, 168 345,
// 224 386, the only shape behind the 0.7 and 0.3); the other tiles showed no such
// gain.  Folded slices (all of K in a tile, in parts) cost FOLD_US a round: down of
// the LLaDA-8B shape, 4 slices, 335 us a round, O 131.
static double tiles_us(int cfg, bool f16, int grid, double k) {
  const int rounds = (grid + 255) / 256;
  constexpr double TILE_US = 5.0, FOLD_US = 20.0;
  double t;   // per round and K 4096
  switch (cfg) {
    case GEMM_NCFG + 1: t = f16 ? 32.0 : 48.0; break;      // 128 x 128
    case GEMM_NCFG + 0: t = f16 ? 0.0 : 75.0; break;       // 128 x 192
    case GEMM_NCFG + 2: t = f16 ? 0.0 : 89.0; break;       // 128 x 256
    case GEMM_NCFG + 3: t = f16 ? 0.0 : rounds == 1 ? 45.0 : 39.0; break;   // 64 x 192
    case GEMM_NCFG + 4: t = f16 ? 0.0 : rounds == 1 ? 33.0 : 28.5; break;   // 64 x 128
    case GEMM_WIDE_128x192: t = f16 ? 40.0 : 0.0; break;
    case GEMM_WIDE_256x192: t = f16 ? 70.0 : 143.0; break;
    case GEMM_WIDE_256x256: t = f16 ? 93.5 : 175.0; break;
    case GEMM_WIDE_FOLD_128x256: t = f16 ? 57.0 : 105.0; break;
    default: t = 0.0;
  }
  const bool shared = cfg == GEMM_NCFG + 3 || cfg == GEMM_NCFG + 4;
  const double fill = cfg == GEMM_WIDE_FOLD_128x256 ? FOLD_US : TILE_US;
  const double last = cfg == GEMM_NCFG + 2 ? 0.7 + 0.3 * (grid - (rounds - 1) * 256) / 256 : 1.0;
  return t == 0.0 ? 0.0 : (rounds - 1 + last) * t * k / 4096 + (shared ? 1 : rounds) * fill;
}

static void tile_size(int cfg, int* bm, int* bn) {
  const bool rows64 = cfg == GEMM_NCFG + 3 || cfg == GEMM_NCFG + 4;
  *bm = cfg == GEMM_WIDE_256x256 || cfg == GEMM_WIDE_256x192 ? 256 : rows64 ? 64 : 128;
  *bn = cfg == GEMM_WIDE_256x256 || cfg == GEMM_WIDE_FOLD_128x256 || cfg == GEMM_NCFG + 2 ? 256
        : cfg == GEMM_NCFG + 1 || cfg == GEMM_NCFG + 4   ? 128
                                                         : 192;
}

static bool one_slice_ok(int cfg, const GemmArgs& a, int epi) {
  return cfg >= GEMM_NCFG + GEMM_NCFG_LDS ? gemm_wide_ok(cfg, a, epi) : gemm_lds_cfg_ok(cfg - GEMM_NCFG, a);
}

// tiles_us of a launch in S slices; the grid counts what the fullest XCD gets of
// the tile order, eight times over.
static double launch_us(int cfg, const GemmArgs& a, int S) {
  int bm, bn;
  tile_size(cfg, &bm, &bn);
  const int grid = gemm_grid_size(a.N / bn, (a.M + bm - 1) / bm, S);
  return tiles_us(cfg, a.f16 != 0, grid, (double)a.K / S);
}

// The one-slice configuration with the least launch_us, and that time; -1 if there is none.
static int one_slice_pick(const GemmArgs& a, int epi, double* cost) {
  int best = -1;
  for (int cfg : {(int)GEMM_WIDE_256x256, (int)GEMM_WIDE_256x192, GEMM_NCFG + 2, (int)GEMM_WIDE_128x192, GEMM_NCFG + 0,
                  GEMM_NCFG + 1, GEMM_NCFG + 3, GEMM_NCFG + 4}) {
    if (!one_slice_ok(cfg, a, epi)) continue;
    const double c = launch_us(cfg, a, 1);
    if (c != 0.0 && (best < 0 || c < 0.98 * *cost)) { best = cfg; *cost = c; }
  }
  return best;
}

// The same for a two-term launch whose slices are workgroups of their own; -1 if there is none.
static int split_pick(const GemmArgs& a, double* cost) {
  int best = -1;
  for (int cfg : {GEMM_NCFG + 0, GEMM_NCFG + 1, GEMM_NCFG + 3, GEMM_NCFG + 4}) {
    if (!gemm_lds_cfg_ok(cfg - GEMM_NCFG, a)) continue;
    const double c = launch_us(cfg, a, a.ksplit);
    if (best < 0 || c < 0.98 * *cost) { best = cfg; *cost = c; }
  }
  return best;
}

int gemm_pick_cfg(const GemmArgs& a, int epi) {
  // One K slice with two-term or fp16 operands: the tile with the least launch_us; of
  // two within 2 % the wider one (so, for example, 256-row gate/up passes take
  // 128 x 192 tiles, one round, 256-row QKV passes 64 x 192 tiles, and the 4096 rows of a serving batch 256 x 256 ones
  // throughout).  An LM head that writes the decision statistics takes the column tile
  // by N alone (256, when N has at least 256 of them), so that their partials do not
  // depend on the row count of a pass or on the terms of its operands (which may change
  // between the passes of a session); one that only stores its logits is chosen
  // like the others (16 x 256 rows of 4096 columns: one round of 256 x 256 tiles, 163 to
  // 180 us, for 216 in 128 x 128; 256 rows of the full vocabulary 480 for 495).
  // Two-term split-K launches choose the same way among the 128- and 64-row tiles
  // of up to 192 columns (down at 120 rows in 4 slices: 64 x 128 tiles 35 us,
  // 128 x 128 45; at 256 rows 63 and 51).  Other split-K launches take 128 x 192
  // tiles when N is a multiple of 192, else 128 x 128; the 128 x 192 tile is not used
  // for slices folded in one workgroup (its second accumulator set does not
  // fit the registers of two waves per SIMD).
  const bool stats = epi == EPI_STORE && a.tstat;
  if (stats && a.N / 256 >= 256 && gemm_lds_cfg_ok(2, a)) return GEMM_NCFG + 2;
  if (!stats && (a.A2 || a.f16) && a.ksplit == 1) {
    double cost;
    const int best = one_slice_pick(a, epi, &cost);
    if (best >= 0) return best;
  }
  if (a.A2 && use_partials(a)) {
    double cost;
    const int best = split_pick(a, &cost);
    if (best >= 0) return best;
  }
  if (a.N % 192 == 0 && gemm_lds_cfg_ok(0, a)) {
    const bool fold = a.ksplit > 1 && !use_partials(a);
    if (!fold) return GEMM_NCFG + 0;
  }
  if (a.N % 128 == 0 && gemm_lds_cfg_ok(1, a)) return GEMM_NCFG + 1;
  // register-staged kernel for the remaining shapes
  const bool bn128 = a.N % 128 == 0 && (epi != EPI_QKV || a.hd % 128 == 0) &&
                     (epi != EPI_SWIGLU || (a.N / 2) % 64 == 0);
  const bool bk64 = a.K % (2 * a.ksplit * 64) == 0;   // even number of 64-wide k tiles per slice
  if (bn128) {
    if (!bk64) return 5;
    return a.M <= 1024 ? 4 : 0;
  }
  if (!bk64) return 6;
  return a.M <= 1024 ? 2 : 3;
}

bool gemm_cfg_ok(int cfg, const GemmArgs& a, int epi) {
  if (cfg < 0 || cfg >= GEMM_NCFG) return false;
  const int BN = kCfgBN[cfg];
  if (a.M <= 0 || a.N % BN || a.ksplit < 1 || a.K % (2 * a.ksplit * kCfgBK[cfg])) return false;
  if (epi == EPI_QKV && (a.hd % BN)) return false;
  if (epi == EPI_SWIGLU && ((a.N / 2) % (BN / 2))) return false;
  return true;
}

bool gemm_args_ok(int epi, const GemmArgs& a) {
  if (!a.A || !a.W || a.M <= 0 || a.N <= 0 || a.K <= 0 || a.ksplit < 1) return false;
  if (a.f16 && (epi != EPI_SWIGLU || a.A2)) return false;   // fp16 operands: single-term gate/up only
  switch (epi) {
    case EPI_STORE: return (a.C && a.ldc >= a.N) || (a.tstat && a.targ && a.zg && a.tg);
    case EPI_RESID: return a.X && a.ldx >= a.N;
    case EPI_SWIGLU: return a.H && a.W2 && a.N % 2 == 0;
    case EPI_QKV:
      // the column mapping divides by hd / 2 and the epilogue indexes every table
      return a.hd > 0 && a.hd % 2 == 0 && a.hq > 0 && a.hkv > 0 && a.N == (a.hq + 2 * a.hkv) * a.hd && a.Qb &&
             a.Kf && a.Vtf && a.Kc && a.Vtc && a.row_dst && a.row_pos && a.rope;
    default: return false;
  }
}

int launch_gemm_bf16_cfg(int epi, int cfg, bool partial, const GemmArgs& a, hipStream_t st) {
  if (!gemm_args_ok(epi, a)) return 1;
  if (cfg >= GEMM_NCFG + GEMM_NCFG_LDS) return partial ? 1 : launch_gemm_wide(epi, cfg, a, st);
  if (cfg >= GEMM_NCFG) return launch_gemm_lds_cfg(epi, cfg - GEMM_NCFG, partial, a, st);
  if (a.f16 || !gemm_cfg_ok(cfg, a, epi)) return 1;   // the register-staged kernel is bf16 only
  if (partial && (!a.part || a.ksplit < 2)) return 1;
  switch (epi) {
    case EPI_STORE: run_epi<EPI_STORE>(cfg, a, partial, st); break;
    case EPI_RESID: run_epi<EPI_RESID>(cfg, a, partial, st); break;
    case EPI_SWIGLU: run_epi<EPI_SWIGLU>(cfg, a, partial, st); break;
    case EPI_QKV: run_epi<EPI_QKV>(cfg, a, partial, st); break;
    default: return 1;
  }
  return 0;
}

// The tiles that whole rounds of CUs run in (gemm_split_rows).
static int rounds_cfg(const GemmArgs& a) { return a.ksplit == 1 ? (int)GEMM_WIDE_256x256 : (int)GEMM_WIDE_FOLD_128x256; }

// Rows [0, m1) of a launch that run as wide tiles in whole rounds of the 256
// CUs, ahead of the rest with its own configuration; 0: one launch.
//
// A launch whose last round is nearly empty pays for a whole one: the 4352 rows
// of a 4096-token refresh are 17 row tiles, 3.19 rounds of QKV tiles.  Rounds of
// 16 row tiles and 256 rows apart took 553 + 53 us against 628.  Split-K launches run
// their rounds in tiles that fold the slices, which saves the partial planes of
// those rows and keeps the bits of separate slices: 4096 rows of O and down in 4
// slices 262 + 37 and 668 + 65 us, for 400 to 435 and 826 to 873 with every row's
// slices apart.  (One 256 x 256 tile over all of K takes 226 and 600, but then a
// row's sums would depend on its place in the pass.)  LAUNCH_US is the drain and
// start of the second launch.
static int gemm_split_rows(const GemmArgs& a, int epi) {
  constexpr double LAUNCH_US = 8.0;
  const int cfg = rounds_cfg(a);
  if (epi == EPI_STORE || !gemm_wide_ok(cfg, a, epi)) return 0;
  int bm, bn;
  tile_size(cfg, &bm, &bn);
  const auto wide = [&](int rounds) { return tiles_us(cfg, a.f16 != 0, rounds * 256, a.K); };
  // one launch of m rows in the context's slices
  const auto plain = [&](int m) {
    GemmArgs r = a;
    r.M = m;
    double c = 0.0;
    if (a.ksplit == 1) return one_slice_pick(r, epi, &c) >= 0 ? c : 1e30;
    // more rows than the partial buffer: 128 x 128 tiles that fold, 1.3 to 1.4 times a one-slice launch
    if (!use_partials(r)) return 1.35 * launch_us(GEMM_NCFG + 1, r, 1);
    if (!a.A2 || split_pick(r, &c) < 0) c = launch_us(GEMM_NCFG + 1, r, a.ksplit);
    // the reduction reads the planes and the destination and writes it at about 4 TB/s
    return c + LAUNCH_US + (double)m * a.N * 4 * (a.ksplit + 2) / 4e6;
  };
  const int nt = a.N / bn, mt_all = a.M / bm;
  double best = 0.98 * plain(a.M);
  int m1 = 0;
  for (int r = 1; (long)r * 256 / nt <= mt_all; ++r) {
    // as many row tiles as r rounds of CUs hold, in equal shares where XCDs split the row tiles
    int mt = (int)((long)r * 256 / nt);
    mt -= mt % tile_py(nt, mt);
    if (mt == 0 || gemm_grid_size(nt, mt, 1) > r * 256) continue;
    const double c = wide(r) + (mt * bm < a.M ? LAUNCH_US + plain(a.M - mt * bm) : 0.0);
    if (c < best) { best = c; m1 = mt * bm; }
  }
  return m1;
}

// Whether launch_gemm_bf16 also runs the RMSNorm that a asks for: the launch has
// one reduction for all its rows, whose kernel holds a row of up to 16 NORM_THREADS columns.
bool gemm_fuses_norm(const GemmArgs& a) {
  if (!a.ngain || a.N % 4 || a.N > 16 * NORM_THREADS || a.ldx % 4 || a.ksplit > 8) return false;
  return use_partials(a) && gemm_split_rows(a, EPI_RESID) == 0;
}

// The arguments of rows [r0, r0 + m) of a launch (r0 a multiple of 128).
static GemmArgs gemm_rows(const GemmArgs& a, int r0, int m) {
  GemmArgs b = a;
  const auto act = [&](const void* p, int ld, int tiled) {
    return p ? (const void*)((const char*)p + (size_t)r0 * (tiled ? 32 : ld) * 2) : nullptr;
  };
  b.M = m;
  b.A = act(a.A, a.lda, a.a_tiled);
  b.A2 = act(a.A2, a.lda, a.a_tiled);
  b.H = (void*)act(a.H, a.ldh, a.h_tiled);
  b.H2 = (void*)act(a.H2, a.ldh, a.h_tiled);
  if (a.X) b.X = a.X + (size_t)r0 * a.ldx;
  if (a.Qb) b.Qb = (char*)a.Qb + (size_t)r0 * a.hd * 2;
  if (a.row_pos) b.row_pos = a.row_pos + r0;
  if (a.row_dst) b.row_dst = a.row_dst + r0;
  b.ngain = nullptr;   // the normalisation of the updated rows runs on all of them together
  return b;
}

// How a launch runs: rows [0, m1) in rounds_cfg tiles, the others in configuration
// cfg (no others when m1 is M), their slices in workgroups of their own or not.
namespace {
struct GemmRoute { int m1, cfg; bool partial; };
}  // namespace

static GemmRoute gemm_route(int epi, const GemmArgs& a) {
  GemmRoute r{gemm_split_rows(a, epi), 0, false};
  if (r.m1 < a.M) {
    const GemmArgs rest = gemm_rows(a, r.m1, a.M - r.m1);
    r.cfg = gemm_pick_cfg(rest, epi);
    r.partial = use_partials(rest);
  }
  return r;
}

int launch_gemm_bf16(int epi, const GemmArgs& a0, hipStream_t st) {
  if (!gemm_args_ok(epi, a0)) return 1;
  GemmArgs a = a0;
  if (!gemm_fuses_norm(a)) a.ngain = nullptr;   // a plain reduction, of rows of any length
  const GemmRoute r = gemm_route(epi, a);
  if (r.m1 == 0) return launch_gemm_bf16_cfg(epi, r.cfg, r.partial, a, st);
  const int rc = launch_gemm_wide(epi, rounds_cfg(a), gemm_rows(a, 0, r.m1), st);
  if (rc || r.m1 == a.M) return rc;
  return launch_gemm_bf16_cfg(epi, r.cfg, r.partial, gemm_rows(a, r.m1, a.M - r.m1), st);
}

std::string gemm_route_text(int epi, const GemmArgs& a) {
  const auto part = [&](int rows, int cfg, bool partial) {
    int bm, bn;
    if (cfg < GEMM_NCFG) { bm = kCfgBM[cfg]; bn = kCfgBN[cfg]; }
    else tile_size(cfg, &bm, &bn);
    std::string t = std::to_string(rows) + " rows " + (cfg < GEMM_NCFG ? "staged " : cfg >= GEMM_NCFG + GEMM_NCFG_LDS ? "wide " : "") +
                    std::to_string(bm) + "x" + std::to_string(bn);
    if (a.ksplit > 1) t += ", " + std::to_string(a.ksplit) + (partial ? " slices" : " folded slices");
    return t;
  };
  const GemmRoute r = gemm_route(epi, a);
  std::string t;
  if (r.m1) t = part(r.m1, rounds_cfg(a), false);
  if (r.m1 < a.M) t += (r.m1 ? "; " : "") + part(a.M - r.m1, r.cfg, r.partial);
  return t;
}

// ---------------------------------------------------------------------------
// fp32 kernel.  KS waves share a tile of 16 RB rows x 16 CB columns and split K:
// wave w takes the 16-wide k chunks w, w + KS, ... with v_mfma_f32_16x16x4_f32,
// the fragments loaded straight from global memory (a lane's float4 holds four
// consecutive k of one row; MFMA i of a chunk multiplies element i of every
// lane, the same k on both sides) and PF chunks requested ahead.  The waves'
// sums are added in wave order through LDS, then the epilogue runs.  The order
// of a sum depends on K alone, so a row's result does not depend on the tile
// or on the rows of the launch.
// Small fp32 models are bound by the chain of global load latencies, so the
// chunks of a row are spread over waves and requested together: 32 rows of the
// tiny model take 5 us at K 256 and 11 us at K 1024, where one 16-wide
// chunk loaded, staged and multiplied at a time took 23 and 85 us; 4096 x 12288
// x 4096 take 4.97 ms (83 TFLOP/s), where 64 x 64 LDS tiles on the vector units
// took 8.19 ms.
constexpr int F32_KS = 8;
template <int EPI, int RB, int CB, int PF>
__global__ __launch_bounds__(64 * F32_KS) void gemm_f32_kernel(GemmArgs a) {
  constexpr int BM = 16 * RB, BN = 16 * CB;
  static_assert(CB % 2 == 0, "pair halves are whole column blocks");
  __shared__ float red[F32_KS][CB * 4][64];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lg = lane >> 4, lc = lane & 15;
  const int tile_n = blockIdx.x, m0 = blockIdx.y * BM;
  // rows past M load row M - 1; those output rows are never stored
  const float* ap[RB];
  const float* wp[CB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) ap[rb] = (const float*)a.A + (size_t)min(m0 + rb * 16 + lc, a.M - 1) * a.lda + lg * 4;
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
    bool second;
    const int wr = brow_index<EPI, BN>(a, tile_n, cb * 16 + lc, &second);
    wp[cb] = (const float*)(second ? a.W2 : a.W) + (size_t)wr * a.ldw + lg * 4;
  }
  f32x4 acc[RB][CB];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nch = a.K / 16;
  for (int c0 = w; c0 < nch; c0 += F32_KS * PF) {
    f32x4 fa[PF][RB], fw[PF][CB];
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      const int k0 = min(c0 + u * F32_KS, nch - 1) * 16;   // past the last chunk: loaded, not multiplied
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) fa[u][rb] = *(const f32x4*)(ap[rb] + k0);
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) fw[u][cb] = *(const f32x4*)(wp[cb] + k0);
    }
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      if (c0 + u * F32_KS >= nch) break;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int cb = 0; cb < CB; ++cb)
            acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[u][rb][i], fw[u][cb][i], acc[rb][cb], 0, 0, 0);
    }
  }
  // accumulator (rb, cb)[i]: row 16 rb + 4 lg + i, tile column 16 cb + lc; wave i < 4 finishes rows 4 lg + i
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    if (rb) __syncthreads();
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int i = 0; i < 4; ++i) red[w][cb * 4 + i][lane] = acc[rb][cb][i];
    __syncthreads();
    const int row = m0 + rb * 16 + lg * 4 + w;
    if (w < 4 && row < a.M) {
      float v[CB];
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        v[cb] = red[0][cb * 4 + w][lane];
#pragma unroll
        for (int s = 1; s < F32_KS; ++s) v[cb] += red[s][cb * 4 + w][lane];
      }
      if constexpr (epi_paired(EPI)) {
#pragma unroll
        for (int cb = 0; cb < CB / 2; ++cb)
          epi_tile_pair<EPI, float, BN>(a, tile_n, cb * 16 + lc, row, v[cb], v[cb + CB / 2]);
      } else {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          const int col = tile_n * BN + cb * 16 + lc;
          if constexpr (EPI == EPI_STORE) epi_store(a, row, col, v[cb]);
          else epi_resid(a, row, col, v[cb]);
        }
      }
    }
  }
}

template <int EPI>
static void run_f32(const GemmArgs& a, hipStream_t st) {
  // 64 x 64 tiles (half the loads per product) once they fill the GPU, 32 x 32 below
  const long big = (long)(a.N / 64) * ((a.M + 63) / 64);
  if (big >= 256) gemm_f32_kernel<EPI, 4, 4, 2><<<dim3(a.N / 64, (a.M + 63) / 64), 64 * F32_KS, 0, st>>>(a);
  else gemm_f32_kernel<EPI, 2, 2, 4><<<dim3(a.N / 32, (a.M + 31) / 32), 64 * F32_KS, 0, st>>>(a);
}

int launch_gemm_f32(int epi, const GemmArgs& a, hipStream_t st) {
  if (!gemm_args_ok(epi, a)) return 1;
  if (a.M <= 0 || a.N % 64 || a.K % 16) return 1;
  if (epi == EPI_QKV && (a.hd % 64)) return 1;
  switch (epi) {
    case EPI_STORE: run_f32<EPI_STORE>(a, st); break;
    case EPI_RESID: run_f32<EPI_RESID>(a, st); break;
    case EPI_SWIGLU: run_f32<EPI_SWIGLU>(a, st); break;
    case EPI_QKV: run_f32<EPI_QKV>(a, st); break;
    default: return 1;
  }
  return 0;
}
