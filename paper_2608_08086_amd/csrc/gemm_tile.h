// Pieces shared by the direct-to-LDS projection GEMMs (gemm_lds.hip, whose
// loader waves feed separate multiply waves, and gemm_wide.hip, whose waves do
// both): the 16-byte direct loads and the LDS tile layout, the staged stores of
// the QKV projection, and the epilogue of an accumulated tile.
#pragma once

#include "gemm_common.h"

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

namespace {

// s_waitcnt immediates (gfx9 encoding)
#define GL_VMCNT(n) (((n) & 15) | (7 << 4) | (15 << 8) | ((((n) >> 4) & 3) << 14))
#define GL_LGKMCNT0 (15 | (7 << 4) | (0 << 8) | (3 << 14))

// M0 is listed as clobbered; no other code of this file keeps a value in it.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void gl_dma16(const void* sbase, unsigned voff, unsigned lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(voff), "s"(sbase), "s"(lds)
               : "memory", "m0");
}
#pragma clang diagnostic pop

__device__ __forceinline__ void gl_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Chunk swizzle of a 64-byte row (four 16-byte chunks), chosen by measurement
// (LDS bank-conflict counter of ds_read_b128 over 16 rows x one chunk): the
// chunk index is XORed with (row / 2) mod 4.
__device__ __forceinline__ int gl_swz(int row) { return (row >> 1) & 3; }

constexpr int BK = 32;      // k chunk per tile (one MFMA k step)
constexpr int CPR = BK / 8; // 16-byte chunks per tile row

// QKV projection, value heads.  A tile whose column pairs are all value pairs
// is staged in LDS as the transposed tile (one row of BM + 8 keys per value
// dimension) and written to V^T in 16-byte chunks along the key axis wherever
// eight consecutive pass rows go to eight consecutive, aligned key columns of
// one buffer; element stores otherwise.  Written one element per lane, the
// transposed layout gives every two-byte store its own cache line, which the
// L2 then reads whole to merge.  The stored values are those of
// epi_tile_pair4.
template <int BN>
__device__ __forceinline__ bool qkv_value_tile(const GemmArgs& a, int tile_n) {
  return tile_n * (BN / 2) >= (a.hq + a.hkv) * (a.hd / 2);
}
constexpr int VT_PAD = 8;
template <int BM, int BN, int NTHREADS>
__device__ __forceinline__ void store_value_tile(const GemmArgs& a, const f16* vs, int tile_n, int m0, int t) {
  constexpr int KS = BM + VT_PAD, KC = BM / 8;
  static_assert(NTHREADS % KC == 0, "a thread keeps one key chunk");
  // this thread's chunk of eight keys is the same for every dimension row it stores
  const int kc = t % KC, k0 = m0 + kc * 8;
  if (k0 >= a.M) return;
  const int nk = min(8, a.M - k0);
  const int dst0 = a.row_dst[k0];
  const bool fresh = dst_is_fresh(dst0);
  const int col0 = fresh ? dst0 : dst_cache_row(dst0);
  f16* vt = (f16*)(fresh ? a.Vtf : a.Vtc);
  const int ld = fresh ? a.ldfresh : a.ldcache;
  bool vec = nk == 8 && col0 % 8 == 0 && ld % 8 == 0 && ((uintptr_t)vt & 15) == 0;
  for (int i = 1; i < 8 && vec; ++i) {
    const int di = a.row_dst[k0 + i];
    vec = dst_is_fresh(di) == fresh && (fresh ? di : dst_cache_row(di)) == col0 + i;
  }
  const int half = a.hd / 2, p0 = tile_n * (BN / 2);
  for (int drow = t / KC; drow < BN; drow += NTHREADS / KC) {
    const int p = p0 + (drow >> 1);
    const int vh = p / half - a.hq - a.hkv, d = p % half + (drow & 1) * half;
    const f16* src = vs + drow * KS + kc * 8;
    if (vec) {
      *(u32x4*)(vt + (size_t)(vh * a.hd + d) * ld + col0) = *(const u32x4*)src;
    } else {
      for (int i = 0; i < nk; ++i) {
        const int di = a.row_dst[k0 + i];
        if (dst_is_fresh(di)) ((f16*)a.Vtf)[(size_t)(vh * a.hd + d) * a.ldfresh + di] = src[i];
        else ((f16*)a.Vtc)[(size_t)(vh * a.hd + d) * a.ldcache + dst_cache_row(di)] = src[i];
      }
    }
  }
}

// QKV projection, query and key heads.  A tile whose column pairs are whole
// query or key heads is staged in LDS as rotated rows (the values of
// epi_tile_pair4) and written with 16-byte stores along each head's
// dimensions, so every store covers whole 128-byte lines.  Written straight
// from the accumulators, a store covers 32 bytes of each of 16 rows, and the
// L2 reads every partly written line from memory first: the query and key
// stores of a 4096-row pass fetched 0.5 GB for 67 MB of output.
template <int BN>
__device__ __forceinline__ bool qkv_qk_tile(const GemmArgs& a, int tile_n) {
  const int half = a.hd / 2;
  return (BN / 2) % half == 0 && (tile_n + 1) * (BN / 2) <= (a.hq + a.hkv) * half &&
         (((uintptr_t)a.Qb | (uintptr_t)a.Kf | (uintptr_t)a.Kc) & 15) == 0;
}
// every tile of a QKV launch is a value tile or a query / key tile
inline bool qkv_all_staged(const GemmArgs& a, int BN) {
  const int half = a.hd / 2;
  return (BN / 2) % half == 0 && (a.hq + a.hkv) * half % (BN / 2) == 0 &&
         (((uintptr_t)a.Qb | (uintptr_t)a.Kf | (uintptr_t)a.Kc) & 15) == 0;
}
constexpr int QK_PAD = 8;
template <int BM, int BN, int NTHREADS>
__device__ __forceinline__ void store_qk_tile(const GemmArgs& a, const f16* qs, int tile_n, int m0, int t) {
  constexpr int RS = BN + QK_PAD, CH = BN / 8;   // staged row stride, 16-byte chunks per row
  const int hd = a.hd, h0 = tile_n * (BN / hd);
  for (int i = t; i < BM * CH; i += NTHREADS) {
    const int r = i / CH, ch = i % CH, row = m0 + r;
    if (row >= a.M) break;                        // i only grows, and so does row
    const int head = h0 + ch * 8 / hd, d = ch * 8 % hd;
    f16* p;
    if (head < a.hq) {
      p = (f16*)a.Qb + ((size_t)head * a.ldq + row) * hd;
    } else {
      const int dst = a.row_dst[row];
      p = dst_is_fresh(dst) ? (f16*)a.Kf + ((size_t)(head - a.hq) * a.ldfresh + dst) * hd
                            : (f16*)a.Kc + ((size_t)(head - a.hq) * a.ldcache + dst_cache_row(dst)) * hd;
    }
    *(u32x4*)(p + d) = *(const u32x4*)(qs + r * RS + ch * 8);
  }
}

// Epilogue of one workgroup tile of BM rows x BN columns whose waves (a grid
// WGN wide) hold C^T fragments: lane (lg, lc) of the wave at (wm, wn) holds in
// acc[rb][cb][e] the element of row wm * WM + 16 rb + lc and tile column
// tc[cb] - lc + 4 lg + e.  QKV_STAGED: whole value, query or key tiles go through
// the SMEM bytes of LDS at smem, which the caller no longer uses once every
// wave has passed the first barrier here; the NT threads of the workgroup (the
// loader waves of gemm_lds.hip included) store them; QKV_ONLY_STAGED: every tile of
// the launch is such a tile (qkv_all_staged).  STATS: the decision
// statistics of an LM-head tile (2 x 2 wave grids only).
template <int BM, int BN, int WGN, int RB, int CB, int EPI, bool QKV_STAGED, bool STATS, int SMEM, int NT,
          bool QKV_ONLY_STAGED = false>
__device__ __forceinline__ void tile_epilogue(const GemmArgs& a, char* smem, int tile_n, int m0, int wm, int wn,
                                              int lane, int tid, const int (&tc)[CB], const f32x4 (&acc)[RB][CB]) {
  constexpr int WM = 16 * RB;
  static_assert(!STATS || WGN == 2, "the statistics partials are per half tile");
  const int lg = lane >> 4, lc = lane & 15;
  // accumulator (rb, cb)[e]: row wm*WM + 16*rb + lc, tile column tb[cb] + e,
  // tb[cb] = tc[cb] - lc + 4*lg (tc evaluated at lane lc = 4*lg)
  if constexpr (QKV_STAGED) {
    if (qkv_value_tile<BN>(a, tile_n)) {
      constexpr int KS = BM + VT_PAD;
      static_assert(BN * KS * 2 <= SMEM, "the staged value tile fits the LDS stages");
      f16* vs = (f16*)smem;
      __syncthreads();   // X_v1
      // tile column c < BN / 2 is pair c (first dimension half), c + BN / 2 its partner
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const int kl = wm * WM + rb * 16 + lc;
#pragma unroll
        for (int cb = 0; cb < CB / 2; ++cb)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int c = tc[cb] - lc + 4 * lg + e;
            vs[(2 * c) * KS + kl] = from_f32<f16>(acc[rb][cb][e]);
            vs[(2 * c + 1) * KS + kl] = from_f32<f16>(acc[rb][cb + CB / 2][e]);
          }
        __builtin_amdgcn_sched_barrier(0);   // one row block's accumulators in flight at a time
      }
      __syncthreads();   // X_v2
      store_value_tile<BM, BN, NT>(a, vs, tile_n, m0, tid);
      return;
    }
    if (QKV_ONLY_STAGED || qkv_qk_tile<BN>(a, tile_n)) {
      constexpr int RS = BN + QK_PAD;
      static_assert(BM * RS * 2 <= SMEM, "the staged query / key tile fits the LDS stages");
      f16* qs = (f16*)smem;
      const int half = a.hd / 2;
      __syncthreads();   // X_q1: every load landed, every fragment read done
      // pair c < BN / 2 of the tile: head c / half of the tile, dimensions j and j + half
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const int r = wm * WM + rb * 16 + lc, row = m0 + r;
        if (row >= a.M) continue;
        const float2* cs = a.rope + (size_t)a.row_pos[row] * half;
        // a row's angles are all requested before the first is used
        float2 ang[CB / 2][4];
#pragma unroll
        for (int cb = 0; cb < CB / 2; ++cb)
#pragma unroll
          for (int e = 0; e < 4; ++e) ang[cb][e] = cs[(tc[cb] - lc + 4 * lg) % half + e];
#pragma unroll
        for (int cb = 0; cb < CB / 2; ++cb) {
          const int c = tc[cb] - lc + 4 * lg, j = c % half;
          f16* q = qs + r * RS + (c / half) * a.hd + j;
          // copied here and not earlier: the accumulators may fill the accumulation registers
          f32x4 v1 = acc[rb][cb], v2 = acc[rb][cb + CB / 2];
          asm volatile("" : "+v"(v1), "+v"(v2));
          f16x4 o1, o2;
          rope_rotate4(v1, v2, ang[cb], &o1, &o2);
          *(f16x4*)q = o1;
          *(f16x4*)(q + half) = o2;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      __syncthreads();   // X_q2
      store_qk_tile<BM, BN, NT>(a, qs, tile_n, m0, tid);
      return;
    }
  }
  if constexpr (STATS) {
    // decision statistics partial (tile tile_n, wave half wn) of each row, from
    // the fp32 results (the values the logits store would write); columns
    // tb[cb] + e are stat_col(BN, wn, lg, cb, e).  All lanes take part in the
    // shuffles; rows past M (clamped loads) are computed and not written.
    if (a.tstat) {
      const int np = 2 * (a.N / BN);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const int row = m0 + wm * WM + rb * 16 + lc;
        const int rowc = min(row, a.M - 1);
        const int orow = a.out_row ? a.out_row[rowc] : rowc;
        const int cur = a.tg[orow];
        float mx = -INFINITY;
        int ix = 0x7fffffff;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int col = tile_n * BN + tc[cb] - lc + 4 * lg + e;
            const float v = acc[rb][cb][e];
            if (col != a.mask_id && (v > mx || (v == mx && col < ix))) { mx = v; ix = col; }
          }
#pragma unroll
        for (int o = 16; o <= 32; o <<= 1) {
          const float m2 = __shfl_xor(mx, o, 64);
          const int i2 = __shfl_xor(ix, o, 64);
          if (m2 > mx || (m2 == mx && i2 < ix)) { mx = m2; ix = i2; }
        }
        float sum = 0.f;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int col = tile_n * BN + tc[cb] - lc + 4 * lg + e;
            const float v = acc[rb][cb][e];
            if (col != a.mask_id) sum += stat_exp(v, mx);
            if (col == cur && row < a.M) a.zg[orow] = v;
          }
        sum += __shfl_xor(sum, 16, 64);   // (s0 + s1), (s2 + s3)
        sum += __shfl_xor(sum, 32, 64);   // (s0 + s1) + (s2 + s3)
        if (lg == 0 && row < a.M) {
          const size_t pi = (size_t)orow * np + 2 * tile_n + wn;
          a.tstat[pi] = make_float2(mx, sum);
          a.targ[pi] = ix;
        }
      }
      if (!a.C) return;
    }
  }
  // one row block after the other, so that only its accumulators are held in
  // ordinary registers
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int row = m0 + wm * WM + rb * 16 + lc;
    if (row >= a.M) continue;
    int tb[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) tb[cb] = tc[cb] - lc + 4 * lg;
    if constexpr (epi_paired(EPI)) {
#pragma unroll
      for (int cb = 0; cb < CB / 2; ++cb) {
        epi_tile_pair4<EPI, bf16, BN>(a, tile_n, tb[cb], row, acc[rb][cb], acc[rb][cb + CB / 2]);
      }
    } else if constexpr (EPI == EPI_STORE) {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) epi_store4(a, row, tile_n * BN + tb[cb], acc[rb][cb]);
    } else {
      // a row's residuals are all read before any is written back: with one
      // wave per SIMD nothing else hides their latency
      f32x4 x[CB];
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) x[cb] = epi_resid_read4(a, row, tile_n * BN + tb[cb]);
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) epi_resid_write4(a, row, tile_n * BN + tb[cb], x[cb] + acc[rb][cb]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

}  // namespace
