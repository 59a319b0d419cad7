// Projection GEMMs, wide tiles: four waves, one per SIMD, which both load and
// multiply, so that a wave has the SIMD's whole register file (a 128 x 128 wave
// tile: 256 accumulation registers for the sums, up to 256 others).
//
// What bounds the fp16 tiles is the path of the direct loads into LDS: the
// texture-data unit they pass through is busy 93 % of the cycles, the matrix
// cores 66 % and the LDS itself 17 % (54 % and 20 % in the 128 x 256 tiles of
// gemm_lds.hip, texture data the same).  Loads move about 23 bytes per busy clock
// and CU there, so the tile that loads least per product wins: per 256 x 256 of
// output and k step of 32, tiles of 128 x 256 load 48 KB, of 256 x 256 32 KB.  Measured
// on the LLaDA-8B gate/up shape: 4096 rows 745-790 -> 607-641 us, 24853 rows
// 4540 -> 3680 us (1.36 PFLOP/s; the loop without any load runs at 1.6, where
// random operands hold the clock down).  Two-term bf16 operands take twice the
// MFMAs for half as much again of loads: matrix cores 68-76 % busy, texture data
// 64-72 %, at a clock of 2.0 GHz; they gain less: 4096 rows, down 557 -> 522 us,
// O 201 -> 189.
//
// Two-term steps: the lo fragments of tile g are read among its hi-term MFMAs;
// then the barrier; then, among the lo-term MFMAs, the weight and hi fragments
// of tile g + 1 replace the old ones and the loads of tile g + NST go to the
// stage of tile g, which no wave reads any more.  Single-term steps keep two
// fragment sets and read tile g + 1 among the MFMAs of tile g.  Reads and loads
// are pinned between MFMAs (at most one of each per pair), so that none comes
// in a burst that would hold up the wave's next MFMA.
//
// FOLD tiles run the K slices of a split context one after the other, 128 x 256 so
// that a second set of sums, the running total, fits beside the accumulators: the
// bits of separate slices without their partial planes, for 112 to 131 us per 256
// tiles and K 4096 where half a round of 256 x 256 tiles takes 100 to 113
// (gemm_split_rows says where).
//
// Addressing, stage layout and epilogues are those of gemm_lds.hip, and so are
// the k order and the bits of every result.
#include <algorithm>

#include "gemm_tile.h"

namespace {

template <int BM, int BN, int WGM, int WGN, int NST, int EPI, bool SPLIT, bool F16, bool FOLD>
__global__ __launch_bounds__(256, 1) void gemm_wide_kernel(GemmArgs a) {
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int RB = WM / 16, CB = WN / 16;
  constexpr int NA = SPLIT ? 2 : 1;
  constexpr int A_SL = BM * CPR, B_SL = BN * CPR;          // 16-byte slots per tile
  constexpr int AI = A_SL / 256, BI = B_SL / 256;          // load instructions per wave per tile
  constexpr int IPT = NA * AI + BI;
  constexpr int STAGE = (NA * A_SL + B_SL) * 16;           // bytes
  static_assert(WGM * WGN == 4 && CB % 2 == 0 && RB >= 1, "bad wave grid");
  static_assert(!F16 || !SPLIT, "fp16 operands are single-term");
  static_assert(A_SL % 256 == 0 && B_SL % 256 == 0, "each wave issues whole load instructions");
  static_assert(BN % (32 * WGN) == 0, "each wave takes 16-column blocks from both tile halves");
  static_assert((NST - 1) * IPT <= 63 && NST >= 3, "vmcnt range");
  static_assert((BN / 2) % (64 / CPR) == 0, "pair halves must not share a load instruction");
  __shared__ __attribute__((aligned(1024))) char smem[NST * STAGE];

  const int n_tiles = a.N / BN, m_tiles = (a.M + BM - 1) / BM;
  int tile_n, tile_m, slice;
  if (!tile_of(blockIdx.x, n_tiles, m_tiles, 1, &tile_n, &tile_m, &slice)) return;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = tile_m * BM;
  const int ntot = a.K / BK;

  // ---- loads ------------------------------------------------------------------
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  unsigned a_go[AI], b_go[BI];
  bool b_hi[BI];
#pragma unroll
  for (int j = 0; j < AI; ++j) {
    const int q = j * 256 + w * 64 + lane, r = q / CPR, pc = q % CPR;
    const int row = min(m0 + r, a.M - 1);
    a_go[j] = ((unsigned)row * (a.a_tiled ? BK : a.lda) + (pc ^ gl_swz(r)) * 8) * 2;
  }
#pragma unroll
  for (int j = 0; j < BI; ++j) {
    const int q = j * 256 + w * 64 + lane, r = q / CPR, pc = q % CPR;
    bool second;
    const int wr = brow_index<EPI, BN>(a, tile_n, r, &second);
    b_go[j] = ((unsigned)wr * (a.w_tiled ? BK : a.ldw) + (pc ^ gl_swz(r)) * 8) * 2;
    b_hi[j] = __builtin_amdgcn_readfirstlane(second ? 1 : 0) != 0;
  }
  const bf16* Abase[2] = {(const bf16*)a.A, (const bf16*)(SPLIT ? a.A2 : a.A)};
  const bf16* Wlo = (const bf16*)a.W;
  const bf16* Whi = (const bf16*)(a.W2 ? a.W2 : a.W);
  const size_t akmul = a.a_tiled ? (size_t)a.lda : 1, wkmul = a.w_tiled ? (size_t)a.ldw : 1;
  // load instruction j (0 .. IPT - 1, a constant) of tile g into stage st
  auto issue1 = [&](int g, int st, int j) __attribute__((always_inline)) {
    const size_t k0 = (size_t)min(g, ntot - 1) * BK;
    const unsigned base = lds0 + (unsigned)(st * STAGE);
    if (j < NA * AI) {
      const int t = j / AI, i = j % AI;
      gl_dma16(Abase[t] + k0 * akmul, a_go[i], base + (unsigned)((t * A_SL + i * 256 + w * 64) * 16));
    } else {
      const int i = j - NA * AI;
      gl_dma16((b_hi[i] ? Whi : Wlo) + k0 * wkmul, b_go[i], base + (unsigned)((NA * A_SL + i * 256 + w * 64) * 16));
    }
  };

  // ---- fragments ----------------------------------------------------------------
  const int lg = lane >> 4, lc = lane & 15;
  const int wm = w / WGN, wn = w % WGN;
  // LDS byte offsets of this lane's fragments within a stage: the swizzle repeats
  // every 8 rows, so fragments 16 rows apart differ by a constant
  const int r0 = wm * WM + lc, t0 = wn * (WN / 2) + lc;
  const unsigned a_lo0 = (unsigned)((r0 * CPR + (lg ^ gl_swz(r0))) * 16);
  const unsigned b_lo0 = (unsigned)((NA * A_SL + t0 * CPR + (lg ^ gl_swz(t0))) * 16);
  auto a_at = [&](const char* stg, int rb) __attribute__((always_inline)) { return *(const bf16x8*)(stg + a_lo0 + rb * 16 * CPR * 16); };
  // tile column of weight block cb (lane lc): blocks 0 .. CB/2 - 1 in the first tile half, their partners in the second
  auto tcol = [](int cb) { return (cb / (CB / 2)) * (BN / 2) + (cb % (CB / 2)) * 16; };
  auto b_at = [&](const char* stg, int cb) __attribute__((always_inline)) { return *(const bf16x8*)(stg + b_lo0 + tcol(cb) * CPR * 16); };

  f32x4 acc[RB][CB];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // acc += W fragment x activation fragment, the accumulator pinned to
  // accumulation registers (left to the register allocator, 84 to 380 copies
  // between the two register files stayed in the loop)
  auto mm = [&](const bf16x8& wf, const bf16x8& xf, f32x4& c) __attribute__((always_inline)) {
    if constexpr (F16) asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(c) : "v"(wf), "v"(xf));
    else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(wf), "v"(xf));
  };
  // 11 wait states from the last MFMA of a loop body to anything behind it: the
  // compiler does not know the assembly writes its accumulator late, and places
  // its copies of accumulators after the loop as it likes (none is inside)
  auto settle = [&]() __attribute__((always_inline)) {
    asm volatile("s_nop 10" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  constexpr int T = RB * CB;   // MFMAs per term and k step

  // FOLD: the K slices of a split context in order, each summed from zero and
  // added to the running total, as the reduction of separate slices adds them
  const int nslices = FOLD ? a.ksplit : 1, kt_slice = ntot / nslices;
  f32x4 tot[FOLD ? RB : 1][FOLD ? CB : 1];
  if constexpr (FOLD) {
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < CB; ++j) tot[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  auto fold = [&]() __attribute__((always_inline)) {
    if constexpr (FOLD) {
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j) {
          tot[i][j] += acc[i][j];
          acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      settle();   // the zeros are written before the next slice's first product reads them
    }
  };

#pragma unroll
  for (int s = 0; s < NST; ++s)
#pragma unroll
    for (int j = 0; j < IPT; ++j) issue1(s, s, j);
  __builtin_amdgcn_s_waitcnt(GL_VMCNT((NST - 1) * IPT));
  gl_barrier();

  if constexpr (SPLIT) {
    bf16x8 fh[RB], fl[RB], fb[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) fb[cb] = b_at(smem, cb);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) fh[rb] = a_at(smem, rb);
    auto step = [&](int g, int st, int stn) __attribute__((always_inline)) {
      const char* cur = smem + st * STAGE;
      const char* nxt = smem + stn * STAGE;
      // hi term; the lo fragments of this tile are read among the first MFMAs
#pragma unroll
      for (int i = 0; i < T; ++i) {
        const int cb = i / RB, rb = i % RB;
        mm(fb[cb], fh[rb], acc[rb][cb]);
        if (i < 2 * RB && (i & 1)) {
          fl[i / 2] = a_at(cur + A_SL * 16, i / 2);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(GL_VMCNT((NST - 2) * IPT) & GL_LGKMCNT0);
      gl_barrier();
      // lo term; the weight and hi fragments of the next tile replace the old
      // ones, and this tile's stage is refilled
#pragma unroll
      for (int i = 0; i < T; ++i) {
        const int cb = i / RB, rb = i % RB;
        mm(fb[cb], fl[rb], acc[rb][cb]);
        if (i < 2 * RB && (i & 1)) fh[i / 2] = a_at(nxt, i / 2);
        if (rb == RB - 1) fb[cb] = b_at(nxt, cb);
        const int d0 = i * IPT / T, d1 = (i + 1) * IPT / T;
        if (d1 > d0) issue1(g + NST, st, d0);
        if ((i & 1) || rb == RB - 1 || d1 > d0) __builtin_amdgcn_sched_barrier(0);
      }
      settle();
    };
    // every step alike, the last included (it refills from a clamped tile): no
    // product is issued outside the loop body
    for (int sl = 0, g = 0, st = 0; sl < nslices; ++sl) {
      for (const int end = g + kt_slice; g < end; ++g) {
        const int stn = st + 1 == NST ? 0 : st + 1;
        step(g, st, stn);
        st = stn;
      }
      fold();
    }
  } else {
    bf16x8 fa[2][RB], fb[2][CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) fb[0][cb] = b_at(smem, cb);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) fa[0][rb] = a_at(smem, rb);
    auto step = [&](int g, int st, int stn, int c) __attribute__((always_inline)) {
      const char* nxt = smem + stn * STAGE;
      __builtin_amdgcn_s_waitcnt(GL_VMCNT((NST - 2) * IPT) & GL_LGKMCNT0);
      gl_barrier();
      constexpr int NR = RB + CB;
#pragma unroll
      for (int i = 0; i < T; ++i) {
        const int cb = i / RB, rb = i % RB;
        mm(fb[c][cb], fa[c][rb], acc[rb][cb]);
        // two thirds of the step's MFMAs carry the reads, all of them the loads
        const int q0 = min(i * NR * 3 / (2 * T), NR), q1 = min((i + 1) * NR * 3 / (2 * T), NR);
        if (q1 > q0) {
          if (q0 < CB) fb[c ^ 1][q0] = b_at(nxt, q0);
          else fa[c ^ 1][q0 - CB] = a_at(nxt, q0 - CB);
        }
        const int d0 = i * IPT / T, d1 = (i + 1) * IPT / T;
        if (d1 > d0) issue1(g + NST, st, d0);
        if (q1 > q0 || d1 > d0) __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    // an even number of steps (K slices are multiples of 64): the fragment set is static
    for (int sl = 0, g = 0, st = 0; sl < nslices; ++sl) {
      for (const int end = g + kt_slice; g < end; g += 2) {
        const int s1 = st + 1 == NST ? 0 : st + 1, s2 = s1 + 1 == NST ? 0 : s1 + 1;
        step(g, st, s1, 0);
        step(g + 1, s1, s2, 1);
        settle();
        st = s2;
      }
      fold();
    }
  }
  __builtin_amdgcn_s_waitcnt(GL_VMCNT(0));   // the trailing loads land before the LDS is reused or released

  int tc[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) tc[cb] = tcol(cb) + t0;
  // 256 x 256 QKV tiles leave no registers for the element-wise stores of a tile
  // that straddles the value heads: only launches without such tiles take them
  // (and even so three registers go through scratch memory between the loop and the stores)
  constexpr bool QKV = EPI == EPI_QKV, ONLY_STAGED = BM * BN == 65536;
  if constexpr (FOLD)
    tile_epilogue<BM, BN, WGN, RB, CB, EPI, QKV, false, NST * STAGE, 256, ONLY_STAGED>(a, smem, tile_n, m0, wm, wn, lane,
                                                                                       tid, tc, tot);
  else
    tile_epilogue<BM, BN, WGN, RB, CB, EPI, QKV, false, NST * STAGE, 256, ONLY_STAGED>(a, smem, tile_n, m0, wm, wn, lane,
                                                                                       tid, tc, acc);
}

}  // namespace


namespace {

template <int BM, int BN, int NST, int EPI, bool SPLIT, bool F16 = false, bool FOLD = false>
void wide(const GemmArgs& a, hipStream_t st) {
  const int grid = gemm_grid_size(a.N / BN, (a.M + BM - 1) / BM, 1);
  gemm_wide_kernel<BM, BN, 2, 2, NST, EPI, SPLIT, F16, FOLD><<<grid, 256, 0, st>>>(a);
}

template <int EPI>
int wide_epi(int c, const GemmArgs& a, hipStream_t st) {
  switch (c) {
    case GEMM_WIDE_256x256:
      if (a.f16) {
        if constexpr (EPI == EPI_SWIGLU) wide<256, 256, 4, EPI, false, true>(a, st);
      } else {
        wide<256, 256, 3, EPI, true>(a, st);
      }
      return 0;
    case GEMM_WIDE_FOLD_128x256:
      if (a.f16) {
        if constexpr (EPI == EPI_SWIGLU) wide<128, 256, 4, EPI, false, true, true>(a, st);
      } else {
        if constexpr (EPI != EPI_STORE) wide<128, 256, 4, EPI, true, false, true>(a, st);
      }
      return 0;
    case GEMM_WIDE_256x192:
      if constexpr (EPI == EPI_SWIGLU) {
        if (a.f16) wide<256, 192, 5, EPI, false, true>(a, st);
        else wide<256, 192, 3, EPI, true>(a, st);
        return 0;
      }
      if constexpr (EPI == EPI_QKV) {
        wide<256, 192, 3, EPI, true>(a, st);
        return 0;
      }
      return 1;
    default:
      if constexpr (EPI == EPI_SWIGLU) {
        wide<128, 192, 4, EPI, false, true>(a, st);
        return 0;
      }
      return 1;
  }
}

}  // namespace

bool gemm_wide_ok(int c, const GemmArgs& a, int epi) {
  // one K slice, or all slices folded; two-term bf16 operands, or single-term fp16 ones (gate/up)
  // (no statistics epilogue: it does not fit beside 256 accumulators)
  if ((epi == EPI_STORE && a.tstat) || (!a.A2 && !a.f16) || a.ksplit < 1 || a.K % (64 * a.ksplit)) return false;
  if ((a.ksplit > 1) != (c == GEMM_WIDE_FOLD_128x256)) return false;
  // 32-bit lane offsets
  if ((size_t)a.N * (a.w_tiled ? BK : a.ldw) * 2 >= (1ull << 32) || (size_t)a.M * (a.a_tiled ? BK : a.lda) * 2 >= (1ull << 32))
    return false;
  switch (c) {
    case GEMM_WIDE_256x256: return a.N % 256 == 0 && (epi != EPI_QKV || qkv_all_staged(a, 256));
    case GEMM_WIDE_256x192: return a.N % 192 == 0 && (epi == EPI_SWIGLU || epi == EPI_QKV);
    case GEMM_WIDE_128x192: return a.N % 192 == 0 && epi == EPI_SWIGLU && a.f16;
    case GEMM_WIDE_FOLD_128x256: return a.N % 256 == 0 && epi != EPI_STORE;
    default: return false;
  }
}

int launch_gemm_wide(int epi, int c, const GemmArgs& a, hipStream_t st) {
  if (!gemm_wide_ok(c, a, epi)) return 1;
  switch (epi) {
    case EPI_STORE: return wide_epi<EPI_STORE>(c, a, st);
    case EPI_RESID: return wide_epi<EPI_RESID>(c, a, st);
    case EPI_SWIGLU: return wide_epi<EPI_SWIGLU>(c, a, st);
    case EPI_QKV: return wide_epi<EPI_QKV>(c, a, st);
    default: return 1;
  }
}
