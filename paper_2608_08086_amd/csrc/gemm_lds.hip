// Projection GEMMs, multistage warp-specialised version.
//
// A workgroup has 8 waves: waves 0-3 multiply (a 2 x 2 or 4 x 1 grid of
// wave tiles, MFMA v_mfma_f32_16x16x32_bf16 -- _f16 for the single-term fp16
// operands of the gate/up projection -- fp32 accumulate), waves 4-7 only
// load.  The loaders move the A (two-term: hi and lo) and W tiles of 32-wide k
// chunks straight from global memory into NST LDS stages
// (global_load_lds_dwordx4, no register staging).  With one wave per SIMD
// doing both jobs, a wave blocked issuing loads into a full memory queue also
// stops issuing MFMAs; separate loader waves keep the MFMA pipes fed.
//
// Addressing.  A direct load writes the 16 bytes of lane l at LDS address
// M0 + 16 l, so the LDS layout is fixed by the slot order and each lane
// fetches the global chunk that belongs in its slot.  Tiles are stored
// row-major with 16-byte chunks XOR-swizzled inside a row (physical chunk =
// logical chunk ^ swz(row)), which keeps the MFMA fragment reads free of bank
// conflicts.  The global address of a slot is a per-lane 32-bit offset that
// never changes plus a wave-uniform 64-bit base that advances by 32 elements
// per tile, so the loaders spend no vector instructions on addresses.
//
// Synchronisation (one barrier per tile, all 8 waves).  The multiply waves
// hold the fragments of tile g in registers (read during tile g - 1) and
// place barrier X_g between the hi-term and lo-term MFMAs of tile g (single
// term: between the MFMAs of the first and second half of its weight blocks);
// after X_g they read the fragments of tile g + 1, overlapping the MFMAs that
// follow X_g.
// A loader arrives at X_g once its loads of tile g + 1 have landed
// (s_waitcnt vmcnt; the loads are issued from inline assembly, outside the
// compiler's own wait tracking) and after X_g loads tile g + NST into the
// stage of tile g, which no wave reads any more.
//
// Results are bitwise identical to the register-staged kernel in gemm.hip:
// the same k order (32-wide chunks in order, hi then lo term per chunk), the
// same split-K slices and the same epilogues.  fp16 operands run only here.
#include <algorithm>

#include "gemm_tile.h"

namespace {

template <int BM, int BN, int WGM, int WGN, int NST, int EPI, bool SPLIT, int MODE, bool F16 = false>
__global__ __launch_bounds__(512, 1) void gemm_lds_kernel(GemmArgs a) {
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int RB = WM / 16, CB = WN / 16;
  constexpr int NA = SPLIT ? 2 : 1;
  constexpr int A_SL = BM * CPR, B_SL = BN * CPR;          // 16-byte slots per tile
  constexpr int AI = A_SL / 256, BI = B_SL / 256;          // load instructions per loader wave per tile
  constexpr int IPT = NA * AI + BI;
  constexpr int STAGE = (NA * A_SL + B_SL) * 16;           // bytes
  constexpr bool PARTIAL = MODE == 2, FOLD = MODE == 1;
  static_assert(WGM * WGN == 4 && CB % 2 == 0 && RB >= 1, "bad wave grid");
  static_assert(!F16 || !SPLIT, "fp16 operands are single-term");
  static_assert(A_SL % 256 == 0 && B_SL % 256 == 0, "each loader wave issues whole load instructions");
  static_assert(BN % (32 * WGN) == 0, "each wave takes 16-column blocks from both tile halves");
  static_assert((NST - 1) * IPT <= 63 && NST >= 2, "vmcnt range");
  // the W / W2 split of a SwiGLU tile falls on a wave-instruction boundary
  static_assert((BN / 2) % (64 / CPR) == 0, "pair halves must not share a load instruction");
  __shared__ __attribute__((aligned(1024))) char smem[NST * STAGE];

  const int n_tiles = a.N / BN, m_tiles = (a.M + BM - 1) / BM;
  int tile_n, tile_m, z;
  if (!tile_of(blockIdx.x, n_tiles, m_tiles, PARTIAL ? a.ksplit : 1, &tile_n, &tile_m, &z)) return;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = tile_m * BM;
  const int kslice = a.K / a.ksplit;
  const int kbeg = PARTIAL ? z * kslice : 0;
  const int nslices = FOLD ? a.ksplit : 1;
  const int kt_slice = (PARTIAL || FOLD ? kslice : a.K) / BK;
  const int ntot = nslices * kt_slice;

  if (w >= 4) {
    // ---- loader waves -------------------------------------------------------
    const int wp = w - 4;
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    // per-lane global byte offsets of the slots this lane fills (rows past M
    // load row M - 1: finite data, and those output rows are never stored)
    unsigned a_go[AI], b_go[BI];
    bool b_hi[BI];
#pragma unroll
    for (int j = 0; j < AI; ++j) {
      const int q = j * 256 + wp * 64 + lane, r = q / CPR, pc = q % CPR;
      const int row = min(m0 + r, a.M - 1);
      a_go[j] = ((unsigned)row * (a.a_tiled ? BK : a.lda) + (pc ^ gl_swz(r)) * 8) * 2;
    }
#pragma unroll
    for (int j = 0; j < BI; ++j) {
      const int q = j * 256 + wp * 64 + lane, r = q / CPR, pc = q % CPR;
      bool second;
      const int wr = brow_index<EPI, BN>(a, tile_n, r, &second);
      b_go[j] = ((unsigned)wr * (a.w_tiled ? BK : a.ldw) + (pc ^ gl_swz(r)) * 8) * 2;
      // uniform over the wave's 64 slots (rows j*256/CPR + wp*64/CPR + [0, 64/CPR))
      b_hi[j] = __builtin_amdgcn_readfirstlane(second ? 1 : 0) != 0;
    }
    const bf16* Abase[2] = {(const bf16*)a.A, (const bf16*)(SPLIT ? a.A2 : a.A)};
    const bf16* Wlo = (const bf16*)a.W;
    const bf16* Whi = (const bf16*)(a.W2 ? a.W2 : a.W);
    // tiles past the last are clamped: redundant loads into stages no wave reads again
    // k-block-major A: the block of k step k0 starts k0 * row-capacity elements in
    const size_t akmul = a.a_tiled ? (size_t)a.lda : 1, wkmul = a.w_tiled ? (size_t)a.ldw : 1;
    auto issue = [&](int g) {
      const int k0 = kbeg + min(g, ntot - 1) * BK;
      const unsigned st = lds0 + (unsigned)((g % NST) * STAGE);
#pragma unroll
      for (int t = 0; t < NA; ++t)
#pragma unroll
        for (int j = 0; j < AI; ++j)
          gl_dma16(Abase[t] + (size_t)k0 * akmul, a_go[j], st + (unsigned)((t * A_SL + j * 256 + wp * 64) * 16));
#pragma unroll
      for (int j = 0; j < BI; ++j)
        gl_dma16((b_hi[j] ? Whi : Wlo) + (size_t)k0 * wkmul, b_go[j], st + (unsigned)((NA * A_SL + j * 256 + wp * 64) * 16));
    };
#pragma unroll
    for (int s = 0; s < NST; ++s) issue(s);
    __builtin_amdgcn_s_waitcnt(GL_VMCNT((NST - 1) * IPT));   // tile 0 landed
    gl_barrier();                                             // X_-1
    for (int g = 0; g + 1 < ntot; ++g) {
      __builtin_amdgcn_s_waitcnt(GL_VMCNT((NST - 2) * IPT)); // tile g + 1 landed
      gl_barrier();                                           // X_g
      issue(g + NST);
    }
    // the trailing loads must land before the workgroup's LDS is released
    __builtin_amdgcn_s_waitcnt(GL_VMCNT(0));
    if constexpr (EPI == EPI_QKV && MODE == 0 && SPLIT) {
      if (qkv_value_tile<BN>(a, tile_n)) {
        __syncthreads();   // X_v1: every load landed, every fragment read done
        __syncthreads();   // X_v2: the multiply waves staged the tile
        store_value_tile<BM, BN, 512>(a, (const f16*)smem, tile_n, m0, tid);
      } else if (qkv_qk_tile<BN>(a, tile_n)) {
        __syncthreads();   // X_q1
        __syncthreads();   // X_q2
        store_qk_tile<BM, BN, 512>(a, (const f16*)smem, tile_n, m0, tid);
      }
    }
    return;
  }

  // ---- multiply waves --------------------------------------------------------
  const int lg = lane >> 4, lc = lane & 15;
  const int wm = w / WGN, wn = w % WGN;
  // LDS byte offsets of this lane's fragment reads within a stage
  unsigned a_lo[RB], b_lo[CB];
  int tc[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) tc[cb] = (cb / (CB / 2)) * (BN / 2) + wn * (WN / 2) + (cb % (CB / 2)) * 16 + lc;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int r = wm * WM + rb * 16 + lc;
    a_lo[rb] = (unsigned)((r * CPR + (lg ^ gl_swz(r))) * 16);
  }
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) b_lo[cb] = (unsigned)((NA * A_SL + tc[cb] * CPR + (lg ^ gl_swz(tc[cb]))) * 16);

  f32x4 acc[RB][CB];
  f32x4 tot[FOLD ? RB : 1][FOLD ? CB : 1];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  if constexpr (FOLD) {
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < CB; ++j) tot[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  bf16x8 fa[2][NA][RB], fb[2][CB];
  auto read_frags = [&](int g, int buf) {
    const char* stg = smem + (g % NST) * STAGE;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) fb[buf][cb] = *(const bf16x8*)(stg + b_lo[cb]);
#pragma unroll
    for (int t = 0; t < NA; ++t)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) fa[buf][t][rb] = *(const bf16x8*)(stg + t * A_SL * 16 + a_lo[rb]);
  };
  // Except for split-K partials, the weight fragment is the MFMA's A operand
  // and the activation fragment its B operand (C^T = W A^T), so that a lane's
  // four accumulator entries are four consecutive output columns of one row,
  // which the epilogue writes with vector stores (gate/up -2 %, LM head -3 %
  // measured).  Partial tiles keep C = A W^T and one store per element: their
  // vector stores would touch 16 rows per instruction instead of 4 and were
  // measured no faster.  Either orientation gives the same bits (each output
  // is the same sum of the same products).
  constexpr bool CT = !PARTIAL;
  // one MFMA of weight fragment wf and activation fragment xf in the tile's
  // orientation (the fragments hold fp16 bits when F16)
  auto mm = [&](const bf16x8& wf, const bf16x8& xf, const f32x4& c) __attribute__((always_inline)) {
    if constexpr (F16) {
      const f16x8 w16 = __builtin_bit_cast(f16x8, wf), x16 = __builtin_bit_cast(f16x8, xf);
      return CT ? __builtin_amdgcn_mfma_f32_16x16x32_f16(w16, x16, c, 0, 0, 0)
                : __builtin_amdgcn_mfma_f32_16x16x32_f16(x16, w16, c, 0, 0, 0);
    } else {
      return CT ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, xf, c, 0, 0, 0)
                : __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf, wf, c, 0, 0, 0);
    }
  };
  auto mfma_term = [&](int buf, int t) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) acc[rb][cb] = mm(fb[buf][cb], fa[buf][t][rb], acc[rb][cb]);
  };
  // Two-term tiles of 64, 96 or 128 columns per wave, except in the folded
  // mode (its second accumulator set leaves no room): one fragment set,
  // refilled in place.  The lo-term fragments of tile g are read during its
  // hi-term MFMAs; after X_g the lo-term MFMAs run weight block by weight
  // block, and each weight fragment of tile g + 1 is read as soon as the
  // MFMAs of its block have taken the old one (the hi-term fragments of tile
  // g + 1 go in among the first blocks), so reads never come in a burst.
  // Measured against two fragment sets (a burst of reads after X_g for 96
  // columns, reads spread one per lo-term MFMA for 64): 128 x 192 tiles 5-10 %
  // faster (LLaDA-8B gate/up and QKV shapes at 256 and 768 rows), 128 x 128
  // tiles 0-3 %, bitwise the same.
  constexpr bool ROLL = NA == 2 && (CB == 4 || CB == 6 || CB == 8) && !FOLD;
  // Single-term tiles (except folded): the MFMAs of the first half of the
  // weight blocks of tile g run before X_g, those of the second half after
  // it.  After X_g the weight fragments of the first half are refilled with
  // those of tile g + 1 at once, each of the second half as soon as its
  // block's MFMAs have taken it, and the activation fragments of tile g + 1 go
  // to the second set in among them.
  constexpr bool PIPE1 = NA == 1 && !FOLD;
  auto mfma_blocks = [&](int buf, int cb0, int cb1) {
#pragma unroll
    for (int cb = cb0; cb < cb1; ++cb)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) acc[rb][cb] = mm(fb[0][cb], fa[buf][0][rb], acc[rb][cb]);
  };
  auto tile_roll = [&](int g, bool more) {
    if constexpr (ROLL) {
      const char* stg = smem + (g % NST) * STAGE;
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
          acc[rb][cb] = mm(fb[0][cb], fa[0][0][rb], acc[rb][cb]);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) fa[0][1][rb] = *(const bf16x8*)(stg + A_SL * 16 + a_lo[rb]);
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
      }
      __builtin_amdgcn_sched_group_barrier(0x008, RB * CB - RB, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (more) {
        __builtin_amdgcn_s_waitcnt(GL_LGKMCNT0);   // this wave's reads of tile g are done
        gl_barrier();                               // X_g
        const char* stn = smem + ((g + 1) % NST) * STAGE;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
#pragma unroll
          for (int rb = 0; rb < RB; ++rb)
            acc[rb][cb] = mm(fb[0][cb], fa[0][1][rb], acc[rb][cb]);
          fb[0][cb] = *(const bf16x8*)(stn + b_lo[cb]);
          if (cb < RB) fa[0][0][cb] = *(const bf16x8*)(stn + a_lo[cb]);
        }
        static_assert(RB <= CB, "the hi-term reads go in among the first RB blocks");
#pragma unroll
        for (int cb = 0; cb < RB; ++cb) {
          __builtin_amdgcn_sched_group_barrier(0x008, RB, 0);   // the MFMAs of block cb
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);    // its weight and one hi-term fragment
        }
#pragma unroll
        for (int cb = RB; cb < CB; ++cb) {
          __builtin_amdgcn_sched_group_barrier(0x008, RB, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      } else {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
          for (int rb = 0; rb < RB; ++rb)
            acc[rb][cb] = mm(fb[0][cb], fa[0][1][rb], acc[rb][cb]);
      }
    }
  };
  auto tile_p1 = [&](int g, int cur, bool more) {
    if constexpr (PIPE1) {
      constexpr int H = CB / 2, NB2 = CB - H;
      mfma_blocks(cur, 0, H);
      if (more) {
        __builtin_amdgcn_s_waitcnt(GL_LGKMCNT0);   // this wave's reads of tile g are done
        gl_barrier();                               // X_g
        const char* stn = smem + ((g + 1) % NST) * STAGE;
#pragma unroll
        for (int cb = 0; cb < H; ++cb) fb[0][cb] = *(const bf16x8*)(stn + b_lo[cb]);
#pragma unroll
        for (int i = 0; i < NB2; ++i) {
          const int cb = H + i;
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) acc[rb][cb] = mm(fb[0][cb], fa[cur][0][rb], acc[rb][cb]);
          fb[0][cb] = *(const bf16x8*)(stn + b_lo[cb]);
#pragma unroll
          for (int rb = RB * i / NB2; rb < RB * (i + 1) / NB2; ++rb)
            fa[cur ^ 1][0][rb] = *(const bf16x8*)(stn + a_lo[rb]);
        }
        __builtin_amdgcn_sched_group_barrier(0x100, H, 0);   // the first half's weight fragments
#pragma unroll
        for (int i = 0; i < NB2; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, RB, 0);   // the MFMAs of block H + i
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);    // its weight fragment
#pragma unroll
          for (int rb = RB * i / NB2; rb < RB * (i + 1) / NB2; ++rb)
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // activation fragments
        }
        __builtin_amdgcn_sched_barrier(0);
      } else {
        mfma_blocks(cur, H, CB);
      }
    }
  };
  // folded slices: two fragment sets, the next tile's read between the terms
  auto tile_body = [&](int g, int cur) {
    mfma_term(cur, 0);
    if (g + 1 < ntot) {
      __builtin_amdgcn_s_waitcnt(GL_LGKMCNT0);   // this wave's reads of tile g are done
      gl_barrier();                               // X_g
      read_frags(g + 1, cur ^ 1);
    }
    if constexpr (NA == 2) mfma_term(cur, 1);
    if constexpr (FOLD) {
      if ((g + 1) % kt_slice == 0) {
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
          for (int j = 0; j < CB; ++j) {
            tot[i][j] += acc[i][j];
            acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
      }
    }
  };
  gl_barrier();                                   // X_-1: tile 0 landed
  if constexpr (ROLL) {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) fb[0][cb] = *(const bf16x8*)(smem + b_lo[cb]);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) fa[0][0][rb] = *(const bf16x8*)(smem + a_lo[rb]);
  } else {
    read_frags(0, 0);
  }
  if constexpr (ROLL) {
    // the last tile peeled off: no branch in the loop body
    for (int g = 0; g + 1 < ntot; ++g) tile_roll(g, true);
    tile_roll(ntot - 1, false);
  } else if constexpr (PIPE1 && CB == 8) {
    // no branch in the loop body: with 128 accumulators the copies of a body
    // with branches do not fit the registers (K is a multiple of 64: gemm_lds_cfg_ok)
    int g = 0;
    for (; g + 2 < ntot; g += 2) {
      tile_p1(g, 0, true);
      tile_p1(g + 1, 1, true);
    }
    tile_p1(g, 0, true);
    tile_p1(g + 1, 1, false);
  } else if constexpr (PIPE1) {
    for (int g = 0; g < ntot; g += 2) {           // fragment buffer parity static in the two halves
      tile_p1(g, 0, g + 1 < ntot);
      if (g + 1 < ntot) tile_p1(g + 1, 1, g + 2 < ntot);
    }
  } else {
    for (int g = 0; g < ntot; g += 2) {           // fragment buffer parity static in the two halves
      tile_body(g, 0);
      if (g + 1 < ntot) tile_body(g + 1, 1);
    }
  }

  if constexpr (PARTIAL) {
    // accumulator (rb, cb)[i]: row wm*WM + 16*rb + 4*lg + i, tile column tc[cb]
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = m0 + wm * WM + rb * 16 + lg * 4 + i;
        if (row >= a.M) continue;
        float* pr = a.part + ((size_t)z * a.M + row) * a.N;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) pr[logical_col<EPI, BN>(a, tile_n, tc[cb])] = acc[rb][cb][i];
      }
    }
    return;
  }
  constexpr bool STAGED = EPI == EPI_QKV && MODE == 0 && SPLIT, STATS = EPI == EPI_STORE && !FOLD && WGN == 2;
  if constexpr (FOLD)
    tile_epilogue<BM, BN, WGN, RB, CB, EPI, STAGED, STATS, NST * STAGE, 512>(a, smem, tile_n, m0, wm, wn, lane, tid, tc, tot);
  else
    tile_epilogue<BM, BN, WGN, RB, CB, EPI, STAGED, STATS, NST * STAGE, 512>(a, smem, tile_n, m0, wm, wn, lane, tid, tc, acc);
}

// The launches gemm_pick_cfg makes: 128 x 192 tiles run one slice of bf16 operands or separate
// slices (fp16 operands of one slice have wide tiles, folded ones spill), 128 x 128 tiles all of them.
template <int BN, int EPI, int MODE>
void lds_mode(const GemmArgs& a, int grid, hipStream_t st) {
  if (a.f16) {
    if constexpr (EPI == EPI_SWIGLU && (BN == 128 || MODE == 2))
      gemm_lds_kernel<128, BN, 2, 2, 4, EPI, false, MODE, true><<<grid, 512, 0, st>>>(a);
  } else if (a.A2) {
    gemm_lds_kernel<128, BN, 2, 2, 4, EPI, true, MODE><<<grid, 512, 0, st>>>(a);
  } else {
    gemm_lds_kernel<128, BN, 2, 2, 4, EPI, false, MODE><<<grid, 512, 0, st>>>(a);
  }
}

template <int BN, int EPI>
void lds_cfg(const GemmArgs& a, bool partial, hipStream_t st) {
  const int grid = gemm_grid_size(a.N / BN, (a.M + 127) / 128, partial ? a.ksplit : 1);
  if (partial) {
    lds_mode<BN, EPI, 2>(a, grid, st);
    launch_gemm_reduce(EPI, a, st);
  } else if (a.ksplit > 1) {
    if constexpr (BN == 128) lds_mode<BN, EPI, 1>(a, grid, st);
  } else {
    lds_mode<BN, EPI, 0>(a, grid, st);
  }
}

struct LdsCfg { int BM, BN; };
const LdsCfg kLds[GEMM_NCFG_LDS] = {
    {128, 192},   // 0: 2 x 2 multiply waves of 64 x 96, 4 stages
    {128, 128},   // 1: 2 x 2 multiply waves of 64 x 64, 4 stages
    {128, 256},   // 2: 2 x 2 multiply waves of 64 x 128, 4 stages, one K slice, two-term (or an LM head's statistics)
    {64, 192},    // 3: 2 x 2 multiply waves of 32 x 96, 4 stages, two-term
    {64, 128},    // 4: 2 x 2 multiply waves of 32 x 64, 4 stages, two-term
};

// 64-row tiles, for launches of few rows.  A workgroup of the small tiles was seen
// to get about 60 bytes per ns into its LDS, however many CUs run and however many
// stages are in flight (4 and 7 alike); why no more is not known (28 bytes per clock;
// texture-data and address units 75 and 70 % busy, matrix cores 41, LDS 17 at 256
// rows).  At that rate a k step of a two-term launch costs
// (2 BM + BN) x 64 bytes: beside two activation terms a row costs twice a
// column, and 64 x 192 loads 20 KB where 128 x 128 loads 24 KB for 4 / 3 of the
// products.  LLaDA-8B QKV at 256 rows (256 workgroups against 192) 55 -> 50 us,
// at 120 rows 64 x 128 tiles 52 -> 39 us; down in 4 slices at 120 rows 45 -> 35 us.
// fp16 launches have one activation term and gain nothing (81 us against 56 in
// 128 x 192 tiles at 256 rows, 46 against 43 at 120).  Slices of separate workgroups only.
template <int BN, int EPI>
void lds_rows64(const GemmArgs& a, bool partial, hipStream_t st) {
  const int grid = gemm_grid_size(a.N / BN, (a.M + 63) / 64, partial ? a.ksplit : 1);
  if (partial) {
    gemm_lds_kernel<64, BN, 2, 2, 4, EPI, true, 2><<<grid, 512, 0, st>>>(a);
    launch_gemm_reduce(EPI, a, st);
  } else {
    gemm_lds_kernel<64, BN, 2, 2, 4, EPI, true, 0><<<grid, 512, 0, st>>>(a);
  }
}

template <int EPI>
void lds_epi(int c, const GemmArgs& a, bool partial, hipStream_t st) {
  switch (c) {
    case 0: lds_cfg<192, EPI>(a, partial, st); break;
    case 1: lds_cfg<128, EPI>(a, partial, st); break;
    case 3: lds_rows64<192, EPI>(a, partial, st); break;
    case 4: lds_rows64<128, EPI>(a, partial, st); break;
    default: {
      // one K slice
      const int grid = gemm_grid_size(a.N / 256, (a.M + 127) / 128, 1);
      if (a.A2) {
        gemm_lds_kernel<128, 256, 2, 2, 4, EPI, true, 0><<<grid, 512, 0, st>>>(a);
      } else {
        if constexpr (EPI == EPI_STORE) gemm_lds_kernel<128, 256, 2, 2, 4, EPI, false, 0><<<grid, 512, 0, st>>>(a);
      }
      break;
    }
  }
}

}  // namespace

int gemm_stats_bn(const GemmArgs& head) {
  GemmArgs a = head;
  float2 asked;
  a.tstat = &asked;   // not read: the configuration of a launch with statistics
  // the configurations whose kernel is gemm_lds_kernel with a 2 x 2 wave grid
  const int cfg = gemm_pick_cfg(a, EPI_STORE) - GEMM_NCFG;
  if (cfg < 0 || a.ksplit != 1 || !gemm_lds_cfg_ok(cfg, a)) return 0;
  return kLds[cfg].BN;
}

bool gemm_lds_cfg_ok(int c, const GemmArgs& a) {
  if (c < 0 || c >= GEMM_NCFG_LDS) return false;
  const LdsCfg& k = kLds[c];
  if (a.M <= 0 || a.N % k.BN || a.ksplit < 1 || a.K % (a.ksplit * BK)) return false;
  // single-term launches only for the statistics, whose column tile must not depend on the terms
  if (c == 2 && ((!a.A2 && (!a.tstat || a.K % 64)) || a.ksplit != 1)) return false;
  if (c >= 3 && !a.A2) return false;
  // 32-bit lane offsets
  if ((size_t)a.N * (a.w_tiled ? BK : a.ldw) * 2 >= (1ull << 32) || (size_t)a.M * (a.a_tiled ? BK : a.lda) * 2 >= (1ull << 32))
    return false;
  return true;
}

int launch_gemm_lds_cfg(int epi, int c, bool partial, const GemmArgs& a, hipStream_t st) {
  if (!gemm_args_ok(epi, a) || !gemm_lds_cfg_ok(c, a)) return 1;
  if (partial && (!a.part || a.ksplit < 2)) return 1;
  if (c == 0 && !partial && (a.ksplit != 1 || a.f16)) return 1;
  if (c == 2 && !a.A2 && epi != EPI_STORE) return 1;
  if (c >= 3 && !partial && (a.ksplit != 1 || a.tstat)) return 1;
  switch (epi) {
    case EPI_STORE: lds_epi<EPI_STORE>(c, a, partial, st); break;
    case EPI_RESID: lds_epi<EPI_RESID>(c, a, partial, st); break;
    case EPI_SWIGLU: lds_epi<EPI_SWIGLU>(c, a, partial, st); break;
    case EPI_QKV: lds_epi<EPI_QKV>(c, a, partial, st); break;
    default: return 1;
  }
  return 0;
}
