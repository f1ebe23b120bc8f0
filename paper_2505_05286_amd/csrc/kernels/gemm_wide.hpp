// bf16 "NT" GEMM C[M,N] = A[M,K] * B[N,K]^T with the weights read straight into registers.
// Instantiated by gemm_wide_*.hip, one epilogue each.
#pragma once

#include "gemm_util.hpp"

namespace hxf {

namespace {

// Macro tiles of 16 TM rows x 16 NW WV columns on the 16x16x32 MFMA: WV wavefronts, each owning all
// the tile's rows and 16 NW of its columns (NW = 4, or 2 where narrow tiles fill the chip: the few
// rows of a decode step, or more rows of an output of a few thousand columns).  The weights go
// straight from memory to registers (a wavefront's columns are its own, so nothing is read twice in a
// workgroup; a packed tile is one contiguous kilobyte per load), R steps of 32 of K ahead; only the
// activations pass through LDS, stages of 64 of K by buffer DMA, NS in flight.
//
// Why: with both operands staged in LDS by eight wavefronts (192 x 256 tiles, 1.1 KB through LDS per
// 32x32x16 MFMA) the wavefronts spent 37-49% of their cycles waiting for those DMAs, with the matrix pipes
// busy 31-52% and LDS reads 19-27% of the time.  Here the weights are requested R steps ahead of their
// use and no barrier stands between, an A fragment feeds four MFMAs and only A is written (0.6 KB):
// 12-28% of the cycles waiting, matrix pipes busy 38% (O) to 62% (gate/up) at a clock that falls from
// 2.26 to 1.97 GHz as they get busier, LDS reads 10-16%.  One
// wavefront per SIMD keeps the accumulators (4 TM registers x 4) in AGPRs and needs its own
// overlap: the A fragments of step k + 1 are read into the registers that step k has just
// used, one LDS read after every NW MFMAs, and the barrier of a stage lies half a stage
// before its first use.  Measured (2080 rows, back to back, against 8 wavefronts with both
// operands in LDS): 57344 x 8192 SwiGLU from row-major activations 1970 -> 1512 us
// (1.29 PFLOP/s), 6144 x 4096 112 -> 89, 4096 x 14336 290 -> 219; 32x32x16 MFMAs on this
// scheme are 5% slower, 8 steps of weights ahead 5-7%, 2 steps 2-4%, two workgroups per CU of
// half the rows 5-10%.  With 8 wavefronts (144 rows x 512 columns, two per SIMD) 8192 x 28672
// takes 847 us against 927 in the best tile of 4: 240 tiles, one round of the chip (three registers
// spill in its loop).
//
// NW = 2 above 128 rows: an A fragment feeds two MFMAs instead of four, but a workgroup fetches half
// the weights per step, which is what bounds it there (16 KB per 0.31 us and CU with 64 x 256 tiles),
// and there are twice as many.  4096 x 14336 at 513 rows: 160 workgroups of 96 x 128 in 92 us, 144
// of 64 x 256 in 141; both operands through LDS took 108.
//
// Up to 128 rows the bytes of the weights are the bound: non-temporal loads where one row of tiles
// reads them (55296 x 5120 at 64 rows 101.4 -> 93.0 us, 128256 x 4096 201 -> 182; the first pass over
// weights just written also waits for the memory-side cache to write back up to 256 MB of them,
// 128256 x 8192 at 64 rows 410 us then and 333 after, whatever the order of the tiles), and against a
// kernel with the weights in LDS: one row 37.5 -> 36.0 us (28672 x 4096) and 19.4 -> 17.3 (4096 x
// 14336), 64 rows 44.5 -> 41.2 and 24.4 -> 24.0, 64 x 128256 x 4096 203 -> 182.
//
// Row-major activations are staged as 8 rows x 128 bytes per DMA (whole cache lines), with the eight
// 16-byte chunks of row r stored in the order chunk ^ (r / 2 % 8), so that the 16 lanes of a fragment
// read touch 16 different 16-byte columns of LDS; packed activations are 1 KB tiles in operand order
// already.  SwiGLU groups logical columns by 64 (32 gate rows, then the 32 matching up rows; by 32
// with NW = 2) so one lane holds both.  Weights are the first MFMA operand, so a lane ends up with 4
// consecutive columns of one row and stores them together.
// SPLIT: grid.y cuts K into chunks of k_chunk (a multiple of 64); each writes its fp32 partial
// [M][N] to slot blockIdx.y of a.partial (SwiGLU: with NW = 2, logical columns in groups of 16 gate
// and 16 up).
// SHORT: K of at most 256 with one row of tiles: all of it is requested at once and multiplied
// after one wait, because the pipeline's start and end (a wait and a barrier per 64 of K, steps over zeros) are a tenth of such a
// call: 1, 2 and 16 rows of 512 x 256 2.65 / 3.4 / 3.6 us against 3.1 / 3.9 / 4.0, 1376 x 256 SwiGLU
// 3.7 / 3.9 / 3.8 against 4.2 / 4.4 / 4.2.  (As a branch of the same kernel it made K = 688 0.3 us
// slower; from 33 rows on it gains nothing.)
template <int TM, int NW, int R, int EPI, bool SPLIT, int WV, int OCC, int CACHE, bool SHORT>
__global__ __launch_bounds__(64 * WV, OCC) void gemm_wide_kernel(GemmArgs a) {
  constexpr int BM = 16 * TM, BN = 16 * NW * WV, NS = 4;
  constexpr int A_BLK = TM * 2, A_PW = (A_BLK + WV - 1) / WV, STAGE = A_BLK * 512;   // 1 KB blocks per stage, per wavefront
  constexpr bool SW = (EPI == EPI_SWIGLU);
  // outstanding loads allowed when stage s + 1 must have landed: the younger stages' DMAs and
  // the weight loads issued since its own DMAs (the first step's of the same pass may have been
  // scheduled before those)
  constexpr int WAIT = (NS - 3) * A_PW + 2 * NW * (NS - 2) - NW;
  static_assert((2 * NS) % R == 0 && WAIT < 64 && NW * R + (NS - 2) * A_PW < 64, "pipeline");
  static_assert(!SW || NW % 2 == 0, "a wavefront holds as many up columns as gate columns");
  static_assert(NS * STAGE * 2 <= 160 * 1024, "stage layout");
  static_assert(!(SW && SPLIT) || NW == 2, "partials hold logical columns in groups of 16 gate and 16 up");
  __shared__ __attribute__((aligned(1024))) bf16_t L0[STAGE], L1[STAGE], L2[STAGE], L3[STAGE];
  auto slot = [&](auto ic) -> bf16_t* {
    constexpr int I = decltype(ic)::value % NS;
    if constexpr (I == 0) return L0; else if constexpr (I == 1) return L1; else if constexpr (I == 2) return L2;
    else return L3;
  };
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
  const int L = xcd_remap(blockIdx.x, tiles_m * tiles_n);
  const int tn = SHORT ? L : L / tiles_m, tm = SHORT ? 0 : L % tiles_m;
  const int m0 = tm * BM, n0 = tn * BN;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kb = SPLIT ? blockIdx.y * (a.k_chunk / 32) : 0;              // first step (32 of K)
  const int kt = (SPLIT ? min(a.kt, kb + a.k_chunk / 32) : a.kt) - kb;   // steps
  const int nst = (kt + 1) / 2;                                          // stages (64 of K)

  // activation DMA: block (row tile rt, kk) of the stage; packed: the tile's half kk; row-major:
  // rows 8 kk .. 8 kk + 7 of the tile (rows past M repeat the last one; never stored)
  const int rows_left = a.M - m0;
  const rsrc_t ra = a.a_packed
      ? make_rsrc(a.A + (size_t)(m0 / 16) * a.kt * 512, (uint32_t)min(TM, (rows_left + 15) / 16) * a.kt * 1024)
      : make_rsrc(a.A + (size_t)m0 * a.lda, (uint32_t)((min(BM, rows_left) - 1) * a.lda + a.K) * 2);
  const int k_end = (a.a_packed ? a.kt * 32 : a.K) - kb * 32 - (nst - 1) * 64;   // of the last stage
  int a_off[A_PW], a_dst[A_PW];
  bool a_in[A_PW];   // the lane's chunk of the last stage lies inside K
#pragma unroll
  for (int u = 0; u < A_PW; ++u) {
    const int b = min(w * A_PW + u, A_BLK - 1), rt = b >> 1, kk = b & 1;
    const int r8 = kk * 8 + (lane >> 3), ch = (lane & 7) ^ (r8 >> 1);
    a_dst[u] = b * 512;
    a_in[u] = (a.a_packed ? kk * 32 : ch * 8) < k_end;
    a_off[u] = 2 * (a.a_packed ? (min(rt, (rows_left - 1) / 16) * a.kt + kk) * 512 + lane * 8
                               : min(rt * 16 + r8, rows_left - 1) * a.lda + ch * 8);
  }
  const int a_step = a.a_packed ? 2048 : 128, a_first = (kb / 2) * a_step;   // bytes per stage (kb is even)
  auto issue_a = [&](int s, bf16_t* base) __attribute__((always_inline)) {
    const int ss = min(s, nst - 1);
    // past the last stage: zeros.  Out of range by or-ing (kOutOfRange is the sign bit): as conditions
    // these became branches that cut the loop into blocks, and the 8-wavefront tile spilled in it
    const int past = s >= nst ? kOutOfRange : 0, last = s == nst - 1 ? kOutOfRange : 0;
#pragma unroll
    for (int u = 0; u < A_PW; ++u)
      buf_dma16(ra, a_off[u] | past | (a_in[u] ? 0 : last), a_first + ss * a_step, base + a_dst[u]);
  };
  // weights: the wavefront's NW column tiles, for SwiGLU NW / 2 of the gate and the same NW / 2 of
  // the up matrix (tiles past N: zeros, or the last one again)
  constexpr int HALF = SW ? NW / 2 : NW;
  const int n_out = SW ? a.N / 2 : a.N, c0 = (n0 + w * NW * 16) / (SW ? 2 : 1);   // output columns, the wavefront's first
  const int b_tiles = (n_out + 15) / 16, bt = min(c0 / 16, b_tiles - 1);
  const uint32_t b_bytes = (uint32_t)min(HALF, b_tiles - bt) * a.kt * 1024;
  const rsrc_t rb0 = make_rsrc(a.B + (size_t)bt * a.kt * 512, b_bytes);
  const rsrc_t rb1 = SW ? make_rsrc(a.B2 + (size_t)bt * a.kt * 512, b_bytes) : rb0;
  int b_off[HALF];
#pragma unroll
  for (int j = 0; j < HALF; ++j) b_off[j] = lane * 16 + j * a.kt * 1024;
  uint4 fb[R][NW];
  auto load_b = [&](auto rc, int k) __attribute__((always_inline)) {
    constexpr int r = decltype(rc)::value % R;
    const int kk = kb + min(k, kt - 1), past = k < kt ? 0 : kOutOfRange;
#pragma unroll
    for (int j = 0; j < NW; ++j)   // past the last step: zeros
      fb[r][j] = buf_load16<CACHE>(j < HALF ? rb0 : rb1, b_off[j % HALF] | past, kk * 1024);
  };
  f32x4 acc[TM][NW];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < NW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 fa[TM];
  // LDS offset of the lane's fragment in a row tile, by step of the stage
  int f_off[2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
    f_off[h] = a.a_packed ? h * 512 + lane * 8
                          : (lane & 15) * 64 + (((h * 4 + (lane >> 4)) ^ ((lane & 15) >> 1)) * 8);
  auto read_a = [&](const bf16_t* base, int i, int h) __attribute__((always_inline)) {
    return as_bf16x8(*reinterpret_cast<const uint4*>(base + i * 1024 + f_off[h]));
  };
  // one step with the weights of ring slot r; reads the next step's fragments as it goes
  auto step = [&](auto rc, const bf16_t* next, int h) __attribute__((always_inline)) {
    constexpr int r = decltype(rc)::value % R;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < NW; ++j) acc[i][j] = mfma16x16x32(as_bf16x8(fb[r][j]), fa[i], acc[i][j]);
      fa[i] = read_a(next, i, h);
    }
    static_for<TM>([&](auto) {
      __builtin_amdgcn_sched_group_barrier(0x008, NW, 0);   // MFMAs
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);    // one LDS read
    });
  };
  if constexpr (SHORT) {
    static_assert(R == 2 * NS && !SPLIT, "a ring slot per step, a stage per slot");
    static_for<R>([&](auto ic) { load_b(ic, decltype(ic)::value); });
    static_for<NS>([&](auto ic) { issue_a(decltype(ic)::value, slot(ic)); });   // past the last: zeros, as the weights
    wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    static_for<NS>([&](auto ic) {
      bf16x8 f[2][TM];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < TM; ++i) f[h][i] = read_a(slot(ic), i, h);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < NW; ++j)
            acc[i][j] = mfma16x16x32(as_bf16x8(fb[2 * decltype(ic)::value + h][j]), f[h][i], acc[i][j]);
    });
  } else {
  static_for<NS - 1>([&](auto ic) {
    issue_a(decltype(ic)::value, slot(ic));
    __builtin_amdgcn_sched_barrier(0);   // the waits below count in this order
  });
  static_for<R>([&](auto ic) { load_b(ic, decltype(ic)::value); });
  __builtin_amdgcn_sched_barrier(0);
  wait_vmcnt<NW * R + (NS - 2) * A_PW>();
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int i = 0; i < TM; ++i) fa[i] = read_a(L0, i, 0);
  step(std::integral_constant<int, 0>{}, L0, 1);
  load_b(std::integral_constant<int, 0>{}, R);
  __builtin_amdgcn_sched_barrier(0);
  // pass s: the second step of stage s (it reads stage s + 1's first fragments) and the first
  // of stage s + 1.  Every LDS read follows, without a branch, the wait for its stage's DMA,
  // and the loop has one exit: otherwise the compiler adds waits for everything in flight.
  // Whole trips of 2 NS steps; a last trip that has at least three steps of its own runs on
  // over zeros (0 x 0 in both operands), which costs less than so many single steps.
  const int s_end = (kt - 1 + 2 * NS - 3) / (2 * NS) * NS;
  int s0 = 0;
  for (; s0 < s_end; s0 += NS) {
    static_for<NS>([&](auto ic) {
      constexpr int J = decltype(ic)::value;
      wait_vmcnt<WAIT>();
      __builtin_amdgcn_s_barrier();
      issue_a(s0 + J + NS - 1, slot(std::integral_constant<int, J + NS - 1>{}));
      const bf16_t* next = slot(std::integral_constant<int, J + 1>{});
      step(std::integral_constant<int, 2 * J + 1>{}, next, 0);
      load_b(std::integral_constant<int, 2 * J + 1>{}, (s0 + J) * 2 + 1 + R);
      __builtin_amdgcn_sched_barrier(0);
      step(std::integral_constant<int, 2 * J + 2>{}, next, 1);
      load_b(std::integral_constant<int, 2 * J + 2>{}, (s0 + J) * 2 + 2 + R);
      __builtin_amdgcn_sched_barrier(0);
    });
  }
  // one or two remaining steps singly, the ring shifted by copies
  auto dyn_slot = [&](int i) -> bf16_t* {
    i %= NS;
    return i == 0 ? L0 : i == 1 ? L1 : i == 2 ? L2 : L3;
  };
  for (int k = 2 * s0 + 1; k < kt; ++k) {
    if (k & 1) {
      wait_vmcnt<0>();
      __builtin_amdgcn_s_barrier();
      issue_a((k >> 1) + NS - 1, dyn_slot((k >> 1) + NS - 1));
    }
    step(std::integral_constant<int, 1>{}, dyn_slot((k >> 1) + (k & 1)), (k & 1) ^ 1);
#pragma unroll
    for (int j = 0; j < NW; ++j) {
#pragma unroll
      for (int r = 1; r < R; ++r) fb[r][j] = fb[(r + 1) % R][j];
    }
    load_b(std::integral_constant<int, 0>{}, k + R);
  }
  wait_vmcnt<0>();
  }

  // lane holds row l % 16 and columns 4 (l / 16) .. + 3 of each 16 x 16 tile
  const int col4 = (lane >> 4) * 4;
  float* P = SPLIT ? a.partial + (size_t)blockIdx.y * a.M * a.N : nullptr;
  const int ld = SPLIT ? a.N : a.ldc;
  // four columns at once where every group of four is whole and aligned
  const bool vec = SW && !SPLIT && a.c_kt ? ((uintptr_t)a.C & 7) == 0
                                : ((ld | a.N) & 3) == 0 && ((SPLIT ? (uintptr_t)P : (uintptr_t)a.C) & 15) == 0;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int row = m0 + i * 16 + (lane & 15);
    if (row >= a.M) continue;
    if constexpr (SW && !SPLIT) {
#pragma unroll
      for (int j = 0; j < HALF; ++j) {
        const int oc = c0 + j * 16 + col4;
        if (oc >= n_out) continue;
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float g = acc[i][j][e];
          o[e] = g / (1.f + __expf(-g)) * acc[i][j + HALF][e];
        }
        bf16_t* c = reinterpret_cast<bf16_t*>(a.C) + (a.c_kt ? packed_elem(row, oc, a.c_kt) : (size_t)row * a.ldc + oc);
        if (vec) {
          *reinterpret_cast<uint2*>(c) = make_uint2(pack_bf2(o[0], o[1]), pack_bf2(o[2], o[3]));
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) c[e] = f2bf(o[e]);
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < NW; ++j) {
        const int col = n0 + (w * NW + j) * 16 + col4;
        if (col >= a.N) continue;
        const size_t o = (size_t)row * ld + col;
        const f32x4 v = acc[i][j];
        if constexpr (EPI == EPI_BF16 && !SPLIT) {
          bf16_t* c = reinterpret_cast<bf16_t*>(a.C) + o;
          if (vec) {
            *reinterpret_cast<uint2*>(c) = make_uint2(pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]));
          } else {
            for (int e = 0; e < 4 && col + e < a.N; ++e) c[e] = f2bf(v[e]);
          }
        } else {
          float* c = (SPLIT ? P : reinterpret_cast<float*>(a.C)) + o;
          constexpr bool ADD = EPI == EPI_RESID && !SPLIT;
          if (vec) {
            float4 x = ADD ? *reinterpret_cast<const float4*>(c) : make_float4(0.f, 0.f, 0.f, 0.f);
            *reinterpret_cast<float4*>(c) = ADD ? make_float4(x.x + v[0], x.y + v[1], x.z + v[2], x.w + v[3])
                                                : make_float4(v[0], v[1], v[2], v[3]);
          } else {
            for (int e = 0; e < 4 && col + e < a.N; ++e) c[e] = ADD ? c[e] + v[e] : v[e];
          }
        }
      }
    }
  }
}

// Shapes: 16 tm rows x 16 nw wv columns.  Weights that one row of tiles reads (tiles_m == 1) are
// fetched with the non-temporal hint (p.once).
template <int TM, int NW, int WV, int CACHE, int EPI, bool SPLIT, bool SHORT = false>
hipError_t launch_wide(const GemmArgs& a, const GemmPlan& p, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  constexpr int BM = 16 * TM, BN = 16 * NW * WV, R = WV == 8 ? 2 : NW == 2 ? 8 : 4, OCC = WV / 4;
  const int nb = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  return launch_ev(gemm_wide_kernel<TM, NW, R, EPI, SPLIT, WV, OCC, CACHE, SHORT>, dim3(nb, p.splits), dim3(64 * WV), st, e0,
                   e1, a);
}

template <int EPI, bool SPLIT>
hipError_t launch_wide_cfg(const GemmArgs& a, const GemmPlan& p, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
#define HXF_WIDE(T, NW, WV, CACHE) \
  case T: return launch_wide<T, NW, WV, CACHE, EPI, SPLIT>(a, p, st, e0, e1);
  if constexpr (!SPLIT) {
    if (p.nw == 2 && p.once && a.kt <= 8 && a.M <= 16 * p.tm) {
      if (p.tm == 1) return launch_wide<1, 2, 4, 2, EPI, false, true>(a, p, st, e0, e1);
      if (p.tm == 2) return launch_wide<2, 2, 4, 2, EPI, false, true>(a, p, st, e0, e1);
    }
  }
  if (p.nw == 2 && p.once) switch (p.tm) {
      HXF_WIDE(1, 2, 4, 2) HXF_WIDE(2, 2, 4, 2) HXF_WIDE(4, 2, 4, 2) HXF_WIDE(8, 2, 4, 2)
    }
  else if (p.nw == 2) switch (p.tm) {
      HXF_WIDE(3, 2, 4, 0) HXF_WIDE(4, 2, 4, 0) HXF_WIDE(5, 2, 4, 0) HXF_WIDE(6, 2, 4, 0) HXF_WIDE(7, 2, 4, 0)
      HXF_WIDE(8, 2, 4, 0) HXF_WIDE(9, 2, 4, 0) HXF_WIDE(10, 2, 4, 0) HXF_WIDE(11, 2, 4, 0) HXF_WIDE(12, 2, 4, 0)
    }
  else if (p.wv == 4 && p.once) switch (p.tm) {
      HXF_WIDE(10, 4, 4, 2) HXF_WIDE(12, 4, 4, 2) HXF_WIDE(14, 4, 4, 2) HXF_WIDE(16, 4, 4, 2)
    }
  else if (p.wv == 4) switch (p.tm) {
      HXF_WIDE(4, 4, 4, 0) HXF_WIDE(5, 4, 4, 0) HXF_WIDE(6, 4, 4, 0) HXF_WIDE(7, 4, 4, 0) HXF_WIDE(8, 4, 4, 0)
      HXF_WIDE(9, 4, 4, 0) HXF_WIDE(10, 4, 4, 0) HXF_WIDE(11, 4, 4, 0) HXF_WIDE(12, 4, 4, 0) HXF_WIDE(13, 4, 4, 0)
      HXF_WIDE(14, 4, 4, 0) HXF_WIDE(15, 4, 4, 0) HXF_WIDE(16, 4, 4, 0)
    }
  // few rows split K with 32 columns per wavefront only, eight wavefronts never do
  if constexpr (!SPLIT) {
    if (p.nw == 4 && p.wv == 4 && p.once) switch (p.tm) {
        HXF_WIDE(1, 4, 4, 2) HXF_WIDE(2, 4, 4, 2) HXF_WIDE(4, 4, 4, 2) HXF_WIDE(6, 4, 4, 2) HXF_WIDE(8, 4, 4, 2)
      }
    if (p.nw == 4 && p.wv == 8) switch (p.tm) { HXF_WIDE(9, 4, 8, 0) }
  }
#undef HXF_WIDE
  return hipErrorInvalidValue;
}

}  // namespace

}  // namespace hxf
