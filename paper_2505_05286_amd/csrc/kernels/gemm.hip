// Dispatch of the bf16 "NT" GEMMs C[M,N] = A[M,K] * B[N,K]^T (fp32 accumulator; bf16 store,
// fp32 residual add, SwiGLU gate*up or fp32 store, or fp32 split-K partials): the choice of
// tile and K split, the split-K reduction and the weight packing.  The kernel is
// gemm_wide_kernel (gemm_wide.hpp).
#include <algorithm>

#include "gemm_util.hpp"

namespace hxf {

namespace {

// 16-byte load from a 16-byte aligned address (one global_load_dwordx4).
__device__ __forceinline__ uint4 load16(const bf16_t* p) {
  const u32x4_t v = *reinterpret_cast<const u32x4_t*>(__builtin_assume_aligned(p, 16));
  return make_uint4(v.x, v.y, v.z, v.w);
}

// Sum split-K partials in a fixed order and apply the epilogue.
template <int EPI>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(GemmArgs a, int S) {
  const int n_out = (EPI == EPI_SWIGLU) ? a.N / 2 : a.N;
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (size_t)a.M * n_out) return;
  const int row = idx / n_out, col = idx % n_out;
  const size_t MN = (size_t)a.M * a.N;
  if (EPI == EPI_SWIGLU) {
    const int lg = (col >> 4) * 32 + (col & 15);
    float g = 0.f, u = 0.f;
    for (int z = 0; z < S; ++z) {
      g += a.partial[z * MN + (size_t)row * a.N + lg];
      u += a.partial[z * MN + (size_t)row * a.N + lg + 16];
    }
    reinterpret_cast<bf16_t*>(a.C)[a.c_kt ? packed_elem(row, col, a.c_kt) : (size_t)row * a.ldc + col] =
        f2bf(g / (1.f + __expf(-g)) * u);
    return;
  }
  float s = 0.f;
  for (int z = 0; z < S; ++z) s += a.partial[z * MN + (size_t)row * a.N + col];
  const size_t o = (size_t)row * a.ldc + col;
  if (EPI == EPI_BF16) reinterpret_cast<bf16_t*>(a.C)[o] = f2bf(s);
  else if (EPI == EPI_RESID) reinterpret_cast<float*>(a.C)[o] += s;
  else reinterpret_cast<float*>(a.C)[o] = s;
}

// The same product with 64-bit addresses and no LDS, for operands whose smallest tile (16 rows, 32
// columns) spans 2 GiB: a wavefront owns 16 rows x 16 output columns (SwiGLU: and their gate and up
// tiles) and reads both operands from memory.  split: grid.z cuts K as in the wide kernel.
template <int EPI>
__global__ __launch_bounds__(256) void gemm_far_kernel(GemmArgs a, int split) {
  constexpr bool SW = EPI == EPI_SWIGLU;
  const int lane = threadIdx.x & 63, n_out = SW ? a.N / 2 : a.N;
  const int c0 = ((int)blockIdx.x * 4 + (int)(threadIdx.x >> 6)) * 16, row = (int)blockIdx.y * 16 + (lane & 15);
  if (c0 >= n_out) return;
  const int64_t kb = split ? (int64_t)blockIdx.z * (a.k_chunk / 32) : 0;
  const int64_t ke = split && kb + a.k_chunk / 32 < a.kt ? kb + a.k_chunk / 32 : a.kt;
  const int r = min(row, a.M - 1);   // rows past M are never stored
  const bf16_t* ap = a.a_packed ? a.A + (size_t)(r / 16) * a.kt * 512 + lane * 8 : a.A + (size_t)r * a.lda + (lane >> 4) * 8;
  const bf16_t* bp = a.B + (size_t)(c0 / 16) * a.kt * 512 + lane * 8;
  const bf16_t* up = SW ? a.B2 + (size_t)(c0 / 16) * a.kt * 512 + lane * 8 : nullptr;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f}, acc2 = acc;
  for (int64_t k = kb; k < ke; ++k) {
    uint4 x = make_uint4(0, 0, 0, 0);
    if (a.a_packed || k * 32 + (lane >> 4) * 8 < a.K) x = load16(ap + k * (a.a_packed ? 512 : 32));
    acc = mfma16x16x32(as_bf16x8(load16(bp + k * 512)), as_bf16x8(x), acc);
    if constexpr (SW) acc2 = mfma16x16x32(as_bf16x8(load16(up + k * 512)), as_bf16x8(x), acc2);
  }
  if (row >= a.M) return;
  // lane holds row l % 16 and columns 4 (l / 16) .. + 3
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int col = c0 + (lane >> 4) * 4 + e;
    if (col >= n_out) continue;
    const size_t o = (size_t)row * a.ldc + col;
    if (split) {   // SwiGLU partials: logical columns in groups of 16 gate and 16 up
      float* P = a.partial + ((size_t)blockIdx.z * a.M + row) * a.N;
      P[SW ? (col >> 4) * 32 + (col & 15) : col] = acc[e];
      if constexpr (SW) P[(col >> 4) * 32 + 16 + (col & 15)] = acc2[e];
    } else if constexpr (SW) {
      reinterpret_cast<bf16_t*>(a.C)[a.c_kt ? packed_elem(row, col, a.c_kt) : o] = f2bf(acc[e] / (1.f + __expf(-acc[e])) * acc2[e]);
    } else if constexpr (EPI == EPI_BF16) {
      reinterpret_cast<bf16_t*>(a.C)[o] = f2bf(acc[e]);
    } else {
      float* c = reinterpret_cast<float*>(a.C) + o;
      *c = EPI == EPI_RESID ? *c + acc[e] : acc[e];
    }
  }
}

template <int EPI>
hipError_t launch_epi(GemmArgs a, const GemmPlan& p, hipStream_t st, bool reduce, hipEvent_t e0, hipEvent_t e1) {
  a.k_chunk = p.k_chunk;
  if (p.tm == 0) {   // no tile fits 32-bit offsets
    const bool more = p.splits > 1 && reduce;
    const dim3 grid(((EPI == EPI_SWIGLU ? a.N / 2 : a.N) + 63) / 64, (a.M + 15) / 16, p.splits);
    hipError_t e = launch_ev(gemm_far_kernel<EPI>, grid, dim3(256), st, e0, more ? nullptr : e1, a, p.splits > 1 ? 1 : 0);
    if (e != hipSuccess || !more) return e;
    const size_t tot = (size_t)a.M * (EPI == EPI_SWIGLU ? a.N / 2 : a.N);
    return launch_ev(splitk_reduce_kernel<EPI>, dim3((tot + 255) / 256), dim3(256), st, nullptr, e1, a, p.splits);
  }
  if (p.splits > 1) {
    if (EPI != EPI_SWIGLU) a.B2 = nullptr;   // B2 marks SwiGLU there
    if (hipError_t e = gemm_wide_split(a, p, st, e0, reduce ? nullptr : e1)) return e;
    if (!reduce) return hipSuccess;
    const size_t tot = (size_t)a.M * (EPI == EPI_SWIGLU ? a.N / 2 : a.N);
    return launch_ev(splitk_reduce_kernel<EPI>, dim3((tot + 255) / 256), dim3(256), st, nullptr, e1, a, p.splits);
  }
  if constexpr (EPI == EPI_BF16) return gemm_wide_bf16(a, p, st, e0, e1);
  if constexpr (EPI == EPI_RESID) return gemm_wide_resid(a, p, st, e0, e1);
  if constexpr (EPI == EPI_SWIGLU) return gemm_wide_swiglu(a, p, st, e0, e1);
  return gemm_wide_f32(a, p, st, e0, e1);
}

// One 16-byte chunk of the packed layout per thread: chunk q is tile q / 64 and,
// inside it, [k/8 = (q % 64) / 16][row = q % 16].
__global__ __launch_bounds__(256) void pack_weight_kernel(const bf16_t* __restrict__ W, int N, int K, int kt,
                                                         bf16_t* __restrict__ out, size_t n_chunks) {
  const size_t q = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= n_chunks) return;
  const size_t tile = q >> 6;
  const int c = (int)(q & 63);
  const int n = (int)(tile / kt) * 16 + (c & 15);
  const int k = (int)(tile % kt) * 32 + (c >> 4) * 8;
  uint4 v = make_uint4(0, 0, 0, 0);
  if (n < N && k < K) v = load16(W + (size_t)n * K + k);
  *reinterpret_cast<uint4*>(out + q * 8) = v;
}

// Estimated time (us) of the wide kernel above 128 rows with tiles of 16 tm x 16 nw wv and K cut
// into pieces of k_chunk: a step of 32 of K takes the longest of the matrix pipe's issue time,
// its power-limited time (which grows with the CUs at work) and the time a CU needs to fetch its
// weights (by rows of tiles: the more of them, the more often a line is already in L2);
// workgroups run in rounds of one per CU; the weights come at tb_s at best; fp32 partials cost
// part_us per MB, written and read back.
//
// Fitted to launches with weights that are not in the caches: 64 (or 128) columns per
// wavefront to 5,900 (13 projection shapes of d 4096-8192, 129-2300 rows), 32 columns to 10,600
// (24 shapes, 129-2300 rows).  It only ranks: over the 28,700 launches of the second sweep its
// error is 18 and 12% rms, 11 and 14% among the launches within a tenth of the best of their
// shape, and the choice is 2.7% slower than the best tile on average, 22% at worst.
struct TileCost {
  double issue0, issue1, power0, power1, fetch[4], start, tb_s_once, tb_s, part_us;
};
constexpr TileCost kCols64{0.136, 0.0304, 0.0665, 0.0475, {0, 0.385, 0.337, 0.312}, 1.1, 5.4, 4.1, 0.42};
constexpr TileCost kCols64Split{0.058, 0.0378, 0.0349, 0.0406, {0, 0.4206, 0.408, 0.3654}, 0.847, 8.73, 4.39, 0.585};
constexpr TileCost kCols32{0.0816, 0.0222, 0.0245, 0.0204, {0.0714, 0.207, 0.164, 0.102}, 1.02, 5.0, 4.61, 0.592};

double wide_time(const TileCost& c, int M, int N, int K, int tm, int nw, int wv, int k_chunk) {
  const int tiles_m = (M + 16 * tm - 1) / (16 * tm), tiles_n = (N + 16 * nw * wv - 1) / (16 * nw * wv);
  const int splits = (K + k_chunk - 1) / k_chunk;
  const int wgs = tiles_m * tiles_n * splits;
  const double eff = (wv == 8 ? 1.75 : 1.0) * (tm == 16 ? 1.044 : 1.0);
  const double steps = k_chunk / 32.0;
  const double fetch = c.fetch[std::min(tiles_m, 4) - 1];
  auto round = [&](int n) {
    return steps * std::max({(c.issue0 + c.issue1 * tm) * eff, (c.power0 + c.power1 * tm) * eff * n / 256.0, fetch}) +
           c.start;
  };
  double t = wgs / 256 * round(256) + (wgs % 256 ? round(wgs % 256) : 0.0);
  t = std::max(t, (double)N * K * 2e-6 / (tiles_m == 1 ? c.tb_s_once : c.tb_s));
  return t + (splits > 1 ? c.part_us * 1e-6 * splits * ((M + 15) / 16 * 16) * (double)N * 4 : 0.0);
}

}  // namespace

size_t packed_weight_elems(int N, int K) { return (size_t)((N + 15) / 16) * 16 * (size_t)((K + 31) / 32) * 32; }

hipError_t pack_weight_launch(const uint16_t* W, int N, int K, uint16_t* out, hipStream_t st) {
  const size_t n_chunks = packed_weight_elems(N, K) / 8;
  hipLaunchKernelGGL(pack_weight_kernel, dim3((unsigned)((n_chunks + 255) / 256)), dim3(256), 0, st,
                     reinterpret_cast<const bf16_t*>(W), N, K, (K + 31) / 32, reinterpret_cast<bf16_t*>(out), n_chunks);
  return hipGetLastError();
}

// Tile and split-K choice.  It depends on M through its 16-row tiles, and on M itself where the
// partials fill or may outgrow the allocation-free array: the last row count of a tile (a multiple of
// 16) or the one before has the tile's largest partials.
//  - Up to 128 rows one row of tiles covers M and the weights' bytes are the bound, so the chip must
//    be full: 128 columns per workgroup and K cut into the most pieces that stay within one workgroup
//    per CU and >= 512 of K each, and shorten the pipeline; outputs of more than 256 such tiles take
//    256 columns unsplit (64 rows: 55296 x 5120 SwiGLU 91.6 us against 96.9, 128256 x 4096 180
//    against 199; below, 28672 x 4096 41.8 against 55.6), except where 128 leave the fullest CU less
//    to do: an eighth up to 32 rows (152064 x 5120: 225 against 242 at one row, 266 against 271 at
//    32, 282 against 275 at 48), a quarter up to 64, where a narrow step also costs more (64 rows:
//    66048 x 8192 218 against 240, 70000 x 8192 223 / 245, 80000 x 4096 123 / 133; at 96 rows of
//    80000 x 5120 173 / 171).  Where the shares are equal 256 are as good or better (one row of
//    100000 x 4096 125 against 138).  Both operands through LDS: 94.6, 198 and 43.3 us for the first
//    three.
//  - Above, tile and split minimise the estimate, over 64 and 32 columns per wavefront: 256-column
//    workgroups leave outputs of a few thousand columns on a part of the chip with long K (down
//    projections, row-major or packed alike), where half the width doubles the workgroups. 4096 x
//    14336: 513 rows 141 us in 64 x 256 tiles, 92 in 96 x 128; 1024 rows 158 and 121; 240 rows 52
//    (four pieces of K) and 44 (four pieces); 5120 x 27648 at 513 rows 276 and 171.  SwiGLU outputs
//    are wide and stay with 64 columns.  Up to 512 rows K may be split (the partials of more rows
//    cost more than the split gains); not for wide outputs, which fill the chip, nor for SwiGLU.
//    Partials outgrow the array of the allocation-free entry point only where they buy much (a
//    million outputs or more, pieces of 2048 of K), so that the shapes it serves do not hang on small
//    gains.
// SwiGLU of a width that is no multiple of 32 has no 64-column form (2 gate and 2 up tiles): 32
// columns per wavefront at any row count.
GemmPlan gemm_plan(int M, int N, int K, int max_splits, bool swiglu, bool own_partials) {
  GemmPlan p;
  const int row_tiles = (M + 15) / 16;
  const bool pairs_only = swiglu && N % 64 != 0;
  if (row_tiles <= 8) {
    const int tiles = (N + 127) / 128;
    p.once = true;
    // the fullest CU's share of the columns, in 128s, with either width
    const int busy2 = (tiles + 255) / 256, busy4 = 2 * (((N + 255) / 256 + 255) / 256);
    const bool even_out = row_tiles <= 2 ? 7 * busy4 >= 8 * busy2 : row_tiles <= 4 && 3 * busy4 >= 4 * busy2;
    p.nw = tiles <= 256 || pairs_only || even_out ? 2 : 4;
    p.tm = row_tiles <= 1 ? 1 : row_tiles <= 2 ? 2 : row_tiles <= 4 ? 4 : p.nw == 4 && row_tiles <= 6 ? 6 : 8;
    int s = 1;
    if (p.nw == 2)
      while (s + 1 <= max_splits && tiles * (s + 1) <= 256 && K / (s + 1) >= 512) ++s;
    // Of up to that many pieces, those that cost least: the pipeline runs 1 + 8 n steps of 32 of K,
    // and one or two steps left over singly, which wait for all their loads and cost about a trip of
    // eight; every piece adds its partials (us per step by row tiles and per MB, fitted to 2,690
    // launches of 100 shapes at 1-128 rows: 0.35% slower than the best split on average, 7% at
    // worst).  One row of 6144 x 4096 in five pieces 13.6 us, in four 13.2; 64 rows 18.7 and 18.0;
    // 5120 x 5120 in six and five 14.2 and 13.8; 128 rows of 4096 x 4096 in eight and four 23.8 and
    // 21.0.
    auto cost = [&](int pieces) {
      const int n = std::min(((K + pieces - 1) / pieces + 63) / 64 * 2, (K + 31) / 32), trips = (n + 4) / 8;
      return (0.03 + 0.01 * p.tm) * (1 + 8 * trips + 8 * std::max(n - 1 - 8 * trips, 0)) +
             (pieces > 1 ? 0.33e-6 * pieces * row_tiles * 16 * (double)N * 4 : 0.0);
    };
    for (int n = s - 1; n >= 1; --n)
      if (cost(n) <= cost(s)) s = n;
    p.k_chunk = ((K + s - 1) / s + 63) / 64 * 64;
    p.splits = (K + p.k_chunk - 1) / p.k_chunk;
    return p;
  }
  const int most = M <= 512 && N < 16384 && !swiglu ? max_splits : 1;
  double best = 0;
  auto consider = [&](const TileCost& cost, int tm, int nw, int wv, int s) {
    const int kc = ((K + s - 1) / s + 63) / 64 * 64;
    const double t = wide_time(cost, M, N, K, tm, nw, wv, kc);
    if (best != 0 && t >= best) return;
    best = t;
    p.tm = tm;
    p.nw = nw;
    p.wv = wv;
    p.once = nw == 4 && row_tiles <= tm;
    p.k_chunk = kc;
    p.splits = (K + kc - 1) / kc;
  };
  auto consider_splits = [&](int tm, int nw) {
    for (int s = 1; s <= most && (s == 1 || K / s >= 512); ++s)
      if (s == 1 || (nw == 4 && K / s >= 2048 && (int64_t)M * N >= 1 << 20) ||
          ((int64_t)s * row_tiles * 16 * N * 4 <= kNoallocPartials &&
           (nw == 4 || own_partials || (int64_t)s * M * N * 4 < kNoallocPartials)))   // (256 x 4096 x 14336 stays refused there)
        consider(nw == 2 ? kCols32 : kCols64, tm, nw, 4, s);
  };
  // heights worth an estimate: the lowest for its rows of tiles (a higher one only costs more), and for
  // one row of 64-column tiles the next even one
  auto lowest = [&](int tm, int first) { return tm == first || (row_tiles + tm - 1) / tm < (row_tiles + tm - 2) / (tm - 1); };
  auto height = [&](int tm) { return row_tiles > tm ? lowest(tm, 4) : tm % 2 == 0 && row_tiles + 2 > tm; };
  if (!pairs_only) {
    for (int tm = 4; tm <= 16; ++tm)
      if (height(tm)) consider_splits(tm, 4);
    // (measured at 129-512 rows too: it wins only where two rows of 144 fit just so, 288 rows of
    // 55296 x 5120 155 us against 174, and is even or slower elsewhere)
    if (M > 512) consider(kCols64, 9, 4, 8, 1);
  }
  if (!swiglu || pairs_only)
    for (int tm = 3; tm <= 12; ++tm)
      if (row_tiles + 1 > tm && lowest(tm, 3)) consider_splits(tm, 2);   // one row of tiles: the height itself
  if (p.splits > 1 && (int64_t)p.splits * M * N * 4 > kNoallocPartials) {
    // The allocation-free entry point refuses this plan whatever its tile: chosen again among those it
    // refuses, by constants fitted up to 512 rows (5120 x 27648 at 251 rows in six pieces 93 us, in the
    // five of the first choice 100; 4096 x 14336 at 256 in seven 50, in five 52).
    best = 0;
    for (int tm = 4; tm <= 16; ++tm)
      for (int s = 2; height(tm) && s <= most && K / s >= 2048; ++s) {
        const int kc = ((K + s - 1) / s + 63) / 64 * 64;
        if ((int64_t)((K + kc - 1) / kc) * row_tiles * 16 * N * 4 > kNoallocPartials) consider(kCols64Split, tm, 4, 4, s);
      }
  }
  return p;
}

hipError_t gemm_launch(const GemmArgs& a, int epi, const GemmPlan& plan, hipStream_t st, bool reduce, hipEvent_t e0,
                       hipEvent_t e1) {
  // A tile addresses its rows and its columns by 32-bit offsets.  Where a row pitch or a K in the
  // millions makes either span 2 GiB, the tallest tile that does not runs, and the 64-bit kernel
  // where no tile does.
  GemmPlan p = plan;
  auto fits = [&](int tm, int nw) {
    const int64_t rows = std::min(16 * tm, a.M);
    return (a.a_packed ? (rows + 15) / 16 * a.kt * 1024 : ((rows - 1) * a.lda + a.K) * 2) < (int64_t)1 << 31 &&
           (int64_t)nw * a.kt * 1024 < (int64_t)1 << 31;
  };
  if (!fits(p.tm, p.nw)) {
    const bool narrow = epi == EPI_SWIGLU && (p.splits > 1 || a.N % 64 != 0);   // no 64-column form
    const GemmPlan was = p;
    p.tm = 0;
    for (int nw : {4, 2}) {
      if (nw == 4 && (narrow || was.nw == 2)) continue;
      for (int tm = std::min(was.tm, nw == 4 ? 16 : 12); p.tm == 0 && tm >= 1; --tm) {
        const bool few = nw == 2 && (tm <= 2 || narrow);   // heights of the few-row form, 1, 2, 4 and 8
        if ((tm < (nw == 4 ? 4 : 3) && !few) || (few && (tm > 8 || (tm & (tm - 1)))) || !fits(tm, nw)) continue;
        p.tm = tm;
        p.nw = nw;
        p.wv = 4;
        p.once = few;
      }
    }
  }
  // packed activations in, or a packed SwiGLU output: K % 32 == 0 and F % 32 == 0
  if ((a.a_packed && (a.K % 32 || (epi == EPI_SWIGLU && a.N % 64 != 0))) ||
      (a.c_kt && (epi != EPI_SWIGLU || a.N % 64 != 0 || a.c_kt * 64 != a.N)))
    return hipErrorInvalidValue;
  switch (epi) {
    case EPI_BF16: return launch_epi<EPI_BF16>(a, p, st, reduce, e0, e1);
    case EPI_RESID: return launch_epi<EPI_RESID>(a, p, st, reduce, e0, e1);
    case EPI_SWIGLU: return launch_epi<EPI_SWIGLU>(a, p, st, reduce, e0, e1);
    default: return launch_epi<EPI_F32>(a, p, st, reduce, e0, e1);
  }
}

}  // namespace hxf
