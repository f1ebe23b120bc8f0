// Greedy sampling (row argmax, lowest index on ties) and a streaming copy used
// as the HBM bandwidth probe.
#include "common.hpp"
#include "kernels.hpp"

namespace hxf {

namespace {

__device__ __forceinline__ void better(float& bv, int& bi, float v, int i) {
  // v beats (bv, bi) if larger, or equal with a lower index; NaN never wins
  if (v > bv || (v == bv && i < bi)) {
    bv = v;
    bi = i;
  }
}

__global__ __launch_bounds__(1024) void argmax_kernel(const float* logits, int32_t* out, int V) {
  __shared__ float sv[16];
  __shared__ int si[16];
  const float* row = logits + (size_t)blockIdx.x * V;
  float bv = -__builtin_huge_valf();
  int bi = 0x7FFFFFFF;
  // One workgroup per row: bound by the comparisons and the latency of its loads, from 200 rows on by
  // memory.  Four float4 in flight per thread; a float4 first gives its maximum (NaN never wins a
  // maximum), and only a larger one than all before replaces the thread's best, so equal values
  // keep the lowest index (a thread's indices ascend).  The best float4 stays in registers and
  // its element is found at the end (reading it again cost a dependent load, and at many rows its
  // traffic: 256 x 128256 26.1 -> 24.5 us, 128 rows 14.2 -> 12.8, 64 rows 10.6 -> 9.8; against comparing
  // every element with its index 24.4, 17.0 and 16.1, one row 13.9 -> 7.3).
  const int n4 = V >> 2;
  const float4* r4 = reinterpret_cast<const float4*>(row);
  int b4 = -1;
  float4 best = make_float4(0.f, 0.f, 0.f, 0.f);
  auto take = [&](const float4& v, int j) __attribute__((always_inline)) {
    const float t = fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w));
    const bool up = t > bv;
    b4 = up ? j : b4;
    best.x = up ? v.x : best.x;
    best.y = up ? v.y : best.y;
    best.z = up ? v.z : best.z;
    bv = fmaxf(bv, t);
  };
  int i = threadIdx.x;
  for (; i + 3 * 1024 < n4; i += 4 * 1024) {
    float4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = r4[i + u * 1024];
#pragma unroll
    for (int u = 0; u < 4; ++u) take(v[u], i + u * 1024);
  }
  for (; i < n4; i += 1024) take(r4[i], i);
  if (b4 >= 0) {
    bi = 4 * b4 + (best.x == bv ? 0 : best.y == bv ? 1 : best.z == bv ? 2 : 3);
  } else {
    // nothing above the type's lowest value: the first element that is not NaN
    for (int j = 4 * threadIdx.x; j < 4 * n4 && bi == 0x7FFFFFFF; j += 4 * 1024)
      for (int e = 3; e >= 0; --e)
        if (row[j + e] == bv) bi = j + e;
  }
  for (int i = 4 * n4 + threadIdx.x; i < V; i += 1024) better(bv, bi, row[i], i);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(bv, o, kWave);
    const int oi = __shfl_xor(bi, o, kWave);
    better(bv, bi, ov, oi);
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    sv[w] = bv;
    si[w] = bi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < 16; ++k) better(bv, bi, sv[k], si[k]);
    out[blockIdx.x] = (bi == 0x7FFFFFFF) ? 0 : bi;
  }
}

__global__ __launch_bounds__(256) void copy_kernel(const uint4* src, uint4* dst, size_t n) {
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * 256;
  for (; i < n; i += stride) dst[i] = src[i];
}

// Streaming read: thread t XORs the 16-byte words it reads (grid-stride, four loads in
// flight per step) into sink[t], so that no load is dead.
__global__ __launch_bounds__(256) void read_kernel(const uint4* src, size_t n, uint32_t* sink) {
  uint32_t acc = 0;
  const size_t stride = (size_t)gridDim.x * 1024;
  for (size_t i = (size_t)blockIdx.x * 1024 + threadIdx.x; i < n; i += stride) {
    uint4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = i + u * 256 < n ? src[i + u * 256] : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int u = 0; u < 4; ++u) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
  }
  sink[(size_t)blockIdx.x * 256 + threadIdx.x] = acc;
}

}  // namespace

hipError_t argmax_launch(const float* logits, int32_t* out, int R, int V, hipStream_t st) {
  if (R <= 0) return hipSuccess;
  hipLaunchKernelGGL(argmax_kernel, dim3(R), dim3(1024), 0, st, logits, out, V);
  return hipGetLastError();
}

hipError_t copy_launch(const void* src, void* dst, size_t bytes, hipStream_t st) {
  const size_t n = bytes / 16;
  if (n == 0) return hipSuccess;
  size_t blocks = (n + 255) / 256;
  if (blocks > 256 * 64) blocks = 256 * 64;
  hipLaunchKernelGGL(copy_kernel, dim3((unsigned)blocks), dim3(256), 0, st, reinterpret_cast<const uint4*>(src),
                     reinterpret_cast<uint4*>(dst), n);
  return hipGetLastError();
}

hipError_t read_launch(const void* src, size_t bytes, uint32_t* sink, hipStream_t st) {
  const size_t n = bytes / 16;
  size_t blocks = (n + 1023) / 1024;
  if (blocks > kReadProbeBlocks) blocks = kReadProbeBlocks;
  if (blocks == 0) blocks = 1;   // no words: every sink word is written as 0
  hipLaunchKernelGGL(read_kernel, dim3((unsigned)blocks), dim3(256), 0, st, reinterpret_cast<const uint4*>(src), n,
                     sink);
  return hipGetLastError();
}

}  // namespace hxf
