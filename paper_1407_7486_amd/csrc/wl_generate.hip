// On-device unit-loop generation: d-loops (Sec. 2.1, Loop Generation,
// Eqs. yn2 and ynk) from a counter-based generator, so that an ensemble is
// created where it is used instead of being copied over PCIe.
//
// Random numbers: Philox4x32-10 as published (Salmon, Moraes, Dror, Shaw,
// "Parallel random numbers: as easy as 1, 2, 3", SC'11), key = the 64-bit
// seed, counter = (block, loop_lo, loop_hi, 0).  Block b gives four words
// w; word w maps to the uniform (w + 0.5) 2^-32, and the pairs (w0, w1),
// (w2, w3) give two standard normals each by Box-Muller:
// r = sqrt(-2 ln u1), (r cos 2 pi u2, r sin 2 pi u2).  Loop l uses normals
// 0 .. 2(N-1)-1 of its own stream, in the order the recursion consumes
// them: level by level (N_k = 2, 4, ..., N), new points in ascending order,
// x then y.  New point p (counting from 0 over all levels) therefore takes
// the normal pair p: block p/2, word pair p%2, x from the cosine, y from the
// sine.  This is the convention of the repository's seeded input
// generator, so the same (seed, loop) gives the same loop up to last-bit
// differences of the FP64 log / cos / sin implementations.
//
// Recursion, per loop of N = 2^m points: y[0] = 0; at level N_k with stride
// h = N/N_k, point i = q h (q odd) is the midpoint of y[i-h] and
// y[(i+h) mod N] plus a normal of standard deviation 1/sqrt(N_k) (the
// heat-bath weight of Eq. ynk); finally the loop's mean is subtracted
// (common centre of mass at 0).  FP64 throughout, stored as FP32.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "wl_internal.h"

namespace wl {
namespace {

constexpr int kGenThreads = 1024;  // most threads of a generating workgroup
constexpr int kSumThreads = 256;   // strides of the centre of mass sums

__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2,
                                              uint32_t c3, uint32_t k0, uint32_t k1,
                                              uint32_t out[4]) {
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k0 += 0x9E3779B9u;  // Weyl key increments
      k1 += 0xBB67AE85u;
    }
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0;
    const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
    c1 = (uint32_t)p1;
    c3 = (uint32_t)p0;
    c0 = n0;
    c2 = n2;
  }
  out[0] = c0;
  out[1] = c1;
  out[2] = c2;
  out[3] = c3;
}

// Sums of x over the workgroup's threads (a fixed tree), to every thread.
template <int N>
__device__ __forceinline__ void block_sums(double (&x)[N], double (*part)[kGenThreads / 64]) {
#pragma unroll
  for (int k = 0; k < N; ++k)
    for (int off = 32; off > 0; off >>= 1) x[k] += __shfl_xor(x[k], off);
  __syncthreads();  // part may still be read
  if (threadIdx.x % 64 == 0)
#pragma unroll
    for (int k = 0; k < N; ++k) part[k][threadIdx.x / 64] = x[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < N; ++k) {
    x[k] = 0.0;
    for (uint32_t w = 0; w < blockDim.x / 64; ++w) x[k] += part[k][w];
  }
}

// Place of point i in LDS: one double of padding per 32, so that the levels'
// strides (powers of two) spread over the banks.
__host__ __device__ constexpr int32_t place(int32_t i) { return i + (i >> 5); }

// One workgroup per loop (grid-stride over loops), both coordinates in one
// pass: the loop's N FP64 x and y values sit in LDS (16.5N bytes).
//   1  every new point's displacement sigma_k z at its place: no point needs
//      another one's, so all threads work on the Philox blocks, logarithms
//      and cosines side by side (a block serves two points).
//   2  the recursion level by level, one addition of the neighbours' midpoint
//      per point, a barrier between levels (within one wave while a level has
//      at most 64 new points).
//   3  the centre of mass; the FP32 points, their segment quantities and the
//      loop's norms, straight from LDS.
// Measured at 16384 x 4096: 1.91 ms with the normals of a level computed
// between its barriers, and kernels of their own for the segments and the
// norms; 1.00 ms in this form, 1.6 GB written.  What bounds it now is the
// arithmetic of step 1.  (Its log, cos and sin stay the library's, and the
// sums' order that of 256 threads: an FP32 coordinate on the edge of a
// rounding would fall the other way with any other last bit, and a plain FP32
// evaluation of an ill-conditioned mean shows that.)
// The FMA contraction is off, as in the CPU generator.
__global__ __launch_bounds__(kGenThreads) __attribute__((amdgpu_waves_per_eu(8))) void k_generate(
    uint64_t seed, int64_t first_loop, int64_t n_loops, int32_t n_ppl,
    float* __restrict__ out_x, float* __restrict__ out_y, float4* __restrict__ seg,
    float2* __restrict__ norm) {
#pragma clang fp contract(off)
  extern __shared__ double v[];
  double* vx = v;
  double* vy = v + place(n_ppl);
  __shared__ double part[2][kGenThreads / 64];
  __shared__ double sum[2][kSumThreads];
  const double two_pi = 6.283185307179586476925286766559;
  const double inv32 = 1.0 / 4294967296.0;
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  const int32_t t = threadIdx.x, nt = blockDim.x;
  for (int64_t l = blockIdx.x; l < n_loops; l += gridDim.x) {
    const uint64_t gl = (uint64_t)(first_loop + l);
    if (t == 0) {
      vx[0] = 0.0;
      vy[0] = 0.0;
    }
    // points 0 .. n_ppl - 2 over all levels: ordinal p belongs to level nk =
    // 2^(floor(log2(p + 1)) + 1), where it is new point p + 1 - nk/2
    for (int32_t bb = t; 2 * bb < n_ppl - 1; bb += nt) {
      uint32_t w[4];
      philox4x32_10((uint32_t)bb, (uint32_t)gl, (uint32_t)(gl >> 32), 0u, k0, k1, w);
#pragma unroll 1
      for (int pr = 0; pr < 2; ++pr) {
        const int32_t p = 2 * bb + pr;
        if (p >= n_ppl - 1) break;
        const int32_t k = 32 - __clz(p + 1);  // nk = 2^k
        const int32_t i = place((2 * (p + 1 - (1 << (k - 1))) + 1) * (n_ppl >> k));
        const double u1 = ((double)(pr ? w[2] : w[0]) + 0.5) * inv32;
        const double u2 = ((double)(pr ? w[3] : w[1]) + 0.5) * inv32;
        const double r = sqrt(-2.0 * log(u1));
        // 1/sqrt(nk): 2^-k/2, its odd powers from 1/sqrt(2) as rounded
        const double sigma = __hiloint2double(
            ((k & 1) ? 0x3fe6a09e : 0x3ff00000) - ((k >> 1) << 20), (k & 1) ? 0x667f3bcc : 0);
        const double zx = r * cos(two_pi * u2);
        const double zy = r * sin(two_pi * u2);
        vx[i] = sigma * zx;
        vy[i] = sigma * zy;
      }
    }
    __syncthreads();
    for (int32_t half = 1; half < n_ppl; half *= 2) {
      const int32_t h = n_ppl / (2 * half);
      for (int32_t q = t; q < half; q += nt) {
        const int32_t i = place((2 * q + 1) * h);
        const int32_t a = place(2 * q * h);
        const int32_t b = q + 1 == half ? 0 : place((2 * q + 2) * h);
        const double mx = 0.5 * (vx[a] + vx[b]);
        const double my = 0.5 * (vy[a] + vy[b]);
        vx[i] = mx + vx[i];
        vy[i] = my + vy[i];
      }
      // while this level and the next have at most 64 points, one wave works
      // on both
      if (half >= 64 || 2 * half >= n_ppl) {
        __syncthreads();
      } else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
    }
    // kSumThreads strided sums over the points, added as a tree
    for (int32_t q = t; q < kSumThreads; q += nt) {
      double sx = 0.0, sy = 0.0;
      for (int32_t i = q; i < n_ppl; i += kSumThreads) {
        sx += vx[place(i)];
        sy += vy[place(i)];
      }
      sum[0][q] = sx;
      sum[1][q] = sy;
    }
    __syncthreads();
    for (int32_t w = kSumThreads / 2; w > 0; w >>= 1) {
      for (int32_t q = t; q < w; q += nt) {
        sum[0][q] += sum[0][q + w];
        sum[1][q] += sum[1][q + w];
      }
      __syncthreads();
    }
    const double mean_x = sum[0][0] / n_ppl, mean_y = sum[1][0] / n_ppl;
    float* ox = out_x + l * n_ppl;
    float* oy = out_y + l * n_ppl;
    float4* os = seg + l * n_ppl;
    double nrm[2] = {0.0, 0.0};
    for (int32_t i = t; i < n_ppl; i += nt) {
      const int32_t i0 = place(i), j = i + 1 == n_ppl ? 0 : place(i + 1);
      const float x0 = (float)(vx[i0] - mean_x), y0 = (float)(vy[i0] - mean_y);
      const float x1 = (float)(vx[j] - mean_x), y1 = (float)(vy[j] - mean_y);
      const float4 q = seg_quantities(x0, y0, x1, y1);
      ox[i] = x0;
      oy[i] = y0;
      os[i] = q;
      nrm[0] += (double)q.w * (double)q.w;
      nrm[1] += (double)q.z * (double)q.z;
    }
    block_sums(nrm, part);  // its barriers also end the reads of v and sum
    if (t == 0) norm[l] = make_float2((float)sqrt(nrm[0]), (float)sqrt(nrm[1]));
  }
}

// Segment array and norms of uploaded loops, one workgroup per loop
// (grid-stride): each point is read from memory once.  Flags non-finite
// input.  65536 x 4096: 1.55 ms, 6.4 GB read and written (the segments and the
// norms in kernels of their own, 2.00).
__global__ __launch_bounds__(256) void k_prep(const float* __restrict__ X,
                                              const float* __restrict__ Y, int64_t n_loops,
                                              int32_t n_ppl, float4* __restrict__ seg,
                                              float2* __restrict__ norm, int* __restrict__ bad) {
  __shared__ double part[2][kGenThreads / 64];
  for (int64_t l = blockIdx.x; l < n_loops; l += gridDim.x) {
    const float* x = X + l * n_ppl;
    const float* y = Y + l * n_ppl;
    double nrm[2] = {0.0, 0.0};
    for (int32_t i = threadIdx.x; i < n_ppl; i += blockDim.x) {
      const int32_t j = i + 1 == n_ppl ? 0 : i + 1;
      const float x0 = x[i], y0 = y[i];
      if (!isfinite(x0) || !isfinite(y0)) *bad = 1;
      const float4 q = seg_quantities(x0, y0, x[j], y[j]);
      seg[l * n_ppl + i] = q;
      nrm[0] += (double)q.w * (double)q.w;
      nrm[1] += (double)q.z * (double)q.z;
    }
    block_sums(nrm, part);
    if (threadIdx.x == 0) norm[l] = make_float2((float)sqrt(nrm[0]), (float)sqrt(nrm[1]));
  }
}

}  // namespace

hipError_t launch_generate(uint64_t seed, int64_t first_loop, int64_t n_loops, int32_t n_ppl,
                           float* d_x, float* d_y, float4* d_seg, float2* d_norm,
                           hipStream_t stream) {
  const int64_t blocks = n_loops < 65536 ? n_loops : 65536;
  const size_t lds = 2 * (size_t)place(n_ppl) * sizeof(double);  // at most 132 KiB (N <= 8192)
  hipError_t e = hipFuncSetAttribute((const void*)k_generate,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  int32_t threads = n_ppl / 4;  // four points per thread, whole waves
  if (threads < 64) threads = 64;
  if (threads > kGenThreads) threads = kGenThreads;
  hipLaunchKernelGGL(k_generate, dim3((uint32_t)blocks), dim3(threads), lds, stream, seed,
                     first_loop, n_loops, n_ppl, d_x, d_y, d_seg, d_norm);
  return hipGetLastError();
}

hipError_t launch_prep(const float* d_x, const float* d_y, int64_t n_loops, int32_t n_ppl,
                       float4* d_seg, float2* d_norm, int* d_bad, hipStream_t stream) {
  const int64_t blocks = n_loops < 65536 ? n_loops : 65536;
  hipLaunchKernelGGL(k_prep, dim3((uint32_t)blocks), dim3(n_ppl <= 64 ? 64 : 256), 0, stream,
                     d_x, d_y, n_loops, n_ppl, d_seg, d_norm, d_bad);
  return hipGetLastError();
}

}  // namespace wl
