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

#include "wl_fma64.h"
#include "wl_internal.h"
#include "wl_poly.h"

namespace wl {
namespace {

constexpr int kGenThreads = 1024;  // most threads of a generating workgroup

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

// log2(x) for x = w + 1/2, w a 32-bit word: x = m 2^e with m in [3/4, 3/2),
// m = (1 + r) / c with c from the table of the nearest multiple of 1/128, r =
// m c - 1 rounded once, and log2(1 + r) = r Q(r), Q of degree 5.  Around m =
// 1 c is 1 and r exact, so the result keeps its relative accuracy there.
__device__ __forceinline__ double log2_word(uint32_t w, const double2* tab) {
  const double x = (double)w + 0.5;
  // m in [3/4, 3/2): the exponent of x (4/3) decides between [1, 3/2) and [3/4, 1)
  int e = (__double2hiint(x) >> 20) - 1023;
  int hi = (__double2hiint(x) & 0x000fffff) | 0x3ff00000;
  if (hi >= 0x3ff80000) {
    hi -= 0x00100000;
    e += 1;
  }
  const double m = __hiloint2double(hi, __double2loint(x));
  const double2 c = tab[(int)rint(fma(128.0, m, -96.0))];
  const double r = fma(m, c.x, -1.0);
  return (double)e +
         fma(r, horner_s_f64<WL_LOG2P1_WIDE_F64_DEG>(WL_LOG2P1_WIDE_F64, r), c.y);
}

// sqrt(x), x > 0 normal, to about an ulp: the hardware estimate of 1/sqrt and
// one third-order step.
__device__ __forceinline__ double root(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double g = x * y;
  const double e = fma(-g, y, 1.0);
  return fma(g, e * fma(0.375, e, 0.5), g);
}

// cos(2 pi u) and sin(2 pi u), u in [0, 1): u = f + j/4, |f| <= 1/8 exact.
__device__ __forceinline__ void sincos2pi(double u, double& s, double& c) {
  const double j = rint(4.0 * u);
  const double f = fma(-0.25, j, u);
  const double v = f * f;
  const double pc = horner_s_f64<WL_COS2PI_F64_DEG>(WL_COS2PI_F64, v);
  const double ps = f * horner_s_f64<WL_SIN2PI_F64_DEG>(WL_SIN2PI_F64, v);
  const int q = (int)j & 3;
  const double a = (q & 1) ? ps : pc, b = (q & 1) ? pc : ps;
  c = (q == 1 || q == 2) ? -a : a;
  s = (q == 2 || q == 3) ? -b : b;
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
// Measured at 16384 x 4096: 1.91 ms as one level of Box-Muller per barrier
// with the library's log, cos and sin, and kernels of their own for the
// segments and the norms; 0.74 ms in this form, 1.6 GB written.  What bounds it
// now is the Philox and FP64 arithmetic of step 1.
// The FMA contraction of the recursion is off, as in the CPU generator.
__global__ __launch_bounds__(kGenThreads) __attribute__((amdgpu_waves_per_eu(8))) void k_generate(
    uint64_t seed, int64_t first_loop, int64_t n_loops, int32_t n_ppl,
    float* __restrict__ out_x, float* __restrict__ out_y, float4* __restrict__ seg,
    float2* __restrict__ norm) {
  extern __shared__ double v[];
  double* vx = v;
  double* vy = v + place(n_ppl);
  __shared__ double part[2][kGenThreads / 64];
  __shared__ double2 tab[97];
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  const int32_t t = threadIdx.x, nt = blockDim.x;
  for (int32_t i = t; i < 97; i += nt)
    tab[i] = make_double2(WL_LOG2_GEN_TAB[2 * i], WL_LOG2_GEN_TAB[2 * i + 1]);
  __syncthreads();
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
        // r = sqrt(-2 ln u1), u1 = (w + 1/2) 2^-32
        const double r = root(1.3862943611198906 * (32.0 - log2_word(pr ? w[2] : w[0], tab)));
        double s, c;
        sincos2pi(((double)(pr ? w[3] : w[1]) + 0.5) * (1.0 / 4294967296.0), s, c);
        // 1/sqrt(nk): 2^-k/2, its odd powers from 1/sqrt(2) as rounded
        const double sigma = __hiloint2double(
            ((k & 1) ? 0x3fe6a09e : 0x3ff00000) - ((k >> 1) << 20), (k & 1) ? 0x667f3bcc : 0);
        vx[i] = sigma * (r * c);
        vy[i] = sigma * (r * s);
      }
    }
    __syncthreads();
    {
#pragma clang fp contract(off)
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
        // levels of at most 64 points are one wave's work
        if (half >= 64 || 2 * half >= n_ppl) {
          __syncthreads();
        } else if (2 * half > 64) {
          __syncthreads();
        } else {
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
      }
    }
    double sum[2] = {0.0, 0.0};
    for (int32_t i = t; i < n_ppl; i += nt) {
      sum[0] += vx[place(i)];
      sum[1] += vy[place(i)];
    }
    block_sums(sum, part);
    const double mean_x = sum[0] / n_ppl, mean_y = sum[1] / n_ppl;
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
    block_sums(nrm, part);  // its barriers also end the reads of v
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
  // four points per thread, one wave at least
  int32_t threads = (n_ppl / 4 + 63) / 64 * 64;
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
