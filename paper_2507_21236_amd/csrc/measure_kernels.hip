// Kernels of the observable and disentangler-environment contractions: FP64
// matrix products over a work list (the contractions of an operator image
// through a tree node, the link Gram matrices, the closing products at the
// lowest common node), leg permutations and fixed-order sums of partials.
#include <hip/hip_runtime.h>

#include "measure.hpp"
#include "mfma_common.hpp"

namespace attn {

// One 64 x 64 tile of C per workgroup: K walked in steps of 16 through LDS,
// each thread accumulating a 4 x 4 block in FP64 (the vector FP64 rate of the
// chip equals its FP64 matrix-core rate).
__global__ __launch_bounds__(256) void k_gemm_jobs(const GMJob* __restrict__ jobs, const int4* __restrict__ wus) {
  __shared__ double As[16][64 + 2];
  __shared__ double Bs[16][64 + 2];
  const int4 wu = wus[blockIdx.x];
  const GMJob& J = jobs[wu.x];
  const double* A = J.A + (int64_t)wu.y * J.sa;
  const double* B = J.B + (int64_t)wu.y * J.sb;
  double* C = J.C + (int64_t)wu.y * J.sc;
  const int m0 = wu.z * 64, n0 = wu.w * 64;
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  double acc[4][4];
#pragma unroll
  for (int r = 0; r < 4; r++)
#pragma unroll
    for (int c = 0; c < 4; c++) acc[r][c] = 0.0;
  // the next K step is on its way into registers while this one is multiplied
  double ra[4], rb[4];
  auto load = [&](int k0) {
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int e = tid + 256 * q;
      const int i = J.ta ? e & 63 : e >> 4, k = J.ta ? e >> 6 : e & 15;
      const int gi = m0 + i, gk = k0 + k;
      const bool in = gi < J.M && gk < J.K;
      const double v = A[in ? (J.ta ? (int64_t)gk * J.lda + gi : (int64_t)gi * J.lda + gk) : 0];
      ra[q] = in ? v : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int e = tid + 256 * q;
      const int j = J.tb ? e >> 4 : e & 63, k = J.tb ? e & 15 : e >> 6;
      const int gj = n0 + j, gk = k0 + k;
      const bool in = gj < J.N && gk < J.K;
      const double v = B[in ? (J.tb ? (int64_t)gj * J.ldb + gk : (int64_t)gk * J.ldb + gj) : 0];
      rb[q] = in ? v : 0.0;
    }
  };
  load(0);
  for (int k0 = 0; k0 < J.K; k0 += 16) {
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int e = tid + 256 * q;
      if (J.ta) As[e >> 6][e & 63] = ra[q];
      else As[e & 15][e >> 4] = ra[q];
      if (J.tb) Bs[e & 15][e >> 4] = rb[q];
      else Bs[e >> 6][e & 63] = rb[q];
    }
    __syncthreads();
    if (k0 + 16 < J.K) load(k0 + 16);
#pragma unroll
    for (int kk = 0; kk < 16; kk++) {
      double a[4], b[4];
#pragma unroll
      for (int r = 0; r < 4; r++) a[r] = As[kk][ty * 4 + r];
#pragma unroll
      for (int c = 0; c < 4; c++) b[c] = Bs[kk][tx * 4 + c];
#pragma unroll
      for (int r = 0; r < 4; r++)
#pragma unroll
        for (int c = 0; c < 4; c++) acc[r][c] = fma(a[r], b[c], acc[r][c]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < 4; r++) {
    const int gi = m0 + ty * 4 + r;
    if (gi >= J.M) continue;
#pragma unroll
    for (int c = 0; c < 4; c++) {
      const int gj = n0 + tx * 4 + c;
      if (gj >= J.N) continue;
      double* p = C + (int64_t)gi * J.ldc + gj;
      *p = J.accumulate ? *p + acc[r][c] : acc[r][c];
    }
  }
}

// The same for results that fill 64 x 64 tiles badly (the images and Gram
// matrices of links up to 32): a 32 x 32 tile per workgroup on
// the matrix cores, the four wavefronts sharing out K inside each step and their
// sums added in order at the end.  A 32 x 32 result of a 64 x 64 tile leaves three
// quarters of its products unused.  Reading A and B bounds it: 512 images of an
// 8 x 8 lattice at m = 32 (K = 1024, 268 MB) took 136 to 150 us, here 82
// (3.3 TB/s); its 64 x 64 correlation matrix 32.6 ms before, 28.8 now.
__global__ __launch_bounds__(256) void k_gemm_jobs32(const GMJob* __restrict__ jobs, const int4* __restrict__ wus) {
  constexpr int KC = 64, ld = 34;
  __shared__ double lds[2 * KC * ld];   // A and B of one step, [k][i]; then the wavefronts' sums
  double* As = lds;
  double* Bs = lds + KC * ld;
  const int4 wu = wus[blockIdx.x];
  const GMJob& J = jobs[wu.x];
  const double* A = J.A + (int64_t)wu.y * J.sa;
  const double* B = J.B + (int64_t)wu.y * J.sb;
  double* C = J.C + (int64_t)wu.y * J.sc;
  const int m0 = wu.z * 32, n0 = wu.w * 32;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l16 = lane & 15, l4 = lane >> 4;
  const int kc = J.K > 32 ? 64 : 32, kw = kc / 4;   // K of a step, and of a wavefront in it
  double ra[8], rb[8];
  auto load = [&](int k0) {
#pragma unroll
    for (int q = 0; q < 8; q++) {
      const int e = tid + 256 * q;
      const int i = J.ta ? e & 31 : e / kc, k = J.ta ? e >> 5 : e % kc;
      const int gi = m0 + i, gk = k0 + k;
      const bool in = i < 32 && k < kc && gi < J.M && gk < J.K;
      const double v = A[in ? (J.ta ? (int64_t)gk * J.lda + gi : (int64_t)gi * J.lda + gk) : 0];
      ra[q] = in ? v : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 8; q++) {
      const int e = tid + 256 * q;
      const int j = J.tb ? e / kc : e & 31, k = J.tb ? e % kc : e >> 5;
      const int gj = n0 + j, gk = k0 + k;
      const bool in = j < 32 && k < kc && gj < J.N && gk < J.K;
      const double v = B[in ? (J.tb ? (int64_t)gj * J.ldb + gk : (int64_t)gk * J.ldb + gj) : 0];
      rb[q] = in ? v : 0.0;
    }
  };
  d4 acc[2][2];
#pragma unroll
  for (int r = 0; r < 2; r++)
#pragma unroll
    for (int c = 0; c < 2; c++) acc[r][c] = d4{0, 0, 0, 0};
  load(0);
  for (int k0 = 0; k0 < J.K; k0 += kc) {
#pragma unroll
    for (int q = 0; q < 8; q++) {
      const int e = tid + 256 * q;
      const int ia = J.ta ? e & 31 : e / kc, ka = J.ta ? e >> 5 : e % kc;
      if (ia < 32 && ka < kc) As[ka * ld + ia] = ra[q];
      const int jb = J.tb ? e / kc : e & 31, kb = J.tb ? e % kc : e >> 5;
      if (jb < 32 && kb < kc) Bs[kb * ld + jb] = rb[q];
    }
    __syncthreads();
    if (k0 + kc < J.K) load(k0 + kc);
    for (int ks = 0; ks < kw; ks += 4) {
      const int k = wave * kw + ks + l4;
      double a[2], b[2];
#pragma unroll
      for (int r = 0; r < 2; r++) a[r] = As[k * ld + 16 * r + l16];
#pragma unroll
      for (int c = 0; c < 2; c++) b[c] = Bs[k * ld + 16 * c + l16];
#pragma unroll
      for (int r = 0; r < 2; r++)
#pragma unroll
        for (int c = 0; c < 2; c++) acc[r][c] = mfma16(a[r], b[c], acc[r][c]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < 2; r++)
#pragma unroll
    for (int c = 0; c < 2; c++)
#pragma unroll
      for (int i = 0; i < 4; i++)
        lds[wave * 1024 + (16 * r + drow<double>(l4, i)) * 32 + 16 * c + l16] = acc[r][c][i];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const int e = tid + 256 * q, gi = m0 + (e >> 5), gj = n0 + (e & 31);
    if (gi >= J.M || gj >= J.N) continue;
    const double v = lds[e] + lds[1024 + e] + lds[2048 + e] + lds[3072 + e];
    double* p = C + (int64_t)gi * J.ldc + gj;
    *p = J.accumulate ? *p + v : v;
  }
}

__global__ __launch_bounds__(256) void k_permute_jobs(const PMJob* __restrict__ jobs) {
  const PMJob& J = jobs[blockIdx.y];
  const int64_t M = (int64_t)J.d0 * J.d1 * J.d2;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < M; e += (int64_t)gridDim.x * 256) {
    const int64_t a = e / ((int64_t)J.d1 * J.d2);
    const int64_t rem = e - a * J.d1 * J.d2;
    const int64_t b = rem / J.d2, c = rem - b * J.d2;
    J.out[(b * J.d0 + a) * J.d2 + c] = J.in[e];
  }
}

__global__ __launch_bounds__(256) void k_sum_parts(const SPJob* __restrict__ jobs) {
  const SPJob& J = jobs[blockIdx.y];
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < J.n; e += (int64_t)gridDim.x * 256) {
    double acc = 0.0;
    for (int q = 0; q < J.nq; q++) acc += J.in[(int64_t)q * J.stride + e];
    J.out[e] = acc;
  }
}

// one workgroup per pair: a strided pass over the two vectors, then a
// reduction across the workgroup in a fixed order
__global__ __launch_bounds__(256) void k_pair_dots(const double* __restrict__ base, const int2* __restrict__ pairs,
                                                   int64_t M, double* __restrict__ out) {
  __shared__ double red[256];
  const int2 pr = pairs[blockIdx.x];
  const double* u = base + (int64_t)pr.x * M;
  const double* v = base + (int64_t)pr.y * M;
  double acc = 0.0;
  for (int64_t e = threadIdx.x; e < M; e += 256) acc = fma(u[e], v[e], acc);
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}

static unsigned grid_for(int64_t n) {
  int64_t g = (n + 255) / 256;
  return (unsigned)(g > 1024 ? 1024 : (g < 1 ? 1 : g));
}

hipError_t launch_gemm_jobs(const GMJob* jobs, const int4* wus, int nwu, int tile, hipStream_t s) {
  if (nwu <= 0) return hipSuccess;
  if (tile == 32) hipLaunchKernelGGL(k_gemm_jobs32, dim3(nwu), dim3(256), 0, s, jobs, wus);
  else hipLaunchKernelGGL(k_gemm_jobs, dim3(nwu), dim3(256), 0, s, jobs, wus);
  return hipGetLastError();
}

hipError_t launch_permute_jobs(const PMJob* jobs, int njob, int64_t maxM, hipStream_t s) {
  if (njob <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_permute_jobs, dim3(grid_for(maxM), njob), dim3(256), 0, s, jobs);
  return hipGetLastError();
}

hipError_t launch_sum_parts(const SPJob* jobs, int njob, int64_t maxn, hipStream_t s) {
  if (njob <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_sum_parts, dim3(grid_for(maxn), njob), dim3(256), 0, s, jobs);
  return hipGetLastError();
}

}  // namespace attn

namespace attn {
hipError_t launch_pair_dots(const double* base, const int2* pairs, int npair, int64_t M, double* out, hipStream_t s) {
  if (npair <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_pair_dots, dim3(npair), dim3(256), 0, s, base, pairs, M, out);
  return hipGetLastError();
}
}  // namespace attn
