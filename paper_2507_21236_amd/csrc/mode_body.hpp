// Mode-product bodies shared by the kernel sources (the staged launches and
// the persistent batched matvec run the same code, so both give the same
// results bit for bit).
#pragma once
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "mfma_common.hpp"

namespace attn {

// ============================================================================ mode product
// Element (i, f) of a (d0, d1, d2) tensor contracted on leg j, where f runs over
// the two other legs in order.
__device__ __forceinline__ int64_t mode_addr(int j, int d0, int d1, int d2, int i, int64_t f) {
  if (j == 0) return (int64_t)i * d1 * d2 + f;
  if (j == 1) {
    const int64_t a = f / d2, c = f - a * d2;
    return a * d1 * d2 + (int64_t)i * d2 + c;
  }
  return f * d2 + i;
}

// out (+)= sum_jobs coef * A x_j in.  wu = (task, 64-wide block of the free
// index f).  A workgroup takes FW = 16 FT (NW / QS) free columns (part `sub` of
// the block when FW < 64) and every row i: its NW wavefronts form
// QS groups of rows by NW / QS groups of FT column tiles.  The input tile
// [i'][f] of a job is staged in LDS, the next job's is already on its way into
// registers while this one is multiplied, and the elements of A run PA steps
// ahead of their products through bounds-checked loads, so a leg that is not a
// multiple of 16, or a last block that is not full, needs no other code (rows
// past the end are zero, results past the end are not stored).  Every output
// entry sums its products in the same order whatever the split.  With a single
// job the output may be the input: a workgroup reads its columns before it
// writes them.
// What bounds it is the latency of the operand loads: a chain has few jobs and
// one launch per stage, so small tiles (many workgroups) are taken up to legs
// of 64 and column pairs above, where each A element then serves two products.
// Three stages of the heaviest 8 x 8 m = 128 node
// (96 products, 51.5 GFLOP): 2.51 ms before the loads ran ahead, 1.09 now.
template <typename T, int NI, int QS = 1, int FT = 1, int NW = 4>
__device__ __forceinline__ void mode_mfma(const MPTask& t, const MPJob* __restrict__ jobs,
                                          const int2 wu, int sub, const T* __restrict__ xbase,
                                          unsigned char* smem_raw) {
  typedef typename V4<T>::type v4;
  constexpr int mjp = 16 * NI, NQ = NI / QS, FW = 16 * FT * (NW / QS), ld = FW + 2;
  constexpr int NT = 64 * NW, NPT = mjp * FW / NT;   // staged elements per thread
  constexpr int PA = NQ > 2 ? 2 : 4;
  T* lds = reinterpret_cast<T*>(smem_raw);
  const int j = t.j, d0 = t.d0, d1 = t.d1, d2 = t.d2;
  const int mj = j == 0 ? d0 : (j == 1 ? d1 : d2);
  const int M = d0 * d1 * d2, F = M / mj, KS = (mj + 3) >> 2;
  const int f0 = wu.y * 64 + (FW < 64 ? FW * sub : 0);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int l16 = lane & 15, l4 = lane >> 4;
  const int tile = (wave / QS) * FT, q0 = (wave % QS) * NQ;
  // byte offset of each staged element in the input, past its end where there is none
  int off[NPT];
#pragma unroll
  for (int u = 0; u < NPT; u++) {
    const int e = threadIdx.x + NT * u;
    const int i = j == 2 ? e % mjp : e / FW, fl = j == 2 ? e / mjp : e % FW;
    off[u] = (i < mj && f0 + fl < F) ? (int)mode_addr(j, d0, d1, d2, i, f0 + fl) * (int)sizeof(T) : M * (int)sizeof(T);
  }
  T pf[NPT];
  auto fetch = [&](int jb) {
    const __amdgpu_buffer_rsrc_t r = block_rsrc(jobs[jb].in ? (const T*)jobs[jb].in : xbase, M);
#pragma unroll
    for (int u = 0; u < NPT; u++) pf[u] = bload<T>(r, off[u]);
  };
  v4 acc[NQ][FT];
#pragma unroll
  for (int q = 0; q < NQ; q++)
#pragma unroll
    for (int c = 0; c < FT; c++) acc[q][c] = v4{0, 0, 0, 0};
  const int ao = (l4 * mj + 16 * q0 + l16) * (int)sizeof(T), astep = 4 * mj * (int)sizeof(T);
  const int j1 = t.job0 + t.njob;
  if (t.job0 < j1) fetch(t.job0);
  for (int jb = t.job0; jb < j1; jb++) {
    const __amdgpu_buffer_rsrc_t ra = block_rsrc((const T*)jobs[jb].A, mj * mj);
    const T coef = (T)jobs[jb].coef;
    T ab[PA][NQ];
    int an = ao;   // the next K step to load, past the end too
#pragma unroll
    for (int u = 0; u < PA; u++, an += astep)
#pragma unroll
      for (int q = 0; q < NQ; q++) ab[u][q] = bload<T>(ra, an + 16 * q * (int)sizeof(T));
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NPT; u++) {
      const int e = threadIdx.x + NT * u;
      const int i = j == 2 ? e % mjp : e / FW, fl = j == 2 ? e / mjp : e % FW;
      if (i < 4 * KS) lds[i * ld + fl] = pf[u];
    }
    __syncthreads();
    if (jb + 1 < j1) fetch(jb + 1);
    const T* xr = lds + l4 * ld + 16 * tile + l16;
    for (int ks = 0; ks < KS; ks += PA) {
#pragma unroll
      for (int u = 0; u < PA; u++) {
        if (ks + u >= KS) break;
        T av[NQ];
#pragma unroll
        for (int q = 0; q < NQ; q++) {
          av[q] = ab[u][q];
          ab[u][q] = bload<T>(ra, an + 16 * q * (int)sizeof(T));
        }
        an += astep;
#pragma unroll
        for (int c = 0; c < FT; c++) {
          const T bop = xr[u * 4 * ld + 16 * c] * coef;
#pragma unroll
          for (int q = 0; q < NQ; q++) acc[q][c] = mfma16(av[q], bop, acc[q][c]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      xr += 4 * PA * ld;
    }
  }
  T* out = (T*)t.out;
#pragma unroll
  for (int c = 0; c < FT; c++) {
    const int f = f0 + 16 * (tile + c) + l16;
    if (f >= F) continue;
#pragma unroll
    for (int q = 0; q < NQ; q++)
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const int r = 16 * (q0 + q) + drow<T>(l4, i);
        if (r >= mj) continue;
        const int64_t ad = mode_addr(j, d0, d1, d2, r, f);
        if (t.accumulate) out[ad] += acc[q][c][i];
        else out[ad] = acc[q][c][i];
      }
  }
}

// Generic mode product: one thread per output element.  wu = (task, first element).
template <typename T>
__device__ __forceinline__ void mode_gen_elem(const MPTask& t, const MPJob* __restrict__ jobs,
                                              int64_t e, const T* __restrict__ xbase) {
  const int j = t.j, d0 = t.d0, d1 = t.d1, d2 = t.d2;
  const int mj = j == 0 ? d0 : (j == 1 ? d1 : d2);
  const int64_t total = (int64_t)d0 * d1 * d2;
  if (e >= total) return;
  const int64_t F = total / mj;
  const int i = (int)(e / F);
  const int64_t f = e - (int64_t)i * F;
  T acc = 0;
  for (int jb = t.job0; jb < t.job0 + t.njob; jb++) {
    const T* in = jobs[jb].in ? (const T*)jobs[jb].in : xbase;
    const T* A = (const T*)jobs[jb].A;
    T sum = 0;
    for (int k = 0; k < mj; k++) sum += A[(int64_t)k * mj + i] * in[mode_addr(j, d0, d1, d2, k, f)];
    acc += (T)jobs[jb].coef * sum;
  }
  T* out = (T*)t.out;
  const int64_t ad = mode_addr(j, d0, d1, d2, i, f);
  if (t.accumulate) out[ad] += acc;
  else out[ad] = acc;
}

}  // namespace attn
