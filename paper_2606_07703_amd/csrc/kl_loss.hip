// KL distillation objective of the indexer and its gradient (Section 6.2):
//
//   kl_i = KL(P_i || softmax(z_i)) = sum_{s<=t_i} P_i(s) (log P_i(s) - z_i(s)) + LSE_i sum P_i
//   LSE_i = log sum_{s<=t_i} exp z_i(s),       loss = (1/n) sum_i kl_i
//   d loss / d z_i(s) = (exp(z_i(s) - LSE_i) sum P_i - P_i(s)) / n   (s <= t_i), 0 after t_i
//
// HBM-bound, one workgroup per supervised row. Rows of up to 16384 keys are
// held in registers by as few threads as take 32 elements each (256 up to 8192
// keys, 512), so that several rows share a CU and one's loads run under
// another's arithmetic and stores. A thread takes the maximum of its z, then
// one exponential per element relative to it, which the gradient reuses: the
// threads' sums are rescaled when they are merged. Against one 1024-thread
// workgroup a row, scalar loads and an online maximum with a branch per
// element, P and z in the caches from the call before: 1024 rows of 8192 keys
// 35.4 -> 18.1 us, of 12000 41.9 -> 30.3, 512 of 16384 26.2 -> 19.1. Longer rows
// stay with that kernel: 1024 threads of the new one fill a CU just the same and
// took 77 us against 73 for 1024 rows of 32768, as it reads nothing twice either
// up to that length.
//
// The P log P - P z sum and sum P accumulate in fp64, since the KL of a good
// student is a small difference of large terms. The mean over rows is a
// second, single-workgroup pass in a fixed order, so the loss is
// deterministic.
#include <math.h>

#include "common.hpp"
#include "kernels.hpp"

namespace sp {
namespace {

constexpr int kKlMean = 1024;     // threads of the mean and of a long row
constexpr int kKlResident = 32;   // elements per thread of a long row kept in registers
constexpr int kKlQuads = 8;       // groups of four elements a thread holds
constexpr int kKlBufferDword3 = 0x00020000;   // raw buffer resource: 32-bit data format

struct KlStats {
  float m;     // running max of z
  float se;    // sum exp(z - m)
  double a;    // sum P (log P - z)
  double sp;   // sum P
};

// One element at a time (long rows).
__device__ __forceinline__ void kl_add(KlStats &st, float zv, float pv) {
  if (zv > st.m) {
    st.se = st.se * __expf(st.m - zv) + 1.f;   // m = -inf gives 0 * ... = 0
    st.m = zv;
  } else {
    st.se += __expf(zv - st.m);
  }
  if (pv > 0.f) st.a += (double)(pv * (__logf(pv) - zv));
  st.sp += (double)pv;
}

__device__ __forceinline__ KlStats kl_merge(KlStats x, KlStats y) {
  const float m = fmaxf(x.m, y.m);
  KlStats r;
  r.m = m;
  r.se = (x.m == -INFINITY ? 0.f : x.se * __expf(x.m - m)) +
         (y.m == -INFINITY ? 0.f : y.se * __expf(y.m - m));
  r.a = x.a + y.a;
  r.sp = x.sp + y.sp;
  return r;
}

__device__ __forceinline__ KlStats kl_shfl(const KlStats &x, int off) {
  KlStats y;
  y.m = __shfl_xor(x.m, off, 64);
  y.se = __shfl_xor(x.se, off, 64);
  y.a = __shfl_xor(x.a, off, 64);
  y.sp = __shfl_xor(x.sp, off, 64);
  return y;
}

// Merged over the workgroup; every thread gets the total.
template <int NT>
__device__ __forceinline__ KlStats kl_total(KlStats st) {
  constexpr int NW = NT / 64;
  __shared__ KlStats red[NW];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) st = kl_merge(st, kl_shfl(st, off));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = st;
  __syncthreads();
  KlStats acc = red[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) acc = kl_merge(acc, red[w]);
  return acc;
}

// VEC: every row starts 16-byte aligned, and a thread's elements are groups
// of four neighbours, loaded through a buffer resource that ends at the row's
// last valid key (what lies past it reads as zeros without touching memory);
// otherwise they lie NT apart and are loaded one by one.
template <int NT, bool VEC>
__global__ __launch_bounds__(NT) void kl_rows_kernel(int S, int n,
                                                     const int32_t *__restrict__ rows,
                                                     const float *__restrict__ P,
                                                     const float *__restrict__ z,
                                                     float *__restrict__ kl,
                                                     float *__restrict__ grad) {
  constexpr int Q = kKlQuads;   // S <= NT * 4 * Q
  const int tid = threadIdx.x;
  const int i = blockIdx.x;
  const int t = rows[i];
  const size_t base = (size_t)i * S;
  float *gi = grad ? grad + base : nullptr;
  if (t < 0 || t >= S) {
    if (kl && tid == 0) kl[i] = 0.f;
    if (gi)
      for (int s = tid; s < S; s += NT) gi[s] = 0.f;
    return;
  }
  const int L = t + 1;
  const float *Pi = P + base;
  const float *zi = z + base;
  auto at = [&](int q, int c) { return VEC ? 4 * (tid + q * NT) + c : tid + (4 * q + c) * NT; };

  float zr[Q][4], pr[Q][4];
  if constexpr (VEC) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const auto rz = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(zi), (short)0,
                                                      (uint32_t)L * 4u, kKlBufferDword3);
    const auto rp = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(Pi), (short)0,
                                                      (uint32_t)L * 4u, kKlBufferDword3);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(rz, (uint32_t)at(q, 0) * 4u, 0, 0);
      const u32x4 b = __builtin_amdgcn_raw_buffer_load_b128(rp, (uint32_t)at(q, 0) * 4u, 0, 0);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        zr[q][c] = __uint_as_float(a[c]);
        pr[q][c] = __uint_as_float(b[c]);
      }
    }
  } else {
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int s = at(q, c);
        zr[q][c] = s < L ? zi[s] : 0.f;
        pr[q][c] = s < L ? Pi[s] : 0.f;
      }
  }
  KlStats st{-INFINITY, 0.f, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < Q; ++q)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (at(q, c) >= L) zr[q][c] = -INFINITY;
      st.m = fmaxf(st.m, zr[q][c]);
    }
  const float mref = st.m == -INFINITY ? 0.f : st.m;
#pragma unroll
  for (int q = 0; q < Q; ++q)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float zv = zr[q][c], pv = pr[q][c];
      if (pv > 0.f) st.a += (double)(pv * (__logf(pv) - zv));   // (0 past the last key)
      st.sp += (double)pv;
      zr[q][c] = __expf(zv - mref);
      st.se += zr[q][c];
    }
  const KlStats tot = kl_total<NT>(st);
  const double lse = (double)tot.m + log((double)tot.se);
  if (kl && tid == 0) kl[i] = (float)(tot.a + lse * tot.sp);
  if (!gi) return;
  // softmax(z)(s) sum P / n = exp(z - mref) * exp(mref - lse) sum P / n
  // (0 for a thread without a finite z, whose mref may lie far above lse, but
  // NaN with the others of its row where the row has no softmax)
  const float f = st.m == -INFINITY && lse > -INFINITY
                      ? 0.f
                      : (float)(exp((double)st.m - lse) * (tot.sp / n));
  const float inv_n = 1.f / n;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    float o[4];
#pragma unroll
    for (int c = 0; c < 4; ++c)   // past the last key 0, whatever the row's sums
      o[c] = at(q, c) < L ? zr[q][c] * f - pr[q][c] * inv_n : 0.f;
    if constexpr (VEC) {
      if (at(q, 0) < S)   // S is a multiple of 4
        *reinterpret_cast<float4 *>(gi + at(q, 0)) = make_float4(o[0], o[1], o[2], o[3]);
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (at(q, c) < S) gi[at(q, c)] = o[c];
    }
  }
}

// Rows of more than 16384 keys: 1024 threads, up to 32768 valid keys in
// registers, longer rows read twice.
__global__ __launch_bounds__(kKlMean) void kl_long_rows_kernel(
    int S, int n, const int32_t *__restrict__ rows, const float *__restrict__ P,
    const float *__restrict__ z, float *__restrict__ kl, float *__restrict__ grad) {
  constexpr int NT = kKlMean, E = kKlResident, NW = NT / 64;
  __shared__ KlStats red[NW];
  __shared__ KlStats total;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i = blockIdx.x;
  const int t = rows[i];
  const size_t base = (size_t)i * S;
  float *gi = grad ? grad + base : nullptr;
  if (t < 0 || t >= S) {
    if (kl && tid == 0) kl[i] = 0.f;
    if (gi)
      for (int s = tid; s < S; s += NT) gi[s] = 0.f;
    return;
  }
  const int L = t + 1;
  const bool resident = L <= NT * E;
  const float *Pi = P + base;
  const float *zi = z + base;

  KlStats st{-INFINITY, 0.f, 0.0, 0.0};
  float zr[E], pr[E];
  if (resident) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int s = tid + e * NT;
      zr[e] = s < L ? zi[s] : -INFINITY;
      pr[e] = s < L ? Pi[s] : 0.f;
    }
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (tid + e * NT < L) kl_add(st, zr[e], pr[e]);
  } else {
    for (int s = tid; s < L; s += NT) kl_add(st, zi[s], Pi[s]);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) st = kl_merge(st, kl_shfl(st, off));
  if (lane == 0) red[wave] = st;
  __syncthreads();
  if (tid == 0) {
    KlStats acc = red[0];
    for (int w = 1; w < NW; ++w) acc = kl_merge(acc, red[w]);
    total = acc;
  }
  __syncthreads();
  const KlStats tot = total;
  const double lse = (double)tot.m + log((double)tot.se);
  if (kl && tid == 0) kl[i] = (float)(tot.a + lse * tot.sp);
  if (!gi) return;
  const float lsef = (float)lse;
  const float spn = (float)(tot.sp / n), inv_n = 1.f / n;
  if (resident) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int s = tid + e * NT;
      if (s < L) gi[s] = __expf(zr[e] - lsef) * spn - pr[e] * inv_n;
    }
  } else {
    for (int s = tid; s < L; s += NT) gi[s] = __expf(zi[s] - lsef) * spn - Pi[s] * inv_n;
  }
  for (int s = L + tid; s < S; s += NT) gi[s] = 0.f;
}

// loss = (1/n) sum_i kl_i, summed in fp64 in a fixed order.
__global__ __launch_bounds__(kKlMean) void kl_mean_kernel(int n, const float *__restrict__ kl,
                                                             float *__restrict__ loss) {
  constexpr int NT = kKlMean, NW = NT / 64;
  __shared__ double red[NW];
  const int tid = threadIdx.x;
  double acc = 0.0;
  for (int i = tid; i < n; i += NT) acc += (double)kl[i];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if ((tid & 63) == 0) red[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) {
    double s = 0.0;
    for (int w = 0; w < NW; ++w) s += red[w];
    loss[0] = (float)(s / n);
  }
}

template <int NT>
void launch_rows(int S, int n, const int32_t *rows, const float *P, const float *z, float *kl,
                 float *grad, hipStream_t st) {
  if (S % 4 == 0)   // the arrays are 16-byte aligned, and then so is every row
    hipLaunchKernelGGL((kl_rows_kernel<NT, true>), dim3(n), dim3(NT), 0, st, S, n, rows, P, z, kl,
                       grad);
  else
    hipLaunchKernelGGL((kl_rows_kernel<NT, false>), dim3(n), dim3(NT), 0, st, S, n, rows, P, z, kl,
                       grad);
}

}  // namespace

hipError_t launch_kl_loss(int S, int n, const int32_t *rows, const float *P, const float *z,
                          float *kl, float *loss, float *grad, hipStream_t st) {
  if (n == 0) return hipSuccess;
  if (S <= 256 * 4 * kKlQuads)
    launch_rows<256>(S, n, rows, P, z, kl, grad, st);
  else if (S <= 512 * 4 * kKlQuads)
    launch_rows<512>(S, n, rows, P, z, kl, grad, st);
  else
    hipLaunchKernelGGL(kl_long_rows_kernel, dim3(n), dim3(kKlMean), 0, st, S, n, rows, P, z, kl,
                       grad);
  if (loss) hipLaunchKernelGGL(kl_mean_kernel, dim3(1), dim3(kKlMean), 0, st, n, kl, loss);
  return hipGetLastError();
}

}  // namespace sp
