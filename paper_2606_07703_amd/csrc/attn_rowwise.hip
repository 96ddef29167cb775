// Row-wise causal GQA attention, dense or restricted to a shared support.
//
// Dense:  o[t,h] = sum_{s<=t} softmax(scale <q[t,h],k[s,g(h)]>) v[s,g(h)]   (Section 3)
// Sparse: the same softmax over U = { s in idx[t/b] : 0 <= s <= t }        (Section 3, 4.2)
//
// One workgroup per (query t, chunk of HPW query heads of one KV group), of one
// or four waves that share the list. A wave is split into four 16-lane groups;
// each group walks every fourth key of the wave's steps and keeps its own
// online-softmax state, with each lane holding d/16 contiguous elements of the
// head dimension. A key row k[s,g,:] is read by one group as a single coalesced
// segment (256 B for bf16 at d=128), and the HPW heads of the chunk reuse it
// from registers. A step loads 1 to 8 keys a group before it uses the first
// (row_keys): with one key a step the walk is a chain of load latencies, which
// many waves hide where the states are small. The partial states are merged
// with cross-group shuffles, then through LDS.
//
// This path serves every shape and dtype; the matrix-core kernels take the bf16
// shapes they are built for.
#include <math.h>

#include "common.hpp"
#include "kernels.hpp"

namespace sp {
namespace {

constexpr float kLazy = 8.f;

// Keys a group takes per step, all loaded before the first is used: what was the
// fastest over lists of 8 to 512 keys (supports; many: k >= 256) and 300 to 2500
// keys (dense). One head of 128 or 256, and supports at d = 256, stay at one: their
// registers are better spent on waves.
template <int D, int HPW, bool SPARSE>
constexpr int row_keys(bool many) {
  if (SPARSE && D == 64) return HPW == 1 ? 2 : many ? 4 : 1;
  if (SPARSE) return D == 128 && HPW == 4 ? 2 : 1;
  if (D == 64) return 4;
  if (D == 128) return HPW == 1 ? 8 : HPW == 2 ? 2 : 4;
  return HPW == 1 ? 1 : 2;
}

// NWK waves share a (query, head chunk): they take the steps, of KEYS keys a
// group, in turn. KEYS = 0: one key a step, its support entry read in the step itself.
template <typename T, int D, int HPW, bool SPARSE, int NWK, int KEYS>
__global__ __launch_bounds__(NWK * 64) void attn_rowwise_kernel(
    int S, int Hq, int Hkv, int G, float scale_log2, const T *__restrict__ q,
    const T *__restrict__ k, const T *__restrict__ v, const int32_t *__restrict__ idx, int kk,
    int b, size_t gstride, T *__restrict__ o, float *__restrict__ lse, KvPages pages, int qo) {
  // q, o and lse are addressed by position: the host shifts them back by qo rows
  constexpr int EPL = D / 16, U = KEYS > 0 ? KEYS : 1;
  const int t = qo + blockIdx.x;
  const int h0 = blockIdx.y * HPW;
  const int j = h0 / G;
  const int lane = threadIdx.x & 63;
  // in a scalar register: the loop's counter and branches are then scalar
  const int wave = NWK > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
  const int grp = lane >> 4;
  const int sub = lane & 15;

  float qr[HPW][EPL];
#pragma unroll
  for (int hh = 0; hh < HPW; ++hh) {
    load_row<EPL>(q + ((size_t)t * Hq + h0 + hh) * D + sub * EPL, qr[hh]);
#pragma unroll
    for (int e = 0; e < EPL; ++e) qr[hh][e] *= scale_log2;
  }
  float m[HPW], l[HPW], acc[HPW][EPL];
#pragma unroll
  for (int hh = 0; hh < HPW; ++hh) {
    m[hh] = -INFINITY;
    l[hh] = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[hh][e] = 0.f;
  }

  const int n = SPARSE ? kk : t + 1;
  const int32_t *ir = SPARSE ? idx + (size_t)j * gstride + (size_t)((t - qo) / b) * kk : nullptr;
  // (a list may hold up to 2^31 - 1 entries, and a step ends past them)
  auto entry = [&](uint32_t base, int u) {
    const uint32_t i = base + 4 * u + grp;
    return SPARSE ? (i < (uint32_t)n ? ir[i] : -1) : (int)i;
  };
  // The running max moves only when a logit exceeds it by 2^kLazy, so the
  // accumulator is rescaled rarely (probabilities stay <= 2^kLazy).
  auto raise = [&](int hh, float top) {
    if (top > m[hh] + kLazy) {
      const float corr = __builtin_amdgcn_exp2f(m[hh] - top);  // m = -inf gives 0
      l[hh] *= corr;
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[hh][e] *= corr;
      m[hh] = top;
    }
  };
  auto add = [&](int hh, float x, const float (&vf)[EPL]) {
    const float pr = __builtin_amdgcn_exp2f(x - m[hh]);
    l[hh] += pr;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[hh][e] = fmaf(pr, vf[e], acc[hh][e]);
  };
  if constexpr (KEYS == 0) {
    static_assert(NWK == 1, "one wave");
    for (uint32_t base = 0; base < (uint32_t)n; base += 4) {
      int s = entry(base, 0);
      bool valid = SPARSE ? s >= 0 && s <= t && s < S : s < n;
      if (SPARSE && valid) {
        s = pages.row(s);   // the K/V row (identity unless the cache is paged)
        valid = s >= 0;
      }
      if (!valid) s = 0;
      const size_t row = ((size_t)s * Hkv + j) * D + sub * EPL;
      float kf[EPL], vf[EPL];
      load_row<EPL>(k + row, kf);
      load_row<EPL>(v + row, vf);
#pragma unroll
      for (int hh = 0; hh < HPW; ++hh) {
        float part = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) part = fmaf(qr[hh][e], kf[e], part);
        const float x = row16_sum(part);
        if (valid) {
          raise(hh, x);
          add(hh, x, vf);
        }
      }
    }
  } else {
    // the support entries of a step are loaded during the step before
    int next[U];
#pragma unroll
    for (int u = 0; u < U; ++u) next[u] = entry(wave * 4 * U, u);
    for (uint32_t base = wave * 4 * U; base < (uint32_t)n; base += NWK * 4 * U) {
      int s[U];
      bool valid[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {   // entry base + 4 u + grp
        s[u] = next[u];
        valid[u] = s[u] < n;
        next[u] = entry(base + NWK * 4 * U, u);
      }
      if (SPARSE) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          valid[u] = s[u] >= 0 && s[u] <= t && s[u] < S;
          if (valid[u]) {
            s[u] = pages.row(s[u]);   // the K/V row (identity unless the cache is paged)
            valid[u] = s[u] >= 0;
          }
        }
      }
      float kf[U][EPL], vf[U][EPL];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const size_t row = ((size_t)(valid[u] ? s[u] : 0) * Hkv + j) * D + sub * EPL;
        load_row<EPL>(k + row, kf[u]);
        load_row<EPL>(v + row, vf[u]);
      }
#pragma unroll
      for (int hh = 0; hh < HPW; ++hh) {
        float x[U], top = -INFINITY;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          float part = 0.f;
#pragma unroll
          for (int e = 0; e < EPL; ++e) part = fmaf(qr[hh][e], kf[u][e], part);
          x[u] = row16_sum(part);
          if (valid[u]) top = fmaxf(top, x[u]);
        }
        raise(hh, top);
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (valid[u]) add(hh, x[u], vf[u]);   // else another's row: skipped, not weighted by 0
      }
    }
  }

  // Merge the four groups' states (lanes sub, sub+16, sub+32, sub+48).
  auto merge = [&](int hh, float mo, float lo, auto other) {
    const float mn = fmaxf(m[hh], mo);
    const float c1 = (m[hh] == -INFINITY) ? 0.f : exp2f(m[hh] - mn);
    const float c2 = (mo == -INFINITY) ? 0.f : exp2f(mo - mn);
    l[hh] = l[hh] * c1 + lo * c2;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[hh][e] = acc[hh][e] * c1 + other(e) * c2;
    m[hh] = mn;
  };
#pragma unroll
  for (int hh = 0; hh < HPW; ++hh) {
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) {
      const float mo = __shfl_xor(m[hh], off, 64);
      const float lo = __shfl_xor(l[hh], off, 64);
      float ao[EPL];
#pragma unroll
      for (int e = 0; e < EPL; ++e) ao[e] = __shfl_xor(acc[hh][e], off, 64);
      merge(hh, mo, lo, [&](int e) { return ao[e]; });
    }
  }
  // Then the waves', in order, into the first.
  if constexpr (NWK > 1) {
    __shared__ float parts[NWK - 1][HPW][EPL + 2][16];
    if (wave > 0 && grp == 0) {
#pragma unroll
      for (int hh = 0; hh < HPW; ++hh) {
        parts[wave - 1][hh][EPL][sub] = m[hh];
        parts[wave - 1][hh][EPL + 1][sub] = l[hh];
#pragma unroll
        for (int e = 0; e < EPL; ++e) parts[wave - 1][hh][e][sub] = acc[hh][e];
      }
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int w = 0; w < NWK - 1; ++w)
#pragma unroll
      for (int hh = 0; hh < HPW; ++hh)
        merge(hh, parts[w][hh][EPL][sub], parts[w][hh][EPL + 1][sub],
              [&](int e) { return parts[w][hh][e][sub]; });
  }
  if (grp == 0) {
#pragma unroll
    for (int hh = 0; hh < HPW; ++hh) {
      const float inv = l[hh] > 0.f ? 1.f / l[hh] : 0.f;
      float out[EPL];
#pragma unroll
      for (int e = 0; e < EPL; ++e) out[e] = acc[hh][e] * inv;
      if (o) store_row<EPL>(o + ((size_t)t * Hq + h0 + hh) * D + sub * EPL, out);
      if (lse && sub == 0)
        lse[(size_t)t * Hq + h0 + hh] = l[hh] > 0.f ? (m[hh] + log2f(l[hh])) * kLn2 : -INFINITY;
    }
  }
}

template <typename T, int D, int HPW, bool SPARSE, int NWK, int U>
hipError_t launch_w(const Prob &p, const void *q, const void *k, const void *v,
                    const int32_t *idx, void *o, float *lse, hipStream_t st, KvPages pages) {
  // chunk rows are addressed by position
  const size_t shift = (size_t)p.qo * p.Hq;
  hipLaunchKernelGGL((attn_rowwise_kernel<T, D, HPW, SPARSE, NWK, U>), dim3(p.nq, p.Hq / HPW),
                     dim3(NWK * 64), 0, st, p.S, p.Hq, p.Hkv, p.G, p.scale * kLog2e,
                     (const T *)q - shift * D, (const T *)k, (const T *)v, idx, SPARSE ? p.k : 0,
                     SPARSE ? p.b : 1, SPARSE ? p.idx_group_stride() : 0,
                     o ? (T *)o - shift * D : nullptr, lse ? lse - shift : nullptr, pages, p.qo);
  return hipGetLastError();
}

// Four waves a query where one each would leave the chip short of waves and
// each gets a step of its own: fp32, one key a step and one wave before, 512
// tokens at 4/2 heads, d = 64, dense 42.3 -> 15.4 us; 1024 at 8/2, d = 128, k =
// 512 97 -> 72. Four waves at 8192 queries times heads, d = 128, k = 256: 100 us,
// one 84. At d = 256 a wave has the registers of two: never for one head, and
// for supports only long ones (1024 tokens at 4/2 heads, k = 64: 28 us with four
// waves, 22 with one; k = 256 52 / 65).
template <typename T, int D, int HPW, bool SPARSE, int U>
hipError_t launch_u(const Prob &p, const void *q, const void *k, const void *v,
                    const int32_t *idx, void *o, float *lse, hipStream_t st, KvPages pages) {
  const int64_t waves = (int64_t)p.nq * (p.Hq / HPW);
  const int keys = SPARSE ? p.k : p.S;
  constexpr int least = D < 256 || !SPARSE ? 16 * U : HPW == 2 ? 256 : 64;
  if constexpr (D < 256 || HPW > 1)
    if (waves <= 2048 && keys >= least)
      return launch_w<T, D, HPW, SPARSE, 4, U>(p, q, k, v, idx, o, lse, st, pages);
  return launch_w<T, D, HPW, SPARSE, 1, U>(p, q, k, v, idx, o, lse, st, pages);
}

template <typename T, int D, int HPW>
hipError_t launch_t(const Prob &p, const void *q, const void *k, const void *v,
                    const int32_t *idx, void *o, float *lse, hipStream_t st, KvPages pages) {
  // One head of 128 or 256, one key a step: reading the entry ahead gains 2 to 26%
  // (2500 tokens at 8/8 heads, d = 128, k = 100 124 -> 101 us), but loses with
  // long supports where the waves all run at once (1024 at 6/2 heads, k = 512 91 ->
  // 103), at d = 256 (300 at 6/2, k = 256 53 -> 59) and over long dense rows there.
  const int64_t waves = (int64_t)p.nq * p.Hq;
  if constexpr (HPW == 1 && D >= 128) {
    if (idx && (D == 256 ? p.k >= 256 : p.k >= 64 && waves > 4096 && waves < 8192))
      return launch_w<T, D, HPW, true, 1, 0>(p, q, k, v, idx, o, lse, st, pages);
    if (D == 256 && !idx && p.S > 2048)
      return launch_w<T, D, HPW, false, 1, 0>(p, q, k, v, idx, o, lse, st, pages);
  }
  if (!idx)
    return launch_u<T, D, HPW, false, row_keys<D, HPW, false>(true)>(p, q, k, v, idx, o, lse, st,
                                                                     pages);
  if (p.k >= 256)
    return launch_u<T, D, HPW, true, row_keys<D, HPW, true>(true)>(p, q, k, v, idx, o, lse, st,
                                                                   pages);
  return launch_u<T, D, HPW, true, row_keys<D, HPW, true>(false)>(p, q, k, v, idx, o, lse, st,
                                                                  pages);
}

template <typename T, int D>
hipError_t launch_d(const Prob &p, const void *q, const void *k, const void *v,
                    const int32_t *idx, void *o, float *lse, hipStream_t st, KvPages pages) {
  if (p.G % 4 == 0) return launch_t<T, D, 4>(p, q, k, v, idx, o, lse, st, pages);
  if (p.G % 2 == 0) return launch_t<T, D, 2>(p, q, k, v, idx, o, lse, st, pages);
  return launch_t<T, D, 1>(p, q, k, v, idx, o, lse, st, pages);
}

}  // namespace

hipError_t launch_attn_rowwise(const Prob &p, const void *q, const void *k, const void *v,
                               const int32_t *idx, void *o, float *lse, hipStream_t st,
                               KvPages pages) {
  if (p.dtype == SP_DTYPE_BF16) {
    if (p.d == 64) return launch_d<bf16, 64>(p, q, k, v, idx, o, lse, st, pages);
    if (p.d == 128) return launch_d<bf16, 128>(p, q, k, v, idx, o, lse, st, pages);
    return launch_d<bf16, 256>(p, q, k, v, idx, o, lse, st, pages);
  }
  if (p.d == 64) return launch_d<float, 64>(p, q, k, v, idx, o, lse, st, pages);
  if (p.d == 128) return launch_d<float, 128>(p, q, k, v, idx, o, lse, st, pages);
  return launch_d<float, 256>(p, q, k, v, idx, o, lse, st, pages);
}

}  // namespace sp
