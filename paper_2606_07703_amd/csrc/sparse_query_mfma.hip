// Sparse GQA attention for per-query (or small-block) supports on bf16 MFMA
// (Section 3 restricted attention; Section 4.2 per-query causal mask;
// Algorithm 2, selection and sparse GQA prefill with b_sel = 1).
//
// Each query owns its support. The gather kernel gives one wave a (query t, KV
// head j) pair and the G query heads of that group (query_attend). Work items
// are laid out so that workgroup i (which runs on XCD i % 8) holds KV head
// i % Hkv: with 8 KV heads each XCD's L2 serves the gathers of one head.
//
// Where the supports cover enough of the keys before them, multiplying every
// key and masking costs less than gathering (launch_sparse_mask_mfma).
#include "attn_rules.hpp"
#include "sparse_query.hpp"

namespace sp {
namespace {

template <int D, int NW>
__global__ __launch_bounds__(NW * 64) void sparse_query_kernel(
    int S, int Hq, int Hkv, int G, int b, int kk, size_t gstride, int n_groups, float scale_log2,
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k,
    const uint16_t *__restrict__ v, const int32_t *__restrict__ idx,
    uint16_t *__restrict__ o, KvPages pages, int qo) {
  // q and o are addressed by position: the host shifts them back by qo rows
  __shared__ __align__(16) QuerySlots<D, NW> sh;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int j = blockIdx.x % Hkv;
  const int grp = n_groups - 1 - blockIdx.x / Hkv;   // longest queries first
  const int t = qo + grp * NW + wave;
  if (t >= S) return;   // no workgroup barrier below: waves are independent
  const int32_t *row = idx + (size_t)j * gstride + (size_t)((t - qo) / b) * kk;
  query_attend<D>(t, j, Hq, Hkv, G, kk, scale_log2, q, k, v, row, o, pages, sh.pos[wave],
                  sh.rows[wave], lane);
}

template <int D>
hipError_t launch_d(const Prob &p, const void *q, const void *k, const void *v,
                    const int32_t *idx, void *o, hipStream_t st, KvPages pages) {
  // waves are independent; at d = 256 two per workgroup keep three
  // workgroups' LDS slots on a CU
  constexpr int NW = D == 256 ? 2 : 4;
  const int n_groups = (p.nq + NW - 1) / NW;
  const size_t shift = (size_t)p.qo * p.Hq * D;   // chunk rows addressed by position
  hipLaunchKernelGGL((sparse_query_kernel<D, NW>), dim3(n_groups * p.Hkv), dim3(NW * 64), 0, st,
                     p.S, p.Hq, p.Hkv, p.G, p.b, p.k, p.idx_group_stride(), n_groups,
                     p.scale * kLog2e,
                     (const uint16_t *)q - shift, (const uint16_t *)k, (const uint16_t *)v, idx,
                     (uint16_t *)o - shift, pages, p.qo);
  return hipGetLastError();
}

}  // namespace

bool sparse_query_mfma_supported(const Prob &p) {
  return p.dtype == SP_DTYPE_BF16 && (p.d == 64 || p.d == 128 || p.d == 256) && p.G <= 16;
}

hipError_t launch_sparse_query_mfma(const Prob &p, const void *q, const void *k, const void *v,
                                    const int32_t *idx, void *o, hipStream_t st, KvPages pages) {
  if (sparse_mask_pays(p)) return launch_sparse_mask_mfma(p, q, k, v, idx, o, st, pages);
  if (p.d == 64) return launch_d<64>(p, q, k, v, idx, o, st, pages);
  if (p.d == 256) return launch_d<256>(p, q, k, v, idx, o, st, pages);
  return launch_d<128>(p, q, k, v, idx, o, st, pages);
}

}  // namespace sp
