// Sparse GQA attention for per-query supports by masked dense tiles (Section 3
// restricted attention; Section 4.2 per-query causal mask).
//
// A gathered support costs k rows of K and V per (query, KV head), through the
// vector-memory path of one CU, with the G heads of the group filling G of 16
// matrix columns. Where the supports cover a good part of the keys before
// their queries it is cheaper to multiply every key, as dense attention does,
// and mask: a tile of K and V then serves 256 / G queries at once. The kernel
// is the dense tile pipeline with a bit per (query, key) in place of the causal
// test, held in LDS for a segment of key tiles at a time: at the
// segment's first step the workgroup clears the bits and sets those of its
// queries' support entries (any order, entries out of [0, t] dropped).
//
// The line between the two kernels is drawn for full support rows. Rows may hold
// sentinels instead: a workgroup whose queries have so few usable entries that
// gathering them takes less than its key tiles finds that in its first fill of
// the bits, or after a part of it, and gathers. Tables of k = 2048 with 16
// entries each, 32768 tokens, 32/8 heads, d = 128: 9.4 -> 2.4 ms (2.05 by the
// gather kernel); k = 512 with 16, 4096 tokens, 16/4: 110 -> 71 us (73); at d = 64,
// k = 1024 with 16, only 93 -> 91 (59), as most of that is the fill.
//
// A weight of zero still multiplies its V row, so an infinite or NaN V entry
// that no query selects would turn outputs to NaN. Rows that come out NaN are
// therefore computed again from the selected rows alone (query_attend).
#include "attn_tile.hpp"
#include "kernels.hpp"
#include "sparse_query.hpp"

namespace sp {
namespace {

// The key tiles of the sequence, masked by a bit per (query, key). The bits of
// a segment of `steps` pipeline steps are in LDS: two words per (tile of the
// segment, query), filled from the support rows at the segment's first step;
// PAGED: and two words per tile of the keys whose page lies in the cache.
template <int NT, bool SPLIT, bool PAGED>
struct MaskedKeys {
  static constexpr bool kLookup = PAGED;   // rows are arithmetic, or read from the page table
  static constexpr bool kBits = true;
  static constexpr bool kTable = PAGED;
  static constexpr bool kNaNs = true;   // rows that come out NaN are computed again
  int ntiles, steps;          // steps of a segment: a power of two
  int t0, nq, TQ;             // the workgroup's queries t0 .. t0 + nq - 1
  const int32_t *table;       // support rows of its KV head, one per b positions from qo
  int qo, b, kk;
  uint32_t *words;            // the segment's bits
  uint32_t lane_bits;         // LDS address of this lane's query within a tile's
  KvPages pages;
  int S;
  uint2 *paged;               // PAGED: the segment's keys on a page of the cache
  int *seen;                  // usable entries, a quarter of them looked at
  int few;                    // so many or fewer are gathered (-1: none)
  // Steps whose row maxima are raised at once, until some 32 selected keys are
  // behind them. Few of a tile's keys are selected, and a maximum of few lags
  // behind the row's: later weights lie above 1, where bf16 is half as fine. With
  // maxima that may lag from the first step on, outputs were 0.1 to 4% further
  // from 64 bits than the gather's where one key in eight or fewer is selected.
  int eager;

  // a tile past the last (see AttnPipe::tile; its bits are clear) takes the
  // last one's rows
  __device__ __forceinline__ int row(int tile, int e) const {
    const int s = (SPLIT ? min(tile, ntiles - 1) : tile) * kAttnKT + e;
    return PAGED ? pages.row(min(s, S - 1)) : s;
  }
  __device__ __forceinline__ int seg_tiles() const { return SPLIT ? 2 * steps : steps; }
  __device__ __forceinline__ uint2 bits(int tile) const {
    // read past the direct-to-LDS tile loads in flight (they never write bits)
    const uint32_t i = (uint32_t)(tile & (seg_tiles() - 1));
    const uint32_t a = lane_bits + i * (uint32_t)(TQ * 8);
    uint2 r;
    if constexpr (PAGED) {
      const uint32_t pa =
          (uint32_t)(size_t)(const __attribute__((address_space(3))) uint2 *)paged + i * 8;
      uint2 in;
      asm volatile("ds_read_b64 %0, %2\n\tds_read_b64 %1, %3\n\ts_waitcnt lgkmcnt(0)"
                   : "=&v"(r), "=&v"(in)
                   : "v"(a), "v"(pa)
                   : "memory");
      r.x &= in.x;
      r.y &= in.y;
    } else {
      asm volatile("ds_read_b64 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(r) : "v"(a) : "memory");
    }
    return r;
  }
  // After the first fill: whether to gather (the same for the whole workgroup).
  __device__ __forceinline__ bool leave() const {
    return __builtin_amdgcn_readfirstlane(*seen) <= few >> 2;   // (one entry in four is seen)
  }
  // Bits of the segment that starts at key tile tile0. (query, 8-entry piece)
  // items, two of a thread's in flight; entries of a piece that share a word
  // (neighbours of an ascending row) are merged before the LDS atomic.
  // Contains barriers: every wave of the workgroup calls it.
  __device__ __forceinline__ void fill(int tile0) const {
    const int tid = threadIdx.x;
    const int n = min(seg_tiles(), ntiles - tile0);
    const int count = ((n + 1) & ~1) * TQ * 2;   // seg_tiles is even
    for (int i = tid * 4; i < count; i += NT * 4)
      *reinterpret_cast<uint4 *>(words + i) = make_uint4(0, 0, 0, 0);
    if constexpr (PAGED) {
      const int lane = tid & 63;
      for (int i = tid >> 6; i < n; i += NT / 64) {
        const int s = (tile0 + i) * kAttnKT + lane;
        const uint64_t in = __ballot(pages.row(min(s, S - 1)) >= 0);
        if (lane == 0) paged[i] = make_uint2((uint32_t)in, (uint32_t)(in >> 32));
      }
    }
    __syncthreads();
    const int s0 = tile0 * kAttnKT, s1 = s0 + n * kAttnKT;
    const int kc = (kk + 7) / 8, items = nq * kc;
    const bool vec = (kk & 3) == 0;   // every row starts 16-byte aligned
    constexpr int U = 2;
    int usable = 0;
#pragma unroll 1
    for (int base = 0; base < items; base += U * NT) {
      const int i0 = base + tid;
      int e[U][8], qq[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int it = i0 + u * NT;
        qq[u] = it < items ? it / kc : 0;
        const int c = (it - qq[u] * kc) * 8;
        const int left = it < items ? kk - c : 0;
        const int32_t *row = table + (size_t)((t0 + qq[u] - qo) / b) * kk + (left > 0 ? c : 0);
        if (vec) {
          const int4 none = make_int4(-1, -1, -1, -1);
          const int4 x = left > 0 ? *reinterpret_cast<const int4 *>(row) : none;
          const int4 y = left > 4 ? *reinterpret_cast<const int4 *>(row + 4) : none;
          e[u][0] = x.x; e[u][1] = x.y; e[u][2] = x.z; e[u][3] = x.w;
          e[u][4] = y.x; e[u][5] = y.y; e[u][6] = y.z; e[u][7] = y.w;
        } else {
#pragma unroll
          for (int x = 0; x < 8; ++x) e[u][x] = x < left ? row[x] : -1;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int t = t0 + qq[u];
        usable += (e[u][0] >= 0 && e[u][0] <= t) + (e[u][4] >= 0 && e[u][4] <= t);
        // ascending rows: most pieces of a wave lie wholly outside the segment
        bool some = false;
#pragma unroll
        for (int x = 0; x < 8; ++x) some |= e[u][x] >= s0 && e[u][x] < s1;
        if (!__any(some)) continue;
        int w[8];
        uint32_t bit[8];
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          const int s = e[u][x], p = s - s0;
          const bool in = s >= s0 && s < s1 && s <= t;
          w[x] = in ? ((p >> 6) * TQ + qq[u]) * 2 + ((p >> 5) & 1) : -1;
          bit[x] = 1u << (p & 31);
        }
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          const bool carry = x < 7 && w[x] == w[x < 7 ? x + 1 : 7];
          if (x < 7) bit[x < 7 ? x + 1 : 7] |= carry ? bit[x] : 0u;
          if (!carry && w[x] >= 0) atomicOr(&words[w[x]], bit[x]);
        }
      }
      // the entries looked at so far may be few enough to leave at once (where
      // the fill is long: the wait takes 3 us of the 4 that a short one does)
      if (tile0 == 0 && base == 0 && items >= 8 * U * NT && few >= 0) {
        tally(usable);
        usable = 0;
        __syncthreads();
        const bool gone =
            __builtin_amdgcn_readfirstlane(*seen) <= few * ((float)(U * NT / 8) / items);
        __syncthreads();   // every wave has read it
        if (gone) return;
      }
    }
    if (tile0 == 0) tally(usable);
    __syncthreads();
  }
  __device__ __forceinline__ void tally(int n) const {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) n += __shfl_xor(n, off, 64);
    if ((threadIdx.x & 63) == 0) atomicAdd(seen, n);
  }
};

template <int D, bool SPLIT>
struct MaskLayout {
  using L = AttnLayout<D>;
  static constexpr int NW = attn_max_waves<D>();
  static constexpr int ROWS = (SPLIT ? NW / 2 : NW) * kAttnQPW;   // query rows per workgroup
  static constexpr int TILES = (SPLIT ? 2 : 1) * L::bytes(true);
  // the segment's bits take what a CU's LDS leaves beside the tiles, 64 KiB at most
  static constexpr int BITS = TILES > 96 * 1024 ? 24 * 1024 : 64 * 1024;
  static constexpr int LDS = TILES + BITS;
  static constexpr int MIN_TQ = ROWS / 16;   // queries at the most heads a group
  // waves that compute NaN rows again: as many as have their slots in the storage
  static constexpr int NF_MAX = LDS / (int)sizeof(QuerySlots<D, 1>);
  static constexpr int NF = NF_MAX < NW ? NF_MAX : NW;
  static_assert(LDS >= L::lds_bytes(true, NW) && LDS >= (int)sizeof(QuerySlots<D, NF>),
                "the output rows and the gather slots reuse the storage");
  static_assert(LDS + ROWS * 4 + BITS / MIN_TQ <= 160 * 1024, "fits the LDS of a CU");
  static_assert(2 * 8 * ROWS <= BITS, "two tiles' bits at one head per group");
};

template <int D, bool SPLIT, bool PAGED>
__global__ __launch_bounds__(attn_max_waves<D>() * 64) SP_ATTN_OCCUPANCY(D) void sparse_mask_kernel(
    int S, int qo, int Hq, int Hkv, int G, int b, int kk, size_t gstride, int TQ, int nqt,
    int seg_tiles, float tile_entries, float query_entries, float scale_log2,
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k,
    const uint16_t *__restrict__ v, const int32_t *__restrict__ idx,
    uint16_t *__restrict__ o, KvPages pages) {
  // q and o are addressed by position: the host shifts them back by qo rows
  using M = MaskLayout<D, SPLIT>;
  constexpr int kNW = M::NW, NT = kNW * 64;
  __shared__ __align__(16) char lds[M::LDS];
  __shared__ uint2 paged[PAGED ? M::BITS / (8 * M::MIN_TQ) : 1];
  __shared__ int again[M::ROWS];   // queries to compute from their selected rows
  __shared__ int seen;

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int h = lane >> 5, n = lane & 31;
  const int j = (int)blockIdx.x % Hkv;
  const int qi = nqt - 1 - (int)blockIdx.x / Hkv;   // longest first
  const int t0 = qo + qi * TQ;
  const int tl = min(t0 + TQ, S) - 1;
  const int nq = tl - t0 + 1;
  const int nrows = nq * G;
  const int row0 = (SPLIT ? wave & 3 : wave) * kAttnQPW;
  const int32_t *table = idx + (size_t)j * gstride;

  QRow<D> qr;
  load_q_row<D>(q, Hq, G, j, t0, row0 + n, nrows, h, qr);
  if (tid < nq) again[tid] = 0;
  if (tid == 0) seen = 0;
  AttnState<D> st;
  const uint32_t bits_a =
      (uint32_t)(size_t)(__attribute__((address_space(3))) char *)(lds + M::TILES);
  // entries that take as long to gather as the key tiles to multiply, at most
  // three quarters of what full rows hold
  const int ntiles = tl / kAttnKT + 1;
  const float worth = ntiles * tile_entries - nq * query_entries;
  const float most = 0.75f * nq * min(t0 + 1, kk);
  const int few = worth <= 0.f ? -1 : (int)(worth < most ? worth : most);
  const int sel = min(kk, tl + 1);   // of the tl + 1 keys
  const MaskedKeys<NT, SPLIT, PAGED> keys{ntiles, SPLIT ? seg_tiles / 2 : seg_tiles,
                                          t0, nq, TQ, table, qo, b, kk,
                                          reinterpret_cast<uint32_t *>(lds + M::TILES),
                                          bits_a + (uint32_t)(qr.t - t0) * 8, pages, S, paged,
                                          &seen, few, (tl + 2 * sel) / (2 * sel)};
  const int kv_rows = PAGED ? pages.num_pages * pages.page_size : S;
  AttnPipe<D, kNW, true, MaskedKeys<NT, SPLIT, PAGED>, SPLIT> pipe(lds, keys, k, v, kv_rows, Hkv,
                                                                   j, scale_log2, 0, qr, st);
  pipe.run();
  const bool left = keys.leave();
  bool nan = false;
  if (!left) {
    if constexpr (SPLIT) {
      attn_merge<D, true>(st, wave, lane, lds);
      if (wave >= 4) qr.valid = false;   // group 0 writes the rows
    }
    // NaN by bit pattern, on values the compiler knows nothing about
    uint32_t top = 0;
#pragma unroll
    for (int dt = 0; dt < AttnLayout<D>::DT; ++dt) {
      settle(st.o[dt]);
#pragma unroll
      for (int e = 0; e < 16; ++e) top = max(top, __float_as_uint(st.o[dt][e]) & 0x7fffffffu);
    }
    nan = qr.valid && top > 0x7f800000u;
    attn_finish<D>(st, qr, Hq, o, nullptr, h, lds);
    if (nan) again[qr.t - t0] = 1;
    drain_memory();   // this wave's rows are written before another wave rewrites them
  }
  if (!__syncthreads_or(nan || left)) return;
  if (wave >= M::NF) return;
  auto &slots = *reinterpret_cast<QuerySlots<D, M::NF> *>(lds);
  for (int i = wave; i < nq; i += M::NF)
    if (left || again[i])
      query_attend<D>(t0 + i, j, Hq, Hkv, G, kk, scale_log2, q, k, v,
                      table + (size_t)((t0 + i - qo) / b) * kk, o, pages, slots.pos[wave],
                      slots.rows[wave], lane);
}

template <int D, bool SPLIT>
hipError_t launch_t(const Prob &p, const void *q, const void *k, const void *v,
                    const int32_t *idx, void *o, hipStream_t st, KvPages pages) {
  using M = MaskLayout<D, SPLIT>;
  const int TQ = M::ROWS / p.G;
  const int nqt = (p.nq + TQ - 1) / TQ;
  const MaskShape m = mask_shape(p);   // (m.split == SPLIT)
  static_assert(M::BITS == 64 * 1024 || M::BITS == 24 * 1024, "as in mask_shape");
  // a workgroup that gathers does so with NF waves, where the gather kernel has
  // 12 / 8 / 6 on a CU at d = 64 / 128 / 256
  constexpr double kCus = 256, kWaves = (D == 64 ? 12.0 : D == 128 ? 8.0 : 6.0) / M::NF;
  const SparseRates r = sparse_rates(p);
  const float tile_entries = (float)(r.step * (SPLIT ? 0.5 * kSplitStep : 1.0) /
                                     (1.15 * kCus * kWaves * r.row)),
              query_entries = (float)(r.query / r.row);
  const size_t shift = (size_t)p.qo * p.Hq * D;   // chunk rows addressed by position
#define SP_MASKED(PAGED)                                                                       \
  hipLaunchKernelGGL((sparse_mask_kernel<D, SPLIT, PAGED>), dim3(nqt * p.Hkv), dim3(M::NW * 64), \
                     0, st, p.S, p.qo, p.Hq, p.Hkv, p.G, p.b, p.k, p.idx_group_stride(), TQ,   \
                     nqt, m.seg_tiles(p), tile_entries, query_entries, p.scale * kLog2e,         \
                     (const uint16_t *)q - shift,                                             \
                     (const uint16_t *)k, (const uint16_t *)v, idx, (uint16_t *)o - shift, pages)
  if (pages.table)
    SP_MASKED(true);
  else
    SP_MASKED(false);
#undef SP_MASKED
  return hipGetLastError();
}

template <int D>
hipError_t launch_d(const Prob &p, const void *q, const void *k, const void *v,
                    const int32_t *idx, void *o, hipStream_t st, KvPages pages) {
  if constexpr (D <= 128)
    if (mask_shape(p).split) return launch_t<D, true>(p, q, k, v, idx, o, st, pages);
  return launch_t<D, false>(p, q, k, v, idx, o, st, pages);
}

}  // namespace

hipError_t launch_sparse_mask_mfma(const Prob &p, const void *q, const void *k, const void *v,
                                   const int32_t *idx, void *o, hipStream_t st, KvPages pages) {
  if (p.d == 64) return launch_d<64>(p, q, k, v, idx, o, st, pages);
  if (p.d == 256) return launch_d<256>(p, q, k, v, idx, o, st, pages);
  return launch_d<128>(p, q, k, v, idx, o, st, pages);
}

}  // namespace sp
