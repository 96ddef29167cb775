// Dense causal GQA attention on bf16 MFMA (Section 3, first equation;
// Algorithm 1, dense scores and normalisers): a flash-attention forward that also returns the
// softmax normaliser lse[t,h] = log sum_{s<=t} exp(scale <q[t,h], k[s,g(h)]>).
//
// One workgroup per (tile of 256/G queries, KV head j; 128/G at head_dim
// 256): its 256 (128) query rows are every (query, head) pair of the tile
// with g(h) = j, so each K/V tile staged in LDS serves all G heads of the
// group. Key tiles below a wave's first
// query need no mask; only tiles reaching the diagonal apply s <= t.
// Workgroups are numbered with the KV head fastest, so consecutive
// workgroups (which the dispatcher spreads over the XCDs) keep one head per
// XCD when Hkv is 8, and query tiles are scheduled longest first (the causal
// work of tile i grows with i), which shortens the tail of the launch.
//
// dense_mfma.hip holds the kernels of whole sequences and of normalisers alone,
// dense_chunk_mfma.hip those of a chunk's output, whose code looks for NaN and is
// built without the assumption that there is none.
//
// With o == nullptr only the normalisers are produced: the P V product and
// the V traffic are skipped (the oracle's first pass needs nothing else).
#pragma once

#include "attn_tile.hpp"
#include "kernels.hpp"

namespace sp {
namespace {

template <bool SPLIT, bool NANS>
struct DenseKeys {
  static constexpr bool kLookup = false;   // rows are arithmetic
  static constexpr bool kBits = false;     // masked by position
  static constexpr bool kTable = false;
  static constexpr bool kNaNs = NANS;
  int ntiles, S;
  // a tile past the last (see AttnPipe::tile) takes the last one's rows, so
  // that its zero weights never meet a value row no query of the tile reads
  __device__ __forceinline__ int row(int tile, int e) const {
    return (SPLIT ? min(tile, ntiles - 1) : tile) * kAttnKT + e;
  }
  __device__ __forceinline__ bool needs_mask(int tile, int wave_tmin) const {
    return tile * kAttnKT + kAttnKT - 1 > wave_tmin;
  }
  __device__ __forceinline__ int4 pos4(int tile, int e0) const {
    const int s = tile * kAttnKT + e0;
    return int4{s, s + 1, s + 2, s + 3};
  }
};

// R query rows of a chunk (positions t, heads `head`, those with need set)
// by one wave, from each row's own keys and in fp32: four 16-lane groups take
// every fourth key each, a lane holds D / 16 dims. Only for rows that the tiles
// left NaN; q and o are addressed by position. Ends early once every output is
// NaN whatever follows.
template <int D, int R>
__device__ __forceinline__ void dense_rows(const int (&t)[R], const int (&head)[R],
                                           const bool (&need)[R], int j, int Hq, int Hkv,
                                           float scale_log2, const uint16_t *__restrict__ q,
                                           const uint16_t *__restrict__ k,
                                           const uint16_t *__restrict__ v,
                                           uint16_t *__restrict__ o, int lane) {
  constexpr int EPL = D / 16, U = 256 / D * 2;   // keys in flight a group
  const int grp = lane >> 4, sub = lane & 15;
  float qf[R][EPL], acc[R][EPL], m[R], l[R];
  int last = -1;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    load_row<EPL>(reinterpret_cast<const bf16 *>(q + ((size_t)t[r] * Hq + head[r]) * D + sub * EPL),
                  qf[r]);
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[r][e] = 0.f;
    m[r] = -INFINITY;
    l[r] = 0.f;
    if (need[r]) last = max(last, t[r]);
  }
#pragma unroll 1
  for (int s0 = 0; s0 <= last; s0 += 4 * U) {
    float kf[U][EPL], vf[U][EPL];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t row = ((size_t)min(s0 + 4 * u + grp, last) * Hkv + j) * D + sub * EPL;
      load_row<EPL>(reinterpret_cast<const bf16 *>(k + row), kf[u]);
      load_row<EPL>(reinterpret_cast<const bf16 *>(v + row), vf[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int r = 0; r < R; ++r) {
        float part = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) part = fmaf(qf[r][e], kf[u][e], part);
        const float x = row16_sum(part) * scale_log2;
        if (s0 + 4 * u + grp > t[r]) continue;   // its values are skipped, not weighted by 0
        const float mn = fmaxf(m[r], x), ref = mn == -INFINITY ? 0.f : mn;
        const float c0 = fast_exp2(m[r] - ref), c1 = fast_exp2(x - ref);
        m[r] = mn;
        l[r] = l[r] * c0 + c1;
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[r][e] = fmaf(c1, vf[u][e], acc[r][e] * c0);
      }
    if ((s0 / (4 * U)) % 8 == 0) {   // every output of the rows NaN in one of the groups?
      bool all = true;
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
          int nan = acc[r][e] != acc[r][e];
          nan |= __shfl_xor(nan, 16, 64);
          nan |= __shfl_xor(nan, 32, 64);
          all = all && (nan || !need[r]);
        }
      if (__all(all)) break;
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) {
      const float mo = __shfl_xor(m[r], off, 64), lo = __shfl_xor(l[r], off, 64);
      const float mn = fmaxf(m[r], mo), ref = mn == -INFINITY ? 0.f : mn;
      const float c0 = fast_exp2(m[r] - ref), c1 = fast_exp2(mo - ref);
      m[r] = mn;
      l[r] = l[r] * c0 + lo * c1;
#pragma unroll
      for (int e = 0; e < EPL; ++e)
        acc[r][e] = acc[r][e] * c0 + __shfl_xor(acc[r][e], off, 64) * c1;
    }
    const float inv = l[r] > 0.f ? 1.f / l[r] : 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[r][e] *= inv;
    if (need[r] && grp == 0)
      store_row<EPL>(reinterpret_cast<bf16 *>(o + ((size_t)t[r] * Hq + head[r]) * D + sub * EPL),
                     acc[r]);
  }
}

// The values a workgroup's rows t0 .. see or its last tile reads, positions 0 ..
// end - 1 of KV head j: kinds[c] of dims 8c .. 8c + 7 gets a bit per dim with a
// NaN (bits 0-7), +inf (8-15) and -inf (16-23) up to position t0, kinds[D / 8 +
// c] after it, *bad the last position after t0 with any. All are cleared by the
// caller.
template <int D, int NT>
__device__ __forceinline__ void dense_value_kinds(int t0, int end, int j, int Hkv,
                                                  const uint16_t *__restrict__ v,
                                                  uint32_t *kinds, int *bad) {
  constexpr int C = D / 8, U = 4;
  const int c = (int)threadIdx.x % C;
  uint32_t mine[2] = {0, 0};
  int last = -1;
  for (int s0 = (int)threadIdx.x / C; s0 < end; s0 += U * (NT / C)) {
    uint4 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      x[u] = ldg16(v + ((size_t)min(s0 + u * (NT / C), end - 1) * Hkv + j) * D + c * 8);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t w[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
      uint32_t here = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t b = (w[e >> 1] >> (16 * (e & 1))) & 0xffffu;
        const uint32_t kind = (b & 0x7fffu) > 0x7f80u ? 0 : b == 0x7f80u ? 8 : b == 0xff80u ? 16 : 32;
        if (kind < 32) here |= 1u << (kind + e);
      }
      const int s = min(s0 + u * (NT / C), end - 1);
      mine[s > t0] |= here;
      if (here && s > t0) last = max(last, s);
    }
  }
#pragma unroll
  for (int x = 0; x < 2; ++x)
    if (mine[x]) atomicOr(&kinds[x * C + c], mine[x]);
  if (last >= 0) atomicMax(bad, last);
}

// SPLIT: see AttnPipe. CHUNK: the queries start at position qo (0 otherwise),
// and the P V product takes the weights in fp32, as three bf16 parts, where
// whole sequences round them to bf16: 1024 queries of 8192 keys, 32/8 heads, d =
// 128, take 215 us so (two parts 174, one key at a time in fp32 3600). A weight
// of zero still multiplies its V row, and an infinite entry each part of its
// weight, so infinite and NaN V entries reach outputs that they should not. Where
// a chunk's rows come out NaN although their weights are numbers, the workgroup
// looks its values over: rows before the last such entry of their tiles are
// computed again from their own keys (dense_rows), unless its dims are NaN anyhow;
// the others see every such entry, and the dims that hold any become what those
// sum up to. Whole sequences are left as the tiles make them.
template <int D, bool WANT_O, bool SPLIT, bool CHUNK>
__global__ __launch_bounds__(attn_max_waves<D>() * 64) SP_ATTN_OCCUPANCY(D) void dense_fwd_kernel(
    int S, int qo, int Hq, int Hkv, int G, int TQ, int nqt, float scale_log2,
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k,
    const uint16_t *__restrict__ v, uint16_t *__restrict__ o, float *__restrict__ lse) {
  // q, o and lse are addressed by position: the host shifts them back by qo rows
  using L = AttnLayout<D>;
  constexpr int kNW = attn_max_waves<D>();
  constexpr int kLds = SPLIT ? 2 * L::bytes(WANT_O) : L::lds_bytes(WANT_O, kNW);
  static_assert(!WANT_O || kLds >= L::lds_bytes(true, kNW), "room for the output rows");
  __shared__ __align__(16) char lds[kLds];
  constexpr bool kAgain = CHUNK && WANT_O;
  constexpr int kRows = (SPLIT ? kNW / 2 : kNW) * kAttnQPW;
  __shared__ int again[kAgain ? kRows : 1];   // query rows that came out NaN
  __shared__ uint32_t kinds[kAgain ? D / 4 : 1];   // see dense_value_kinds
  __shared__ int bad;

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int h = lane >> 5, n = lane & 31;
  const int j = (int)blockIdx.x % Hkv;
  const int qi = nqt - 1 - (int)blockIdx.x / Hkv;
  const int t0 = (CHUNK ? qo : 0) + qi * TQ;
  const int tl = min(t0 + TQ, S) - 1;
  const int nrows = (tl - t0 + 1) * G;
  const int row0 = (SPLIT ? wave & 3 : wave) * kAttnQPW;

  QRow<D> qr;
  load_q_row<D>(q, Hq, G, j, t0, row0 + n, nrows, h, qr);
  AttnState<D> st;
  if constexpr (kAgain) {
    if (tid < kRows) again[tid] = 0;
    if (tid < D / 4) kinds[tid] = 0;
    if (tid == 0) bad = -1;
  }
  using Keys = DenseKeys<SPLIT, kAgain>;
  const Keys keys{tl / kAttnKT + 1, S};
  const int wave_tmin = t0 + min(row0, nrows - 1) / G;
  AttnPipe<D, kNW, WANT_O, Keys, SPLIT, CHUNK && WANT_O> pipe(
      lds, keys, k, v, S, Hkv, j, scale_log2, wave_tmin, qr, st);
  pipe.run();
  if constexpr (SPLIT) {
    attn_merge<D, WANT_O>(st, wave, lane, lds);
    if (wave >= 4) qr.valid = false;   // group 0 writes the rows
  }
  if constexpr (kAgain) {
    // NaN by bit pattern, on values the compiler knows nothing about
    uint32_t top = 0;
#pragma unroll
    for (int dt = 0; dt < L::DT; ++dt) {
      settle(st.o[dt]);
#pragma unroll
      for (int e = 0; e < 16; ++e) top = max(top, __float_as_uint(st.o[dt][e]) & 0x7fffffffu);
    }
    // (weights that are NaN leave every dim NaN, as they should)
    const float l = half_sum(st.l);
    const bool nan = qr.valid && top > 0x7f800000u && l == l;
    attn_finish<D>(st, qr, Hq, o, lse, h, lds);
    if (nan) again[row0 + n] = 1;
    drain_memory();   // this wave's rows are written before another wave rewrites them
    if (!__syncthreads_or(nan)) return;
    dense_value_kinds<D, kNW * 64>(t0, min(keys.ntiles * kAttnKT, S), j, Hkv, v, kinds, &bad);
    __syncthreads();
    // whether rows before the last bad entry have to be computed again: not
    // if the dims it and its like are in are NaN from entries all rows see
    uint32_t fresh = 0;
    for (int c = 0; c < D / 8; ++c) {
      const uint32_t seen = kinds[c], later = kinds[D / 8 + c];
      fresh |= (later | later >> 8 | later >> 16) & ~(seen | (seen >> 8 & seen >> 16)) & 0xffu;
    }
    constexpr int R = 4;   // rows a wave takes at once
    for (int i0 = wave * R; i0 < nrows; i0 += kNW * R) {
      int t[R], head[R];
      bool need[R], any = false;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int i = min(i0 + r, nrows - 1);
        t[r] = t0 + i / G;
        head[r] = j * G + i % G;
        const bool nans = i0 + r < nrows && again[i] != 0;
        need[r] = nans && fresh != 0 && t[r] < bad;
        any = any || need[r];
        if (!nans || need[r]) continue;
        for (int d = lane; d < D; d += 64) {
          const uint32_t kind =
              (kinds[d >> 3] | (t[r] < bad ? 0u : kinds[D / 8 + (d >> 3)])) >> (d & 7);
          const bool pos = kind >> 8 & 1, neg = kind >> 16 & 1;
          if ((kind & 1) || pos || neg)
            o[((size_t)t[r] * Hq + head[r]) * D + d] =
                (kind & 1) || (pos && neg) ? 0x7fc0 : pos ? 0x7f80 : 0xff80;
        }
      }
      if (any) dense_rows<D, R>(t, head, need, j, Hq, Hkv, scale_log2, q, k, v, o, lane);
    }
  } else {
    attn_finish<D>(st, qr, Hq, WANT_O ? o : nullptr, lse, h, lds);
  }
}

template <int D, bool SPLIT, bool WANT_O, bool CHUNK>
hipError_t launch_dense(const Prob &p, const void *q, const void *k, const void *v, void *o,
                        float *lse, hipStream_t st) {
  constexpr int kNW = attn_max_waves<D>();
  const int TQ = ((SPLIT ? kNW / 2 : kNW) * kAttnQPW) / p.G;
  const int nqt = (p.nq + TQ - 1) / TQ;
  const size_t shift = (size_t)p.qo * p.Hq;   // chunk rows addressed by position
  hipLaunchKernelGGL((dense_fwd_kernel<D, WANT_O, SPLIT, CHUNK>), dim3(nqt * p.Hkv),
                     dim3(kNW * 64), 0, st, p.S, p.qo, p.Hq, p.Hkv, p.G, TQ, nqt,
                     p.scale * kLog2e, (const uint16_t *)q - shift * D, (const uint16_t *)k,
                     (const uint16_t *)v, o ? (uint16_t *)o - shift * D : nullptr,
                     lse ? lse - shift : nullptr);
  return hipGetLastError();
}

// Whether a launch splits the keys between the wave groups.
template <int D>
bool dense_split(const Prob &p) {
  constexpr int kRows = attn_max_waves<D>() * kAttnQPW;
  return D <= 128 && p.G <= kRows / 2 && few_workgroups(p, kRows / p.G);
}

// One of the launches above, by the problem's head dimension and split.
template <bool WANT_O, bool CHUNK>
hipError_t launch_dense_d(const Prob &p, const void *q, const void *k, const void *v, void *o,
                          float *lse, hipStream_t st) {
  if (p.d == 256) return launch_dense<256, false, WANT_O, CHUNK>(p, q, k, v, o, lse, st);
  if (p.d == 64)
    return dense_split<64>(p) ? launch_dense<64, true, WANT_O, CHUNK>(p, q, k, v, o, lse, st)
                              : launch_dense<64, false, WANT_O, CHUNK>(p, q, k, v, o, lse, st);
  return dense_split<128>(p) ? launch_dense<128, true, WANT_O, CHUNK>(p, q, k, v, o, lse, st)
                             : launch_dense<128, false, WANT_O, CHUNK>(p, q, k, v, o, lse, st);
}

}  // namespace
}  // namespace sp
