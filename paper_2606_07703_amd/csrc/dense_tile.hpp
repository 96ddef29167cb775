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

// One query row by one wave, from keys 0 .. t alone and in fp32: four 16-lane
// groups take every fourth key each, a lane holds D / 16 dims. Only for rows
// of a chunk that the tiles left NaN; q and o are addressed by position.
template <int D>
__device__ __forceinline__ void dense_row(int t, int head, int j, int Hq, int Hkv,
                                          float scale_log2, const uint16_t *__restrict__ q,
                                          const uint16_t *__restrict__ k,
                                          const uint16_t *__restrict__ v,
                                          uint16_t *__restrict__ o, int lane) {
  constexpr int EPL = D / 16;
  const int grp = lane >> 4, sub = lane & 15;
  const size_t at = ((size_t)t * Hq + head) * D + sub * EPL;
  float qf[EPL], acc[EPL], m = -INFINITY, l = 0.f;
  load_row<EPL>(reinterpret_cast<const bf16 *>(q + at), qf);
#pragma unroll
  for (int e = 0; e < EPL; ++e) acc[e] = 0.f;
  // adds a partial state (mo, lo, other) scaled to the common maximum
  auto merge = [&](float mo, float lo, auto other) {
    const float mn = fmaxf(m, mo), ref = mn == -INFINITY ? 0.f : mn;
    const float c0 = fast_exp2(m - ref), c1 = fast_exp2(mo - ref);
    l = l * c0 + lo * c1;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] = acc[e] * c0 + other(e) * c1;
    m = mn;
  };
#pragma unroll 1
  for (int s0 = 0; s0 <= t; s0 += 4) {
    const int s = s0 + grp;
    const size_t row = ((size_t)min(s, t) * Hkv + j) * D + sub * EPL;
    float kf[EPL], vf[EPL], part = 0.f;
    load_row<EPL>(reinterpret_cast<const bf16 *>(k + row), kf);
    load_row<EPL>(reinterpret_cast<const bf16 *>(v + row), vf);
#pragma unroll
    for (int e = 0; e < EPL; ++e) part = fmaf(qf[e], kf[e], part);
    const float x = row16_sum(part) * scale_log2;
    if (s <= t) merge(x, 1.f, [&](int e) { return vf[e]; });
  }
#pragma unroll
  for (int off = 16; off <= 32; off <<= 1) {
    const float mo = __shfl_xor(m, off, 64), lo = __shfl_xor(l, off, 64);
    float ao[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) ao[e] = __shfl_xor(acc[e], off, 64);
    merge(mo, lo, [&](int e) { return ao[e]; });
  }
  const float inv = l > 0.f ? 1.f / l : 0.f;
#pragma unroll
  for (int e = 0; e < EPL; ++e) acc[e] *= inv;
  if (grp == 0) store_row<EPL>(reinterpret_cast<bf16 *>(o + at), acc);
}

// SPLIT: see AttnPipe. CHUNK: the queries start at position qo (0 otherwise),
// and the P V product takes the weights to 2^-18, where whole sequences round
// them to bf16. A weight of zero still multiplies its V row, so an infinite or
// NaN V entry after a query would turn its output to NaN: a chunk's rows that
// come out NaN are computed again from their own keys (dense_row).
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
  __shared__ int again[kAgain ? kRows : 1];   // query rows to compute from their own keys

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
  if constexpr (kAgain)
    if (tid < kRows) again[tid] = 0;
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
    const bool nan = qr.valid && top > 0x7f800000u;
    attn_finish<D>(st, qr, Hq, o, lse, h, lds);
    if (nan) again[row0 + n] = 1;
    drain_memory();   // this wave's rows are written before another wave rewrites them
    if (!__syncthreads_or(nan)) return;
    for (int i = wave; i < nrows; i += kNW)
      if (again[i])
        dense_row<D>(t0 + i / G, j * G + i % G, j, Hq, Hkv, scale_log2, q, k, v, o, lane);
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
