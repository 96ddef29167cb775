// Fused per-query indexer scoring and top-k selection (Section 6.3 score;
// Section 6.4 and Algorithm 2, scoring, selection and sparse prefill with b_sel = 1; Section 4.1 TopK):
// the top-k of z[t, s] = ReLU(scale <q_idx[t], k_idx[s]>) over s <= t, for
// every query t, without ever storing the S x S score matrix.
//
// Selection is the same as sp_topk_select on the stored scores: for a row
// with L = t+1 > k positions, the Wf = min(W, k) most recent positions are
// forced and k' = k - Wf are taken from [0, L - Wf) in the order (score
// descending, position ascending); output rows are ascending, -1 padded.
//
// One workgroup takes 32 queries through a whole radix select over the
// order-preserving uint32 keys of the fp32 scores, 10 bits a digit, with the
// scores recomputed on the matrix cores in every pass:
//   * histogram passes: the waves walk the key tiles in turn and count the keys
//     that match their row's prefix in LDS (16-bit counters, a row of them per
//     query); then a wave per row picks the digit that holds the k'-th largest
//     key. A row whose chosen bin holds exactly the keys still needed is
//     settled: every key with that prefix is taken. The passes end when every
//     row is (usually after three of the four).
//   * emission: the waves write two bits per (query, key), above the threshold
//     and on it, to LDS, 8192 keys at a time; a wave per row then turns the
//     words into positions in order, with prefix sums of their bit counts.
// The score of a (query, key) pair is bit-identical in every pass (the same
// MFMA chain and epilogue, the one of the stored scores), which keeps the
// passes consistent.
//
// A wave loads its key tiles straight into an LDS slot of its own: the next
// tile is in flight while the current one, in registers, is multiplied and
// counted, and no barrier is needed inside a pass. One kernel in place of ten
// with 64-query x 4096-key items and global partial histograms: d_idx 128, 4096
// tokens at k = 512 710 -> 100 us, 8192 at k = 2048 733 -> 183 us, 32768 3.55 ->
// 1.36 ms (scoring into a buffer and selecting from it: 1.39 ms). Below about 16K
// tokens the longest workgroup, which has twice the mean work, sets the time; over
// the whole launch at 8192 tokens the vector units are busy 29% of the cycles, LDS
// 16% (nearly half of that bank conflicts of the counters), the matrix cores 7%,
// and a wave waits 41% of its time.
#include <math.h>

#include "common.hpp"
#include "kernels.hpp"
#include "mfma.hpp"

namespace sp {
namespace {

constexpr int kFQ = 32;            // queries per workgroup
constexpr int kFW = 8;             // waves
constexpr int kFBits = 10;         // bits per digit (the fourth has the last two)
constexpr int kFHistRow = 513;     // words of a row's 1024 16-bit counters, padded by one
constexpr int kFSeg = 8192;        // keys per emission segment
constexpr int kFSegRow = kFSeg / 32 + 1;   // words of a row's bits, padded by one
constexpr int kFSlot = 8192;       // bytes of a wave's LDS slot
constexpr int kFBufferDword3 = 0x00020000;   // raw buffer resource: 32-bit data format

struct FzProb {
  int S, k, Wf, relu;
  float scale;
};

template <int DI>
struct FzTile {
  static constexpr int KW = DI == 256 ? 16 : 32;   // keys per tile of a wave
  static constexpr int KT = KW / 16;               // 16-key MFMA rows
  static constexpr int KS = DI / 32;               // MFMA k-steps
  static constexpr int RB = DI * 2;                // row bytes
  static constexpr int SLOTS = DI / 8;             // 16-byte slots per row
  static constexpr int CH = KW * RB / 1024;        // 1 KiB direct loads per tile
  static_assert(KW * RB <= kFSlot, "a tile fits the wave's slot");
  // 16-byte slot c of row r is stored at c ^ swz(r): the 16 rows of an operand
  // read fall on distinct banks
  __device__ __forceinline__ static int swz(int r) { return DI == 64 ? (r >> 1) & 7 : r & 15; }

  __device__ __forceinline__ static void offsets(int lane, uint32_t (&off)[CH]) {
#pragma unroll
    for (int q = 0; q < CH; ++q) {
      const int row = (q * 64 + lane) / SLOTS, c = (q * 64 + lane) % SLOTS;
      off[q] = (uint32_t)(row * RB + (c ^ swz(row)) * 16);
    }
  }
  // keys k0 .. k0 + KW - 1 into the slot; those past S - 1 load zeros
  __device__ __forceinline__ static void issue(uint32_t slot, const uint16_t *ki, int S, int k0,
                                               const uint32_t (&off)[CH]) {
    const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(ki), (short)0,
                                                      (uint32_t)S * RB, kFBufferDword3);
#pragma unroll
    for (int q = 0; q < CH; ++q)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rs, (__attribute__((address_space(3))) void *)(size_t)(slot + q * 1024), 16,
          off[q] + (uint32_t)k0 * RB, 0, 0, 0);
  }
};

__device__ __forceinline__ uint32_t or4(uint32_t x) {   // over lanes l, l^16, l^32, l^48
  const auto a = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  const uint32_t y = a[0] | a[1];
  const auto c = __builtin_amdgcn_permlane16_swap(y, y, false, false);
  return c[0] | c[1];
}

// LDS accesses that run while direct loads are in flight: inline, as the
// compiler would wait for those loads first. Drained by fz_lds_done.
__device__ __forceinline__ void fz_lds_add(uint32_t a, uint32_t x) {
  asm volatile("ds_add_u32 %0, %1" : : "v"(a), "v"(x) : "memory");
}
__device__ __forceinline__ void fz_lds_put32(uint32_t a, uint32_t x) {
  asm volatile("ds_write_b32 %0, %1" : : "v"(a), "v"(x) : "memory");
}
__device__ __forceinline__ void fz_lds_put16(uint32_t a, uint32_t x) {
  asm volatile("ds_write_b16 %0, %1" : : "v"(a), "v"(x) : "memory");
}
__device__ __forceinline__ void fz_lds_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// What a lane keeps of its two queries (columns c16 of query tiles 0 and 1).
struct FzLane {
  int nc[2];              // candidates of the row (0: none to look at)
  uint32_t prefix[2], pmask[2];
};

template <int DI, bool RELU>
__global__ __launch_bounds__(kFW * 64) void fz_select_kernel(FzProb f,
                                                             const uint16_t *__restrict__ qi,
                                                             const uint16_t *__restrict__ ki,
                                                             int32_t *__restrict__ idx) {
  using T = FzTile<DI>;
  constexpr int KT = T::KT, KS = T::KS, KW = T::KW;
  constexpr int kWords = kFQ * kFHistRow > 2 * kFQ * kFSegRow ? kFQ * kFHistRow
                                                              : 2 * kFQ * kFSegRow;
  __shared__ __align__(16) char slots[kFW][kFSlot];
  __shared__ uint32_t words[kWords];   // histograms, then the emission's bits
  __shared__ uint32_t st_prefix[kFQ], st_pmask[kFQ], st_left[kFQ];
  __shared__ int st_open[kFQ];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, c16 = lane & 15;
  const int t0 = ((int)gridDim.x - 1 - (int)blockIdx.x) * kFQ;   // longest first
  const int t_last = min(t0 + kFQ, f.S) - 1;
  const int kp = f.k - f.Wf;

  // rows with at most k positions take them all; the others' forced window
  for (int r = wave; t0 + r <= t_last; r += kFW) {
    const int L = t0 + r + 1;
    int32_t *out = idx + (size_t)(t0 + r) * f.k;
    if (L <= f.k)
      for (int c = lane; c < f.k; c += 64) out[c] = c < L ? c : -1;
    else
      for (int c = lane; c < f.Wf; c += 64) out[kp + c] = L - f.Wf + c;
  }
  if (t_last + 1 <= f.k || kp == 0) return;   // nothing to choose
  if (tid < kFQ) {
    st_prefix[tid] = 0u;
    st_pmask[tid] = 0u;
    st_left[tid] = (uint32_t)kp;
    st_open[tid] = t0 + tid <= t_last && t0 + tid + 1 > f.k;
  }

  bf16x8 qb[2][KS];
#pragma unroll
  for (int qt = 0; qt < 2; ++qt)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      qb[qt][ks] = as_bf16x8(
          ldg16(qi + (size_t)min(t0 + qt * 16 + c16, f.S - 1) * DI + ks * 32 + g * 8));
  const uint32_t slot =
      (uint32_t)(size_t)(__attribute__((address_space(3))) char *)&slots[wave][0];
  const uint32_t words_a = (uint32_t)(size_t)(__attribute__((address_space(3))) uint32_t *)words;
  uint32_t off[T::CH], kread[KS];
  T::offsets(lane, off);
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    kread[ks] = slot + (uint32_t)(c16 * T::RB + ((ks * 4 + g) ^ T::swz(c16)) * 16);
  const int ncmax = t_last + 1 - f.Wf;
  // every open row has candidates up to here: tiles below need no position test
  const int ncmin = max(t0 + 1, f.k + 1) - f.Wf;

  // Walks this wave's tiles of keys [k_begin, k_end), body(k0, key): key[qt][kt][r]
  // is the key of query 16 qt + c16 and position k0 + 16 kt + 4 g + r.
  auto walk = [&](int k_begin, int k_end, auto body) {
    int k0 = k_begin + wave * KW;
    if (k0 < k_end) T::issue(slot, ki, f.S, k0, off);
    for (; k0 < k_end; k0 += kFW * KW) {
      __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the tile has landed
      asm volatile("" ::: "memory");
      bf16x8 a[KT][KS];
#pragma unroll
      for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          asm volatile("ds_read_b128 %0, %1 offset:%2"
                       : "=v"(a[kt][ks])
                       : "v"(kread[ks]), "i"(kt * 16 * T::RB));
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0][0]) : : "memory");
#pragma unroll
      for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(a[kt][ks]));
      // the tile is in registers: the slot takes the next one
      if (k0 + kFW * KW < k_end) T::issue(slot, ki, f.S, k0 + kFW * KW, off);
      uint32_t key[2][KT][4];
#pragma unroll
      for (int qt = 0; qt < 2; ++qt)
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
          f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) acc = mfma16(a[kt][ks], qb[qt][ks], acc);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float z = acc[r] * f.scale;
            // a ReLU'd score is +0, -0 or positive: both zeros share one key
            key[qt][kt][r] = RELU ? __float_as_uint(fmaxf(z, 0.f)) | 0x80000000u : float_key(z);
          }
        }
      body(k0, key);
    }
  };

  FzLane ln;
  auto load_rows = [&]() {   // the lane's rows; ones not looked at match no key
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
      const int r = qt * 16 + c16;
      const bool open = st_open[r] != 0;
      ln.nc[qt] = open ? t0 + r + 1 - f.Wf : 0;
      ln.prefix[qt] = open ? st_prefix[r] : 1u;
      ln.pmask[qt] = open ? st_pmask[r] : 0u;
    }
  };

  // ------------------------------------------------------------ histograms
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = pass == 3 ? 0 : 32 - kFBits * (pass + 1);
    const uint32_t dmask = pass == 3 ? 3u : (1u << kFBits) - 1u;
    for (int i = tid; i < kFQ * kFHistRow; i += kFW * 64) words[i] = 0u;
    __syncthreads();
    load_rows();
    uint32_t row_a[2];
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) row_a[qt] = words_a + (uint32_t)((qt * 16 + c16) * kFHistRow) * 4;
    auto count = [&](auto first_, auto full_, int k0, const uint32_t (&key)[2][KT][4]) {
      constexpr bool FIRST = decltype(first_)::value, FULL = decltype(full_)::value;
#pragma unroll
      for (int qt = 0; qt < 2; ++qt)
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const uint32_t kv = key[qt][kt][r];
            bool in = true;
            if constexpr (!FULL) in = k0 + 16 * kt + 4 * g + r < ln.nc[qt];
            if constexpr (!FIRST) in = in && (kv & ln.pmask[qt]) == ln.prefix[qt];
            // counter d is the half d % 2 of word d / 2
            const uint32_t d = (kv >> shift) & dmask;
            const uint32_t a = row_a[qt] + (d >> 1) * 4, one = 1u << ((d & 1u) * 16);
            if (FIRST && FULL)
              fz_lds_add(a, one);
            else if (in)
              fz_lds_add(a, one);
          }
    };
    // in the first pass every row of a full tile counts, also those not open
    walk(0, ncmax, [&](int k0, const uint32_t (&key)[2][KT][4]) {
      const bool full = k0 + KW <= ncmin;
      if (pass == 0) {
        if (full) count(std::true_type{}, std::true_type{}, k0, key);
        else count(std::true_type{}, std::false_type{}, k0, key);
      } else {
        if (full) count(std::false_type{}, std::true_type{}, k0, key);
        else count(std::false_type{}, std::false_type{}, k0, key);
      }
    });
    fz_lds_done();
    __syncthreads();
    // the digit of each open row: lane l owns bins 16 l .. 16 l + 15
    int open = 0;
    for (int r = wave; r < kFQ; r += kFW) {
      if (!st_open[r]) continue;   // uniform over the wave
      uint32_t cnt[16], mine = 0;
#pragma unroll
      for (int w = 0; w < 8; ++w) {
        const uint32_t x = words[r * kFHistRow + 8 * lane + w];
        cnt[2 * w] = x & 0xffffu;
        cnt[2 * w + 1] = x >> 16;
        mine += cnt[2 * w] + cnt[2 * w + 1];
      }
      uint32_t incl = mine;   // over this lane's bins and all higher ones
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t x = __shfl_down(incl, o, 64);
        if (lane + o < 64) incl += x;
      }
      const uint32_t need = st_left[r];
      uint32_t above = incl - mine;
      const bool here = above < need && incl >= need;
      uint32_t bin = 0, left = 0, in_bin = 0;
      if (here) {
#pragma unroll
        for (int e = 15; e >= 0; --e) {
          if (above < need && above + cnt[e] >= need) {
            bin = (uint32_t)(16 * lane + e);
            left = need - above;
            in_bin = cnt[e];
          }
          above += cnt[e];
        }
      }
      const uint64_t who = __ballot(here);
      const int owner = who ? __ffsll((unsigned long long)who) - 1 : 0;
      bin = __shfl(bin, owner, 64);
      left = __shfl(left, owner, 64);
      in_bin = __shfl(in_bin, owner, 64);
      const bool settled = left == in_bin || pass == 3;
      if (lane == 0) {
        st_prefix[r] |= bin << shift;
        st_pmask[r] |= dmask << shift;
        st_left[r] = left;
        st_open[r] = settled ? 0 : 1;
      }
      open |= !settled;
    }
    if (!__syncthreads_or(open)) break;
  }

  // -------------------------------------------------------------- emission
  if (tid < kFQ) st_open[tid] = t0 + tid <= t_last && t0 + tid + 1 > f.k;
  __syncthreads();
  load_rows();
  uint32_t done_gt[kFQ / kFW] = {}, done_eq[kFQ / kFW] = {};   // of this wave's rows
  int32_t *stage = reinterpret_cast<int32_t *>(slots[wave]);
  for (int s0 = 0; s0 < ncmax; s0 += kFSeg) {
    walk(s0, min(s0 + kFSeg, ncmax), [&](int k0, const uint32_t (&key)[2][KT][4]) {
      uint32_t gt[2] = {0u, 0u}, eq[2] = {0u, 0u};
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) {
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const uint32_t m = key[qt][kt][r] & ln.pmask[qt];
            gt[qt] |= m > ln.prefix[qt] ? 1u << (16 * kt + r) : 0u;
            eq[qt] |= m == ln.prefix[qt] ? 1u << (16 * kt + r) : 0u;
          }
        const int n = ln.nc[qt] - k0;   // candidates from this tile on
        const uint32_t in = n >= 32 ? ~0u : n <= 0 ? 0u : (1u << n) - 1u;
        gt[qt] = or4(gt[qt] << (4 * g)) & in;
        eq[qt] = or4(eq[qt] << (4 * g)) & in;
      }
      // lane group g writes one of the four words: above or on, query tile
      const uint32_t w = g == 0 ? gt[0] : g == 1 ? gt[1] : g == 2 ? eq[0] : eq[1];
      const uint32_t row = (uint32_t)((g >> 1) * kFQ + (g & 1) * 16 + c16) * kFSegRow;
      const uint32_t p = (uint32_t)(k0 - s0);
      if constexpr (KW == 32)
        fz_lds_put32(words_a + (row + (p >> 5)) * 4, w);
      else
        fz_lds_put16(words_a + (row + (p >> 5)) * 4 + (p & 16) / 8, w);
    });
    fz_lds_done();
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kFQ / kFW; ++i) {
      const int r = wave + i * kFW;
      if (t0 + r > t_last || t0 + r + 1 <= f.k) continue;   // uniform over the wave
      const int nw = (min(t0 + r + 1 - f.Wf - s0, kFSeg) + 31) / 32;
      const uint32_t left = st_left[r];
      int32_t *out = idx + (size_t)(t0 + r) * f.k;
      for (int w0 = 0; w0 < nw; w0 += 64) {
        const int w = w0 + lane;
        // (the half of a row's last word past its tiles may be unwritten)
        const int n_in = t0 + r + 1 - f.Wf - s0 - w * 32;
        const uint32_t in = n_in >= 32 ? ~0u : n_in <= 0 ? 0u : (1u << n_in) - 1u;
        uint32_t take = w < nw ? words[r * kFSegRow + w] & in : 0u;
        uint32_t eq = w < nw ? words[(kFQ + r) * kFSegRow + w] & in : 0u;
        const uint32_t cg = (uint32_t)__popc(take), ce = (uint32_t)__popc(eq);
        uint32_t incl = (cg << 16) | ce;   // at most 2048 of each
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const uint32_t x = __shfl_up(incl, o, 64);
          if (lane >= o) incl += x;
        }
        const uint32_t total = __shfl(incl, 63, 64);
        const uint32_t my_eq = done_eq[i] + (incl & 0xffffu) - ce;
        const uint32_t eq0 = min(done_eq[i], left), used = min(my_eq, left);
        uint32_t neq = min(left - used, ce);
        if (neq == ce) {
          take |= eq;
        } else {
          for (; neq > 0; --neq) {
            const uint32_t low = eq & (0u - eq);
            take |= low;
            eq ^= low;
          }
        }
        // chosen positions in order, staged in the wave's slot
        uint32_t at = (incl >> 16) - cg + used - eq0;
        while (take) {
          stage[at++] = s0 + w * 32 + __builtin_ctz(take);
          take &= take - 1u;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const uint32_t n = (total >> 16) + min(done_eq[i] + (total & 0xffffu), left) - eq0;
        const uint32_t o0 = done_gt[i] + eq0;
        for (uint32_t c = lane; c < n; c += 64)
          if (o0 + c < (uint32_t)kp) out[o0 + c] = stage[c];   // always true for consistent counts
        done_gt[i] += total >> 16;
        done_eq[i] += total & 0xffffu;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
    }
    __syncthreads();   // the words are read: the next segment may overwrite them
  }
}

template <int DI>
hipError_t launch_di(const FzProb &f, const void *qi, const void *ki, int32_t *idx,
                     hipStream_t st) {
  const dim3 grid((f.S + kFQ - 1) / kFQ);
  const uint16_t *q = (const uint16_t *)qi, *k = (const uint16_t *)ki;
  if (f.relu)
    hipLaunchKernelGGL((fz_select_kernel<DI, true>), grid, dim3(kFW * 64), 0, st, f, q, k, idx);
  else
    hipLaunchKernelGGL((fz_select_kernel<DI, false>), grid, dim3(kFW * 64), 0, st, f, q, k, idx);
  return hipGetLastError();
}

}  // namespace

// The size the entry points state and check (512 bytes per query and 4096-key
// chunk, 144 per query, in 256-byte units). The kernel keeps its histograms in
// LDS and touches none of it.
size_t indexer_topk_workspace(const Prob &p) {
  auto al = [](size_t b) { return (b + 255) & ~size_t(255); };
  const size_t S = (size_t)p.S;
  return al(16 * S) + al(512 * ((S + 4095) / 4096) * S) + 2 * al(64 * S);
}

// 16-bit counters hold a row's candidates
bool indexer_topk_supported(const Prob &p) {
  return p.dtype == SP_DTYPE_BF16 && (p.di == 64 || p.di == 128 || p.di == 256) && p.b == 1 &&
         p.S <= 65535 && p.iscale >= 0.f;
}

hipError_t launch_indexer_topk(const Prob &p, const void *qi, const void *ki, int32_t *idx,
                               void *, hipStream_t st) {
  FzProb f{p.S, p.k, p.W < p.k ? p.W : p.k, p.relu, p.iscale};
  if (p.di == 64) return launch_di<64>(f, qi, ki, idx, st);
  if (p.di == 128) return launch_di<128>(f, qi, ki, idx, st);
  return launch_di<256>(f, qi, ki, idx, st);
}

hipError_t launch_indexer_topk_static(const Prob &p, const void *qi, const void *ki,
                                      int32_t *idx, hipStream_t st) {
  return launch_indexer_topk(p, qi, ki, idx, nullptr, st);
}

}  // namespace sp
