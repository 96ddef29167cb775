// Head-collapsed indexer front end on bf16 MFMA (Section 6.3, projection and
// score equations; Algorithm 2, indexer projection and its key normalisation, RoPE and query scale):
//
//   q_idx[t] = RoPE(W_Q x_t, pos0 + t)
//   k_idx[t] = RoPE(LN(W_K x_t), pos0 + t),  LN over d_idx with gamma, beta
//   RoPE(a, p): the pair (a[c], a[c + d_idx/2]) turns by p * theta^(-2c/d_idx)
//
// project_ring_kernel computes C = x W^T for a tile of tokens and columns.
// The fp32 C tile is then parked in LDS and the epilogue works a token row at
// a time: each lane holds one rotation pair, takes the LayerNorm statistics of
// the key row with a wave reduction, rotates, and writes bf16. Angles are
// formed and range-reduced in fp64 (positions reach 1e5 and beyond) before a
// float sincos.
//
// project_kernel serves weights of 4 GiB or more, past the ring kernel's
// 32-bit offsets: one workgroup per 64 tokens computes both projections with
// W = [W_Q; W_K] ([2 d_idx, d_model]); x and W tiles go through
// double-buffered LDS (register staged), eight waves each own 2 d_idx / 8
// output columns of all 64 tokens.
#include <math.h>

#include "common.hpp"
#include "kernels.hpp"
#include "mfma.hpp"

namespace sp {
namespace {

constexpr int kPT = 64;    // tokens per workgroup
constexpr int kPW = 8;     // waves

template <int DI>
struct ProjLayout {
  static constexpr int KPK = DI == 256 ? 32 : 64;    // model columns per k-chunk (LDS fit)
  static constexpr int N = 2 * DI;                    // output columns (q then k)
  static constexpr int RB = KPK * 2 + 16;             // padded row bytes of an LDS tile
  static constexpr int XBYTES = kPT * RB;
  static constexpr int WBYTES = N * RB;
  static constexpr int BUF = XBYTES + WBYTES;
  static constexpr int CT = N / kPW / 16;             // 16-column tiles per wave
  static constexpr int CSTRIDE = N + 4;               // floats per token row of the C tile
  static constexpr int CBYTES = kPT * CSTRIDE * 4;
  static constexpr int LDS = (2 * BUF > CBYTES ? 2 * BUF : CBYTES);
};

// Epilogue on the fp32 C tile parked in LDS (token-major, cstride floats per
// token): one (token, q or k) row per wave step, lane pairs c, c + DI/2.
// PARTS = 1: the tile holds columns q then k; 2: only those of `part`.
template <int DI, int TOK, int NWAVE, int PARTS>
__device__ __forceinline__ void project_epilogue(const float *cl, int cstride, int S, int t0,
                                                 int pos0, float theta, float eps,
                                                 const float *__restrict__ gamma,
                                                 const float *__restrict__ beta,
                                                 uint16_t *__restrict__ qo,
                                                 uint16_t *__restrict__ ko, int part, int wave,
                                                 int lane) {
  constexpr int H = DI / 2;
  constexpr int PPL = (H + 63) / 64;   // pairs per lane
  double inv_freq[PPL];
  float gam[PPL][2], bet[PPL][2];
#pragma unroll
  for (int u = 0; u < PPL; ++u) {
    const int c = lane + u * 64;
    inv_freq[u] = exp2(-(2.0 * c / DI) * log2((double)theta));
    gam[u][0] = c < H ? gamma[c] : 0.f;
    gam[u][1] = c < H ? gamma[c + H] : 0.f;
    bet[u][0] = c < H ? beta[c] : 0.f;
    bet[u][1] = c < H ? beta[c + H] : 0.f;
  }
  const double two_pi = 6.283185307179586;
  for (int row = wave; row < (PARTS == 1 ? 2 * TOK : TOK); row += NWAVE) {
    const int tl = PARTS == 1 ? row >> 1 : row, is_k = PARTS == 1 ? row & 1 : part;
    const int t = t0 + tl;
    if (t >= S) continue;   // wave-uniform
    const float *cr = cl + tl * cstride + (PARTS == 1 ? is_k * DI : 0);
    float lo[PPL], hi[PPL];
#pragma unroll
    for (int u = 0; u < PPL; ++u) {
      const int c = lane + u * 64;
      lo[u] = c < H ? cr[c] : 0.f;
      hi[u] = c < H ? cr[c + H] : 0.f;
    }
    if (is_k) {
      float s = 0.f;
#pragma unroll
      for (int u = 0; u < PPL; ++u) s += lo[u] + hi[u];
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
      const float mean = s / DI;
      float v = 0.f;
#pragma unroll
      for (int u = 0; u < PPL; ++u) {
        const int c = lane + u * 64;
        if (c < H) {
          v += (lo[u] - mean) * (lo[u] - mean);
          v += (hi[u] - mean) * (hi[u] - mean);
        }
      }
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
      const float inv = 1.f / sqrtf(v / DI + eps);
#pragma unroll
      for (int u = 0; u < PPL; ++u) {
        lo[u] = (lo[u] - mean) * inv * gam[u][0] + bet[u][0];
        hi[u] = (hi[u] - mean) * inv * gam[u][1] + bet[u][1];
      }
    }
    uint16_t *out = (is_k ? ko : qo) + (size_t)t * DI;
    const double p = (double)pos0 + t;
#pragma unroll
    for (int u = 0; u < PPL; ++u) {
      const int c = lane + u * 64;
      if (c >= H) continue;
      double ang = p * inv_freq[u];
      ang -= two_pi * rint(ang / two_pi);
      float sn, cs;
      sincosf((float)ang, &sn, &cs);
      out[c] = float_to_bf16(lo[u] * cs - hi[u] * sn);
      out[c + H] = float_to_bf16(hi[u] * cs + lo[u] * sn);
    }
  }
}

template <int DI>
__global__ __launch_bounds__(kPW * 64) void project_kernel(
    int S, int dm, int pos0, float theta, float eps, const uint16_t *__restrict__ x,
    const uint16_t *__restrict__ wq, const uint16_t *__restrict__ wk,
    const float *__restrict__ gamma, const float *__restrict__ beta, uint16_t *__restrict__ qo,
    uint16_t *__restrict__ ko) {
  using L = ProjLayout<DI>;
  constexpr int NT = kPW * 64, N = L::N, RB = L::RB, CT = L::CT, kPK = L::KPK;
  constexpr int XP = kPT * kPK / 8;     // 16-byte pieces of an x tile
  constexpr int WP = N * kPK / 8;       // ... of a W tile
  constexpr int XPER = (XP + NT - 1) / NT, WPER = (WP + NT - 1) / NT;
  __shared__ __align__(16) char lds[L::LDS];

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int g = lane >> 4, c16 = lane & 15;
  const int t0 = blockIdx.x * kPT;

  uint4 xs[XPER], ws[WPER];
  auto load = [&](int k0) {
#pragma unroll
    for (int i = 0; i < XPER; ++i) {
      const int c = tid + i * NT;
      if (c < XP) {
        const int row = c / (kPK / 8), col = c % (kPK / 8);
        const int t = min(t0 + row, S - 1);
        xs[i] = ldg16(x + (size_t)t * dm + k0 + col * 8);
      }
    }
#pragma unroll
    for (int i = 0; i < WPER; ++i) {
      const int c = tid + i * NT;
      if (c < WP) {
        const int row = c / (kPK / 8), col = c % (kPK / 8);
        const uint16_t *w = row < DI ? wq + (size_t)row * dm : wk + (size_t)(row - DI) * dm;
        ws[i] = ldg16(w + k0 + col * 8);
      }
    }
  };
  auto store = [&](char *buf) {
#pragma unroll
    for (int i = 0; i < XPER; ++i) {
      const int c = tid + i * NT;
      if (c < XP) sts16(buf + (c / (kPK / 8)) * RB + (c % (kPK / 8)) * 16, xs[i]);
    }
#pragma unroll
    for (int i = 0; i < WPER; ++i) {
      const int c = tid + i * NT;
      if (c < WP)
        sts16(buf + L::XBYTES + (c / (kPK / 8)) * RB + (c % (kPK / 8)) * 16, ws[i]);
    }
  };

  f32x4 acc[4][CT];
#pragma unroll
  for (int rt = 0; rt < 4; ++rt)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int nk = dm / kPK;
  load(0);
  store(lds);
  __syncthreads();
  for (int it = 0; it < nk; ++it) {
    const bool more = it + 1 < nk;
    if (more) load((it + 1) * kPK);
    const char *buf = lds + (it & 1) * L::BUF;
#pragma unroll
    for (int ks = 0; ks < kPK / 32; ++ks) {
      bf16x8 a[4], b[CT];
#pragma unroll
      for (int rt = 0; rt < 4; ++rt)
        a[rt] = as_bf16x8(lds16(buf + (rt * 16 + c16) * RB + ks * 64 + g * 16));
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
        b[ct] = as_bf16x8(lds16(buf + L::XBYTES + ((wave * CT + ct) * 16 + c16) * RB +
                                ks * 64 + g * 16));
#pragma unroll
      for (int rt = 0; rt < 4; ++rt)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = mfma16(a[rt], b[ct], acc[rt][ct]);
    }
    if (more) store(lds + ((it + 1) & 1) * L::BUF);
    __syncthreads();
  }

  // Park C (token-major, fp32) in LDS: lane (g, c16) holds tokens
  // 16rt + 4g + r of column (wave*CT + ct)*16 + c16.
  float *cl = reinterpret_cast<float *>(lds);
#pragma unroll
  for (int rt = 0; rt < 4; ++rt)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        cl[(rt * 16 + g * 4 + r) * L::CSTRIDE + (wave * CT + ct) * 16 + c16] = acc[rt][ct][r];
  __syncthreads();

  project_epilogue<DI, kPT, kPW, 1>(cl, L::CSTRIDE, S, t0, pos0, theta, eps, gamma, beta, qo, ko,
                                    0, wave, lane);
}

// Ring kernel: TOK tokens times N output columns per workgroup, N = 2 d_idx
// (PARTS = 1: q and k together) or d_idx (PARTS = 2: one of them; LayerNorm
// and the rotation pairs stay within a part). x and W tiles of 64 model
// columns go straight from memory into a ring of LDS stages, NS - 1 of them
// in flight. A row of a stage is one 128-byte line (1 KiB load = 8 whole
// lines; the 64-byte rows of a 32-column stage were served at half the rate),
// its 16-byte slot c stored at c ^ ((row / 2) % 8) so that the 16 rows of an
// operand read at one slot hit distinct banks. Eight waves: WT along tokens,
// WO along columns, the rest split the k-steps of a stage; they run
// v_mfma_f32_32x32x16_bf16 with tokens as A rows and output columns as B rows;
// the operand reads are inline so the compiler adds no wait for the direct
// loads still in flight.
//
// Every workgroup takes in (TOK + N) model rows, and the host picks the tile by
// rounds of workgroups times intake, which orders the tiles' times. It is no
// constant bound: by the times below the intake is 13.7 TB/s over the chip at 4096
// tokens, 11.6, 10.1 and 8.3 TB/s at 32768. What limits the short launches is not
// one unit: at 4096 tokens the matrix cores are busy 11% of the cycles, the vector
// units 20, LDS 13 (no bank conflict), the L2s serve 12.4 TB/s with 85% hits, and
// a wave waits 39% of its time. Against 128 tokens x 2 d_idx columns in 32-column
// stages for every length, d_model 4096, d_idx 128, x and W in the caches from the
// call before: 4096 tokens (32 x 128 tiles) 91.6 -> 24.7 us, 8192 (64 x 128) 92.4 ->
// 34.8, 16384 (128 x 128) 94.5 -> 53.1, 32768 (128 x 256) 111.7 -> 97.4; d_idx 256
// (64 tokens x 512, register staged before): 4096 119 -> 38, 32768 271 -> 176. In a
// layer step, where other stages have used the caches, 32768 tokens take 130 us by
// either kernel.
constexpr int kRK = 64;         // model columns per stage
constexpr int kRW = 8;          // waves
constexpr int kProjBufferDword3 = 0x00020000;   // raw buffer resource: 32-bit data format

template <int DI, int TOK, int PARTS>
struct RingLayout {
  static constexpr int N = PARTS == 1 ? 2 * DI : DI;   // output columns
  static constexpr int SLOTS = kRK / 8;                // 16-byte slots per row
  static constexpr int RB = SLOTS * 16;                // row bytes (128)
  static constexpr int CH = (TOK + N) * RB / 1024;     // 1 KiB direct loads per stage
  static constexpr int CPW = (CH + kRW - 1) / kRW;     // per wave, one less past the EXTRA first
  static constexpr int EXTRA = CH % kRW;
  static constexpr int STAGE = (TOK + N) * RB;
  static constexpr int NS = 152 * 1024 / STAGE < 7 ? 152 * 1024 / STAGE : 7;
  // wave grid: 64x64 wave tiles where the tile has them, else 32-row sides
  static constexpr int WT = TOK >= 64 ? 2 : 1;
  static constexpr int WO = N / 32 < kRW / WT ? N / 32 : kRW / WT;
  static constexpr int WK = kRW / (WT * WO);           // k-steps of a stage split WK ways
  static constexpr int BT = TOK / WT / 32, BO = N / WO / 32;   // 32x32 blocks per wave
  static constexpr int KS = kRK / 16 / WK;             // k-steps per wave and stage
  static constexpr int CSTRIDE = N + 4;                // floats per token row of the C tile
  static constexpr int CBYTES = TOK * CSTRIDE * 4;
  static constexpr int LDS = NS * STAGE > CBYTES ? NS * STAGE : CBYTES;
  static_assert(TOK % 8 == 0 && DI % 8 == 0, "a chunk is rows of one array");
  static_assert(NS >= 3 && KS >= 1 && LDS <= 160 * 1024, "fits the LDS of a CU");
  static_assert((NS - 2) * CPW < 64, "vmcnt is six bits");
};

// vmcnt(n) alone (expcnt and lgkmcnt left at their maxima)
constexpr int vm_wait_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

// Direct loads of a stage. Chunk q covers 8 rows of the stage (TOK of x, then
// the W rows); lane l writes LDS bytes [1024 q + 16 l, + 16): row 8 q + l / 8,
// whose slot l % 8 holds column slot (l % 8) ^ ((row / 2) % 8). Token rows past
// the sequence end read the last row (their outputs are not written). A lane's
// offsets are fixed but for the stage's first column.
template <int DI, int TOK, int PARTS>
struct RingDma {
  using L = RingLayout<DI, TOK, PARTS>;
  __device__ __forceinline__ static int chunk(int wave, int p) { return wave + p * kRW; }
  // chunk p of this wave exists (uniform over the wave)
  __device__ __forceinline__ static bool has(int wave, int p) {
    return L::EXTRA == 0 || p < L::CPW - 1 || wave < L::EXTRA;
  }
  __device__ __forceinline__ static void offsets(int S, int dm, int t0, int wave, int lane,
                                                 uint32_t (&off)[L::CPW]) {
#pragma unroll
    for (int p = 0; p < L::CPW; ++p) {
      const int row = chunk(wave, p) * 8 + (lane >> 3);
      const uint32_t cb = (uint32_t)((lane & 7) ^ ((row >> 1) & 7)) * 16;
      const int r = row < TOK ? min(row, S - 1 - t0) : (row - TOK) % DI;
      off[p] = (uint32_t)r * (uint32_t)dm * 2u + cb;
    }
  }
  // xt: the tile's first token row, of which xrows exist
  __device__ __forceinline__ static void issue(uint32_t stage, int it, int xrows, int dm, int part,
                                               const uint16_t *xt, const uint16_t *wq,
                                               const uint16_t *wk, int wave,
                                               const uint32_t (&off)[L::CPW]) {
    const uint32_t kb = (uint32_t)it * (kRK * 2u);
#pragma unroll
    for (int p = 0; p < L::CPW; ++p) {
      const int q = chunk(wave, p), row = q * 8;
      const bool is_x = row < TOK, is_k = PARTS == 1 ? row >= TOK + DI : part == 1;
      const uint16_t *base = is_x ? xt : is_k ? wk : wq;
      const uint32_t bytes = (uint32_t)(is_x ? xrows : DI) * (uint32_t)dm * 2u;
      const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(base), (short)0,
                                                        bytes, kProjBufferDword3);
      if (has(wave, p))
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rs, (__attribute__((address_space(3))) void *)(size_t)(stage + q * 1024), 16,
            off[p] + kb, 0, 0, 0);
    }
  }
};

template <int DI, int TOK, int PARTS>
__global__ __launch_bounds__(kRW * 64) void project_ring_kernel(
    int S, int dm, int pos0, float theta, float eps, const uint16_t *__restrict__ x,
    const uint16_t *__restrict__ wq, const uint16_t *__restrict__ wk,
    const float *__restrict__ gamma, const float *__restrict__ beta, uint16_t *__restrict__ qo,
    uint16_t *__restrict__ ko) {
  using L = RingLayout<DI, TOK, PARTS>;
  using Dma = RingDma<DI, TOK, PARTS>;
  constexpr int BT = L::BT, BO = L::BO, KS = L::KS, RB = L::RB, NS = L::NS, CPW = L::CPW;
  __shared__ __align__(16) char lds[L::LDS];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int wt = wave % L::WT, wo = (wave / L::WT) % L::WO, wks = wave / (L::WT * L::WO);
  // the two parts of a token tile are 8 workgroups apart: one XCD, whose L2
  // then holds the tile's x for the second
  const int part = PARTS == 1 ? 0 : ((int)blockIdx.x >> 3) & 1;
  const int tile = PARTS == 1 ? (int)blockIdx.x
                              : ((int)blockIdx.x >> 4) * 8 + ((int)blockIdx.x & 7);
  const int t0 = tile * TOK;
  if (t0 >= S) return;   // the whole workgroup
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) char *)&lds[0];

  uint32_t off[CPW];
  Dma::offsets(S, dm, t0, wave, lane, off);
  const uint16_t *xt = x + (size_t)t0 * dm;
  const int xrows = min(TOK, S - t0);
  auto issue = [&](int it) {
    Dma::issue(lds0 + (it % NS) * L::STAGE, it, xrows, dm, part, xt, wq, wk, wave, off);
  };
  const int nk = dm / kRK;
#pragma unroll
  for (int st = 0; st < NS - 1; ++st)
    if (st < nk) issue(st);

  f32x16 acc[BT][BO];
#pragma unroll
  for (int bt = 0; bt < BT; ++bt)
#pragma unroll
    for (int bo = 0; bo < BO; ++bo) acc[bt][bo] = f32x16{};
  // per-lane LDS offsets within a stage: A rows (tokens), B rows (columns);
  // row bases are multiples of 32, so a lane's swizzle is (n / 2) % 8, and
  // k-step ks reads column slot 2 ks + h
  const uint32_t xrow = (uint32_t)(wt * BT * 32 + n) * RB;
  const uint32_t wrow = (uint32_t)(TOK + wo * BO * 32 + n) * RB;
  uint32_t kso[KS];
#pragma unroll
  for (int i = 0; i < KS; ++i)
    kso[i] = (uint32_t)((2 * (wks * KS + i) + h) ^ ((n >> 1) & 7)) * 16;
  for (int it = 0; it < nk; ++it) {
    // this wave's loads of stage it have landed (later stages may still fly)
    if (it + NS - 2 >= nk)
      __builtin_amdgcn_s_waitcnt(vm_wait_imm(0));
    else if (Dma::has(wave, CPW - 1))
      __builtin_amdgcn_s_waitcnt(vm_wait_imm((NS - 2) * CPW));
    else
      __builtin_amdgcn_s_waitcnt(vm_wait_imm((NS - 2) * (CPW - 1)));
    // every wave's loads of stage it have landed and stage it - 1 is fully
    // read (each wave waited for its own reads before its products): a bare
    // barrier, as the fence of a full one would also wait for the loads of
    // the later stages
    __builtin_amdgcn_s_barrier();
    if (it + NS - 1 < nk) issue(it + NS - 1);
    const uint32_t sbase = lds0 + (it % NS) * L::STAGE;
    bf16x8 fa[KS][BT], fb[KS][BO];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uint32_t xa = sbase + xrow + kso[ks], wa = sbase + wrow + kso[ks];
#pragma unroll
      for (int bt = 0; bt < BT; ++bt)
        asm volatile("ds_read_b128 %0, %1 offset:%2"
                     : "=v"(fa[ks][bt])
                     : "v"(xa), "i"(bt * 32 * RB));
#pragma unroll
      for (int bo = 0; bo < BO; ++bo)
        asm volatile("ds_read_b128 %0, %1 offset:%2"
                     : "=v"(fb[ks][bo])
                     : "v"(wa), "i"(bo * 32 * RB));
    }
    static_for<0, KS>([&](auto I) {
      // reads complete in order: k-step ks needs all but the later k-steps' reads
      constexpr int ks = decltype(I)::value;
      asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(fa[ks][0]) : "i"((KS - 1 - ks) * (BT + BO)));
#pragma unroll
      for (int bt = 1; bt < BT; ++bt) asm volatile("" : "+v"(fa[ks][bt]));
#pragma unroll
      for (int bo = 0; bo < BO; ++bo) asm volatile("" : "+v"(fb[ks][bo]));
#pragma unroll
      for (int bt = 0; bt < BT; ++bt)
#pragma unroll
        for (int bo = 0; bo < BO; ++bo) acc[bt][bo] = mfma32(fa[ks][bt], fb[ks][bo], acc[bt][bo]);
    });
  }
  __builtin_amdgcn_s_waitcnt(vm_wait_imm(0));
  __syncthreads();   // the ring is free: park C (token-major, fp32), the k-shares in order
  float *cl = reinterpret_cast<float *>(lds);
#pragma unroll
  for (int w = 0; w < L::WK; ++w) {
    if (wks == w) {
#pragma unroll
      for (int bt = 0; bt < BT; ++bt)
#pragma unroll
        for (int bo = 0; bo < BO; ++bo)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int tl = (wt * BT + bt) * 32 + 8 * (e >> 2) + 4 * h + (e & 3);
            float *c = cl + tl * L::CSTRIDE + (wo * BO + bo) * 32 + n;
            *c = w ? *c + acc[bt][bo][e] : acc[bt][bo][e];
          }
    }
    __syncthreads();
  }
  project_epilogue<DI, TOK, kRW, PARTS>(cl, L::CSTRIDE, S, t0, pos0, theta, eps, gamma, beta, qo,
                                        ko, part, wave, lane);
}

struct ProjArgs {
  int S, dm, pos0;
  float theta, eps;
  const uint16_t *x, *wq, *wk;
  const float *gamma, *beta;
  uint16_t *qo, *ko;
  hipStream_t st;
};

// Model rows a CU takes in with this tile: rounds of workgroups (one per CU
// at a time) times rows per workgroup.
template <int DI, int TOK, int PARTS>
int64_t ring_intake(int S) {
  constexpr int kCus = 256;
  const int64_t wgs = ((int64_t)S + TOK - 1) / TOK * PARTS;
  return (wgs + kCus - 1) / kCus * (TOK + RingLayout<DI, TOK, PARTS>::N);
}

template <int DI, int TOK, int PARTS>
hipError_t launch_ring(const ProjArgs &a) {
  const int tiles = (a.S + TOK - 1) / TOK;
  const int grid = PARTS == 1 ? tiles : (tiles + 7) / 8 * 16;
  hipLaunchKernelGGL((project_ring_kernel<DI, TOK, PARTS>), dim3(grid), dim3(kRW * 64), 0, a.st,
                     a.S, a.dm, a.pos0, a.theta, a.eps, a.x, a.wq, a.wk, a.gamma, a.beta, a.qo,
                     a.ko);
  return hipGetLastError();
}

// The tile of least intake, the larger one on a tie.
template <int DI>
hipError_t launch_tile(const ProjArgs &a) {
  if constexpr (DI == 256) {
    const int64_t c128 = ring_intake<DI, 128, 2>(a.S), c64 = ring_intake<DI, 64, 2>(a.S),
                  c32 = ring_intake<DI, 32, 2>(a.S);
    if (c128 <= c64 && c128 <= c32) return launch_ring<DI, 128, 2>(a);
    if (c64 <= c32) return launch_ring<DI, 64, 2>(a);
    return launch_ring<DI, 32, 2>(a);
  } else {
    const int64_t c1 = ring_intake<DI, 128, 1>(a.S), c128 = ring_intake<DI, 128, 2>(a.S),
                  c64 = ring_intake<DI, 64, 2>(a.S), c32 = ring_intake<DI, 32, 2>(a.S);
    if (c1 <= c128 && c1 <= c64 && c1 <= c32) return launch_ring<DI, 128, 1>(a);
    if (c128 <= c64 && c128 <= c32) return launch_ring<DI, 128, 2>(a);
    if (c64 <= c32) return launch_ring<DI, 64, 2>(a);
    return launch_ring<DI, 32, 2>(a);
  }
}

template <int DI>
hipError_t launch_di(const ProjArgs &a) {
  // the ring kernel's offsets within a weight matrix and a tile are 32-bit
  constexpr int kRows = DI < 128 ? 128 : DI;
  if ((uint64_t)kRows * (uint64_t)a.dm * 2u < (1ull << 32)) return launch_tile<DI>(a);
  hipLaunchKernelGGL((project_kernel<DI>), dim3((a.S + kPT - 1) / kPT), dim3(kPW * 64), 0, a.st,
                     a.S, a.dm, a.pos0, a.theta, a.eps, a.x, a.wq, a.wk, a.gamma, a.beta, a.qo,
                     a.ko);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_indexer_project(int S, int di, int dm, int pos0, float theta, float eps,
                                  const void *x, const void *wq, const void *wk,
                                  const float *gamma, const float *beta, void *qo, void *ko,
                                  hipStream_t st) {
  const ProjArgs a{S,  dm,    pos0, theta,          eps,            (const uint16_t *)x,
                   (const uint16_t *)wq, (const uint16_t *)wk, gamma, beta, (uint16_t *)qo,
                   (uint16_t *)ko, st};
  if (di == 64) return launch_di<64>(a);
  if (di == 128) return launch_di<128>(a);
  return launch_di<256>(a);
}

}  // namespace sp
