// Which attention kernel serves a problem, by estimates of their times: rules of
// sizes alone, host code that needs no device (a test calls them).
#pragma once

#include "kernels.hpp"

namespace sp {

// Whether one workgroup's key tiles, and not the even share of all of them
// over the CUs, set the length of the launch: the longest workgroup takes
// S / 64 steps, the average one about (qo + S) / 128. A split step serves as
// many query rows times keys as an unsplit one but loads twice the tile bytes
// (about 1.4 times the time), so the longest has to be 1.6 times the share.
// Split against unsplit, 32/8 heads, d = 128: 1024 queries of 8192 keys
// (ratio 2.1) 215 / 307 us, 2048 tokens (2.0) 44 / 50, 4096 at 16/4 heads (2.0) 76
// / 94; past the line 3072 tokens (1.3) 92 / 82, 4000 (1.0) 144 / 121, 4096 rows of
// 8192 (1.0) 659 / 619, though 2048 of 4096 (1.3) 172 / 185.
inline bool few_workgroups(const Prob &p, int TQ) {
  constexpr int kCus = 256;
  const int64_t wgs = (int64_t)((p.nq + TQ - 1) / TQ) * p.Hkv;
  return 8 * wgs * ((int64_t)p.qo + p.S) < 5 * 2 * (int64_t)kCus * p.S;
}

// What the two kernels of per-query supports take, in us, fitted to their times
// over sequences of 1K to 32K tokens and their last 1K rows, k 64 to 2048, 1 to 16
// heads a group.
struct SparseRates {
  double row;     // gather: per selected row and KV head
  double query;   // ... per query and KV head, with its support row's copy to LDS
  double step;    // masked: a 64-key step of 256 query rows (128 at d = 256)
  double fill;    // ... its masks, per support entry and CU of a segment of the keys
};
constexpr double kSplitStep = 1.3;   // a split step of half the rows against a whole one

inline SparseRates sparse_rates(const Prob &p) {
  const double pieces = (p.k + 511) / 512;   // the support row is copied 512 entries at a time
  if (p.d == 64) return {12e-6, 0.7e-3 + 0.15e-3 * pieces, 1.55, 0.35e-3};
  if (p.d == 128) return {24e-6, 1.3e-3 + 0.2e-3 * pieces, 2.1, 0.35e-3};
  return {73e-6, 2.0e-3 + 0.3e-3 * pieces, 2.8, 0.35e-3};
}

// The masked kernel's workgroups: query rows, whether they split the keys, and
// bytes of LDS for the masks.
struct MaskShape {
  int rows, bits;
  bool split;
  int tq(const Prob &p) const { return rows / p.G; }
  // key tiles of a segment: the most whose masks fit, a power of two
  int seg_tiles(const Prob &p) const {
    int n = 2;
    while (2 * n * 8 * tq(p) <= bits) n *= 2;
    return n;
  }
};
inline MaskShape mask_shape(const Prob &p) {
  const int rows = p.d == 256 ? 128 : 256;
  const bool split = p.d != 256 && few_workgroups(p, rows / p.G);
  return {split ? 128 : rows, p.d == 64 || (p.d == 128 && !split) ? 64 * 1024 : 24 * 1024, split};
}

// Whether masked tiles serve a problem of per-query supports sooner than the
// gather. The masked kernel takes its steps as long as its longest workgroup or
// the even share of all of them, and reads every support entry once a segment
// of its keys, on no more CUs than it has workgroups. The factor keeps what was
// measured slower out; a paged cache, whose masked steps are up to 1.25 times
// as long, has the same line. Gathered / masked, us: 4096 tokens, 16/4 heads, d = 128,
// k = 512: 246 / 101; 8192, 32/8, k = 1024: 1512 / 594; 32768, 32/8, k = 2048: 15.7
// / 9.5 ms; on the other side 1024 rows at 15360, 32/8, k = 1024: 226 / 326; 8192
// tokens at 16/2 heads, k = 512: 242 / 293; 2048 at 32/8, k = 64: 46 / 51; 1024 rows
// at 3072, 8/8 heads, k = 1024: 219 / 299.
inline bool sparse_mask_pays(const Prob &p) {
  constexpr double kCus = 256;
  const double S = p.S, qo = p.qo, nq = p.nq, k = p.k, Hkv = p.Hkv;
  const double cut = k < qo ? 0 : (k < S ? k : S) - qo;   // rows that see fewer than k keys
  const double entries = nq * k - cut * (k - qo - 0.5 * cut);
  const SparseRates r = sparse_rates(p);
  const MaskShape m = mask_shape(p);
  const int TQ = m.tq(p);
  // (a workgroup counts its support entries, eight at a time, in 32 bits)
  if ((int64_t)TQ * (((int64_t)p.k + 7) / 8) > (1 << 30)) return false;
  const double gather = Hkv * (entries * r.row + nq * r.query);
  const double longest = (S + 63) / 64, mean = (qo + S) / 128;
  const double wgs = ((p.nq + TQ - 1) / TQ) * Hkv;
  const double share = wgs * mean / kCus;
  const double steps = (longest > share ? longest : share) * (m.split ? 0.5 * kSplitStep : 1.0);
  const double segs = 0.5 + mean / m.seg_tiles(p) > 1 ? 0.5 + mean / m.seg_tiles(p) : 1;
  const double masked =
      steps * r.step + r.fill * entries * Hkv * segs / (wgs < kCus ? wgs : kCus);
  return 1.15 * masked < gather;
}

}  // namespace sp
