// Which fp32 attention kernel a launch takes, and in which shape: plain host code.
#pragma once
#include <cmath>

namespace amskv {

// waves of a workgroup of the kernel in attend_f32.hip
constexpr int waves_of(int split) { return split == 8 ? 8 : 4; }

// Which variant: the one with the least modelled time.  A workgroup serves one (b,h), so a launch has as many of them per (b,h) as
// its query blocks fill, and they go to the CUs in rounds of what fits there (LDS).  A round takes a start, and per key block
// that a wave walks either the latency of one block's chain or, with more waves on a SIMD, what the matrix pipe needs for
// all of theirs, whichever is longer (a wave without query rows counts too: it fetches and waits at the barriers).  us, fitted to the
// eight variants on 1600 shapes (1 to 4096 (b,h), 1 to 2500 queries, 1 to 6000 keys): the choice loses 0.5 % against the best
// of the eight on average and 21 % at most.  (Counted as though several (b,h) shared a workgroup it lost 4.4 % and 92 %: 4096 (b,h), 64
// x 65 keys 134 us against 75.)
struct F32Cost {
  double base, start, start_split, latency, work;
  int resident;  // workgroups of four waves on a CU
};
struct F32Choice {
  int qt, split;
  int parts;  // > 0: the kernel of attend_f32_parts.hip, with that many waves of 32 query rows
};
// attend_f32_parts.hip, per key block: `latency` at least, or `per` and `work` for each active wave on a SIMD; a round that leaves CUs
// without a workgroup is faster by up to `idle` (the clock is higher)
struct F32PartsCost {
  int rows, split, resident;
  double base, start, latency, per, work, idle;
};
inline F32Choice choose_f32(int head_dim, long long bh, int t_q, int t_kv, float softmax_scale) {
  static const F32Cost rows16{2.2, 0.55, 2.0, 1.5, 0.65, 4}, rows32{1.55, 2.45, 5.5, 2.65, 2.2, 2}, rows16_d128{1.1, 1.1, 4.6, 2.05, 1.5, 2};
  F32Choice best{16, 1, 0};
  double least = 1e300;
  for (int qt = head_dim == 64 ? 32 : 16; qt >= 16; qt /= 2)
    for (int split = 1; split <= 8; split *= 2) {
      // (four 16-row units to a workgroup that do not split keys: one workgroup per (b,h) at head dim 64.  With more query rows the other
      // kernel or a split was the faster one in each of 3 million shapes: 1 to 60000 (b,h), 1 to 8192 queries, up to 20000 more keys.)
      if (head_dim == 64 && split == 1 && (qt == 32 || t_q > 64)) continue;
      const F32Cost& c = head_dim == 128 ? rows16_d128 : qt == 32 ? rows32 : rows16;
      const int waves = waves_of(split), units = waves / split, blocks = (t_kv + qt - 1) / qt;
      const long long groups = bh * (((t_q + qt - 1) / qt + units - 1) / units);
      const int resident = c.resident * 4 / waves, walk = (blocks + split - 1) / split;
      auto round = [&](long long n) {
        return (split == 1 ? c.start : c.start_split) + walk * std::fmax(c.latency, (double)(n * waves / 4) * c.work);
      };
      const long long per_round = 256LL * resident, rest = groups % per_round;
      const double t = c.base + (double)(groups / per_round) * round(resident) + (rest ? round((rest + 255) / 256) : 0.0);
      if (t < least) {
        least = t;
        best = F32Choice{qt, split, 0};
      }
    }
  // (a wave of the other kernel holds 32 queries, and below 128 of them it has never won)
  if (t_q <= 32 || bh * ((t_q + 31) / 32) < 128) return best;
  // (its scores are exact to 2^-67 beside their roundings, which a scale this large would bring up)
  if (softmax_scale > 0x1p30f) return best;
  // The kernel of bf16 parts, where it is modelled to be the faster one: roughly from 500 blocks of 32 queries on.  (The 16-row variants
  // take 1.15 of their model there, which the margin makes up for in part.)  Fitted to 2000 shapes (8 to 4096 (b,h), 33 to 2500 queries,
  // 33 to 6000 keys): the choice takes 1.007 of the best of all variants on average at head dim 64, 1.001 at 128, and 1.03 and 1.04 of what
  // it takes without this kernel at most.  256 (b,h), us, without / with: 64 x 155 14.6 / 12.0, 100 x 255 30 / 19, 256 x 680 110 / 65.
  static const F32PartsCost parts64[] = {{8, 1, 1, 0.32, 4.15, 0.1, 0.87, 0.88, 0.17}, {4, 1, 2, 0.97, 4.48, 1.58, 1.09, 0.77, 0.33},
                                      {4, 2, 1, 0.0, 7.12, 0.81, 1.51, 0.57, 0.27}};
  static const F32PartsCost parts128{4, 1, 1, 0.0, 9.0, 2.93, 0.0, 3.12, 0.1};
  least *= head_dim == 64 && best.qt == 16 ? 1.05 : 0.95;
  for (int i = 0; i < (head_dim == 64 ? 3 : 1); ++i) {
    const F32PartsCost& c = head_dim == 64 ? parts64[i] : parts128;
    const int q_blocks = (t_q + 31) / 32, tiles = (q_blocks + c.rows - 1) / c.rows, walk = ((t_kv + 31) / 32 + c.split - 1) / c.split;
    const double on_simd = (double)q_blocks / tiles * c.split / 4;  // active waves of a workgroup
    auto round = [&](long long n, double busy) {
      return (c.start + walk * std::fmax(c.latency, c.per + (double)n * on_simd * c.work)) * (1 - c.idle * (1 - busy));
    };
    const long long groups = bh * tiles, per_round = 256LL * c.resident, rest = groups % per_round;
    const double t = c.base + (double)(groups / per_round) * round(c.resident, 1.0) +
                     (rest ? round((rest + 255) / 256, std::fmin(1.0, (double)rest / 256)) : 0.0);
    if (t < least) {
      least = t;
      best = F32Choice{32, c.split, c.rows};
    }
  }
  return best;
}

}  // namespace amskv
