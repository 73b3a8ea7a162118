// fp32 per-scale attention (Section 3.1) on the bf16 matrix pipe, for launches with work enough to be bound by it: every
// operand goes in as three bf16 parts (x = hi + mid + lo, each the rounded rest of the ones before: 24 bits, and bf16 has
// fp32's range), and a product is six of theirs -- lo*hi, hi*lo, mid*mid, mid*hi, hi*mid, hi*hi; what is left out is below
// 2^-24 of it.  Sums stay in fp32, probabilities are formed in fp32 and split like the inputs.
//
// Why: v_mfma_f32_32x32x16_bf16 has 16 times the rate of v_mfma_f32_32x32x2_f32, and it adds eight products exactly before it rounds
// its accumulator (to nearest): faster, and closer to the exact sums.  Against the kernel of attend_f32.hip in the form that took these
// launches before, us in a long run of launches (rel error against 64 bits): 256 (b,h), 256 x 680 110 -> 65 (4.8e-7 -> 2.0e-7), 169 x 424
// 64 -> 38 (3.9 -> 1.7e-7), 100 x 255 30 -> 19 (2.0 -> 1.3e-7); 64 (b,h), 1024 x 2645 389 -> 219 (9.3 -> 3.6e-7); head dim 128, 256 (b,h), 256 x 680
// 221 -> 151 (4.9 -> 2.0e-7), 32 (b,h), 1024 x 1621 256 -> 159 (7.4 -> 3.0e-7).  (The first few launches after a pause, and those between
// smaller ones in a pass, take a tenth more: 256 x 680 73.)  One accumulator for all of a score's large products is 4 % faster, and less
// exact than that kernel where one channel outweighs the others (1.6e-6 for 1.5e-6; as it is 1.1e-6).
// What bounds it at the large sizes is the matrix pipe next to the power limit: busy 51 % of the SIMD cycles at 256 x 680 and 59 % at 1024 x
// 2645, at 1.8 GHz (1.05 and 1.2 PFLOP/s of bf16 products; a loop of nothing but these instructions on random data runs at 1.6 PFLOP/s
// and 1.6 GHz), vector ALUs 44 and 47 %.  A second tile in flight and a raised wave priority for half of the waves changed nothing (+-2 %).
//
// Work.  A workgroup has kRowWaves * kSplit waves: kRowWaves of them hold 32 query rows of one (b,h) each, kSplit of them share a
// row group and take the blocks of a tile (kSplit * 32 keys) in turn, with softmax statistics of their own that meet in LDS at the end.
// Transposed formulation as everywhere (S^T = K Q^T, O^T += V^T P^T: a lane holds 16 keys of one query, its probabilities already are
// the second product's B operand).  Per block: the score products of block b next to the splitting of tile t + 1, then the second
// product of block b - 1 next to the softmax of block b.
//
// Memory.  K and V rows come through registers (a tile ahead, an even share per wave): the split is done once per workgroup, and
// stores of the current scale's rows (fused append) take them from there.  The parts go to a ring of three tiles in LDS -- being
// filled, in use, and the one whose V is still multiplied -- one barrier per tile; swizzle and transposing reads as in the streaming
// bf16 kernel, on each part.
//
// Large numbers.  From 2^59 on the products of parts of Q and K may overflow; every lane keeps the largest magnitude of theirs that it
// has split.  In V a magnitude from 2^95 on, scaled (below), or a sum that overflows, leaves sums in O that are not finite, in all rows.  A
// workgroup that sees either does its work again on the fp32 matrix instructions, which give such inputs, infinities too, what the
// formula has.  (256 (b,h), 256 x 680, such a value in each: 196 us instead of 65.  A maximum over V too, beside the scaling: 0.4 %
// of a stack of layers on 16 images.)
// Small numbers.  bf16 has subnormals, in steps of 2^-133, and the matrix cores take them: a part is off by 2^-134 at most.  V is split
// scaled, which keeps all bits of every normal number.  In a score that error, times 2^59 and 2 D, is below 2^-66, nothing next to
// the rounding of the exponential unless the softmax scale is huge (the dispatch leaves those to attend_f32.hip).  In a probability it is
// less than what every kernel here loses where the exponential falls below 2^-126, which the instruction gives as 0.
#include "amskv_internal.hpp"

namespace amskv {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// lag of the softmax reference and the sum that has it looked at again: as in attend_f32.hip
constexpr float kMaxLag = 6.0f;
constexpr float kTripSum = 1024.0f;
// Q and K lie below this: no product of parts, and no sum of them, comes near fp32's largest number.  (Products of parts have either
// sign: where they overflow, a score that is -inf, or finite, would be the sum of two opposite infinities.)
constexpr float kLarge = 0x1p59f;
// V is split times this, and O divided by it: bf16 goes down in steps of 2^-133, so that the parts of a number below 2^-109 would be short
// of bits.
constexpr float kScaleV = 0x1p32f;

#define AMSKV_LDS __attribute__((address_space(3)))
__device__ __forceinline__ bf16x4 lds_read_tr16(const char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((AMSKV_LDS bf16x4*)(p));
}
template <int D>
__device__ __forceinline__ constexpr int swizzle(int row) {
  return D == 64 ? (row & 7) : (((row & 3) << 1) | ((row >> 2) & 1) | (row & 8));
}
__device__ __forceinline__ unsigned pack(float a, float b) {
  bf16x2 x;
  x[0] = (__bf16)a;
  x[1] = (__bf16)b;
  unsigned w = __builtin_bit_cast(unsigned, x);
  asm("" : "+v"(w));  // (the compiler would round the lower one a second time rather than shift the pair)
  return w;
}
__device__ __forceinline__ float low(unsigned w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float high(unsigned w) { return __uint_as_float(w & 0xffff0000u); }
// a pair of numbers as three bf16 parts each
__device__ __forceinline__ void split2(float a, float b, unsigned& hi, unsigned& mid, unsigned& lo) {
  hi = pack(a, b);
  a -= low(hi);
  b -= high(hi);
  mid = pack(a, b);
  a -= low(mid);
  b -= high(mid);
  lo = pack(a, b);
}
__device__ __forceinline__ float max3_abs(float m, float a, float b) {
  asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(a), "v"(b));
  return m;
}
constexpr int kRing = 3;
constexpr int kMostWhole = 0;  // left-over (b,h) always in equal shares (place()): 0.98 to 1.02 of the time of whole ones up to 32 workgroups an XCD, 48 0.76 to 0.61
constexpr int lds_bytes(int D, int split) { return kRing * split * 6 * 32 * D * 2; }

// what a launch's workgroups have in common
struct Call {
  const float* q;
  float* o;
  char *kc, *vc;
  int t_q;
  long long cap_tokens;
  float scale_log2e;
  int n_qtiles;
};

// Rows of K~ and V~ on their way from memory to LDS: a tile at a time through registers, a share per wave.
template <int D, int kWaves, int kSplit>
struct Stage {
  static constexpr int RB = D * 4, CPR = D / 4;  // bytes and 16-byte pieces of a row
  static constexpr int TK = 32 * kSplit, kRowsPerLoad = 64 / CPR;
  static constexpr int kLoads = TK / kRowsPerLoad / kWaves;  // per wave and tensor
  static_assert(kLoads >= 1 && kLoads * kRowsPerLoad * kWaves == TK, "the waves share a tile evenly");
  const SegTable& seg;
  const ExtKV& ext_kv;
  char *kb, *vb;
  const char *xk, *xv;
  long long x_tok;
  int wave, row0, pos, t_kv, n_qtiles, q_tile;
  int seg_end = 0, seg_delta = 0;
  bool write_back;
  f32x4 raw[2][kLoads];  // K and V
  __device__ __forceinline__ Stage(const Call& call, const SegTable& seg, const ExtKV& ext_kv, const CallerIo& io, long long bh, int q_tile)
      : seg(seg), ext_kv(ext_kv), q_tile(q_tile) {
    const long long x_unit = unit_offset(io.kv, bh, io.heads);  // borrowed current scale, if any
    kb = call.kc + bh * call.cap_tokens * RB;
    vb = call.vc + bh * call.cap_tokens * RB;
    xk = (const char*)ext_kv.k + x_unit;
    xv = (const char*)ext_kv.v + x_unit;
    x_tok = io.kv.tok;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    row0 = (threadIdx.x & 63) / CPR;
    pos = (threadIdx.x & 63) % CPR;
    t_kv = seg.total;
    n_qtiles = call.n_qtiles;
    write_back = writes_back(ext_kv, seg.total, seg.ext_start);
  }
  __device__ __forceinline__ int row(int k) const { return (k * kWaves + wave) * kRowsPerLoad + row0; }  // of load k, in the tile
  __device__ __forceinline__ void fetch(int tile) {
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
      const int j0 = tile * TK + (k * kWaves + wave) * kRowsPerLoad;
      if (__builtin_expect(j0 >= seg_end && j0 < t_kv, 0)) {
        seg_end = seg.virt_start[0] + seg.len[0], seg_delta = seg.phys_off[0] - seg.virt_start[0];
        for (int i = 1; i < seg.n; ++i)
          if (j0 >= seg.virt_start[i]) {
            seg_end = seg.virt_start[i] + seg.len[i];
            seg_delta = seg.phys_off[i] - seg.virt_start[i];
          }
        if (j0 >= seg.ext_start) {
          seg_end = t_kv;
          seg_delta = -seg.ext_start;
        }
      }
      const bool in_ext = j0 >= seg.ext_start;
      const long long st = in_ext ? x_tok : (long long)RB;
      if (__builtin_expect(j0 + kRowsPerLoad <= seg_end && st < (1ll << 24), 1)) {
        const long long at = (long long)(j0 + seg_delta) * st;
        const unsigned off = row0 * (unsigned)st + 16 * pos;
        raw[0][k] = *reinterpret_cast<const f32x4*>((in_ext ? xk : kb) + at + off);
        raw[1][k] = *reinterpret_cast<const f32x4*>((in_ext ? xv : vb) + at + off);
      } else {
        bool ext;
        const long long at = locate_row(seg, min(j0 + row0, t_kv - 1), ext);
        raw[0][k] = *reinterpret_cast<const f32x4*>((ext ? xk + at * x_tok : kb + at * RB) + 16 * pos);
        raw[1][k] = *reinterpret_cast<const f32x4*>((ext ? xv + at * x_tok : vb + at * RB) + 16 * pos);
      }
    }
  }
  // what is rare about a tile in the registers: rows of the current scale to store, rows past the end to clear
  __device__ __forceinline__ void touch_up(int tile) {
    const bool ends = (tile + 1) * TK > t_kv;
    const bool mine = write_back && (tile + 1) * TK > seg.ext_start && tile % n_qtiles == q_tile;
    if (__builtin_expect(!(ends || mine), 1)) return;
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
      const int j = tile * TK + row(k);
      if (mine) {
        const int to = write_back_row(ext_kv, j, t_kv, seg.ext_start);
        if (j >= seg.ext_start && to >= 0) {
          *reinterpret_cast<f32x4*>(kb + (long long)to * RB + 16 * pos) = raw[0][k];
          *reinterpret_cast<f32x4*>(vb + (long long)to * RB + 16 * pos) = raw[1][k];
        }
      }
      if (j >= t_kv) raw[0][k] = raw[1][k] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
};

// The same sums on the fp32 matrix instructions, for a workgroup that has met a number that its parts cannot stand for.  Waves of the first slice compute, all of them fetch.
template <int D, int kRowWaves, int kSplit>
__device__ __forceinline__ void attend_unit_wide(const Call& call, const SegTable& seg, const ExtKV& ext_kv, const CallerIo& io,
                                                 long long bh, int q_tile, char* lds) {
  constexpr int kWaves = kRowWaves * kSplit, DB = D / 32, kRow = D + 4;  // floats of a row in LDS
  Stage<D, kWaves, kSplit> stage(call, seg, ext_kv, io, bh, q_tile);
  const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
  const int q_base = (q_tile * kRowWaves + stage.wave) * 32, t_kv = seg.total;
  const bool active = stage.wave < kRowWaves && q_base < call.t_q;
  const int n_tiles = (t_kv + stage.TK - 1) / stage.TK;
  float* fk = reinterpret_cast<float*>(lds);
  float* fv = fk + stage.TK * kRow;
  static_assert(2 * 32 * kSplit * kRow * 4 <= lds_bytes(D, kSplit), "the tile fits");
  const char* q_row = (const char*)call.q + unit_offset(io.q, bh, io.heads) + (long long)min(q_base + r, call.t_q - 1) * io.q.tok;
  f32x16 oacc[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int v = 0; v < 16; ++v) oacc[d][v] = 0.f;
  float run_ref = -INFINITY, run_sum = 0.f;
  for (int t = 0; t < n_tiles; ++t) {
    stage.fetch(t);
    stage.touch_up(t);
#pragma unroll
    for (int k = 0; k < stage.kLoads; ++k) {
      *reinterpret_cast<f32x4*>(fk + stage.row(k) * kRow + 4 * stage.pos) = stage.raw[0][k];
      *reinterpret_cast<f32x4*>(fv + stage.row(k) * kRow + 4 * stage.pos) = stage.raw[1][k];
    }
    __syncthreads();
    for (int b = 0; b < kSplit && active && t * stage.TK + 32 * b < t_kv; ++b) {
      const float* bk = fk + 32 * b * kRow;
      const float* bv = fv + 32 * b * kRow;
      f32x16 s;
#pragma unroll
      for (int v = 0; v < 16; ++v) s[v] = 0.f;
      for (int i = 0; i < D / 2; i += 4) {  // lane half h: channels D/2 * h ..; a partial sum takes eight products
        const f32x4 a = *reinterpret_cast<const f32x4*>(bk + r * kRow + D / 2 * h + i);
        const f32x4 b = *reinterpret_cast<const f32x4*>(q_row + 4 * (D / 2 * h + i));
        f32x16 part;
#pragma unroll
        for (int v = 0; v < 16; ++v) part[v] = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) part = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], part, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] += part[v];
      }
      float mx = -INFINITY;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        if (t * stage.TK + 32 * b + 8 * (v >> 2) + 4 * h + (v & 3) >= t_kv) s[v] = -INFINITY;
        mx = fmaxf(mx, s[v]);
      }
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const bool move = mx > run_ref;
      const float alpha = move ? __builtin_amdgcn_exp2f((run_ref - mx) * call.scale_log2e) : 1.f;
      if (move) run_ref = mx;
      const float ref = run_ref == -INFINITY ? 0.f : run_ref;  // no reference yet: every score so far is -inf and weighs 0
      float sum = 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        s[v] = __builtin_amdgcn_exp2f((s[v] - ref) * call.scale_log2e);
        sum += s[v];
      }
      run_sum = run_sum * alpha + sum;
#pragma unroll
      for (int d = 0; d < DB; ++d) {
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[d][v] *= alpha;
#pragma unroll
        for (int v = 0; v < 16; ++v)
          oacc[d] = __builtin_amdgcn_mfma_f32_32x32x2f32(bv[(8 * (v >> 2) + 4 * h + (v & 3)) * kRow + 32 * d + r], s[v], oacc[d], 0, 0, 0);
      }
    }
    __syncthreads();
  }
  const float inv = 1.0f / (run_sum + __shfl_xor(run_sum, 32, 64));
  if (!active || q_base + r >= call.t_q) return;
  char* o_row = (char*)call.o + unit_offset(io.o, bh, io.heads) + (long long)(q_base + r) * io.o.tok;
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      f32x4 x;
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = oacc[d][4 * c + e] * inv;
      *reinterpret_cast<f32x4*>(o_row + 4 * (32 * d + 8 * c + 4 * h)) = x;
    }
}

template <int D, int kRowWaves, int kSplit>
__device__ __forceinline__ bool attend_unit(const Call& call, const SegTable& seg, const ExtKV& ext_kv, const CallerIo& io, long long bh,
                                            int q_tile, char* lds, float2 (*stat)[32], int* wide_flag) {
  constexpr int kWaves = kRowWaves * kSplit;
  constexpr int KS = D / 16, DB = D / 32;
  constexpr int PB = D * 2;                  // bytes of a row, one part
  constexpr int kPart = 32 * PB;             // one part of a 32-key block
  constexpr int kTensor = 3 * kPart, kBlk = 2 * kTensor, kTile = kSplit * kBlk;
  constexpr int TK = 32 * kSplit;
  constexpr int CPR = D / 4;                 // 16-byte pieces of an fp32 row
  constexpr int kRowsPerLoad = 64 / CPR;
  constexpr int kLoads = TK / kRowsPerLoad / kWaves;  // per wave and tensor
  static_assert(kLoads >= 1 && kLoads * kRowsPerLoad * kWaves == TK, "the waves share a tile evenly");
  constexpr bool kAllOfK = kLoads == 1 || D == 128;  // registers for the K parts of both steps of a pair of sums at once

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int r = lane & 31, h = lane >> 5;
  const int slice = kSplit == 1 ? 0 : wave / kRowWaves;
  const int t_q = call.t_q, n_qtiles = call.n_qtiles;
  const float scale_log2e = call.scale_log2e;
  const int q_base = (q_tile * kRowWaves + wave - slice * kRowWaves) * 32;
  const bool active = q_base < t_q;
  const int t_kv = seg.total;
  const int n_tiles = (t_kv + TK - 1) / TK, n_blocks = (t_kv + 31) / 32;
  const int n_mine = !active ? 0 : kSplit == 1 ? n_blocks : (n_blocks - slice + kSplit - 1) / kSplit;
  Stage<D, kRowWaves * kSplit, kSplit> stage(call, seg, ext_kv, io, bh, q_tile);
  f32x4 (&raw)[2][kLoads] = stage.raw;
  const int row0 = stage.row0, pos = stage.pos;
  // ---- registers -> parts in LDS (V's scaled)
  float top = 0.f;  // largest magnitude in K and Q that this lane has split
  constexpr int kPieces = 2 * kLoads;
  auto put_piece = [&](int slot, int piece) __attribute__((always_inline)) {
    const int k = piece >> 1, t = piece & 1;
    const int row = (k * kWaves + wave) * kRowsPerLoad + row0;
    char* dst = lds + slot + (kSplit == 1 ? 0 : (row >> 5) * kBlk) + (row & 31) * PB + 16 * ((pos >> 1) ^ swizzle<D>(row & 31)) + 8 * (pos & 1);
    f32x4 x = raw[t][k];
    u32x2 p[3];
    unsigned a, b, c, d, e, f;
    if (t == 0) {
      top = max3_abs(top, x[0], x[1]);
      top = max3_abs(top, x[2], x[3]);
    } else {
      x *= kScaleV;
    }
    split2(x[0], x[1], a, b, c);
    split2(x[2], x[3], d, e, f);
    p[0] = u32x2{a, d}, p[1] = u32x2{b, e}, p[2] = u32x2{c, f};
#pragma unroll
    for (int i = 0; i < 3; ++i) *reinterpret_cast<u32x2*>(dst + t * kTensor + i * kPart) = p[i];
  };
  auto put = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kPieces; ++i) put_piece(slot, i);
  };

  stage.fetch(0);
  // Q parts: B operand of S^T = K Q^T; lane (r,h) holds Q[row r][16t + 8h .. +8)
  bf16x8 qf[3][KS];
  if (active) {
    const char* q_row = (const char*)call.q + unit_offset(io.q, bh, io.heads) + (long long)min(q_base + r, t_q - 1) * io.q.tok;
    f32x4 x[KS][2];
#pragma unroll
    for (int t = 0; t < KS; ++t)
#pragma unroll
      for (int i = 0; i < 2; ++i) x[t][i] = *reinterpret_cast<const f32x4*>(q_row + 64 * t + 32 * h + 16 * i);
#pragma unroll
    for (int t = 0; t < KS; ++t) {
      u32x4 w[3];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        unsigned a, b, c;
        const float x0 = x[t][i >> 1][2 * (i & 1)], x1 = x[t][i >> 1][2 * (i & 1) + 1];
        top = max3_abs(top, x0, x1);
        split2(x0, x1, a, b, c);
        w[0][i] = a, w[1][i] = b, w[2][i] = c;
      }
#pragma unroll
      for (int i = 0; i < 3; ++i) qf[i][t] = __builtin_bit_cast(bf16x8, w[i]);
    }
  }

  f32x16 oacc[DB], osml[DB];  // O^T: sums of the products of the high parts, and of the others
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      oacc[d][v] = 0.f;
      osml[d][v] = 0.f;
    }
  float run_ref = -INFINITY, run_sum = 0.f;
  bf16x8 pf[2][3];  // probabilities of the block before, in parts

  const int tr_key = 4 * h + ((lane & 15) >> 2);
  const int tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  int v_base[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d) {
    const int col = 32 * d + tr_col;
    v_base[d] = kTensor + tr_key * PB + 16 * ((col >> 3) ^ swizzle<D>(tr_key)) + 2 * (col & 7);
  }
  auto hi_off = [](int d) { return 8 * PB + (D == 64 ? 0 : (d < 2 ? 128 : -128)); };
  int k_off[KS];
#pragma unroll
  for (int t = 0; t < KS; ++t) k_off[t] = r * PB + 16 * ((2 * t + h) ^ swizzle<D>(r));

  auto mul = [](bf16x8 a, bf16x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); };

  // The five products of parts beside hi * hi: parts of the first and of the second operand.
  constexpr int kA[5] = {2, 0, 1, 1, 0}, kB[5] = {0, 2, 1, 0, 1};
  // Scores of a block.  Partial sums of 32 channels, the small products of a sum before its large ones: a matrix instruction
  // rounds its accumulator after every eight products, at the size it has by then.  Two sums are formed in turn.
  f32x16 s;
  auto scores = [&](const char* blk, int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int half = 0; half < KS / 4; ++half) {
      f32x16 c[2];
      bf16x8 k[2][2][3];  // [step][sum]
#pragma unroll
      for (int v = 0; v < 16; ++v) c[0][v] = c[1][v] = 0.f;
      auto load_k = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 2; x >= 0; --x)
#pragma unroll
          for (int e = 0; e < 2; ++e) k[i][e][x] = *reinterpret_cast<const bf16x8*>(blk + x * kPart + k_off[4 * half + i + 2 * e]);
      };
      load_k(0);
      if constexpr (kAllOfK) {
        load_k(1);
        __builtin_amdgcn_sched_barrier(0);  // all on their way before the first product (the scheduler would spare registers)
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int t = 4 * half + i;
        if (!kAllOfK && i == 1) load_k(1);
#pragma unroll
        for (int j = 0; j < 5; ++j)
#pragma unroll
          for (int e = 0; e < 2; ++e) c[e] = mul(k[i][e][kA[j]], qf[kB[j]][t + 2 * e], c[e]);
#pragma unroll
        for (int n = 0; n < kPieces; ++n)
          if (n * (KS / 2) / kPieces == 2 * half + i) put_piece(slot, n);
      }
#pragma unroll
      for (int i = 1; i >= 0; --i)
#pragma unroll
        for (int e = 0; e < 2; ++e) c[e] = mul(k[i][e][0], qf[0][4 * half + i + 2 * e], c[e]);
#pragma unroll
      for (int v = 0; v < 16; ++v) s[v] = half == 0 ? c[0][v] + c[1][v] : s[v] + (c[0][v] + c[1][v]);
    }
  };
  auto mask = [&](int j0) __attribute__((always_inline)) {
    if (__builtin_expect(j0 + 32 > t_kv, 0)) {
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (j0 + 8 * (v >> 2) + 4 * h + (v & 3) >= t_kv) s[v] = -INFINITY;
    }
  };
  float p[16];
  auto form = [&](int u, float ref, float& sum) __attribute__((always_inline)) {
#pragma unroll
    for (int v = 8 * u; v < 8 * u + 8; ++v) {
      p[v] = __builtin_amdgcn_exp2f((s[v] - ref) * scale_log2e);
      sum += p[v];
    }
  };
  auto parts = [&](int u) __attribute__((always_inline)) {
    u32x4 w[3];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      unsigned a, b, c;
      split2(p[8 * u + 2 * i], p[8 * u + 2 * i + 1], a, b, c);
      w[0][i] = a, w[1][i] = b, w[2][i] = c;
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) pf[u][i] = __builtin_bit_cast(bf16x8, w[i]);
  };
  // O^T += V^T P^T over 16 keys of a block
  auto multiply_v = [&](const char* blk, int u) __attribute__((always_inline)) {
#pragma unroll
    for (int d0 = 0; d0 < DB; d0 += 2) {
      bf16x8 a[2][3];
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int x = 0; x < 3; ++x) {
          const char* vp = blk + v_base[d0 + e] + x * kPart + 16 * u * PB;
          const bf16x4 lo = lds_read_tr16(vp), hi = lds_read_tr16(vp + hi_off(d0 + e));
          a[e][x] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
#pragma unroll
      for (int e = 0; e < 2; ++e) oacc[d0 + e] = mul(a[e][0], pf[u][0], oacc[d0 + e]);
#pragma unroll
      for (int j = 0; j < 5; ++j)
#pragma unroll
        for (int e = 0; e < 2; ++e)  // (two row blocks in turn: neighbours do not wait for one another)
          osml[d0 + e] = mul(a[e][kA[j]], pf[u][kB[j]], osml[d0 + e]);
    }
  };
  // the reference was not good enough (always so in the first block)
  auto move_reference = [&](float& sum) __attribute__((always_inline)) {
    float mx = s[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[v]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const bool move = (mx - run_ref) * scale_log2e > kMaxLag;
    const float alpha = move ? __builtin_amdgcn_exp2f((run_ref - mx) * scale_log2e) : 1.f;
    run_sum *= alpha;
    run_ref = move ? mx : run_ref;
    const float ref = run_ref == -INFINITY ? 0.f : run_ref;
    sum = 0.f;
    form(0, ref, sum);
    form(1, ref, sum);
    parts(0);
    parts(1);
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        oacc[d][v] *= alpha;
        osml[d][v] *= alpha;
      }
  };

  stage.touch_up(0);
  put(0);
  if (1 < n_tiles) stage.fetch(1);
  __syncthreads();
  auto next_slot = [](int slot) { return slot == (kRing - 1) * kTile ? 0 : slot + kTile; };
  int before = 0, now = 0, next = kTile;  // ring positions of the tile whose V is multiplied, the one in use, the one being filled
  for (int t = 0; t < n_tiles; ++t) {
    if (t + 1 < n_tiles) stage.touch_up(t + 1);
    const bool has = t < n_mine;
    const char* blk = lds + now + slice * kBlk;
    if (has) {
      scores(blk, next);
    } else if (t + 1 < n_tiles) {
      put(next);
    }
    if (t + 2 < n_tiles) stage.fetch(t + 2);
    if (has) {
      mask(32 * (t * kSplit + slice));
      float sum = INFINITY;
      if (t > 0) {
        sum = 0.f;
        const char* old = lds + before + slice * kBlk;
        multiply_v(old, 0);
        form(0, run_ref, sum);
        form(1, run_ref, sum);
        parts(0);
        multiply_v(old, 1);
        parts(1);
      }
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(sum <= kTripSum)) != 0, 0)) move_reference(sum);
      run_sum += sum;
    }
    __syncthreads();
    if (has) before = now;
    now = next;
    next = next_slot(next);
  }
  if (n_mine > 0) {
    multiply_v(lds + before + slice * kBlk, 0);
    multiply_v(lds + before + slice * kBlk, 1);
  }
  float finite = 0.f;  // stays 0 if they all are
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      oacc[d][v] += osml[d][v];
      finite = fmaf(oacc[d][v], 0.f, finite);
    }
  if (top >= kLarge || !(finite == 0.f)) *wide_flag = 1;
  __syncthreads();
  if (*wide_flag != 0) return true;
  float total = run_sum + __shfl_xor(run_sum, 32, 64);
  char* o_row = (char*)call.o + unit_offset(io.o, bh, io.heads) + (long long)(q_base + r) * io.o.tok;
  const bool row_ok = q_base + r < t_q;
  if constexpr (kSplit == 1) {
    const float inv = 1.0f / total * (1.0f / kScaleV);
    if (!active) return false;
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        f32x4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = oacc[d][4 * c + e] * inv;
        if (row_ok) *reinterpret_cast<f32x4*>(o_row + 4 * (32 * d + 8 * c + 4 * h)) = x;
      }
  } else {
    constexpr int kChunks = 4 * DB;
    static_assert(kWaves * kChunks * 1024 <= lds_bytes(D, kSplit), "the parked results fit");
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      f32x4 x;
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = oacc[c >> 2][4 * (c & 3) + e];
      *reinterpret_cast<f32x4*>(lds + (wave * kChunks + c) * 1024 + lane * 16) = x;
    }
    if (h == 0) stat[wave][r] = make_float2(run_ref, total);
    __syncthreads();
    const int w0 = wave - slice * kRowWaves;
    float best = -INFINITY;
#pragma unroll
    for (int p = 0; p < kSplit; ++p) best = fmaxf(best, stat[w0 + p * kRowWaves][r].x);
    float weight[kSplit], sum = 0.f;
#pragma unroll
    for (int p = 0; p < kSplit; ++p) {
      const float2 y = stat[w0 + p * kRowWaves][r];
      weight[p] = __builtin_amdgcn_exp2f((y.x - best) * scale_log2e);
      sum = fmaf(weight[p], y.y, sum);
    }
    const float inv = 1.0f / sum * (1.0f / kScaleV);
#pragma unroll
    for (int c0 = 0; c0 < kChunks; c0 += kSplit) {
      const int c = c0 + slice;
      f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int p = 0; p < kSplit; ++p) {
        const f32x4 y = *reinterpret_cast<const f32x4*>(lds + ((w0 + p * kRowWaves) * kChunks + c) * 1024 + lane * 16);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = fmaf(weight[p], y[e], x[e]);
      }
      x *= inv;
      if (active && row_ok) *reinterpret_cast<f32x4*>(o_row + 4 * (32 * (c >> 2) + 8 * (c & 3) + 4 * h)) = x;
    }
  }
  return false;
}

template <int D, int kRowWaves, int kSplit, int kOcc>
__global__ __launch_bounds__(64 * kRowWaves * kSplit, kOcc) void attend_f32_parts_kernel(
    const float* __restrict__ q, float* __restrict__ o, float* __restrict__ kc, float* __restrict__ vc, int t_q,
    long long cap_tokens, SegTable seg, ExtKV ext_kv, CallerIo io, float scale_log2e, int n_bh, int n_qtiles, int n_whole) {
  fetch_arguments<kAttentionArguments>();
  __shared__ __align__(1024) char lds[lds_bytes(D, kSplit)];
  __shared__ float2 stat[kSplit > 1 ? kRowWaves * kSplit : 1][32];
  __shared__ int wide_flag;
  const Place at = place<true>(blockIdx.x, n_bh, n_qtiles, n_whole);
  const int bh_i = at.bh, q_tile = at.tile;
  if (bh_i >= n_bh) return;  // whole workgroup
  if (threadIdx.x == 0) wide_flag = 0;  // (read and written again behind barriers only)
  const Call call{q, o, (char*)kc, (char*)vc, t_q, cap_tokens, scale_log2e, n_qtiles};
  if (__builtin_expect(attend_unit<D, kRowWaves, kSplit>(call, seg, ext_kv, io, bh_i, q_tile, lds, stat, &wide_flag), 0))
    attend_unit_wide<D, kRowWaves, kSplit>(call, seg, ext_kv, io, bh_i, q_tile, lds);
}

template <int D, int kRowWaves, int kSplit, int kOcc>
hipError_t launch(const void* q, void* o, void* kc, void* vc, int bh, int t_q, int64_t cap_tokens, const SegTable& seg,
                  const ExtKV& ext, const CallerIo& io, float c, hipStream_t st) {
  const int n_qtiles = (t_q + 32 * kRowWaves - 1) / (32 * kRowWaves);
  const int n_whole = whole_units(bh, n_qtiles, kMostWhole);
  dim3 grid(placed_grid(bh, n_qtiles, n_whole)), block(64 * kRowWaves * kSplit);
  hipLaunchKernelGGL((attend_f32_parts_kernel<D, kRowWaves, kSplit, kOcc>), grid, block, 0, st, (const float*)q, (float*)o, (float*)kc,
                     (float*)vc, t_q, (long long)cap_tokens, seg, ext, io, c, bh, n_qtiles, n_whole);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_attend_f32_parts(int row_waves, int split, const void* q, void* o, void* kc, void* vc, int bh, int t_q, int head_dim,
                                   int64_t cap_tokens, const SegTable& seg, const ExtKV& ext, const CallerIo& io, float softmax_scale,
                                   hipStream_t st) {
  const float c = softmax_scale * 1.4426950408889634f;
  // head dim 128: ~470 registers, one wave per SIMD (eight waves of 256 registers spill)
  if (head_dim == 128) return launch<128, 4, 1, 1>(q, o, kc, vc, bh, t_q, cap_tokens, seg, ext, io, c, st);
  if (split == 2) return launch<64, 4, 2, 2>(q, o, kc, vc, bh, t_q, cap_tokens, seg, ext, io, c, st);
  return row_waves == 8 ? launch<64, 8, 1, 2>(q, o, kc, vc, bh, t_q, cap_tokens, seg, ext, io, c, st)
                        : launch<64, 4, 1, 2>(q, o, kc, vc, bh, t_q, cap_tokens, seg, ext, io, c, st);
}

}  // namespace amskv
