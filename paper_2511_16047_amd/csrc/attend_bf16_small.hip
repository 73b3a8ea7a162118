// bf16 per-scale attention where a (b,h) has little work or the (b,h) are few (Section 3.1's per-step attention): the
// launch is bound by memory latency and by the serial chain of a unit's key blocks, not by bandwidth or the matrix cores, so
// the design goal is to have every unit of the launch resident at once and its chain short.
//
// One WAVE owns one unit = (b, h, block of 32 query rows), or (kSplit > 1) the waves of a workgroup share one, each taking
// every kSplit-th block of 32 keys with softmax statistics of its own; their partial results meet in LDS once, behind one
// barrier.  Otherwise the waves of a workgroup are independent.  K fragments are loaded straight from the cache into
// registers in the A-operand layout of v_mfma_f32_32x32x16_bf16 (lane (r,h) reads 16 bytes of key row r), so K never touches
// LDS; LDS holds two 32-key blocks of V per wave, which the transposing read ds_read_b64_tr_b16 needs as its source and
// which direct-to-LDS loads fill without passing through registers (that is what lets four waves per SIMD be resident at
// head dim 64).  The loads of a wave's next block are issued right after the first product has consumed the K registers, so
// they overlap the softmax and the second product.  Same transposed formulation (S^T = K Q^T, O^T += V^T P^T) and the same
// segment-table walk as the streaming kernel; plain online softmax.
//
// kDensity: the softmax mass on each group of keys (Section 4.1) as a by-product.  A wave sums its probabilities per group in
// fp32 as the key stream passes; where a group ends it parks (sum, the maximum it refers to) in LDS, and at the end
// everything parked moves to the common maximum.  (Coarse scales, 1920 units: 8.7 us for the stand-alone density kernel and
// 8.4 for the attention -> 11.2 for both.)
#include "amskv_internal.hpp"

namespace amskv {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// 16-byte chunk as a native vector: arrays of it stay in registers (HIP's uint4 struct did not)
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// waves of a workgroup: four units, or the four or eight slices of one
constexpr int waves_of(int split) { return split == 8 ? 8 : 4; }
// query blocks on the fullest XCD up to which a (b,h) stays on one (place()).  Equal shares over whole (b,h): fewer than 8 (b,h), up to 4
// blocks 1.03 of the time (6 us a launch), 8 1.08, 16 1.01, 20 to 28 0.99, 32 0.96, 64 0.66; more (b,h): 0.99 to 1.01 up to 32, 48 0.72.
constexpr int kMostWhole = 8;

#define AMSKV_LDS __attribute__((address_space(3)))

__device__ __forceinline__ bf16x4 lds_read_tr16(const char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((AMSKV_LDS bf16x4*)(p));
}

// One wave-wide direct-to-LDS load: lane i's 16 bytes at `g` land at lds_wave_base + 16*i (wave-uniform base,
// through M0).  Inline assembly: the compiler does not count it among its outstanding loads, which is safe
// here because every V load is issued BEFORE the K register loads of the same block -- loads complete in
// order, so the wait the compiler places in front of the first use of those K registers covers it.
__device__ __forceinline__ void lds_dma16(const char* g, char* lds_wave_base) {
  const unsigned m0v = (unsigned)(size_t)(AMSKV_LDS char*)lds_wave_base;
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(m0v) : "memory", "m0");
}

__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// The compiler tracks the wait states a matrix instruction needs before an ordinary vector
// instruction may read its result, but not for a read from inside inline assembly (max3 above).
// Called on the accumulator between the two, this holds the wave for the 11 wait states that an
// 8-pass v_mfma_f32_32x32x16_bf16 requires (one to spare); taking the accumulator as an in/out operand pins
// it after the matrix instructions and before every later use.
__device__ __forceinline__ void settle_mfma(f32x16& acc) { asm volatile("s_nop 11" : "+v"(acc)); }

// Register budget: four waves per SIMD at head dim 64 and two at 128 are the most that fit without spilling;
// every step up in resident waves measured faster on these latency-bound launches.
template <int D, int kSplit, bool kDensity>
__global__ __launch_bounds__(64 * waves_of(kSplit), !kDensity ? (D == 64 ? 4 : 2) : kSplit > 1 ? 1 : D == 64 ? 3 : 2) void attend_bf16_small_kernel(
    const __bf16* __restrict__ q, __bf16* __restrict__ o, char* __restrict__ kc, char* __restrict__ vc,
    int t_q, long long cap_tokens, SegTable seg, ExtKV ext_in, CallerIo io, float scale_log2e, int n_qblk, int n_bh, int n_whole,
    GroupEnds groups, float* __restrict__ partial) {
  fetch_arguments<kAttentionArguments>();
  const ExtKV ext_kv = chosen(ext_in);
  constexpr int kWaves = waves_of(kSplit);
  constexpr int RB = D * 2;
  constexpr int CPR = D / 8;
  constexpr int KS = D / 16;
  constexpr int DB = D / 32;
  constexpr int VCH = 32 * CPR / 64;  // 16-byte chunks of a 32-key V block per lane
  // The form that also takes steps of more than 32 queries sums the probabilities in fp32 as they are, like the streaming
  // kernel it stands in for there.  The others sum the bf16 values that the second product multiplies, two at a time.
  constexpr bool kSumUnrounded = kSplit == 8;

  __shared__ __align__(1024) char lds_v[kWaves][2][32 * RB];  // per wave: the block in use and the one in flight
  __shared__ float2 stat[kSplit > 1 ? kWaves : 1][32];        // split: reference and sum of every slice's rows
  __shared__ float2 park[kDensity ? kWaves : 1][kDensity ? AMSKV_MAX_SCALES : 1][32];  // density: sum and its reference

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int slice = kSplit == 1 ? 0 : wave;
  // without a split: launched with one block of queries only
  const Place place_of = kSplit == 1 ? Place{(int)(blockIdx.x * kWaves) + wave, 0} : place<true>(blockIdx.x, n_bh, n_qblk, n_whole);
  const int q_blk = place_of.tile;
  const long long bh = place_of.bh;
  if (bh >= n_bh) return;  // without a split nothing below synchronises across waves; with one, the whole workgroup leaves
  const int r = lane & 31, h = lane >> 5;
  const int q_base = q_blk * 32;
  const int t_kv = seg.total;
  const int n_blocks = (t_kv + 31) / 32;
  char* kb = kc + bh * cap_tokens * RB;
  char* vb = vc + bh * cap_tokens * RB;
  const long long x_unit = unit_offset(io.kv, bh, io.heads);  // borrowed current scale, if any
  const char* xk = (const char*)ext_kv.k + x_unit;
  const char* xv = (const char*)ext_kv.v + x_unit;
  const long long x_tok = io.kv.tok;
  const char* q_unit = (const char*)q + unit_offset(io.q, bh, io.heads);
  char* o_unit = (char*)o + unit_offset(io.o, bh, io.heads);
  const bool write_back = writes_back(ext_kv, seg.total, seg.ext_start) && q_base == 0;

  bf16x8 qf[KS];
  {
    const int row = min(q_base + r, t_q - 1);
#pragma unroll
    for (int t = 0; t < KS; ++t) qf[t] = *reinterpret_cast<const bf16x8*>(q_unit + row * io.q.tok + 32 * t + 16 * h);
  }

  bf16x8 kf[KS];
  // lane i of V load k fills chunk position i % CPR of row k * (64 / CPR) + i / CPR with the global chunk that the
  // XOR swizzle (same as the streaming kernel's at head dim 64) assigns to that position
  auto load_block = [&](int g, int buffer) {
    const int j0 = 32 * g;
    char* dst = lds_v[wave][buffer];
    // The rows this lane fetches -- VCH of V, one of K -- and where they sit: one walk of the segment table for all of them,
    // four entries per step.  (One walk per row and one entry at a time was a chain of up to 25 scalar-load waits in front of
    // the first load: 16-layer stack on one image 1076 -> 1016 us a pass.)
    int at[VCH + 1], delta[VCH + 1];
#pragma unroll
    for (int k = 0; k <= VCH; ++k) {
      at[k] = min(j0 + (k < VCH ? k * (64 / CPR) + lane / CPR : r), t_kv - 1);
      delta[k] = 0;
    }
    for (int i0 = 0; i0 < seg.n; i0 += 4) {
#pragma unroll
      for (int i = i0; i < i0 + 4; ++i) {
        const int from = i < seg.n ? seg.virt_start[i] : 0x7fffffff, by = seg.phys_off[i] - seg.virt_start[i];
#pragma unroll
        for (int k = 0; k <= VCH; ++k) delta[k] = at[k] >= from ? by : delta[k];
      }
    }
#pragma unroll
    for (int k = 0; k < VCH; ++k) {
      const int row = k * (64 / CPR) + lane / CPR, c = (lane % CPR) ^ (row & 7);
      const char* p = at[k] >= seg.ext_start ? xv + (at[k] - seg.ext_start) * x_tok : vb + (long long)(at[k] + delta[k]) * RB;
      lds_dma16(p + 16 * c, dst + k * 1024);
    }
    const char* kp = at[VCH] >= seg.ext_start ? xk + (at[VCH] - seg.ext_start) * x_tok : kb + (long long)(at[VCH] + delta[VCH]) * RB;
#pragma unroll
    for (int t = 0; t < KS; ++t) kf[t] = *reinterpret_cast<const bf16x8*>(kp + 32 * t + 16 * h);
  };
  if (kSplit == 1 || slice < n_blocks) load_block(slice, 0);

  f32x16 oacc[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int v = 0; v < 16; ++v) oacc[d][v] = 0.f;
  float run_max = -INFINITY, run_sum = 0.f;

  const int tr_key = 4 * h + ((lane & 15) >> 2);
  const int tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);

  // density: group the stream is in, its end, where the part of it that this block holds begins, sum so far
  int group = 0, next_end = kDensity ? groups.end[0] : 0;
  float in_group = 0.f;
  auto park_group = [&]() {
    const float x = half_sum(in_group);  // the lane halves hold different keys of a query
    if (h == 0) park[wave][group][r] = make_float2(x, run_max);
    in_group = 0.f;
    ++group;
    next_end = group < groups.n ? groups.end[group] : 0x7fffffff;
  };

  int buffer = 0;
  for (int g = slice; g < n_blocks; g += kSplit, buffer ^= 1) {
    // every load of block g (the V rows in LDS and the K registers) has landed; an explicit point, because the
    // compiler does not know that the V loads wrote LDS and could otherwise move reads of it above its own wait
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const char* my_v = lds_v[wave][buffer];
    f32x16 sacc;
#pragma unroll
    for (int v = 0; v < 16; ++v) sacc[v] = 0.f;
#pragma unroll
    for (int t = 0; t < KS; ++t) sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t], qf[t], sacc, 0, 0, 0);
    if (write_back) {
      // fused append: this unit also fills the current scale's slot from the registers it just used
      const int j0 = 32 * g;
      const int k_to = write_back_row(ext_kv, j0 + r, t_kv, seg.ext_start);
      if (k_to >= 0) {
        char* dst = kb + (long long)k_to * RB + 16 * h;
#pragma unroll
        for (int t = 0; t < KS; ++t) *reinterpret_cast<bf16x8*>(dst + 32 * t) = kf[t];
      }
#pragma unroll
      for (int k = 0; k < VCH; ++k) {
        const int row = k * (64 / CPR) + lane / CPR, c = (lane % CPR) ^ (row & 7);
        const int v_to = write_back_row(ext_kv, j0 + row, t_kv, seg.ext_start);
        if (v_to >= 0)
          *reinterpret_cast<u32x4*>(vb + (long long)v_to * RB + 16 * c) =
              *reinterpret_cast<const u32x4*>(my_v + k * 1024 + 16 * lane);
      }
    }
    if (g + kSplit < n_blocks) load_block(g + kSplit, buffer ^ 1);  // in flight during the softmax and the second product

    if (g == n_blocks - 1 && (t_kv & 31) != 0) {
      const int valid = t_kv & 31;
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (8 * (v >> 2) + 4 * h + (v & 3) >= valid) sacc[v] = -INFINITY;
    }
    settle_mfma(sacc);
    float mx = max3(sacc[0], sacc[1], sacc[2]);
#pragma unroll
    for (int v = 3; v < 15; v += 2) mx = max3(mx, sacc[v], sacc[v + 1]);
    const float other = __shfl_xor(max3(mx, sacc[15], sacc[15]), 32, 64);
    mx = max3(mx, sacc[15], other);
    const float new_max = fmaxf(run_max, mx);
    const float alpha = __builtin_amdgcn_exp2f((run_max - new_max) * scale_log2e);
    const float mc = new_max * scale_log2e;
    run_max = new_max;
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
    float sum = run_sum * alpha, sum2 = 0.f;
    bf16x8 pf[2];
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      const float p0 = __builtin_amdgcn_exp2f(fmaf(sacc[v], scale_log2e, -mc));
      const float p1 = __builtin_amdgcn_exp2f(fmaf(sacc[v + 1], scale_log2e, -mc));
      if constexpr (kDensity) {
        sacc[v] = p0;
        sacc[v + 1] = p1;
      }
      bf16x2 pk;
      pk[0] = (__bf16)p0;
      pk[1] = (__bf16)p1;
      if constexpr (kSumUnrounded) {
        sum += p0;
        sum2 += p1;
      } else {
        sum = __builtin_amdgcn_fdot2_f32_bf16(pk, ones, sum, false);
      }
      pf[v >> 3][v & 7] = pk[0];
      pf[v >> 3][(v & 7) + 1] = pk[1];
    }
    run_sum = kSumUnrounded ? sum + sum2 : sum;
    if constexpr (kDensity) {
      in_group *= alpha;
      // keys [from, to) of the block belong to the group
      auto take = [&](int from, int to) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int key = 8 * (v >> 2) + 4 * h + (v & 3);
          in_group += key >= from && key < to ? sacc[v] : 0.f;
        }
      };
      int from = 0;
      while (next_end <= 32 * g + 32) {  // (an end in front of this block lies in another slice's block)
        const int to = max(next_end - 32 * g, 0);
        take(from, to);
        park_group();
        from = to;
      }
      take(from, 32);
    }
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int v = 0; v < 16; ++v) oacc[d][v] *= alpha;

    __builtin_amdgcn_wave_barrier();  // the V rows written above by all lanes are read below
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int d = 0; d < DB; ++d) {
        const int key0 = 16 * u + tr_key, key1 = key0 + 8, col = 32 * d + tr_col;
        const bf16x4 lo = lds_read_tr16(my_v + key0 * RB + 16 * ((col >> 3) ^ (key0 & 7)) + 2 * (col & 7));
        const bf16x4 hi = lds_read_tr16(my_v + key1 * RB + 16 * ((col >> 3) ^ (key1 & 7)) + 2 * (col & 7));
        bf16x8 a;
        a[0] = lo[0]; a[1] = lo[1]; a[2] = lo[2]; a[3] = lo[3];
        a[4] = hi[0]; a[5] = hi[1]; a[6] = hi[2]; a[7] = hi[3];
        oacc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pf[u], oacc[d], 0, 0, 0);
      }
    __builtin_amdgcn_wave_barrier();  // ... and are overwritten by the next iteration
  }

  if constexpr (kDensity)
    while (group < groups.n) park_group();
  float total = run_sum + __shfl_xor(run_sum, 32, 64);
  const int row = q_base + r;
  __bf16* dst = reinterpret_cast<__bf16*>(o_unit + min(row, t_q - 1) * io.o.tok);
  float top = run_max, weight[kSplit];
  if constexpr (kSplit == 1) {
    const float inv = 1.0f / total;
    // The lane halves hold alternate 8-byte pieces of a row (columns 8g + 4h ..); one lane swap per register pairs
    // them up, so that every lane stores 16 bytes and the two lanes of a row 32 contiguous bytes.
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
        bf16x4 wa, wb;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          wa[e] = (__bf16)(oacc[d][8 * k + e] * inv);
          wb[e] = (__bf16)(oacc[d][8 * k + 4 + e] * inv);
        }
        const u32x2 a = __builtin_bit_cast(u32x2, wa), b = __builtin_bit_cast(u32x2, wb);
        const auto s0 = __builtin_amdgcn_permlane32_swap(a[0], b[0], false, false);
        const auto s1 = __builtin_amdgcn_permlane32_swap(a[1], b[1], false, false);
        const u32x4 w = {s0[0], s1[0], s0[1], s1[1]};
        if (row < t_q) *reinterpret_cast<u32x4*>(dst + 32 * d + 16 * k + 8 * h) = w;
      }
  } else {
    // Every slice parks its O^T where its V blocks were (the same number of bytes; 16 per lane, consecutive lanes) and then
    // puts its share of the row pieces together from all slices.
    constexpr int kChunks = 4 * DB;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      f32x4 x;
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = oacc[c >> 2][4 * (c & 3) + e];
      *reinterpret_cast<f32x4*>(&lds_v[wave][0][0] + c * 1024 + lane * 16) = x;
    }
    if (h == 0) stat[wave][r] = make_float2(run_max, total);  // -inf, 0 for a slice without blocks: it weighs 0
    __syncthreads();
#pragma unroll
    for (int p = 0; p < kSplit; ++p) top = fmaxf(top, stat[p][r].x);
    total = 0.f;
#pragma unroll
    for (int p = 0; p < kSplit; ++p) {
      weight[p] = __builtin_amdgcn_exp2f((stat[p][r].x - top) * scale_log2e);
      total = fmaf(weight[p], stat[p][r].y, total);
    }
    const float inv = 1.0f / total;
#pragma unroll
    for (int c0 = 0; c0 < kChunks; c0 += kSplit) {
      const int c = c0 + slice;
      f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int p = 0; p < kSplit; ++p) {
        const f32x4 y = *reinterpret_cast<const f32x4*>(&lds_v[p][0][0] + c * 1024 + lane * 16);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = fmaf(weight[p], y[e], x[e]);
      }
      bf16x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = (__bf16)(x[e] * inv);
      if (row < t_q) *reinterpret_cast<bf16x4*>(dst + 8 * c + 4 * h) = w;  // chunk c: columns 8c + 4h ..
    }
  }
  if constexpr (kDensity) {
    // mass of the unit on group p = sum over its rows of (sum of exp over the group) / (sum over all groups)
    auto mass = [&](int p) {
      float x = 0.f;
#pragma unroll
      for (int w = 0; w < kSplit; ++w) {
        const float2 y = park[kSplit == 1 ? wave : w][p][r];
        x = fmaf(y.x, __builtin_amdgcn_exp2f((y.y - top) * scale_log2e), x);
      }
      return x;
    };
    float all = 0.f;  // (either lane half takes every second group)
    for (int p = h; p < groups.n; p += 2) all += mass(p);
    const float inv_all = row < t_q ? 1.0f / half_sum(all) : 0.f;
    for (int p0 = 2 * slice; p0 < groups.n; p0 += 2 * kSplit) {
      const int p = p0 + h;
      const float m = group_sum<32>(mass(min(p, groups.n - 1)) * inv_all);  // over the 32 query rows
      if (r == 0 && p < groups.n) partial[(bh * n_qblk + q_blk) * AMSKV_MAX_SCALES + p] = m;
    }
  }
}

template <int D, int kSplit, bool kDensity>
hipError_t launch_one(const void* q, void* o, void* kc, void* vc, int bh, int t_q, int64_t cap_tokens, const SegTable& seg,
                      const ExtKV& ext, const CallerIo& io, float c, const GroupEnds& groups, float* partial, hipStream_t st) {
  const int n_qblk = (t_q + 31) / 32;
  constexpr int kWaves = waves_of(kSplit);
  const int n_whole = whole_units(bh, n_qblk, kMostWhole);
  if (kSplit == 1 && n_qblk != 1) return hipErrorInvalidValue;  // (the dispatch splits wherever a unit has more queries)
  const unsigned grid = kSplit == 1 ? (unsigned)(((long long)bh * n_qblk + kWaves - 1) / kWaves)
                                    : placed_grid(bh, n_qblk, n_whole);
  hipLaunchKernelGGL((attend_bf16_small_kernel<D, kSplit, kDensity>), dim3(grid), dim3(64 * kWaves), 0, st, (const __bf16*)q,
                     (__bf16*)o, (char*)kc, (char*)vc, t_q, (long long)cap_tokens, seg, ext, io, c, n_qblk, bh, n_whole, groups, partial);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attend_bf16_small(const void* q, void* o, void* kc, void* vc, int bh, int t_q,
                                    int head_dim, int64_t cap_tokens, const SegTable& seg, const ExtKV& ext,
                                    const CallerIo& io, float softmax_scale, int split, const GroupEnds& groups, float* partial,
                                    hipStream_t st) {
  const float c = softmax_scale * 1.4426950408889634f;
  auto go = [&](auto f) { return f(q, o, kc, vc, bh, t_q, cap_tokens, seg, ext, io, c, groups, partial, st); };
  if (head_dim == 64) {
    if (split == 8) return partial ? go(launch_one<64, 8, true>) : go(launch_one<64, 8, false>);
    if (split == 4) return partial ? go(launch_one<64, 4, true>) : go(launch_one<64, 4, false>);
    return partial ? go(launch_one<64, 1, true>) : go(launch_one<64, 1, false>);
  }
  if (split > 1) return partial ? go(launch_one<128, 4, true>) : go(launch_one<128, 4, false>);
  return partial ? go(launch_one<128, 1, true>) : go(launch_one<128, 1, false>);
}

}  // namespace amskv
