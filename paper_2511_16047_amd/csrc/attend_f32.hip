// fp32 per-scale attention over the resident segments (Section 3.1: the queries of scale s attend to the cached
// scales and to their own scale; no mask inside a step), everything in fp32.  Launches with little work; the others go to
// attend_f32_parts.hip (attend_f32_choice.hpp).
//
// What bounds it: all query rows of a (b,h) share its keys, so wherever there are enough units the fp32 matrix pipe
// (v_mfma_f32_32x32x2_f32 and 16x16x4: 157 TFLOP/s nominal, 154 measured on a large product) is the limit, not memory;
// with few units it is the chain of a wave's key blocks.  Measured: 16 (b,h), 256 queries x 680 keys 124 -> 14 us (one image)
// against a kernel that kept four lanes to a query row and fed the vector ALUs from LDS and had one serial chain of keys for
// each of 64 workgroups.
//
// Formulation.  A unit is (b, h, block of QT query rows), QT = 32 or 16.  Per block of QT keys the transposed scores
// S^T = K Q^T (M = keys, N = queries) leave every lane with the scores of ONE query, so the softmax is in-lane plus an
// exchange between the 64/QT lane groups -- and the accumulator registers already are, one by one, the B operands of
// O^T += V^T P^T: register v of lane group g holds the key the matrix instruction of step v expects from that group.
// The head dim is dealt to the lane groups in runs (group g of H holds channels [g*D/H, (g+1)*D/H) of its K and Q
// rows), so a lane reads 16-byte pieces; the rows of V are read whole, D/QT channels per lane.
//
// Memory.  K and V blocks come through LDS with direct-to-LDS loads (whole rows, coalesced; the 16-byte chunks of K rows are
// XOR-swizzled on the global side so that 16 lanes reading one chunk of 16 rows hit 16 different bank groups).  (K straight
// from memory into registers touches 16 lines per quarter wave and instruction and kept the matrix pipe at half its rate.)
// The four waves of a workgroup that each hold a block of query rows of one (b,h) walk the same keys and fetch each block
// once, a quarter per wave, into a ring: two blocks on the way, one in use, one whose V is still multiplied, one barrier per
// block.  Against a stream per wave (four times the traffic from L2 and one block of slack), on launches that attend_f32_parts.hip has
// taken over since and before a dot product was 16 partial sums (which cost 5 to 10 %): 256 (b,h), 256 x 680 118 -> 108 us, 169 x 424
// 65 -> 61; head dim 128, 32 (b,h), 1024 x 1621 269 -> 241.
// Where a unit's keys are split over waves every wave has a stream of its own: K of its next block is requested behind the
// score products, V behind the second product, each half a block ahead of its use, and nothing in the loop synchronises waves.
//
// Few units (one image): the keys of a unit are dealt block by block to kSplit waves of a workgroup, each with its
// own online softmax; their partial results meet in LDS once, behind one barrier.
#include "amskv_internal.hpp"
#include "attend_f32_choice.hpp"

namespace amskv {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// the running reference of the softmax may lag the true maximum by this many powers of two before the accumulators
// are rescaled: probabilities stay far below overflow, of no consequence to fp32's relative precision
constexpr float kMaxLag = 6.0f;
// sum of a lane's (at most 16) new probabilities above which the reference is looked at again: 16 * 2^kMaxLag
constexpr float kTripSum = 1024.0f;

template <int QT>
struct Mfma;
template <>
struct Mfma<32> {
  typedef f32x16 Acc;
  static constexpr int NV = 16;
  __device__ static __forceinline__ int row(int v, int g) { return 8 * (v >> 2) + 4 * g + (v & 3); }
  __device__ static __forceinline__ Acc mul(float a, float b, Acc c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
};
template <>
struct Mfma<16> {
  typedef f32x4 Acc;
  static constexpr int NV = 4;
  __device__ static __forceinline__ int row(int v, int g) { return 4 * g + v; }
  __device__ static __forceinline__ Acc mul(float a, float b, Acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
};

// split: per wave a block of K and one of V (the K piece later holds the wave's partial result), and its softmax statistics;
// else a ring of blocks for the workgroup
constexpr int kRing = 4;
// workgroups on the fullest XCD up to which a (b,h) stays on one (place()).  Equal shares over whole (b,h): up to 4 1.03 to 1.06 of the
// time (7 to 11 us a launch), 8 1.01 to 1.05, 12 to 32 0.99 to 1.04, 48 0.84 to 0.53.
constexpr int kMostWhole = 32;
constexpr int lds_bytes(int D, int QT, int split) {
  return split > 1 ? waves_of(split) * (2 * QT * D * 4 + QT * 8) : kRing * 2 * QT * D * 4;
}

#define AMSKV_LDS __attribute__((address_space(3)))

// One wave-wide direct-to-LDS load: lane i's 16 bytes at base + lane_off land at lds_wave_base + 16*i (both bases
// wave-uniform).  Inline assembly with explicit waits: see the streaming bf16 kernel.
__device__ __forceinline__ void lds_dma16_s(const char* base, unsigned lane_off, char* lds_wave_base) {
  const unsigned m0v = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(AMSKV_LDS char*)lds_wave_base);
  const unsigned long long b = (unsigned long long)base;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)b), hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
  const unsigned long long bs = ((unsigned long long)hi << 32) | lo;
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_off), "s"(bs), "s"(m0v) : "memory", "m0");
}
__device__ __forceinline__ void lds_dma16(const char* g, char* lds_wave_base) {
  const unsigned m0v = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(AMSKV_LDS char*)lds_wave_base);
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(m0v) : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// every LDS read of this wave has returned: what follows may overwrite what they read
__device__ __forceinline__ void wait_lds_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

template <int D, int QT, int kSplit, bool kShares>
__global__ __launch_bounds__(64 * waves_of(kSplit), 2) void attend_f32_kernel(
    const float* __restrict__ q, float* __restrict__ o, float* __restrict__ kc, float* __restrict__ vc, int t_q,
    long long cap_tokens, SegTable seg, ExtKV ext_kv, CallerIo io, float scale_log2e, int n_bh, int n_parts, int n_whole) {
  fetch_arguments<kAttentionArguments>();
  typedef Mfma<QT> M;
  constexpr int H = 64 / QT;         // lane groups
  constexpr int DL = D / H;          // channels of a K or Q row one lane holds
  constexpr int NC = DL / 4;         // ... in 16-byte pieces
  constexpr int NDB = D / QT;        // row blocks of O^T; channels of a V row one lane holds
  constexpr int NV = M::NV;
  constexpr int RB = D * 4;
  constexpr int kWaves = waves_of(kSplit);
  constexpr int kUnits = kWaves / kSplit;  // units per workgroup
  constexpr int CPR = D / 4;            // 16-byte chunks of a row
  constexpr int kRowsPerLoad = 64 / CPR;
  constexpr int kLoads = QT / kRowsPerLoad;  // direct-to-LDS loads of a block, per tensor
  constexpr int kBlk = QT * RB;
  __shared__ __align__(1024) char lds[lds_bytes(D, QT, kSplit)];

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int r = lane % QT, g = lane / QT;
  const int slice = wave % kSplit;
  const Place place_of = place<kShares>(blockIdx.x, n_bh, n_parts, n_whole);
  const int part = place_of.tile;
  const long long bh = place_of.bh;
  if (bh >= n_bh) return;  // whole workgroup
  const int q_base = (part * kUnits + wave / kSplit) * QT;
  const bool active = q_base < t_q;
  const int t_kv = seg.total;
  const int n_blocks = (t_kv + QT - 1) / QT;
  char* kb = (char*)kc + bh * cap_tokens * RB;
  char* vb = (char*)vc + bh * cap_tokens * RB;
  const long long x_unit = unit_offset(io.kv, bh, io.heads);  // borrowed current scale, if any
  const char* xk = (const char*)ext_kv.k + x_unit;
  const char* xv = (const char*)ext_kv.v + x_unit;
  // fused append: the blocks of the current scale are dealt to the units of the (b,h), so that none lags behind
  const bool write_back = writes_back(ext_kv, seg.total, seg.ext_start);
  const int n_qblk = (t_q + QT - 1) / QT, my_qblk = kSplit == 1 ? part : q_base / QT;
  constexpr bool kShared = kSplit == 1;  // the waves of the workgroup walk the same blocks and fetch them together
  char* lds_k = lds + (kShared ? 0 : wave * 2 * kBlk);  // shared: ring slot of the block in use
  char* lds_v = lds_k + kBlk;                           // shared: ring slot of the block whose V is multiplied
  constexpr int kMyLoads = kShared ? kLoads / kWaves : kLoads;  // direct-to-LDS loads of this wave, per block and tensor
  static_assert(kMyLoads >= 1 && (!kShared || kMyLoads * kWaves == kLoads), "the waves share a block evenly");
  const int first_load = kShared ? wave * kMyLoads : 0;

  f32x4 qf[NC];
  if (active) {
    const char* q_row = (const char*)q + unit_offset(io.q, bh, io.heads) + (long long)min(q_base + r, t_q - 1) * io.q.tok;
#pragma unroll
    for (int i = 0; i < NC; ++i) qf[i] = *reinterpret_cast<const f32x4*>(q_row + 4 * DL * g + 16 * i);
  }

  // Rows of key block b -> LDS.  Lane i of load k fills chunk position i % CPR of row k * kRowsPerLoad + i / CPR; for K
  // that position holds global chunk position ^ (row & 15).  A block inside one segment (wave-uniform, nearly always)
  // is addressed from one scalar base; elsewhere every lane looks its row up (rows past the end re-read the last one).
  // Both are left with exactly kMyLoads loads in flight.
  // The segment looked up last is kept: the table is walked again only when a block begins outside it.
  int seg_lo = 0, seg_end = 0, seg_delta = 0;
  auto load = [&](int b, bool is_v) {
    const int j0 = b * QT;
    char* dst = kShared ? lds + (b % kRing) * 2 * kBlk + (is_v ? kBlk : 0) : is_v ? lds_v : lds_k;
    if (__builtin_expect(j0 < seg_lo || j0 >= seg_end, 0)) {
      seg_lo = seg.virt_start[0], seg_end = seg_lo + seg.len[0], seg_delta = seg.phys_off[0] - seg_lo;
      for (int i = 1; i < seg.n; ++i)
        if (j0 >= seg.virt_start[i]) {
          seg_lo = seg.virt_start[i];
          seg_end = seg_lo + seg.len[i];
          seg_delta = seg.phys_off[i] - seg_lo;
        }
      if (j0 >= seg.ext_start) {
        seg_lo = seg.ext_start;
        seg_end = t_kv;
        seg_delta = -seg.ext_start;
      }
    }
    const bool in_ext = j0 >= seg.ext_start;
    const long long st = in_ext ? io.kv.tok : (long long)RB;
    const int row0 = lane / CPR, pos = lane % CPR;
    if (__builtin_expect(j0 + QT <= seg_end && st < (1ll << 24), 1)) {
      const char* base = (in_ext ? (is_v ? xv : xk) : (is_v ? vb : kb)) + (long long)(j0 + seg_delta) * st;
#pragma unroll
      for (int k = first_load; k < first_load + kMyLoads; ++k) {
        const int row = k * kRowsPerLoad + row0;
        lds_dma16_s(base, row * (unsigned)st + 16 * (is_v ? pos : pos ^ (row & 15)), dst + k * 1024);
      }
      return;
    }
#pragma unroll
    for (int k = first_load; k < first_load + kMyLoads; ++k) {
      const int row = k * kRowsPerLoad + row0;
      bool ext;
      const long long at = locate_row(seg, min(j0 + row, t_kv - 1), ext);
      const char* p = ext ? (is_v ? xv : xk) + at * io.kv.tok : (is_v ? vb : kb) + at * RB;
      lds_dma16(p + 16 * (is_v ? pos : pos ^ (row & 15)), dst + k * 1024);
    }
  };
  // Fused append: the rows of the current scale go from LDS to their slot as they pass.  Lane i re-reads the 16 bytes
  // its own loads fetched.
  // Returns whether it issued exactly kLoads stores (the counted waits behind it then need not wait for them).
  auto store_rows = [&](int b, bool is_v) {
    const int j0 = b * QT;
    if (j0 + QT <= seg.ext_start || b % (kShared ? n_parts : n_qblk) != my_qblk) return false;
    const char* src = kShared ? lds + (b % kRing) * 2 * kBlk + (is_v ? kBlk : 0) : is_v ? lds_v : lds_k;
    char* dst = is_v ? vb : kb;
    const int row0 = lane / CPR, pos = lane % CPR;
    if (__builtin_expect(j0 >= seg.ext_start && j0 >= ext_kv.wb_from && j0 + QT <= t_kv, 1)) {  // every row moves by wb_delta
      dst += (long long)(j0 + ext_kv.wb_delta) * RB;
#pragma unroll
      for (int k = first_load; k < first_load + kMyLoads; ++k) {
        const int row = k * kRowsPerLoad + row0;
        *reinterpret_cast<f32x4*>(dst + row * RB + 16 * (is_v ? pos : pos ^ (row & 15))) =
            *reinterpret_cast<const f32x4*>(src + k * 1024 + 16 * lane);
      }
      return true;
    }
#pragma unroll
    for (int k = first_load; k < first_load + kMyLoads; ++k) {
      const int row = k * kRowsPerLoad + row0, j = j0 + row;
      const int to = write_back_row(ext_kv, j, t_kv, seg.ext_start);
      if (j >= seg.ext_start && to >= 0)
        *reinterpret_cast<f32x4*>(dst + (long long)to * RB + 16 * (is_v ? pos : pos ^ (row & 15))) =
            *reinterpret_cast<const f32x4*>(src + k * 1024 + 16 * lane);
    }
    return false;
  };

  typename M::Acc oacc[NDB];
#pragma unroll
  for (int d = 0; d < NDB; ++d)
#pragma unroll
    for (int v = 0; v < NV; ++v) oacc[d][v] = 0.f;
  float run_ref = -INFINITY, run_sum = 0.f;  // softmax reference (a score); the lane's own sum of 2^((s - reference) * c)
  float pf[NV];                              // probabilities of the block before
  float alpha = 1.f;                         // factor the accumulators still have to be moved by
  bool moved = false;
  bool stored_v = false;  // the step before stored V rows in front of its V loads

  // All but the youngest kLoads loads, and the stores right in front of those, are done.
  auto wait_younger = [](bool stored) {
    if (stored) wait_vmcnt<2 * kLoads>();
    else wait_vmcnt<kLoads>();
  };
  // O^T += V^T P^T of the block whose V is in LDS and whose probabilities are pf.  `valid` (the last block only): how many of
  // its rows are keys; the others hold the last key again and weigh 0, which would make NaN of an infinity there.
  auto multiply_v = [&](int v, int valid = QT) {
    const char* vp = lds_v + M::row(v, g) * RB + (NDB == 2 ? 8 : 16) * r;
    float a[NDB];
    if constexpr (NDB == 2) {
      const float2 x = *reinterpret_cast<const float2*>(vp);
      a[0] = x.x;
      a[1] = x.y;
    } else {
#pragma unroll
      for (int i = 0; i < NDB / 4; ++i) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(vp + 16 * QT * i);
#pragma unroll
        for (int e = 0; e < 4; ++e) a[4 * i + e] = x[e];
      }
    }
    if (__builtin_expect(valid < QT, 0)) {
#pragma unroll
      for (int d = 0; d < NDB; ++d) a[d] = M::row(v, g) < valid ? a[d] : 0.f;
    }
#pragma unroll
    for (int d = 0; d < NDB; ++d) oacc[d] = M::mul(a[d], pf[v], oacc[d]);
  };
  auto rescale = [&]() {
    if (__builtin_expect(moved, 0)) {
#pragma unroll
      for (int d = 0; d < NDB; ++d)
#pragma unroll
        for (int v = 0; v < NV; ++v) oacc[d][v] *= alpha;
    }
  };

  // One key block: its scores, its softmax next to the second product of the block before (they share no data, so the
  // vector work runs in the shadow of the matrix instructions), then the fetch of its V behind that product.
  auto step = [&](int b, bool first) {
    const int j0 = b * QT;
    const bool more = b + kSplit < n_blocks;
    rescale();
    if (!kShared && !first) wait_younger(stored_v);  // K of this block; V of the block before may still be on the way
    // A dot product is 16 partial sums (eight in a 32-row unit) that meet in additions: an accumulator that takes all D
    // products rounds D times, and at the size the sum has by then.  So the error is no larger than that of a kernel whose
    // four lanes per query summed fours on the vector ALU.  rel against 64 bits, one accumulator (16-row units: four) / these
    // / the four lanes: 32-row units 32 x 32 keys 2.40e-7 / 1.53e-7 / 1.65e-7, 256 x 424 4.66 / 3.93 / 3.97, 1024 x 1621 7.83 /
    // 7.39 / 7.44; 16-row units 25 x 55 1.48 / 1.38 / 1.83, head dim 128 2 x 4 0.97 / 0.85 / 0.85, 256 x 680 5.00 / 4.89 / 4.94.
    // us, before / now: 256 (b,h), 256 x 680 105 / 113 (16 sums in the 32-row unit too: 120), head dim 128 209 / 221; 16 (b,h)
    // 13.5 / 14.5; 64 (b,h), 1024 x 2645 348 / 387.
    constexpr int kChain = QT == 32 ? 4 : D / 16 / H;  // matrix instructions of one partial sum (two or four products each)
    typename M::Acc s;
#pragma unroll
    for (int i = 0; i < NC; i += kChain) {
      f32x4 kv[kChain];
#pragma unroll
      for (int u = 0; u < kChain; ++u) kv[u] = *reinterpret_cast<const f32x4*>(lds_k + r * RB + 16 * ((NC * g + i + u) ^ (r & 15)));
      typename M::Acc four;
#pragma unroll
      for (int e0 = 0; e0 < 4; e0 += 2) {
        typename M::Acc part[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
#pragma unroll
          for (int v = 0; v < NV; ++v) part[e][v] = 0.f;
#pragma unroll
          for (int u = 0; u < kChain; ++u) part[e] = M::mul(kv[u][e0 + e], qf[i + u][e0 + e], part[e]);
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) four[v] = e0 == 0 ? part[0][v] + part[1][v] : four[v] + (part[0][v] + part[1][v]);
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) s[v] = i == 0 ? four[v] : s[v] + four[v];
      asm volatile("" : "+v"(s));  // added here, not where the scores are used: 16 partial sums would not fit the registers
    }
    bool stored_k = false;
    if constexpr (!kShared) {
      stored_k = write_back && store_rows(b, false);
      wait_lds_reads();
      if (more) load(b + kSplit, false);
    }
    if (__builtin_expect(j0 + QT > t_kv, 0)) {
#pragma unroll
      for (int v = 0; v < NV; ++v)
        if (j0 + M::row(v, g) >= t_kv) s[v] = -INFINITY;
    }
    // The probabilities are formed against the reference of the blocks before; their sum tells whether that was good
    // enough.  Only where it was not (always in the first block) is the maximum taken.
    float sum = INFINITY;
    if (!first) {
      if constexpr (!kShared) {
        if (more) wait_younger(stored_k);  // V of the block before; the next K may still be on the way
        else wait_vmcnt<0>();
      }
      sum = 0.f;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        multiply_v(v);
        pf[v] = __builtin_amdgcn_exp2f((s[v] - run_ref) * scale_log2e);
        sum += pf[v];
      }
      if constexpr (!kShared) {
        stored_v = write_back && store_rows(b - kSplit, true);
        wait_lds_reads();
      }
    }
    if constexpr (!kShared) load(b, true);
    moved = __builtin_amdgcn_ballot_w64(!(sum <= kTripSum)) != 0;
    if (__builtin_expect(moved, 0)) {
      float mx = s[0];
#pragma unroll
      for (int v = 1; v < NV; ++v) mx = fmaxf(mx, s[v]);
#pragma unroll
      for (int m = QT; m < 64; m <<= 1) mx = fmaxf(mx, __shfl_xor(mx, m, 64));
      const bool move = (mx - run_ref) * scale_log2e > kMaxLag;
      alpha = move ? __builtin_amdgcn_exp2f((run_ref - mx) * scale_log2e) : 1.f;  // 0 on the first block
      run_sum *= alpha;
      run_ref = move ? mx : run_ref;
      const float ref = run_ref == -INFINITY ? 0.f : run_ref;  // no reference yet: every score so far is -inf and weighs 0
      sum = 0.f;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        pf[v] = __builtin_amdgcn_exp2f((s[v] - ref) * scale_log2e);  // the key at the reference weighs exactly 1
        sum += pf[v];
      }
      if (first) moved = false;  // the accumulators are zero
    }
    run_sum += sum;
  };
  if constexpr (kShared) {
    // Two blocks are on their way while one is in use and the V of the one before it still is: the barrier of block b
    // makes it readable and frees the slot of block b - 2, which block b + 2 is requested into.
    for (int b = 0; b < 2 && b < n_blocks; ++b) {
      load(b, false);
      load(b, true);
    }
    if (active) {
#pragma unroll
      for (int i = 0; i < NC; ++i) asm volatile("" : "+v"(qf[i]));  // the Q rows have landed
    }
    for (int b = 0; b < n_blocks; ++b) {
      if (b + 1 < n_blocks) wait_vmcnt<2 * kMyLoads>();  // (stores in between only make this stricter)
      else wait_vmcnt<0>();
      __syncthreads();
      if (write_back) {
        store_rows(b, false);
        store_rows(b, true);
      }
      if (b + 2 < n_blocks) {
        load(b + 2, false);
        load(b + 2, true);
      }
      if (active) {
        lds_k = lds + (b % kRing) * 2 * kBlk;
        lds_v = lds + ((b + kRing - 1) % kRing) * 2 * kBlk + kBlk;
        step(b, b == 0);
      }
    }
    if (!active) return;
    rescale();
    lds_v = lds + ((n_blocks - 1) % kRing) * 2 * kBlk + kBlk;
#pragma unroll
    for (int v = 0; v < NV; ++v) multiply_v(v, t_kv - (n_blocks - 1) * QT);
  } else if (active && slice < n_blocks) {
    load(slice, false);
#pragma unroll
    for (int i = 0; i < NC; ++i) asm volatile("" : "+v"(qf[i]));  // the Q rows have landed, and
    wait_vmcnt<0>();                                              // the first K
    step(slice, true);
    int b = slice + kSplit;
    for (; b < n_blocks; b += kSplit) step(b, false);
    rescale();
    wait_vmcnt<0>();
#pragma unroll
    for (int v = 0; v < NV; ++v) multiply_v(v, t_kv - (b - kSplit) * QT);
    if (write_back) store_rows(b - kSplit, true);
  }

  // oacc[d][v] is channel 2*row(v,g) + d of query row r where O^T has two row blocks, else channel
  // 4*QT*(d/4) + 4*row(v,g) + d%4 (as the V operand was read): runs of four consecutive channels either way.
  float total = run_sum;
#pragma unroll
  for (int m = QT; m < 64; m <<= 1) total += __shfl_xor(total, m, 64);
  constexpr int kChunks = NV * NDB / 4;
  char* o_row = (char*)o + unit_offset(io.o, bh, io.heads) + (long long)(q_base + r) * io.o.tok;
  const bool row_ok = q_base + r < t_q;
  // chunk c: four consecutive channels, from channel(c) on
  auto value = [&](int c, int e) { return NDB == 2 ? oacc[e & 1][2 * c + (e >> 1)] : oacc[4 * (c / NV) + e][c % NV]; };
  auto channel = [&](int c) { return NDB == 2 ? 2 * M::row(2 * c, g) : 4 * QT * (c / NV) + 4 * M::row(c % NV, g); };
  if constexpr (kSplit == 1) {
    const float inv = 1.0f / total;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      f32x4 x;
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = value(c, e) * inv;
      if (row_ok) *reinterpret_cast<f32x4*>(o_row + 4 * channel(c)) = x;
    }
  } else {
    // partial results of the slices: every wave parks its own, then takes a share of the channels of all
    float* stat = reinterpret_cast<float*>(lds + kWaves * 2 * kBlk);  // [wave][2][QT]: reference, sum
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      f32x4 x;
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = value(c, e);
      *reinterpret_cast<f32x4*>(lds_k + c * 1024 + lane * 16) = x;
    }
    if (g == 0) {
      stat[(2 * wave) * QT + r] = run_ref;  // -inf, sum 0 for a slice without blocks
      stat[(2 * wave + 1) * QT + r] = total;
    }
    __syncthreads();
    const int w0 = wave - slice;
    float top = -INFINITY;
#pragma unroll
    for (int p = 0; p < kSplit; ++p) top = fmaxf(top, stat[2 * (w0 + p) * QT + r]);
    float weight[kSplit], sum = 0.f;
#pragma unroll
    for (int p = 0; p < kSplit; ++p) {
      weight[p] = __builtin_amdgcn_exp2f((stat[2 * (w0 + p) * QT + r] - top) * scale_log2e);
      sum = fmaf(weight[p], stat[(2 * (w0 + p) + 1) * QT + r], sum);
    }
    const float inv = 1.0f / sum;
#pragma unroll
    for (int c0 = 0; c0 < kChunks; c0 += kSplit) {
      const int c = c0 + slice;
      if (kChunks % kSplit != 0 && c >= kChunks) break;
      f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int p = 0; p < kSplit; ++p) {
        const f32x4 y = *reinterpret_cast<const f32x4*>(lds + (w0 + p) * 2 * kBlk + c * 1024 + lane * 16);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = fmaf(weight[p], y[e], x[e]);
      }
      x *= inv;
      if (active && row_ok) *reinterpret_cast<f32x4*>(o_row + 4 * channel(c)) = x;
    }
  }
}

template <int D, int QT, int kSplit>
hipError_t launch(const void* q, void* o, void* kc, void* vc, int bh, int t_q, int64_t cap_tokens, const SegTable& seg,
                  const ExtKV& ext, const CallerIo& io, float c, hipStream_t st) {
  constexpr int kWaves = waves_of(kSplit), kUnits = kWaves / kSplit;
  const int n_parts = ((t_q + QT - 1) / QT + kUnits - 1) / kUnits;
  constexpr bool kOnePart = D == 64 && kSplit == 1;  // at most 64 queries (choose_f32())
  if (kOnePart && n_parts > 1) return hipErrorInvalidValue;
  const int n_whole = whole_units(bh, n_parts, kMostWhole);
  dim3 grid(placed_grid(bh, n_parts, n_whole)), block(64 * kWaves);
  const auto kernel = !kOnePart && n_whole < bh ? attend_f32_kernel<D, QT, kSplit, !kOnePart> : attend_f32_kernel<D, QT, kSplit, false>;
  hipLaunchKernelGGL(kernel, grid, block, 0, st, (const float*)q, (float*)o, (float*)kc, (float*)vc,
                     t_q, (long long)cap_tokens, seg, ext, io, c, bh, n_parts, n_whole);
  return hipGetLastError();
}

template <int D, int QT>
hipError_t launch_split(int split, const void* q, void* o, void* kc, void* vc, int bh, int t_q, int64_t cap_tokens,
                        const SegTable& seg, const ExtKV& ext, const CallerIo& io, float c, hipStream_t st) {
  switch (split) {
    case 1:  // (32-row units always split their keys)
      if constexpr (QT == 16) return launch<D, QT, 1>(q, o, kc, vc, bh, t_q, cap_tokens, seg, ext, io, c, st);
      return hipErrorInvalidValue;
    case 2: return launch<D, QT, 2>(q, o, kc, vc, bh, t_q, cap_tokens, seg, ext, io, c, st);
    case 4: return launch<D, QT, 4>(q, o, kc, vc, bh, t_q, cap_tokens, seg, ext, io, c, st);
    default: return launch<D, QT, 8>(q, o, kc, vc, bh, t_q, cap_tokens, seg, ext, io, c, st);
  }
}

}  // namespace

hipError_t launch_attend_f32(const void* q, void* o, void* kc, void* vc, int bh, int t_q,
                             int head_dim, int64_t cap_tokens, const SegTable& seg, const ExtKV& ext,
                             const CallerIo& io, float softmax_scale, hipStream_t st) {
  const float c = softmax_scale * 1.4426950408889634f;
  const F32Choice x = choose_f32(head_dim, bh, t_q, seg.total, softmax_scale);
  if (x.parts) return launch_attend_f32_parts(x.parts, x.split, q, o, kc, vc, bh, t_q, head_dim, cap_tokens, seg, ext, io, softmax_scale, st);
  if (head_dim == 128) return launch_split<128, 16>(x.split, q, o, kc, vc, bh, t_q, cap_tokens, seg, ext, io, c, st);
  return x.qt == 32 ? launch_split<64, 32>(x.split, q, o, kc, vc, bh, t_q, cap_tokens, seg, ext, io, c, st)
                    : launch_split<64, 16>(x.split, q, o, kc, vc, bh, t_q, cap_tokens, seg, ext, io, c, st);
}

}  // namespace amskv
