// Inter-scale similarity (Eq. 3): scale s-1 is resized bilinearly to the grid of scale s on
// the fly (never materialised) and compared with scale s, straight from the cache.
// Each token row is read with 16-byte loads by consecutive lanes.
// Reduction order is fixed (lanes of a token -> lanes of a wave -> waves in order -> strided lanes and an xor tree over
// batch), so the result is deterministic from run to run.
#include "amskv_internal.hpp"

namespace amskv {
namespace {

constexpr int kStaticMaxUnits = AMSKV_STATIC_MAX_UNITS;
constexpr int kMaxDevices = 64;

template <bool BF16>
struct Chunk;  // one 16-byte piece of a token row, widened to fp32

template <>
struct Chunk<true> {
  static constexpr int N = 8;
  float v[8];
  __device__ __forceinline__ void load(const char* p) {
    const uint4 r = *reinterpret_cast<const uint4*>(p);
    const unsigned w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __uint_as_float(w[i] << 16);
      v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
};

template <>
struct Chunk<false> {
  static constexpr int N = 4;
  float v[4];
  __device__ __forceinline__ void load(const char* p) {
    const float4 r = *reinterpret_cast<const float4*>(p);
    v[0] = r.x; v[1] = r.y; v[2] = r.z; v[3] = r.w;
  }
};

// Source coordinate of the bilinear resize with half-pixel centres, clamped to the grid; scale = n_in / n_out.
__device__ __forceinline__ void taps(int dst, int n_in, float scale, int& i0, int& i1, float& lam) {
  float src = ((float)dst + 0.5f) * scale - 0.5f;
  src = fminf(fmaxf(src, 0.f), (float)(n_in - 1));
  const float f = floorf(src);
  i0 = (int)f;
  i1 = min(i0 + 1, n_in - 1);
  lam = src - f;
}

// Sum over the lanes of a wave, in every one of them: lane l takes l^32, then l^16, l^8, ... l^1, each step on the vector ALU.  (Lanes that
// agree modulo 8 may take the one four lanes back in their row of 16 for l^4.)
__device__ __forceinline__ float wave_sum(float x) {
  x = half_sum(x);
  const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_int(x), __float_as_int(x), false, false);
  x = __int_as_float(sw[0]) + __int_as_float(sw[1]);
  x = add_lane<0x128>(x);  // row_ror:8
  x = add_lane<0x124>(x);  // row_ror:4
  x = add_lane<0x4E>(x);   // quad_perm 2 3 0 1
  return add_lane<0xB1>(x);  // quad_perm 1 0 3 2
}

// grid: (B*H / kUnits, tensors); kThreads threads per (b,h) of one tensor (0 = keys, 1 = values), kUnits (b,h) to a workgroup.
// partial[(tensor*BH + bh)*4 + {0,1,2,3}] = sum_t cos_t, sum a.b, sum |a|^2, sum |b|^2.
// Bound: HBM at the fine scales (the rows of scale s once, those of s-1 once and from L2 after that), next to the vector
// ALU, so what a token costs beside its multiply-adds is kept down: the four bilinear weights are formed once per token,
// sums over its lanes run on the ALU, and the cosine's square roots and quotient, which every lane of a wave would execute
// for the one lane that needs them, run once for kLanes passes, each lane of a token keeping the sums of one of them.
// (di, dj): how far one pass moves a thread's token on the grid.
template <bool BF16, int kLanes, int kThreads, int kUnits>
__global__ __launch_bounds__(kThreads * kUnits) void similarity_partial_kernel(
    ScaleRef cur_ref, ScaleRef prev_ref, int n_bh, int heads, int h_cur, int w_cur, int h_prev, int w_prev, float scale_h, float scale_w,
    int di, int dj, float* __restrict__ partial) {
  static_assert(kUnits == 1 || kThreads == 64, "a (b,h) of several to a workgroup has one wave: nothing synchronises them");
  fetch_arguments<2 * sizeof(ScaleRef) + 40>();
  const int thread = kUnits == 1 ? threadIdx.x : threadIdx.x & 63;
  const long long bh = kUnits == 1 ? blockIdx.x : blockIdx.x * kUnits + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (kUnits > 1 && bh >= n_bh) return;
  const char* cur = (const char*)(blockIdx.y ? cur_ref.v : cur_ref.k) + unit_offset(cur_ref.map, bh, heads) +
                    cur_ref.off_tokens * cur_ref.map.tok;
  const char* prev = (const char*)(blockIdx.y ? prev_ref.v : prev_ref.k) + unit_offset(prev_ref.map, bh, heads) +
                     prev_ref.off_tokens * prev_ref.map.tok;
  const long long cur_tok = cur_ref.map.tok, prev_tok = prev_ref.map.tok;
  const int sub = thread % kLanes;  // which 16-byte piece of the row
  const int slot = thread / kLanes;
  constexpr int kPerPass = kThreads / kLanes;
  const int t_cur = h_cur * w_cur;
  cur += sub << 4;
  prev += sub << 4;

  float acc_cos = 0.f, acc_ab = 0.f, acc_aa = 0.f, acc_bb = 0.f;
  float kept_ab = 0.f, kept_aa = 0.f, kept_bb = 0.f;  // the token whose cosine this lane takes next
  auto take_cosine = [&]() {
    acc_cos += kept_ab / fmaxf(sqrtf(kept_aa) * sqrtf(kept_bb), 1e-12f);  // 0 where nothing is kept
    kept_ab = kept_aa = kept_bb = 0.f;
  };
  int i = slot / w_cur, j = slot - i * w_cur, pass = 0;
  for (int t0 = 0; t0 < t_cur; t0 += kPerPass) {
    const int t = t0 + slot;
    float ab = 0.f, aa = 0.f, bb = 0.f;
    if (t < t_cur) {
      int r0, r1, c0, c1;
      float lr, lc;
      taps(i, h_prev, scale_h, r0, r1, lr);
      taps(j, w_prev, scale_w, c0, c1, lc);
      Chunk<BF16> a, p00, p01, p10, p11;
      a.load(cur + t * cur_tok);
      p00.load(prev + (r0 * w_prev + c0) * prev_tok);
      p01.load(prev + (r0 * w_prev + c1) * prev_tok);
      p10.load(prev + (r1 * w_prev + c0) * prev_tok);
      p11.load(prev + (r1 * w_prev + c1) * prev_tok);
      const float w00 = (1.f - lr) * (1.f - lc), w01 = (1.f - lr) * lc, w10 = lr * (1.f - lc), w11 = lr * lc;
#pragma unroll
      for (int e = 0; e < Chunk<BF16>::N; ++e) {
        const float b = fmaf(w11, p11.v[e], fmaf(w10, p10.v[e], fmaf(w01, p01.v[e], w00 * p00.v[e])));
        ab = fmaf(a.v[e], b, ab);
        aa = fmaf(a.v[e], a.v[e], aa);
        bb = fmaf(b, b, bb);
      }
    }
    acc_ab += ab;
    acc_aa += aa;
    acc_bb += bb;
    ab = group_sum<kLanes>(ab);
    aa = group_sum<kLanes>(aa);
    bb = group_sum<kLanes>(bb);
    if (sub == pass) {
      kept_ab = ab;
      kept_aa = aa;
      kept_bb = bb;
    }
    if (++pass == kLanes) {
      take_cosine();
      pass = 0;
    }
    i += di;
    j += dj;
    if (j >= w_cur) {
      j -= w_cur;
      ++i;
    }
  }
  take_cosine();

  // workgroup sum in a fixed order: xor tree over the lanes of a wave, then the waves in ascending order
  float acc[4] = {acc_cos, acc_ab, acc_aa, acc_bb};
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q] = wave_sum(acc[q]);
  float* out = partial + ((long long)blockIdx.y * n_bh + bh) * 4;
  if constexpr (kThreads == 64) {
    if (thread == 0) *reinterpret_cast<float4*>(out) = make_float4(acc[0], acc[1], acc[2], acc[3]);
    return;
  }
  __shared__ float red[kThreads / 64][4];
  if ((threadIdx.x & 63) == 0)
    for (int q = 0; q < 4; ++q) red[threadIdx.x >> 6][q] = acc[q];
  __syncthreads();
  if (threadIdx.x < 4) {
    float total = red[0][threadIdx.x];
    for (int w = 1; w < kThreads / 64; ++w) total += red[w][threadIdx.x];
    out[threadIdx.x] = total;
  }
}

template <bool BF16, int kLanes, int kThreads, int kUnits = 1>
hipError_t launch_partial(const ScaleRef& cur, const ScaleRef& prev, int bh, int heads, int h_cur, int w_cur, int h_prev, int w_prev,
                          float* partial_ws, hipStream_t st) {
  constexpr int kPerPass = kThreads / kLanes;
  hipLaunchKernelGGL((similarity_partial_kernel<BF16, kLanes, kThreads, kUnits>), dim3((bh + kUnits - 1) / kUnits, cur.v && prev.v ? 2 : 1),
                     dim3(kThreads * kUnits), 0, st, cur, prev, bh, heads, h_cur, w_cur, h_prev, w_prev, (float)h_prev / (float)h_cur, (float)w_prev / (float)w_cur,
                     kPerPass / w_cur, kPerPass % w_cur, partial_ws);
  return hipGetLastError();
}

// totals[(tensor*H + h)*4 + q] = sum over b of partial[(tensor*B*H + b*H + h)*4 + q].
// One 64-lane workgroup per (tensor, h): lane i sums batch entries i, i+64, ... in ascending
// order, then a fixed xor tree joins the lanes -- the same order on every run.
__global__ __launch_bounds__(64) void similarity_total_kernel(const float* __restrict__ partial, int batch, int heads,
                                                              float* __restrict__ totals) {
  const int h = blockIdx.x % heads, tn = blockIdx.x / heads;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int b = threadIdx.x; b < batch; b += 64) {
    const float4 x = *reinterpret_cast<const float4*>(partial + (((long long)tn * batch + b) * heads + h) * 4);
    acc[0] += x.x; acc[1] += x.y; acc[2] += x.z; acc[3] += x.w;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q] = wave_sum(acc[q]);
  if (threadIdx.x == 0)
    *reinterpret_cast<float4*>(totals + ((long long)tn * heads + h) * 4) = make_float4(acc[0], acc[1], acc[2], acc[3]);
}

// Algorithm 1's test on the device: flag = (mean over heads of the mean cosine < theta), from the per-head sums the
// kernel above left (totals[h*4] = sum of the per-token cosines of K).  The arithmetic is spelled out so that the
// host, given the same sums, would decide the same: per head the quotient in double rounded to float, their mean
// in double, compared with theta in double.  (One lane for the quotients too took 4.8 us a launch, this 4.2.)
__global__ __launch_bounds__(64) void theta_flag_kernel(const float* __restrict__ totals, int heads, double n_tok, float theta,
                                                        int32_t* __restrict__ flag, int32_t* __restrict__ flag_host) {
  __shared__ double quotient[64];
  double mean = 0.0;
  for (int h0 = 0; h0 < heads; h0 += 64) {  // the quotients side by side, their sum in order
    const int here = min(64, heads - h0);
    if ((int)threadIdx.x < here) quotient[threadIdx.x] = (double)(float)((double)totals[(h0 + threadIdx.x) * 4] / n_tok);
    __syncthreads();
    if (threadIdx.x == 0)
      for (int h = 0; h < here; ++h) mean += quotient[h];
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  mean /= heads;
  const int32_t word = mean < (double)theta ? 1 : 0;
  *flag = word;       // for the launch behind this one
  *flag_host = word;  // pinned host memory: the host reads it behind the event, no transfer
}

// Partial-sum workspace of the entry point that allocates nothing: per (tensor, b, h) four floats, for up to
// kStaticMaxUnits = batch * heads units and both tensors (512 KB).  Every device the library runs on holds its
// own copy for the life of the process.
__device__ __align__(256) float scratch[2 * kStaticMaxUnits * 4];

// Device address of `scratch` on the current device, looked up once per device (the array's name is only a
// host-side handle).
hipError_t scratch_address(float** out) {
  static float* address[kMaxDevices];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  float* p = __atomic_load_n(&address[dev], __ATOMIC_ACQUIRE);
  if (!p) {
    e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    __atomic_store_n(&address[dev], p, __ATOMIC_RELEASE);  // every caller looks up the same value
  }
  *out = p;
  return hipSuccess;
}

}  // namespace

hipError_t launch_similarity_static(const ScaleRef& cur, const ScaleRef& prev, int batch, int heads, int head_dim,
                                    int dtype, int h_cur, int w_cur, int h_prev, int w_prev, float* out_dev,
                                    hipStream_t st) {
  if ((long long)batch * heads > kStaticMaxUnits) return hipErrorInvalidValue;  // the caller checks first
  float* ws = nullptr;
  hipError_t e = scratch_address(&ws);
  if (e != hipSuccess) return e;
  // every partial sum the totals kernel reads is written by the partial kernel of the same call: nothing to clear
  return launch_similarity(cur, prev, batch, heads, head_dim, dtype, h_cur, w_cur, h_prev, w_prev, ws, out_dev, st);
}

hipError_t launch_similarity(const ScaleRef& cur, const ScaleRef& prev, int batch, int heads, int head_dim,
                             int dtype, int h_cur, int w_cur, int h_prev, int w_prev, float* partial_ws,
                             float* out_dev, hipStream_t st) {
  const int tensors = (cur.v && prev.v) ? 2 : 1;
  const int bh = batch * heads;
  // Few (b,h) with rows of some length: four times the threads, so that a row takes a quarter of the passes.  The sums of the
  // keys keep their bits whether the values are asked for or not, so the rule looks at the (b,h) alone.  1024 over 256
  // threads, time, keys / keys and values, by KB of scale s per (b,h): 12 KB 0.95 / 0.95-1.08 up to 240 (b,h), 1.07 / 1.2 at 448;
  // 16-25 KB 0.84-0.97 / 0.84-1.1 up to 240, 1.0-1.1 / 1.05-1.24 at 448; 32-64 KB 0.67-0.88 / 0.67-0.99 up to 240, 0.8-0.98 /
  // 0.93-1.1 at 448; 128 KB and more 0.4-0.65 / 0.4-0.84, 0.7-0.83 / 0.9-1.0; up to 8 KB 1.07-1.3 / 1.07-1.7 everywhere.
  const long long row = (long long)h_cur * w_cur * head_dim * (dtype == AMSKV_DTYPE_BF16 ? 2 : 4);
  const bool few = bh < (row >= 32 << 10 ? 512 : row >= 16 << 10 ? 256 : 0);
  // Many (b,h) with few rows: a wave each, four to a workgroup; with four waves to a (b,h) the launch takes as long as its waves take to
  // start.  A pass of the wave takes 1 KB: up to four of them, and as many (b,h) as make up for the longer chain.  us, keys and values and
  // their totals, four waves / one, by bytes of scale s: 7680 (b,h) 512 23.2 / 11.8, 1152 24.8 / 15.2, 2048 26.4 / 17.9, 3200 30.9 / 29.8, 4608
  // 40.5 / 40.8; 1920 (b,h) 9.7 / 6.3, 10.1 / 7.5, 10.2 / 7.8, 11.3 / 10.4, 13.4 / 12.5, 6272 15.6 / 15.8, 8192 17.2 / 18.7; 576 (b,h) 6.9 / 5.9,
  // 7.0 / 6.4, 7.1 / 6.5, 7.4 / 7.9; 128 (b,h) 6.0 / 5.5, 6.1 / 6.3, 6.0 / 6.1, 6.1 / 7.6.
  const bool waves = row <= 4096 && row <= 4ll * bh;
  auto go = [&](auto f_many, auto f_few, auto f_waves) {
    return (waves ? f_waves : few ? f_few : f_many)(cur, prev, bh, heads, h_cur, w_cur, h_prev, w_prev, partial_ws, st);
  };
  hipError_t e;
  if (dtype == AMSKV_DTYPE_BF16)
    e = head_dim == 64 ? go(launch_partial<true, 8, 256>, launch_partial<true, 8, 1024>, launch_partial<true, 8, 64, 4>)
                       : go(launch_partial<true, 16, 256>, launch_partial<true, 16, 1024>, launch_partial<true, 16, 64, 4>);
  else
    e = head_dim == 64 ? go(launch_partial<false, 16, 256>, launch_partial<false, 16, 1024>, launch_partial<false, 16, 64, 4>)
                       : go(launch_partial<false, 32, 256>, launch_partial<false, 32, 1024>, launch_partial<false, 32, 64, 4>);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(similarity_total_kernel, dim3(tensors * heads), dim3(64), 0, st, (const float*)partial_ws, batch,
                     heads, out_dev);
  return hipGetLastError();
}

hipError_t launch_theta_flag(const float* totals_dev, int heads, double n_tok, float theta, int32_t* flag_dev,
                             int32_t* flag_host_pinned, hipStream_t st) {
  hipLaunchKernelGGL(theta_flag_kernel, dim3(1), dim3(64), 0, st, totals_dev, heads, n_tok, theta, flag_dev, flag_host_pinned);
  return hipGetLastError();
}

}  // namespace amskv
