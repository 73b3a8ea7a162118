// Bandwidth-bound cache kernels: evict + compact + append (Algorithm 1's append and rolling
// step, Algorithm 2's eviction, at scale and at token granularity) and the read-back export.
// All traffic is 16-byte vector loads/stores, consecutive lanes on consecutive chunks.
#include "amskv_internal.hpp"

namespace amskv {
namespace {

constexpr int kThreads = 256;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// What an iteration does to one (b,h) row of one tensor, as ranges of 16-byte chunks in the order they are carried
// out: first the survivors that slide toward offset 0 (sources inside the row), then what is kept of the new scale
// (sources in the caller's tensor).  Range i covers chunks [begin[i], begin[i+1]) of the concatenation of all ranges.
constexpr int kMaxRanges = AMSKV_MAX_SCALES + 2;
struct CopyList {
  int32_t n_moves, n, total;
  int32_t begin[kMaxRanges];  // chunks
  int32_t src[kMaxRanges];    // tokens: of the row, or of the new scale
  int32_t dst[kMaxRanges];    // tokens of the row
};

__device__ __forceinline__ void wait_all_vector_loads() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// One workgroup owns one (b,h) row of one tensor (blockIdx.y: 0 = K, 1 = V).  Its chunks, taken in list order, are
// loaded kChunks per thread at a time; once every load of such a pass has returned (the barrier) they are stored.
// Destinations ascend with the list.  A moved chunk's destination lies below its source, so a store can only hit the
// source of a chunk of the same or an earlier pass; the new scale lands behind the survivors, perhaps where one of them
// used to be, and comes last.
// Bound: HBM.  Most iterations are one pass (up to 256 x 8 or 1024 x 8 chunks, 32 or 128 KB), so all loads of a row --
// survivors and new scale alike -- are in flight at once and the row pays the memory latency once.  Compaction and
// append as two launches (and 16 KB passes through LDS, where the compiler had put the staging array) took 4.6 ms of a
// pass of the ragged 12-layer stack at batch 64, this kernel and append_kernel take 2.7 (63 us for the average step of
// the last two scales, 1536 (b,h), about 5 TB/s read + write); on one image a step's compaction 6-14 -> 5 us.
template <int kBlock, int kChunks>
__global__ __launch_bounds__(kBlock) void roll_kernel(char* __restrict__ kc, char* __restrict__ vc,
                                                      const char* __restrict__ k_new, const char* __restrict__ v_new,
                                                      int row_shift, long long cap_tokens, CopyList cl, RowMap src_map,
                                                      int heads) {
  fetch_arguments<4 * 8 + 16 + sizeof(CopyList) + sizeof(RowMap)>();
  const long long bh = blockIdx.x;
  char* base = (blockIdx.y ? vc : kc) + ((bh * cap_tokens) << row_shift);
  const char* ext = (blockIdx.y ? v_new : k_new) + unit_offset(src_map, bh, heads);
  const int cpr_shift = row_shift - 4;

  for (int c0 = 0; c0 < cl.total; c0 += kBlock * kChunks) {
    int src_tok[kChunks], dst_tok[kChunks], piece[kChunks], moved_end = cl.n_moves < cl.n ? cl.begin[cl.n_moves] : cl.total;
#pragma unroll
    for (int u = 0; u < kChunks; ++u) src_tok[u] = dst_tok[u] = piece[u] = 0;
    for (int i = 0; i < cl.n; ++i) {  // the range of every chunk (uniform values, one walk for all chunks of the thread)
      const int begin = cl.begin[i], src = cl.src[i], dst = cl.dst[i];
#pragma unroll
      for (int u = 0; u < kChunks; ++u) {
        const int rel = c0 + u * kBlock + (int)threadIdx.x - begin;
        if (rel >= 0) {
          src_tok[u] = src + (rel >> cpr_shift);
          dst_tok[u] = dst + (rel >> cpr_shift);
          piece[u] = (rel & ((1 << cpr_shift) - 1)) << 4;
        }
      }
    }
    u32x4 buf[kChunks];
#pragma unroll
    for (int u = 0; u < kChunks; ++u) {
      const int c = c0 + u * kBlock + (int)threadIdx.x;
      if (c < cl.total) {
        const char* p = c < moved_end ? base + ((long long)src_tok[u] << row_shift) : ext + src_tok[u] * src_map.tok;
        buf[u] = *reinterpret_cast<const u32x4*>(p + piece[u]);
      }
    }
    if (cl.n_moves > 0) {  // uniform; without moves nothing that is read is ever written
      wait_all_vector_loads();
      __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < kChunks; ++u)
      if (c0 + u * kBlock + (int)threadIdx.x < cl.total)
        *reinterpret_cast<u32x4*>(base + ((long long)dst_tok[u] << row_shift) + piece[u]) = buf[u];
  }
}

// Append without compaction: tokens [src_first, src_first + t_new) of every (b,h) row of the new scale (the caller's
// tensors, rows located by src_map) go to their slot of that row; the token-granular trim of Algorithm 2 keeps a scale
// in part, hence the range.  blockIdx.y: 0 = K, 1 = V.  A workgroup takes `rows` whole rows where they are short (one
// token of head dim 64 is 128 bytes), else an equal part of one, so every launch runs full workgroups.
// Bound: HBM.  The position of a chunk comes from one multiplication (`inv` = 2^32 / chunks of a row, rounded up, exact
// for the kRowChunks positions of a workgroup) and shifts; with two 64-bit divisions per chunk and the staging array in
// LDS a launch took 18 us before it moved anything to speak of (1920 rows of 16 tokens: 20.3 us, 7.1 now; of 64 tokens:
// 25.7, 14.8 now = 4.2 TB/s read + write).
constexpr int kChunksPerThread = 4;
constexpr int kRowChunks = kThreads * kChunksPerThread;
__global__ __launch_bounds__(kThreads) void append_kernel(char* __restrict__ kc, char* __restrict__ vc,
                                                          const char* __restrict__ k_new, const char* __restrict__ v_new,
                                                          int row_shift, long long cap_tokens, int chunks, unsigned inv,
                                                          int rows, int parts, int dst_new, int src_first, RowMap src_map,
                                                          int heads, int n_bh) {
  fetch_arguments<4 * 8 + 16 + 24 + sizeof(RowMap)>();
  char* cache = blockIdx.y ? vc : kc;
  const char* src = blockIdx.y ? v_new : k_new;
  const int cpr_shift = row_shift - 4;
  const unsigned group = parts == 1 ? blockIdx.x : blockIdx.x / (unsigned)parts;
  const int first = (int)(blockIdx.x - group * parts) * kRowChunks;  // of the row's chunks (0 where rows are taken whole)
  const int total = parts == 1 ? rows * chunks : chunks - first;     // this workgroup's chunks
  u32x4 buf[kChunksPerThread];
  long long to[kChunksPerThread];
#pragma unroll
  for (int u = 0; u < kChunksPerThread; ++u) {
    const int i = u * kThreads + (int)threadIdx.x;
    to[u] = -1;
    if (i < total) {
      const int row = parts == 1 ? (int)__umulhi((unsigned)i, inv) : 0;
      const int c = first + i - row * chunks, tok = c >> cpr_shift, piece = (c & ((1 << cpr_shift) - 1)) << 4;
      const long long bh = (long long)group * rows + row;
      if (bh < n_bh) {
        to[u] = ((bh * cap_tokens + dst_new + tok) << row_shift) + piece;
        buf[u] = *reinterpret_cast<const u32x4*>(src + unit_offset(src_map, bh, heads) + (src_first + tok) * src_map.tok + piece);
      }
    }
  }
#pragma unroll
  for (int u = 0; u < kChunksPerThread; ++u)
    if (to[u] >= 0) *reinterpret_cast<u32x4*>(cache + to[u]) = buf[u];
}

// Gather the resident segments, ascending and back to back, into [BH][T_kept][row].
__global__ __launch_bounds__(kThreads) void export_kernel(const char* __restrict__ kc,
                                                          const char* __restrict__ vc, char* __restrict__ k_out,
                                                          char* __restrict__ v_out, int row_bytes,
                                                          long long cap_tokens, SegTable seg, ExtKV ext_kv,
                                                          RowMap ext_map, int heads) {
  const long long bh = blockIdx.x;
  const char* base = (blockIdx.y ? vc : kc) + bh * cap_tokens * row_bytes;
  const char* xbase = (const char*)(blockIdx.y ? ext_kv.v : ext_kv.k) + unit_offset(ext_map, bh, heads);
  char* out = blockIdx.y ? v_out : k_out;
  if (!out) return;
  out += bh * (long long)seg.total * row_bytes;
  const int cpr = row_bytes >> 4;
  const int n = seg.total * cpr;
  for (int c = threadIdx.x; c < n; c += kThreads) {
    const int tok = c / cpr, piece = c - tok * cpr;
    bool ext;
    const long long at = locate_row(seg, tok, ext);
    const char* src = ext ? xbase + at * ext_map.tok : base + at * row_bytes;
    *reinterpret_cast<uint4*>(out + ((long long)c << 4)) = *reinterpret_cast<const uint4*>(src + (piece << 4));
  }
}

}  // namespace

hipError_t launch_append(void* kc, void* vc, const void* k_new, const void* v_new, int bh, int row_bytes,
                         int64_t cap_tokens, const MoveList& mv, int t_new, int dst_new, int src_first,
                         const RowMap& src_map, int heads, hipStream_t st) {
  const bool copies = k_new && t_new > 0;  // else the scale is borrowed: compaction only
  if (mv.n > 0) {
    NewRanges nr{};
    if (copies) {
      nr.n = 1;
      nr.src_first[0] = src_first;
      nr.dst[0] = dst_new;
      nr.len[0] = t_new;
    }
    return launch_roll(kc, vc, k_new, v_new, bh, row_bytes, cap_tokens, mv, nr, src_map, heads, st);
  }
  if (!copies) return hipSuccess;
  const int row_shift = __builtin_ctz((unsigned)row_bytes);  // 128, 256 or 512 bytes
  const int chunks = t_new << (row_shift - 4);               // at most 2^25 (t_new <= 2^20)
  const int rows = chunks <= kRowChunks ? kRowChunks / chunks : 1;
  const int parts = (chunks + kRowChunks - 1) / kRowChunks;
  const unsigned inv = (unsigned)((0x100000000ull + chunks - 1) / chunks);
  const unsigned grid = (unsigned)((bh + rows - 1) / rows) * (unsigned)parts;
  hipLaunchKernelGGL(append_kernel, dim3(grid, 2), dim3(kThreads), 0, st, (char*)kc, (char*)vc, (const char*)k_new,
                     (const char*)v_new, row_shift, (long long)cap_tokens, chunks, inv, rows, parts, dst_new, src_first, src_map,
                     heads, bh);
  return hipGetLastError();
}

hipError_t launch_roll(void* kc, void* vc, const void* k_new, const void* v_new, int bh, int row_bytes,
                       int64_t cap_tokens, const MoveList& mv, const NewRanges& nr, const RowMap& src_map, int heads,
                       hipStream_t st) {
  const int row_shift = __builtin_ctz((unsigned)row_bytes);
  CopyList cl{};
  auto add = [&](int src, int dst, int len, bool move) {
    if (len <= 0) return;
    // survivors that lay back to back and still do are one range
    const int last = cl.n - 1;
    const int last_len = last >= 0 ? (cl.total - cl.begin[last]) >> (row_shift - 4) : 0;
    if (move && last >= 0 && cl.src[last] + last_len == src && cl.dst[last] + last_len == dst) {
      cl.total += len << (row_shift - 4);
      return;
    }
    cl.begin[cl.n] = cl.total;
    cl.src[cl.n] = src;
    cl.dst[cl.n] = dst;
    ++cl.n;
    if (move) cl.n_moves = cl.n;
    cl.total += len << (row_shift - 4);
  };
  for (int i = 0; i < mv.n; ++i) add(mv.src[i], mv.dst[i], mv.len[i], true);
  for (int i = 0; i < nr.n; ++i) add(nr.src_first[i], nr.dst[i], nr.len[i], false);
  if (cl.total == 0) return hipSuccess;
  auto go = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3(bh, 2), dim3(threads), 0, st, (char*)kc, (char*)vc, (const char*)k_new, (const char*)v_new,
                       row_shift, (long long)cap_tokens, cl, src_map, heads);
    return hipGetLastError();
  };
  // the smallest workgroup that takes the row in one pass; few rows get the threads of a large one
  if (cl.total <= 1024 && bh >= 128) return go(roll_kernel<256, 4>, 256);
  if (cl.total <= 2048 && bh >= 128) return go(roll_kernel<256, 8>, 256);
  return go(roll_kernel<1024, 8>, 1024);
}

hipError_t launch_export(const void* kc, const void* vc, void* k_out, void* v_out, int bh, int row_bytes,
                         int64_t cap_tokens, const SegTable& seg, const ExtKV& ext, const RowMap& ext_map, int heads,
                         hipStream_t st) {
  dim3 grid(bh, 2), block(kThreads);
  hipLaunchKernelGGL(export_kernel, grid, block, 0, st, (const char*)kc, (const char*)vc, (char*)k_out,
                     (char*)v_out, row_bytes, (long long)cap_tokens, seg, ext, ext_map, heads);
  return hipGetLastError();
}

}  // namespace amskv
