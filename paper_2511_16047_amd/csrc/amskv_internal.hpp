// Internal declarations shared by the host layer and the kernel launchers of libamskv.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "amskv.h"

namespace amskv {

// Resident segments of one layer as the attention kernel walks them: segment i holds
// `len[i]` tokens; in the virtual concatenation K~ of Section 3.1's per-step attention it
// covers rows [virt_start[i], virt_start[i]+len[i]); in the layer's K/V regions it sits at
// token offset phys_off[i].  Passed to kernels by value (lives in scalar registers).
// A borrowed current scale (read in place from the caller's K/V, never copied) is always the
// last segment: it covers virtual rows [ext_start, total) and its rows come from the external
// pointers handed to the kernel next to the table; ext_start == total when nothing is borrowed.
struct SegTable {
  int32_t n;
  int32_t total;      // sum of len = T_kv
  int32_t ext_start;  // first virtual row of the borrowed segment (== total: none)
  int32_t virt_start[AMSKV_MAX_SCALES];
  int32_t phys_off[AMSKV_MAX_SCALES];
  int32_t len[AMSKV_MAX_SCALES];
};

// Groups of keys of the virtual concatenation, for the attention density: group i covers virtual rows
// [end[i-1], end[i]) (from 0 for the first); end[n-1] == SegTable::total.
struct GroupEnds {
  int32_t n;
  int32_t end[AMSKV_MAX_SCALES];
};

// External (borrowed) K and V of the current scale in the caller's buffers (rows located by
// CallerIo::kv), or null pointers.
// The attention kernel can also write rows it streams into the layer's K/V regions (the append fused into the
// attention of its step; in the token modes a whole iteration of Algorithm 1 -- survivors slide toward offset 0,
// what stays of the new scale lands behind them): row j of the virtual concatenation goes to token offset
// j + wb_delta when j >= wb_from, and to token offset j when ext_start <= j < wb_head_end.  Nothing is written with
// wb_from >= total and wb_head_end <= ext_start (kNoWriteBack, 0).  A destination never lies above its source row,
// and rows are streamed in ascending order by the one workgroup (or wave) that owns the unit, so a row is
// overwritten only after that owner has fetched it; callers ask for cached rows to be moved only for launches
// with one owner per unit (attend_owns_unit).
// When the outcome of the iteration hangs on an Eq. 3 test that is decided on the device just before the launch,
// both outcomes are handed over: alt_if points at the device word the test leaves (non-zero: the layer is
// cache-demanding, the budget grows) and the alt_ triple replaces the wb_ triple when it is set.
constexpr int32_t kNoWriteBack = 0x7fffffff;
struct ExtKV {
  const void* k;
  const void* v;
  int32_t wb_from, wb_delta, wb_head_end;
  const int32_t* alt_if;
  int32_t alt_from, alt_delta, alt_head_end;
};
__host__ __device__ inline bool writes_back(const ExtKV& e, int total, int ext_start) {
  return e.wb_from < total || e.wb_head_end > ext_start;
}
#if defined(__HIPCC__)
// the write-back the launch is to perform, the device's decision applied (uniform over the launch)
__device__ inline ExtKV chosen(ExtKV e) {
  if (e.alt_if != nullptr && *e.alt_if != 0) {
    e.wb_from = e.alt_from;
    e.wb_delta = e.alt_delta;
    e.wb_head_end = e.alt_head_end;
  }
  e.alt_if = nullptr;
  return e;
}
#endif
// token offset row j is written to, or -1
__host__ __device__ inline int write_back_row(const ExtKV& e, int j, int total, int ext_start) {
  if (j >= total) return -1;
  if (j >= e.wb_from) return j + e.wb_delta;
  return j >= ext_start && j < e.wb_head_end ? j : -1;
}

// Where the rows of a tensor owned by the caller sit: row t of unit (b, h) starts, in bytes from
// the tensor's base, at b*batch + h*head + t*tok (the D channels of a row are contiguous).
// Head-major [B][H][T][D] gives {H*T*D, T*D, D} * element size; token-major [B][T][..H*D..] with a
// token stride of `tok` elements gives {T*tok, D, tok} * element size.
struct RowMap {
  int64_t batch, head, tok;
};

// Maps of the tensors one attention call touches besides the cache: Q, O and the current scale's
// own K/V when it is read in place (ExtKV); `heads` splits the unit index bh into (b, h).
struct CallerIo {
  RowMap q, o, kv;
  int32_t heads;
};

// Token ranges that slide toward lower offsets when scales are evicted (COMPACT layout),
// in ascending order of offset; dst < src for every entry.
struct MoveList {
  int32_t n;
  int32_t src[AMSKV_MAX_SCALES];
  int32_t dst[AMSKV_MAX_SCALES];
  int32_t len[AMSKV_MAX_SCALES];
};

// Token ranges of the newest scale that Algorithm 2's trim keeps (its head while the cache is still
// shorter than the condensed part, and its tail): tokens [src_first, src_first + len) go to offset dst.
struct NewRanges {
  int32_t n;
  int32_t src_first[2];
  int32_t dst[2];
  int32_t len[2];
};

// Workgroup id -> unit (b,h) and query tile; bh >= n_bh: none.  Consecutive ids go round-robin to the 8 XCDs, each with its own L2,
// so the query tiles of one (b,h) are given ids 8 apart: they run on one XCD back to back, the second one finds K~ and V~ in that
// L2 -- and so does the first what the append in front of the launch left there, whose workgroups are dealt to the XCDs in the same
// way.  The units that are left when n_bh is no multiple of 8 would keep as many XCDs busy: if that puts more than `most` tiles on
// an XCD, which has 32 CUs, their tiles are dealt to all 8 in equal shares.  us: bf16, 4 (b,h), 1600 x 4240 47 -> 27, 9 (b,h), 576 x 1152
// 16.5 -> 10.0; fp32, head dim 128, 1 (b,h), 1600 x 1612 170 -> 44, 9 (b,h), 1600 x 1600 274 -> 144.  (Equal shares of all units: as fast,
// but a layer of fp32 on one image loses what the append left, 113 -> 118 us.)  With few tiles the L2 counts for more; each kernel has
// its own `most`, measured beside it.
struct Place {
  int bh, tile;
};
// units that stay on one XCD each: all of them, rounded up to whole groups of 8, or the whole groups only
inline int whole_units(int n_bh, int n_tiles, int most) {
  return n_tiles > 1 && ((long long)n_bh + 7) / 8 * n_tiles > most ? n_bh & ~7 : (int)(((long long)n_bh + 7) / 8 * 8);
}
// kShares: n_whole < n_bh is possible.  (The fp32 kernel of small launches comes in both forms: one layer on one image takes 112.5 us
// with the branch and 112.0 without, whose runs differ by 0.2.  bf16 in both forms: nothing that goes beyond what runs differ by, 1.000 of
// the time at 16 layers on 1 and on 32 images, 1.001 at six layers on 256.)
template <bool kShares>
__host__ __device__ inline Place place(unsigned id, int n_bh, int n_tiles, int n_whole) {
  const unsigned per_group = 8u * n_tiles, group = id / per_group, within = id - group * per_group;
  Place at{(int)(group * 8 + (within & 7)), (int)(within >> 3)};
  if (kShares && __builtin_expect((int)(group * 8 + 8) > n_whole, 0)) {
    const unsigned all = (n_bh - group * 8) * n_tiles, share = all >> 3, more = all & 7, xcd = within & 7, nth = within >> 3;
    if (nth >= share + (xcd < more ? 1 : 0)) return {n_bh, 0};
    const unsigned item = xcd * share + (xcd < more ? xcd : more) + nth, unit = item / (unsigned)n_tiles;
    at = {(int)(group * 8 + unit), (int)(item - unit * n_tiles)};
  }
  return at;
}
// workgroups of a launch that gives n_tiles of them to each (b,h)
inline unsigned placed_grid(int n_bh, int n_tiles, int n_whole) {
  const long long left = n_bh > n_whole ? n_bh - n_whole : 0;
  return (unsigned)((long long)n_whole * n_tiles + (left * n_tiles + 7) / 8 * 8);
}

#if defined(__HIPCC__)
// Asks for every 64-byte line of the kernel's arguments (the first kBytes of them) at once, and waits.  The arguments of a launch are
// cold, and the compiler loads them piece by piece as it needs them, behind the branches that need them: a workgroup waited for four or
// five such misses in a row, 0.3 us each.  us a pass, before / with it: 16 bf16 layers on one image 1016 / 853 (160 launches), on 32
// images 2073 / 1941, one fp32 layer on one image 112.1 / 105.8 (20), six layers on 256 images 7494 / 7406 (72).
template <int kBytes>
__device__ __forceinline__ void fetch_arguments() {
  typedef const __attribute__((address_space(4))) int* Args;
  const Args p = (Args)__builtin_amdgcn_kernarg_segment_ptr();
  auto line = [&](int i) { return p[16 * i < kBytes / 4 ? 16 * i : kBytes / 4 - 1]; };
  static_assert(kBytes <= 9 * 64, "lines asked for below");
  asm volatile("" ::"s"(line(0)), "s"(line(1)), "s"(line(2)), "s"(line(3)), "s"(line(4)), "s"(line(5)), "s"(line(6)), "s"(line(7)),
               "s"(line(8)));
}
// the arguments of an attention kernel up to its CallerIo: what every workgroup needs before its first load.  (The numbers behind it mostly share its
// last line; the ends of the density's groups and `partial` are loaded where a group ends, and the kernels that copy by a table or form the fp32
// density by itself do without this.)
constexpr int kAttentionArguments = 4 * 8 + 16 + sizeof(SegTable) + sizeof(ExtKV) + sizeof(CallerIo);

// x plus its value in the lane that the cross-lane pattern pairs with this one, on the vector ALU
template <int kPattern>
__device__ __forceinline__ float add_lane(float x) {
  return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kPattern, 0xf, 0xf, false));
}

// Sum over the kLanes (8, 16 or 32) consecutive lanes of an aligned group, in every one of them: pairs, quads, then
// mirrored halves of 8 and of 16 lanes (whose quads, and then halves, already agree).
template <int kLanes>
__device__ __forceinline__ float group_sum(float x) {
  x = add_lane<0xB1>(x);   // quad_perm 1 0 3 2
  x = add_lane<0x4E>(x);   // quad_perm 2 3 0 1
  x = add_lane<0x141>(x);  // row_half_mirror
  if (kLanes >= 16) x = add_lane<0x140>(x);  // row_mirror
  if (kLanes >= 32) x += __shfl_xor(x, 16, 64);
  return x;
}

// Sum of x over the two lane halves (lanes l and l^32), in every lane.
__device__ __forceinline__ float half_sum(float x) {
  const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_int(x), __float_as_int(x), false, false);
  return __int_as_float(sw[0]) + __int_as_float(sw[1]);
}
#endif

#if defined(__HIPCC__)
// Byte offset of row 0 of unit bh = b*heads + h inside a caller tensor.
__device__ __forceinline__ long long unit_offset(const RowMap& m, long long bh, int heads) {
  if (m.batch == m.head * heads) return bh * m.head;  // units back to back (head-major tensors): no division
  const unsigned b = (unsigned)bh / (unsigned)heads;   // bh < 2^24 (checked at create)
  return (long long)b * m.batch + (long long)((unsigned)bh - b * (unsigned)heads) * m.head;
}

// Virtual row j of K~/V~ -> row index inside the layer's cache region of this (b,h), or, for a
// row of the borrowed segment, row index inside the external tensor of this (b,h) (ext = true).
__device__ __forceinline__ int locate_row(const SegTable& seg, int j, bool& ext) {
  ext = j >= seg.ext_start;
  int delta = -seg.ext_start;
  if (!ext) {
    delta = 0;
    for (int g = 0; g < seg.n; ++g)
      if (j >= seg.virt_start[g]) delta = seg.phys_off[g] - seg.virt_start[g];
  }
  return j + delta;
}
#endif

// ---- kernel launchers (each validates nothing: the host layer has checked shapes) ----
// kc/vc are written only where writes_back() says so (fused append, moves of cached rows)
hipError_t launch_attend_bf16(const void* q, void* o, void* kc, void* vc, int bh,
                              int t_q, int head_dim, int64_t cap_tokens, const SegTable& seg,
                              const ExtKV& ext, const CallerIo& io, float softmax_scale, hipStream_t st);
// The launch gives every (b,h) to one workgroup (or, on the coarse scales, one wave) where it writes over cached rows: the
// condition for asking it to move any (ExtKV).  The dispatch sees from the tables whether a launch does; others may share a (b,h).
bool attend_owns_unit(int head_dim, int t_q);
// The attention of a step with the attention density of its queries as a by-product: as launch_attend_bf16, plus
// the per-head masses of the groups in out_dev (heads * AMSKV_MAX_SCALES floats; workspace as for launch_density).
hipError_t launch_attend_density_bf16(const void* q, void* o, void* kc, void* vc, int batch, int heads, int t_q, int head_dim,
                                      int64_t cap_tokens, const SegTable& seg, const ExtKV& ext, const CallerIo& io,
                                      float softmax_scale, const GroupEnds& groups, float* partial_ws, float* out_dev,
                                      hipStream_t st);
// split: how many waves share the key blocks of a 32-row unit (1; 4; 8 at head dim 64); partial: nullptr, or the workspace
// that takes the masses of `groups`
hipError_t launch_attend_bf16_small(const void* q, void* o, void* kc, void* vc, int bh, int t_q,
                                    int head_dim, int64_t cap_tokens, const SegTable& seg,
                                    const ExtKV& ext, const CallerIo& io, float softmax_scale, int split,
                                    const GroupEnds& groups, float* partial, hipStream_t st);
hipError_t launch_attend_f32(const void* q, void* o, void* kc, void* vc, int bh,
                             int t_q, int head_dim, int64_t cap_tokens, const SegTable& seg,
                             const ExtKV& ext, const CallerIo& io, float softmax_scale, hipStream_t st);
// the same in bf16 parts (attend_f32_parts.hip); row_waves: waves of 32 query rows per workgroup (8 or 4), split: waves that share
// their key blocks (1; 2 with 4 row waves); head dim 128 has 4 and 1
hipError_t launch_attend_f32_parts(int row_waves, int split, const void* q, void* o, void* kc, void* vc, int bh, int t_q, int head_dim,
                                   int64_t cap_tokens, const SegTable& seg, const ExtKV& ext, const CallerIo& io, float softmax_scale,
                                   hipStream_t st);
// k_new == nullptr: compaction only (the new scale is borrowed, nothing to copy); otherwise tokens
// [src_first, src_first + t_new) of the new scale (rows located by src_map) go to offset dst_new
hipError_t launch_append(void* kc, void* vc, const void* k_new, const void* v_new, int bh,
                         int row_bytes, int64_t cap_tokens, const MoveList& mv, int t_new,
                         int dst_new, int src_first, const RowMap& src_map, int heads, hipStream_t st);
// One iteration of Algorithm 1 at token granularity in one launch: the surviving ranges slide down (mv), then
// the kept ranges of the new scale (rows located by src_map) are copied behind them
hipError_t launch_roll(void* kc, void* vc, const void* k_new, const void* v_new, int bh, int row_bytes,
                       int64_t cap_tokens, const MoveList& mv, const NewRanges& nr, const RowMap& src_map, int heads,
                       hipStream_t st);
// k_out/v_out are head-major [BH][T_kept][row]; ext_map locates the rows of a borrowed scale
hipError_t launch_export(const void* kc, const void* vc, void* k_out, void* v_out, int bh,
                         int row_bytes, int64_t cap_tokens, const SegTable& seg, const ExtKV& ext,
                         const RowMap& ext_map, int heads, hipStream_t st);
// A whole scale, wherever it lives: base pointers of the tensor holding it (the layer's cache
// regions or the caller's K/V), the map of that tensor's rows, and the token offset of the scale
// inside each (b,h) row range; v may be null (keys only)
struct ScaleRef {
  const void* k;
  const void* v;
  RowMap map;
  int32_t off_tokens;
};
hipError_t launch_similarity(const ScaleRef& cur, const ScaleRef& prev, int batch, int heads,
                             int head_dim, int dtype, int h_cur, int w_cur, int h_prev, int w_prev,
                             float* partial_ws, float* out_dev, hipStream_t st);

// the same with the partial sums in the library's static device array instead of partial_ws; batch * heads
// must not exceed AMSKV_STATIC_MAX_UNITS.  Calls no allocating routine.
hipError_t launch_similarity_static(const ScaleRef& cur, const ScaleRef& prev, int batch, int heads,
                                    int head_dim, int dtype, int h_cur, int w_cur, int h_prev, int w_prev,
                                    float* out_dev, hipStream_t st);

// attention density: pieces = one table entry per group of keys (nothing merged); partial_ws holds
// batch*heads*ceil(t_q/32)*AMSKV_MAX_SCALES floats, out_dev heads*AMSKV_MAX_SCALES floats
hipError_t launch_density(const void* q, const void* kc, int batch, int heads, int t_q, int head_dim, int dtype,
                          int64_t cap_tokens, const SegTable& pieces, const ExtKV& ext, const CallerIo& io,
                          float softmax_scale, float* partial_ws, float* out_dev, hipStream_t st);
// Algorithm 1's test decided on the device: *flag_dev = (mean over heads of totals_dev[h*4] / n_tok) < theta
hipError_t launch_theta_flag(const float* totals_dev, int heads, double n_tok, float theta, int32_t* flag_dev,
                             int32_t* flag_host_pinned, hipStream_t st);
// its second stage alone: out[h][p] = mean over the batch of the sum over the query blocks of partial_ws
hipError_t launch_density_total(const float* partial_ws, int batch, int heads, int n_qblk, int n_groups, float* out_dev,
                                hipStream_t st);

}  // namespace amskv
