// Decode attention on the packed 3-bit cache for groups of 8 query heads per
// KV head (App. A; Table 2 A-D; Sec. 3.4), gfx950.  The same kernel runs on
// 2- and 4-bit records (Algorithm 1 at b = 2, 4); the notes below describe
// the 3-bit case, the others differ only in how a lane's slice of a record
// splits into code pairs.
//
// Work decomposition: one 512-thread workgroup (8 waves, two per SIMD) per
// (split of 16 * nbat positions, KV head g, sequence b), the grid's three
// dimensions; the split's nbat batches of 16 positions are dealt to the 8
// waves in contiguous runs of nbat / 8 or nbat / 8 + 1 batches.  With one
// workgroup per CU the SIMDs carry equal work.  A wave's loads (query,
// rotation parameters, both scale arrays and the keys of all its batches,
// then each batch's values as its scores start) are issued in the order the
// data is used, so each wait covers only the data it needs and the waves
// compute while the rest of the cache is still arriving.  In grids of one
// round the loads do not wait for the sequence length (see the kernel).
// The fused step adds one workgroup per (b, g) for the new token.
//
// The two contractions of a batch are dense 8-head x 128-dim x 16-position
// products and run on the matrix cores (v_mfma_f32_16x16x32_f16):
//
//  QK (Table 2 A): S[t][n] = sum_k Khat[t][k] Qt[k][n], rows t = 16 positions,
//    columns n = 16, k = 32 dims per instruction.  The fp32 rotated query is
//    split into fp16 hi + lo parts: columns 0..7 hold the 8 heads' hi parts,
//    columns 8..15 their lo parts, and lanes n and n ^ 8 add their products,
//    so the scores carry ~22 bits.
//    A lane (t, gk) supplies 8 dims 32gk+8kb..+7 of position t, i.e. 4
//    consecutive 6-bit fields (2 codes each) of its 12-byte slice of the
//    record; each field indexes a 64-entry LDS table holding the pair of
//    fp16 codebook levels, which is directly the MFMA operand dword.
//  PV (Table 2 C): O[(h, s)][u] = sum_(t, s') P'[(h, s)][(t, s')] Vhat[(t, s')][u]
//    with rows (head h, slot s) and columns u = 16 dim pairs per instruction.
//    The operand dword of position t is the decoded field (v_{2F}, v_{2F+1});
//    row (h, s) carries the fp16 weight in half s of its dword and zero in
//    the other half, so row (h, 0) accumulates dim 2F and row (h, 1) dim
//    2F+1.  Lane group gk of the PV operands holds positions 4gk..4gk+3,
//    exactly the rows the QK accumulator left in that lane group, so the
//    weights never leave their lanes.  Each weight is split into fp16 hi +
//    lo parts, one product each: with the weights rounded to fp16 once the
//    outputs of long contexts drift past 2e-3 of the fp64 result.
//
// Softmax (Table 2 B) is two-phase per wave: all QK products of the wave's
// positions first (scores kept in registers), one max per head, then the
// weights and the PV products; scores are in log2 units (the rotated query
// is pre-scaled by scale * log2 e) so exp2 is a single instruction.  The
// value scales s^V are divided by the wave's largest value scale before the
// fp16 conversion, keeping the weights in [0, 2^15].
//
// Merge: the 8 waves merge in LDS; with several splits per (b, g) each
// workgroup writes its partial (m, l, O) per head and a second kernel merges
// them, divides by the sum and applies the single inverse rotation
// R^T = H_128 M^T (Table 2 D); with one split the workgroup does it itself.
#include <hip/hip_runtime.h>
#include <math.h>

#include "iq_g8_split.h"

namespace iq {
namespace {

// The decode kernel.  Rows of a sequence: (KV head g, head group vg) with vg
// < ceil(group / 8); row (g, vg) serves query heads g * group + 8 vg + 0 ..
// nh - 1 (nh = 8, fewer in the last head group when group is not a multiple
// of 8), whose other query rows of the products are zero and unused.
//
// One-round grids (kWide false; at most one workgroup per CU): grid (split,
// row, sequence b), one work item per workgroup, bound by latency (the
// loads go out before the length is read).  The fused step (kAppend) adds
// split index n_splits per (b, row) for the new token.
//
// Grids of several rounds (kWide): gridDim.x persistent workgroups.  The
// work items are the fused step's new tokens (batch * rows of them, kAppend)
// and then the live splits, enumerated sequence by sequence (a sequence of
// clamped length L has ceil(L / split_len) live splits, each with its rows;
// exactly one when there is a single split, so that an empty sequence still
// gets its zero row); workgroup w takes items w, w + gridDim.x, ...  The
// lengths are read 64 at a time (one per lane) and turned into item offsets
// by a prefix sum across the lanes; every wave computes the same mapping.
// Splits past a length take no workgroup, and the merge kernel reads only
// the splits before each length.
//
// kPaged: the cache is a page pool (PageTable); capacity is then the logical
// capacity max_pages * page_size, and every batch of 16 positions and the
// new token's slot are located through the page table.
//
// kBits: the records' code width, 3 (the paper's cache) or 2 / 4 (Algorithm
// 1 with C_2 / C_4: records of 32 / 64 bytes).  Paged pools hold 3-bit
// records only.
//
// kRope: the content / RoPE sub-block split (Sec. 5, "MLA/RoPE hard
// blocker"): each key also has a 64-dim positional part in fp16
// (k_rope [b][rope row][capacity][64], rope row g, or 0 when rope_shared),
// never rotated or quantized, and each query head a positional part
// (q_rope [b][head][64] fp32); the score adds their dot product.  Decode
// only (no append), contiguous 3-bit caches; the three arguments of the
// append (k_new, v_new, new_f16) carry k_rope, q_rope and rope_shared.
//
// kAnyGroup: `group` query heads per KV head (1 .. 16) in head groups of 8;
// otherwise exactly 8 (the argument is not read).
template <int NB, bool kAppend, bool kWide, bool kPaged, int kBits, bool kRope = false,
          bool kAnyGroup = false>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(kWide && !kRope ? 4 : 2)))
void decode_g8_kernel(
    const float* __restrict__ q, uint8_t* __restrict__ k_codes, float* __restrict__ k_norms,
    uint8_t* __restrict__ v_codes, float* __restrict__ v_norms,
    const int32_t* __restrict__ seq_lens, const float* __restrict__ quats,
    float* __restrict__ partials, float* __restrict__ out, int64_t capacity, int max_seq_len,
    int n_kv_heads, int n_splits, int split_len, float qscale, CodebookB<kBits> cb,
    const void* __restrict__ k_new, const void* __restrict__ v_new, int new_f16,
    int32_t* __restrict__ status, PageTable pages, int group, int batch,
    int32_t* __restrict__ lens0) {
  static_assert(kBits == 3 || !kPaged, "paged pools hold 3-bit records");
  static_assert(!kRope || (!kAppend && !kPaged && kBits == 3 && kAnyGroup),
                "the positional split runs on contiguous 3-bit caches, decode only");
  // the arguments gathered for the device functions (the pointers keep the
  // kernel parameters' no-alias property: the lengths, for one, are then
  // read through the scalar cache)
  const G8Args<kBits> a{q,        k_codes,  k_norms, v_codes,    v_norms,     seq_lens,
                        quats,    partials, out,     capacity,   max_seq_len, n_kv_heads,
                        n_splits, split_len, qscale, cb,         k_new,       v_new,
                        new_f16,  status,   pages,   group,      batch,       lens0};
  __shared__ __attribute__((aligned(16))) G8Smem<kBits, kRope, !kWide> sm;
  const int gsize = kAnyGroup ? a.group : kHeads;
  const int vshift = kAnyGroup && gsize > kHeads ? 1 : 0;
  const int n_rows = a.n_kv_heads << vshift;

  if constexpr (!kWide) {
    const int split = blockIdx.x, yrow = blockIdx.y, b = blockIdx.z;
    const int g = yrow >> vshift, vg = yrow & vshift;
    const int bgv = b * n_rows + yrow;
    if constexpr (kAppend) {
      if (split == a.n_splits) {
        append_token<kPaged, kBits, kRope>(sm, a, gsize, g, vg, b, new_token_partial(a, bgv),
                                           true);
        return;
      }
    }
    attend_split<NB, kAppend, false, kPaged, kBits, kRope>(sm, a, gsize, split, g, vg, b, bgv,
                                                          0, true);
  } else {
    wide_items<NB, kAppend, kPaged, kBits, kRope>(sm, a, gsize, n_rows, vshift, true, -1);
  }
}
}  // namespace

// Split plan of the group-8 path: splits per (sequence, KV head) and their
// length (a multiple of 16).  A workgroup covers at most 8 waves x 5 batches
// x 16 = 640 positions (at 640 every wave has 5 batches and every SIMD the
// same load; a cap of 560 left three SIMDs with one batch more than the
// fourth for the same per-item time); while the grid is small (<= 4 rounds of one workgroup per CU) the
// split count is raised so that the grid, with the fused step's append
// workgroup per (sequence, KV head), fills whole rounds, but a split keeps at
// least one batch per wave.  n_rows: the (KV head, head group) rows of the
// grid per sequence (n_kv_heads * ceil(group / 8)).
void g8_plan(int64_t batch, int64_t n_rows, int64_t max_seq_len, int* nb, int64_t* n_splits,
             int64_t* split_len) {
  constexpr int64_t kCus = 256;
  constexpr int64_t kMaxLen = 640;
  const int64_t t = max_seq_len > 0 ? max_seq_len : 1;
  const int64_t bg = batch * n_rows > 0 ? batch * n_rows : 1;
  int64_t s = (t + kMaxLen - 1) / kMaxLen;
  const int64_t wgs = bg * (s + 1);
  if (wgs <= 4 * kCus) {
    const int64_t rounds = (wgs + kCus - 1) / kCus;
    int64_t s_fill = (rounds * kCus) / bg - 1;
    const int64_t s_min_len = (t + 16 * kWaves - 1) / (16 * kWaves);   // >= 1 batch per wave
    if (s_fill > s_min_len) s_fill = s_min_len;
    if (s_fill > s) s = s_fill;
  }
  int64_t len = (t + s - 1) / s;
  len = (len + 15) / 16 * 16;
  s = (t + len - 1) / len;
  *split_len = len;
  *n_splits = s;
  const int64_t nbat = len / 16;
  *nb = static_cast<int>((nbat + kWaves - 1) / kWaves);
}

hipError_t launch_decode_g8(int nb, int64_t n_splits, int64_t split_len, const float* q,
                            uint8_t* k_codes, float* k_norms, uint8_t* v_codes, float* v_norms,
                            int32_t* seq_lens, int64_t capacity, int64_t max_seq_len,
                            const float* quats, int64_t batch, int64_t n_kv_heads,
                            int64_t group, float scale, float* out, float* partials,
                            const StepAppend* append, const PageTable* pages, int bits,
                            hipStream_t stream, const iq_codebook_t* cb,
                            const RopeKeys* rope) {
  if (bits != 3 && pages) return hipErrorInvalidValue;
  if (rope && (append || pages || bits != 3)) return hipErrorInvalidValue;
  if (group < 1 || group > 2 * kHeads) return hipErrorInvalidValue;
  // partials per (sequence, KV head, head group): the splits, and the fused
  // step's new token
  const int64_t n_rows = n_kv_heads * ((group + kHeads - 1) / kHeads);
  const int64_t n_parts = append ? n_splits + 1 : n_splits;
  // Up to 5 batches per wave the kernel needs at most 128 VGPRs and ~55 KB of
  // LDS, so two workgroups fit on a CU.  A grid of at most one round gets one
  // workgroup per work item, and its LDS request is padded so that no CU
  // takes two while another idles.  Larger grids run two persistent
  // workgroups per CU over the work items (fewer when there are fewer
  // items): one workgroup's prologue and merge then run beside the other's
  // attention, and splits past a length take no workgroup.
  constexpr int64_t kCus = 256;
  const bool wide = n_parts * n_rows * batch > kCus;
  // The span kernel where lines can be long: the longest rows give each wave of
  // two workgroups per CU at least 12 batches (3 of its chunks), with positional
  // keys each wave of one workgroup per CU at least 8.  (Only the kernel knows
  // the lengths: short lines of such calls take the fixed splits there.)  Full
  // rows just above the line, fixed splits / span kernel: steps of 16 x 8 rows
  // of 6400 (12.5 batches per wave) 40.8 / 37.2 us, 32 x 2 rows of 12544 37.7 /
  // 36.3, decode of these 38.9 / 30.7 and 33.2 / 30.4; with positional keys 4 x
  // 16 rows of 4112 (8 batches) 22.8 / 20.5, 8 x 8 rows 24.0 / 20.7.  Below it
  // (8 batches per wave, 4 bits, 8 x 4 rows of 16K) 30.5 / 30.2 to 32.4.
  const int64_t span_wgs = (rope ? 1 : 2) * kCus;
  const int64_t span_line = span_wgs * kWaves * (rope ? 8 : 12);
  if (wide && n_splits > 1 && batch * n_rows * ((max_seq_len + 15) / 16) >= span_line) {
    SpanPlan sp;
    if (span_plan(batch, n_rows, n_splits, max_seq_len, span_wgs, split_len, &sp) && sp.workers == span_wgs)
      return launch_decode_span(sp, n_splits, q, k_codes, k_norms, v_codes, v_norms, seq_lens,
                                capacity, max_seq_len, quats, batch, n_kv_heads, group, scale,
                                out, partials, append, pages, bits, stream, cb, rope);
  }
  const size_t lds_pad = wide ? 0 : kOneWorkgroupPadBytes;
  const int64_t n_items = n_parts * n_rows * batch;
  if (n_items > (int64_t{1} << 30)) return hipErrorInvalidValue;   // 32-bit item indices
  // (the positional split's wide instances hold one workgroup per CU)
  const int64_t workers = (rope ? 1 : 2) * kCus;
  const dim3 grid = wide ? dim3(static_cast<unsigned>(n_items < workers ? n_items : workers))
                         : dim3(static_cast<unsigned>(n_parts), static_cast<unsigned>(n_rows),
                                static_cast<unsigned>(batch));
  const dim3 block(kThreads);
  const float qscale = scale * kLog2e;
  const void* k_new = append ? append->k_new : nullptr;
  const void* v_new = append ? append->v_new : nullptr;
  const int new_f16 = append ? append->f16 : 0;
  int32_t* status = append ? append->status : nullptr;
  const PageTable pt = pages ? *pages : PageTable{nullptr, 0, 4, 1};
  // the positional split passes its arguments in the append's three
  const void* k_side = rope ? static_cast<const void*>(rope->k_rope) : k_new;
  const void* v_side = rope ? static_cast<const void*>(rope->q_rope) : v_new;
  const int flag = rope ? rope->shared : new_f16;
  const bool any_group = group != kHeads;
  // fused steps on grids of several rounds: each sequence's length at the
  // step's start, after the partials (the merge's count of live splits)
  int32_t* const lens0 =
      wide && append && n_parts > 1
          ? reinterpret_cast<int32_t*>(reinterpret_cast<char*>(partials) +
                                       g8_partial_region_bytes(batch, n_rows, n_splits))
          : nullptr;
#define IQ_LAUNCH_G8_K(NB_, APP_, WIDE_, PAGED_, BITS_, ROPE_, ANY_)                           \
  hipLaunchKernelGGL((decode_g8_kernel<NB_, APP_, WIDE_, PAGED_, BITS_, ROPE_, ANY_>), grid,     \
                     block, lds_pad, stream, q, k_codes, k_norms, v_codes, v_norms, seq_lens,   \
                     quats, partials, out, capacity, static_cast<int>(max_seq_len),             \
                     static_cast<int>(n_kv_heads), static_cast<int>(n_splits),                  \
                     static_cast<int>(split_len), qscale, codebook_for<BITS_>(cb), k_side,      \
                     v_side, flag, status, pt, static_cast<int>(group), static_cast<int>(batch), \
                     lens0)
#define IQ_LAUNCH_G8_WPB(NB_, APP_, WIDE_, PAGED_, BITS_)         \
  if (any_group) {                                                \
    IQ_LAUNCH_G8_K(NB_, APP_, WIDE_, PAGED_, BITS_, false, true);  \
  } else {                                                        \
    IQ_LAUNCH_G8_K(NB_, APP_, WIDE_, PAGED_, BITS_, false, false); \
  }
#define IQ_LAUNCH_G8_W(NB_, APP_, WIDE_)                \
  if (pages) {                                          \
    IQ_LAUNCH_G8_WPB(NB_, APP_, WIDE_, true, 3);        \
  } else if (bits == 2) {                               \
    IQ_LAUNCH_G8_WPB(NB_, APP_, WIDE_, false, 2);       \
  } else if (bits == 4) {                               \
    IQ_LAUNCH_G8_WPB(NB_, APP_, WIDE_, false, 4);       \
  } else {                                              \
    IQ_LAUNCH_G8_WPB(NB_, APP_, WIDE_, false, 3);       \
  }
#define IQ_LAUNCH_G8(NB_, APP_)          \
  if (wide) {                            \
    IQ_LAUNCH_G8_W(NB_, APP_, true)      \
  } else {                               \
    IQ_LAUNCH_G8_W(NB_, APP_, false)     \
  }
#define IQ_LAUNCH_G8_NB(APP_)            \
  switch (nb) {                          \
    case 1: IQ_LAUNCH_G8(1, APP_); break; \
    case 2: IQ_LAUNCH_G8(2, APP_); break; \
    case 3: IQ_LAUNCH_G8(3, APP_); break; \
    case 4: IQ_LAUNCH_G8(4, APP_); break; \
    default: IQ_LAUNCH_G8(5, APP_); break; \
  }
#define IQ_LAUNCH_G8_ROPE(NB_)                              \
  if (wide) {                                               \
    IQ_LAUNCH_G8_K(NB_, false, true, false, 3, true, true);  \
  } else {                                                  \
    IQ_LAUNCH_G8_K(NB_, false, false, false, 3, true, true); \
  }
  if (rope) {
    switch (nb) {
      case 1: IQ_LAUNCH_G8_ROPE(1); break;
      case 2: IQ_LAUNCH_G8_ROPE(2); break;
      case 3: IQ_LAUNCH_G8_ROPE(3); break;
      case 4: IQ_LAUNCH_G8_ROPE(4); break;
      default: IQ_LAUNCH_G8_ROPE(5); break;
    }
  } else if (append) {
    IQ_LAUNCH_G8_NB(true)
  } else {
    IQ_LAUNCH_G8_NB(false)
  }
#undef IQ_LAUNCH_G8_ROPE
#undef IQ_LAUNCH_G8_NB
#undef IQ_LAUNCH_G8
#undef IQ_LAUNCH_G8_W
#undef IQ_LAUNCH_G8_WPB
#undef IQ_LAUNCH_G8_K
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // the partials of every (sequence, query head) merged by a second launch,
  // which in the fused step also advances the lengths
  if (n_parts > 1) {
    const dim3 mgrid(static_cast<unsigned>(n_kv_heads * group), static_cast<unsigned>(batch));
    // grids of several rounds leave the splits past each length unwritten:
    // their merge reads the live ones only.  Rows of more than 64 partials
    // (one sequence's long context over few KV heads) are read in passes of
    // 128 or 256 partials by variants that hold them all in registers (fewer
    // waves per SIMD: for merge grids of at most 256 workgroups)
    const bool wide_pass = n_parts > 64 && n_kv_heads * group * batch <= kCus;
#define IQ_LAUNCH_MERGE_U(APP_, ANY_, LIVE_, U_)                                               \
  hipLaunchKernelGGL((merge_g8_kernel<APP_, 1, ANY_, LIVE_, U_>), mgrid, dim3(kMergeThreads), 0, \
                     stream, partials, quats, out, static_cast<int>(n_kv_heads),                \
                     static_cast<int>(n_parts), seq_lens, capacity, static_cast<int>(group),    \
                     static_cast<int>(split_len), static_cast<int>(max_seq_len), lens0)
#define IQ_LAUNCH_MERGE_L(APP_, ANY_, LIVE_)        \
  if (wide_pass && n_parts > 128) {                 \
    IQ_LAUNCH_MERGE_U(APP_, ANY_, LIVE_, 32);       \
  } else if (wide_pass) {                           \
    IQ_LAUNCH_MERGE_U(APP_, ANY_, LIVE_, 16);       \
  } else {                                          \
    IQ_LAUNCH_MERGE_U(APP_, ANY_, LIVE_, 8);        \
  }
#define IQ_LAUNCH_MERGE(APP_, ANY_)        \
  if (wide) {                              \
    IQ_LAUNCH_MERGE_L(APP_, ANY_, true)    \
  } else {                                 \
    IQ_LAUNCH_MERGE_L(APP_, ANY_, false)   \
  }
    if (append && any_group) {
      IQ_LAUNCH_MERGE(true, true)
    } else if (append) {
      IQ_LAUNCH_MERGE(true, false)
    } else if (any_group) {
      IQ_LAUNCH_MERGE(false, true)
    } else {
      IQ_LAUNCH_MERGE(false, false)
    }
#undef IQ_LAUNCH_MERGE
#undef IQ_LAUNCH_MERGE_L
#undef IQ_LAUNCH_MERGE_U
    e = hipGetLastError();
  }
  return e;
}

}  // namespace iq
