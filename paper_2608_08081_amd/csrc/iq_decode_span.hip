// Decode attention on the packed cache for grids of many work items (large
// batches, long contexts): the attention of iq_decode_g8.hip (operands,
// matrix products, softmax weights and merge are the same) with the work cut
// into as many equal pieces as the chip holds workgroups, instead of into
// splits of a fixed length.  gfx950.
//
// Work decomposition: a sequence's positions, in batches of 16, follow each
// other row by row (row = KV head x head group of 8 query heads) and sequence
// by sequence; two persistent workgroups per CU each take an equal run of
// this line (short lines: fixed splits, see decode_span_kernel).  A run holds
// one row's part, or the end of a row, whole rows and the start of another;
// the part of one row in one run is a span.  Rows are longer by kRowBatches
// than their positions, for what a span costs besides its batches; the
// workgroup whose run holds a row's start also appends the row's new token
// (fused step).
//
// Inside a span each wave walks its own stretch of batches, kSpanBatches at a
// time (two-phase softmax per chunk, running maximum between chunks), and the
// waves meet only at the span's end.  The next chunk's keys are loaded into
// the registers of the current ones once the scores are done, the next values
// once the current ones are multiplied, so every wave has loads in flight
// through all of its arithmetic.  Value codes are loaded straight in the
// products' layout (a dword per record and lane) and need no LDS staging.
//
// Why: with fixed splits of 640 positions an item took 9.7 us, of which the
// scores and values were 4.6; the rest was the item's query rotation and first
// loads, its merge of the 8 waves and the wait between items.  A run pays
// these once per span (about 4300 positions on the batch-64 step).  What
// bounds it: 128 rows of 16K and of 32K positions differ by 51.8 us, 4.3 TB/s,
// which is also what the kernel reaches with its arithmetic taken out (fixed
// splits: 73.5 us); the arithmetic alone, on cached records, takes 0.85 of
// the whole, split evenly over the table lookups (LDS), the vector and the
// matrix units.  Batch-64 step (2048..32768 positions, 2 rows): 81.7 -> 68.0
// us.
#include <hip/hip_runtime.h>
#include <math.h>

#include "iq_g8_split.h"

namespace iq {
namespace {

// 16-position batches per chunk of a wave: 4 keeps the prefetched keys and
// values within the 128 VGPRs of two workgroups per CU.
constexpr int kSpanBatches = 4;
static_assert(16 * kSpanBatches == 64, "a chunk's scales are one per lane");
// a wave's time for a new key or value, in its batches
constexpr int kCompressBatches = 2;
// buffer descriptors: raw, unformatted dwords
constexpr int kBufferFlags = 0x00020000;
// smallest value-scale unit (see span_chunk): keeps 2^14 / unit finite
constexpr uint32_t kMinScaleBits = (127u - 100u) << 23;

struct SpanStage {
  float ks[64];                   // key scales of the chunk's positions
  float vs[64];                   // value scales times 2^14 / unit, 0 past the end
  float fac[kHeads];              // rescale factors of the heads' outputs
};

// LDS of the kernel, the pair table first (see G8Smem).
template <int kBits, bool kRope>
struct SpanSmem {
  uint32_t lut[1 << (2 * kBits)];
  uint32_t qop[2][kHeads][kQRowWords];
  uint32_t qop_r[kRope ? 2 : 1][kHeads][kRope ? kRopeRowWords : 1];   // positional operands
  int qexp[kHeads];
  float wave_ml[kWaves][2][kHeads];
  uint32_t new_rec[2][4 * kBits];   // the row's new token: its records,
  float new_scale[2];               // scales and the rotated queries
  f32x4_t new_q[kHeads][kDim / 4];
  union {
    SpanStage stage[kWaves];
    f32x4_t wave_o[kWaves][4][64];
  };
};

// v of this lane's row and of the other row of its pair of 16-lane rows (in
// either order), and the same for the halves of the wave: vector
// instructions only, the permute unit stays free for the table lookups.
// (The results go through plain integers: a bit cast of a vector's element
// reads element 0.)
__device__ __forceinline__ f32x2_t row_pair(float v) {
  const uint32_t x = __builtin_bit_cast(uint32_t, v);
  const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  const uint32_t r0 = r[0], r1 = r[1];
  return f32x2_t{__builtin_bit_cast(float, r0), __builtin_bit_cast(float, r1)};
}
__device__ __forceinline__ f32x2_t half_pair(float v) {
  const uint32_t x = __builtin_bit_cast(uint32_t, v);
  const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  const uint32_t r0 = r[0], r1 = r[1];
  return f32x2_t{__builtin_bit_cast(float, r0), __builtin_bit_cast(float, r1)};
}
// Largest / sum over the lanes l, l ^ 16, l ^ 32, l ^ 48 (one column's four
// lane groups).
__device__ __forceinline__ float cols_max(float v) {
  const f32x2_t a = row_pair(v);
  const f32x2_t b = half_pair(fmaxf(a[0], a[1]));
  return fmaxf(b[0], b[1]);
}
__device__ __forceinline__ float cols_sum(float v) {
  const f32x2_t a = row_pair(v);
  const f32x2_t b = half_pair(a[0] + a[1]);
  return b[0] + b[1];
}

// PV operand dwords of lane u = col for records 4 gk + r: pairs F = 4 u + nb
// (nb = 0..3), i.e. dims 8 u .. 8 u + 7, bits 8 b u .. of the record.  w[r]:
// the dword at byte b u of record 4 gk + r, or the record's last dword where
// that one would reach past its end (2 and 3 bits, u = 15), which vsh then
// shifts down.
template <int kBits>
__device__ __forceinline__ void window_pairs(const uint32_t* lut, const uint32_t (&w)[4],
                                             uint32_t vsh, u32x4_t (&vb)[4]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if constexpr (kBits == 3) {
      const uint32_t win = w[r] >> vsh, wu = w[r] >> (vsh + 4);
      vb[0][r] = lut_at(lut, low6x4<0>(win));
      vb[1][r] = lut_at(lut, top6x4<0>(wu));
      vb[2][r] = lut_at(lut, low6x4<1>(wu));
      vb[3][r] = lut_at(lut, top6x4<2>(win));
    } else if constexpr (kBits == 4) {
      vb[0][r] = lut_at(lut, byte4x4<0>(w[r]));
      vb[1][r] = lut_at(lut, byte4x4<1>(w[r]));
      vb[2][r] = lut_at(lut, byte4x4<2>(w[r]));
      vb[3][r] = lut_at(lut, byte4x4<3>(w[r]));
    } else {
      const uint32_t x = w[r] >> vsh;
      const uint32_t lo = x << 2, hi = x >> 2;
      vb[0][r] = lut_at(lut, nib4x4<0>(lo));
      vb[1][r] = lut_at(lut, nib4x4<0>(hi));
      vb[2][r] = lut_at(lut, nib4x4<1>(lo));
      vb[3][r] = lut_at(lut, nib4x4<1>(hi));
    }
  }
}

// What a wave carries from chunk to chunk.  m: largest score so far of head
// col % 8, in the head's scaled domain (see attend_wave); l: this lane's
// share of the head's sum of weights; unit: the power of two at or below the
// largest value scale so far (its bits), the outputs being in units of unit /
// 2^14.
template <int kBits, bool kRope>
struct SpanState {
  float m, l;
  uint32_t unit;
  f32x4_t o[4];
  uint32_t kw[kSpanBatches][kBits], vw[kSpanBatches][4];
  float ks, vs;   // lane j: position j of the chunk
  u32x4_t rk[kRope ? kSpanBatches : 1][2];   // positional keys (see attend_wave)
};

// One chunk: the batches held in s.kw / s.vw / s.ks / s.vs, nvalid positions
// (kFull: all of them).  next_keys / next_values issue the next chunk's loads
// into the same registers as soon as these are free.
template <bool kFull, int kBits, bool kRope, class NextKeys, class NextValues>
__device__ __forceinline__ void span_chunk(SpanState<kBits, kRope>& s, SpanStage& st,
                                           const u32x4_t (&qb)[4], const u32x4_t (&qbr)[2],
                                           const uint32_t* lut, int lane,
                                           int col, int grp, int nvalid, uint32_t vsh, float qdown,
                                           NextKeys next_keys, NextValues next_values) {
  constexpr int NB = kSpanBatches;
  const bool upper = col >= 8;
  const int rs = upper ? 2 : 0;
  // ---- the chunk's scales to LDS, the values' in units of unit / 2^14 -----
  uint32_t unit;
  {
    const float v = kFull || lane < nvalid ? s.vs : 0.f;
    unit = __builtin_bit_cast(uint32_t, wave64_max(v)) & 0x7F800000u;
    unit = unit > s.unit ? unit : s.unit;
    // 2^14 / unit, exactly
    const float up = __builtin_bit_cast(float, ((127u + 127u + 14u) << 23) - unit);
    st.ks[lane] = s.ks;
    st.vs[lane] = v * up;
  }
  wave_lds_fence();
  // ---- scores (Table 2 A) --------------------------------------------------
  f32x2_t sc[NB];
  float m = s.m;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    if (!kFull && 16 * i >= nvalid) break;
    u32x4_t a[4];
    key_pairs<kBits>(lut, s.kw[i], a);
    f32x4_t acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) acc = mfma(a[kb], qb[kb], acc);
    // lane (col, grp) holds positions 4 grp + r, the hi parts' products for
    // col < 8 and the lo parts' otherwise; it keeps positions rs and rs + 1
    f32x2_t xs;
    if constexpr (kRope) {
      const f32x4_t ks = *reinterpret_cast<const f32x4_t*>(&st.ks[16 * i + 4 * grp]);
      f32x4_t accr = f32x4_t{0.f, 0.f, 0.f, 0.f};
      accr = mfma(s.rk[i][0], qbr[0], accr);
      accr = mfma(s.rk[i][1], qbr[1], accr);
      f32x4_t x = acc * ks + accr;
#pragma unroll
      for (int r = 0; r < 4; ++r) x[r] += xor_lane<8>(x[r]);
      xs = upper ? f32x2_t{x[2], x[3]} : f32x2_t{x[0], x[1]};
    } else {
      // (s^K (hi + lo) rounded once: the scores' rounding is most of the error;
      // lo is below 2^10, so that an infinite s^K gives hi's infinity, not NaN)
      const f32x2_t ks = *reinterpret_cast<const f32x2_t*>(&st.ks[16 * i + 4 * grp + rs]);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        // (a rotation by 8 in each row of 16 lanes, into its upper or lower half
        // only; plain floats first, see row_pair)
        const float f0 = acc[j], f2 = acc[2 + j];
        const int a0 = __builtin_bit_cast(int, f0), a2 = __builtin_bit_cast(int, f2);
        const float hi = __builtin_bit_cast(
            float, __builtin_amdgcn_update_dpp(a0, a2, 0x128, 0xF, 0xC, false));
        const float lo = __builtin_bit_cast(
            float, __builtin_amdgcn_update_dpp(a2, a0, 0x128, 0xF, 0x3, false));
        xs[j] = __builtin_fmaf(hi, ks[j], lo * __builtin_amdgcn_fmed3f(ks[j], 0.f, 0x1p117f));
      }
    }
    if (!kFull && 16 * i + 16 > nvalid) {
#pragma unroll
      for (int j = 0; j < 2; ++j) xs[j] = (16 * i + 4 * grp + rs + j < nvalid) ? xs[j] : -INFINITY;
    }
    sc[i] = xs;
    m = fmaxf(fmaxf(m, xs[0]), xs[1]);
  }
  next_keys();
  m = cols_max(fmaxf(m, xor_lane<8>(m)));
  // ---- a new maximum or unit: what is summed so far, rescaled --------------
  if (unit != s.unit || __any(m > s.m)) {
    // (nothing finite so far: 0, which leaves a NaN sum NaN)
    const float f = s.m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((s.m - m) * qdown);
    s.l *= f;
    // the old unit over the new, exactly (0 if beyond the exponent range)
    const int de = static_cast<int>(s.unit >> 23) - static_cast<int>(unit >> 23) + 127;
    const float fu =
        de > 0 ? __builtin_bit_cast(float, static_cast<uint32_t>(de) << 23) : 0.f;
    if (lane < kHeads) st.fac[lane] = f * fu;
    wave_lds_fence();
    // rows 4 grp + r of the outputs are heads 4 (grp % 2) + r
    const f32x4_t fr = *reinterpret_cast<const f32x4_t*>(&st.fac[4 * (grp & 1)]);
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) s.o[nb] *= fr;
    s.m = m;
    s.unit = unit;
  }
  wave_lds_fence();
  // ---- weights (Table 2 B) and values (Table 2 C), as in attend_wave -------
  const uint32_t sel_hi = upper ? 0x01000808u : 0x08080504u;
  // (every score so far -inf: weights exp2(-inf) = 0; scores that are NaN,
  // which the maximum passes over, give NaN weights and so a NaN sum)
  const float mq = m == -INFINITY ? 0.f : -m * qdown;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    if (!kFull && 16 * i >= nvalid) break;
    const f32x2_t wv = *reinterpret_cast<const f32x2_t*>(&st.vs[16 * i + 4 * grp + rs]);
    uint32_t pk[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[i][j], qdown, mq));
      s.l += e;
      // hi and lo parts of the product, both to nearest (cut instead, the
      // outputs of rows up to 6000 positions were 2 to 9 % further from 64
      // bits, and it took two instructions more)
      const _Float16 ph = static_cast<_Float16>(e * wv[j]);
      const _Float16 pl =
          static_cast<_Float16>(__builtin_fmaf(e, wv[j], -static_cast<float>(ph)));
      pk[j] = __builtin_bit_cast(uint32_t, half2_t{ph, pl});
    }
    const uint32_t pp0 = static_cast<uint32_t>(
        __builtin_amdgcn_mov_dpp(static_cast<int>(pk[0]), 0x128, 0xF, 0xF, true));
    const uint32_t pp1 = static_cast<uint32_t>(
        __builtin_amdgcn_mov_dpp(static_cast<int>(pk[1]), 0x128, 0xF, 0xF, true));
    const u32x4_t pw_hi = u32x4_t{__builtin_amdgcn_perm(pk[0], pp0, sel_hi),
                                  __builtin_amdgcn_perm(pk[1], pp1, sel_hi),
                                  __builtin_amdgcn_perm(pp0, pk[0], sel_hi),
                                  __builtin_amdgcn_perm(pp1, pk[1], sel_hi)};
    uint32_t sel_lo = sel_hi;
    asm volatile("" : "+v"(sel_lo));
    sel_lo |= 0x02020202u;
    const u32x4_t pw_lo = u32x4_t{__builtin_amdgcn_perm(pk[0], pp0, sel_lo),
                                  __builtin_amdgcn_perm(pk[1], pp1, sel_lo),
                                  __builtin_amdgcn_perm(pp0, pk[0], sel_lo),
                                  __builtin_amdgcn_perm(pp1, pk[1], sel_lo)};
    u32x4_t vb[4];
    window_pairs<kBits>(lut, s.vw[i], vsh, vb);
    // the matrix products of a wave go out together: other waves' lookups
    // then find the LDS free
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) s.o[nb] = mfma(pw_hi, vb[nb], s.o[nb]);
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) s.o[nb] = mfma(pw_lo, vb[nb], s.o[nb]);
    __builtin_amdgcn_s_setprio(0);
  }
  next_values();
  // the next chunk's staging stays behind this chunk's reads
  wave_lds_fence();
}

// One span: batches a0 .. a1 - 1 of row (KV head g, head group vg) of
// sequence b, whose clamped length is len (a1 <= ceil(len / 16)); the partial
// (m, l, O) of its heads goes to `part`.  append: also the row's new token,
// to part_new (then a span may have no batches): two waves compress it while
// the others attend, and its score is taken when the span ends, so that the
// append adds a fraction of a microsecond to the span (as a work item of its
// own it took 4 us of the workgroup, 32 to 48 batches' time).
//
// kRope: the content / RoPE sub-block split of decode_g8_kernel (decode only,
// contiguous 3-bit caches; the append's three arguments carry k_rope, q_rope
// and rope_shared).
template <bool kAppend, bool kPaged, int kBits, bool kRope>
__device__ __forceinline__ void attend_span(SpanSmem<kBits, kRope>& sm, const G8Args<kBits>& a,
                                            int gsize, int g, int vg, int b, int a0, int a1, int len,
                                            float* part, bool append, float* part_new) {
  constexpr int NB = kSpanBatches;
  constexpr int kRB = record_bytes<kBits>();
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));   // recomputed per span (see attend_split)
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int col = lane & 15, grp = lane >> 4;
  const int n_q_heads = a.n_kv_heads * gsize;
  const int hq0 = g * gsize + kHeads * vg;
  const int nh = gsize - kHeads * vg < kHeads ? gsize - kHeads * vg : kHeads;
  const int qh = (tid >> 5) & 7, qblk = tid & 31;
  const f32x4_t qload = *reinterpret_cast<const f32x4_t*>(
      a.q + (static_cast<int64_t>(b) * n_q_heads + hq0 + (qh < nh ? qh : nh - 1)) * kDim +
      4 * qblk);
  const f32x4_t qv = qh < nh ? qload : f32x4_t{0.f, 0.f, 0.f, 0.f};
  f32x4_t qrv = f32x4_t{0.f, 0.f, 0.f, 0.f};   // positional dims 4 qblk .. (qblk < 16)
  if constexpr (kRope) {
    const f32x4_t t = *reinterpret_cast<const f32x4_t*>(
        static_cast<const float*>(a.v_new) +
        (static_cast<int64_t>(b) * n_q_heads + hq0 + (qh < nh ? qh : nh - 1)) * kRopeDim +
        4 * (qblk & 15));
    qrv = (qh < nh && qblk < 16) ? t : f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
  const f32x4_t* qpar = reinterpret_cast<const f32x4_t*>(
      a.quats + static_cast<int64_t>(g) * kQuatFloats + 8 * qblk);
  const f32x4_t ql = qpar[0], qr = qpar[1];
  const int64_t row = kPaged ? 0 : static_cast<int64_t>(b * a.n_kv_heads + g) * a.capacity;
  const uint8_t* kc = a.k_codes + row * kRB;
  const uint8_t* vc = a.v_codes + row * kRB;
  const float* kn = a.k_norms + row;
  const float* vn = a.v_norms + row;

  // this wave's stretch: positions p .. p + left - 1
  // (the two that compress a new token take kCompressBatches less)
  const int nbat = a1 - a0;
  int nb_late = nbat / kWaves, n_early = kWaves;
  if (kAppend && append) {
    nb_late = (nbat + 2 * kCompressBatches) / kWaves - kCompressBatches;
    nb_late = nb_late > 0 ? nb_late : 0;
    n_early = kWaves - 2;
  }
  const int n_deal = nbat - (kWaves - n_early) * nb_late;   // to the first n_early waves
  const int nb_base = n_deal / n_early, nb_rem = n_deal % n_early;
  const int nb_w = wave >= n_early ? nb_late : nb_base + (wave < nb_rem ? 1 : 0);
  int p = 16 * (a0 + (wave >= n_early ? n_deal + (wave - n_early) * nb_late
                                      : wave * nb_base + (wave < nb_rem ? wave : nb_rem)));
  const int end = p + 16 * nb_w < len ? p + 16 * nb_w : len;
  int left = nb_w > 0 ? end - p : 0;
  // start of its last batch: every load starts at or before it, so loaded
  // batches lie in the row (the capacity is a multiple of 16)
  const int last16 = left > 0 ? (end - 1) & ~15 : (a1 > 0 ? 16 * (a1 - 1) : 0);

  // paged: lane j keeps the page of batch page_t / 16 + j (an entry outside
  // the pools becomes page 0), loaded 64 batches at a time through the vector
  // cache: scalar loads in the loop would share their counter with the
  // lookups and stall these until they return.  page_deltas gives the record
  // deltas of the chunk at `at` (see attend_split).
  int pages_l = 0, page_t = p;
  auto load_pages = [&](int at) {
    const PageTable& pages = a.pages;
    page_t = at;
    const int t = at + 16 * lane < last16 ? at + 16 * lane : last16;
    const int pg = pages.tables[static_cast<int64_t>(b) * pages.max_pages +
                                (t >> pages.page_shift)];
    pages_l = static_cast<uint32_t>(pg) < static_cast<uint32_t>(pages.n_pages) ? pg : 0;
  };
  auto page_deltas = [&](int at, int64_t(&dlt)[NB]) {
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      dlt[i] = 0;
      if constexpr (kPaged) {
        const int t = at + 16 * i < last16 ? at + 16 * i : last16;
        const int64_t page = __builtin_amdgcn_readlane(pages_l, ((at - page_t) >> 4) + i);
        dlt[i] = ((page * a.n_kv_heads + g) << a.pages.page_shift) -
                 static_cast<int64_t>((t >> a.pages.page_shift) << a.pages.page_shift);
      }
    }
  };
  const int koff = col * kRB + 4 * kBits * grp;
  int64_t dlt[NB];
  SpanState<kBits, kRope> s;
  const int cap = static_cast<int>(a.capacity);
  // records of the batch at t: lane (t, gk) takes dwords b gk .. b gk + b - 1
  // of record t, through a buffer descriptor that ends with the row (lanes
  // past it read 0) and needs no per-lane address arithmetic
  auto load_records = [&](const uint8_t* base, int64_t d, int t, uint32_t(&w)[kBits]) {
    const int n = kPaged || cap - t > 16 ? 16 : cap - t;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(base + (d + t) * kRB), 0, n * kRB, kBufferFlags);
    if constexpr (kBits == 4) {
      const auto v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, koff, 0, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) w[j] = v[j];
    } else if constexpr (kBits == 3) {
      const auto v = __builtin_amdgcn_raw_buffer_load_b96(rsrc, koff, 0, 0);
#pragma unroll
      for (int j = 0; j < 3; ++j) w[j] = v[j];
    } else {
      const auto v = __builtin_amdgcn_raw_buffer_load_b64(rsrc, koff, 0, 0);
#pragma unroll
      for (int j = 0; j < 2; ++j) w[j] = v[j];
    }
  };
  // the scale of this lane's position of the chunk at `at`
  auto load_scale = [&](const float* base, int at) -> float {
    if constexpr (kPaged) {
      const int jb = lane >> 4;
      const int tj = (at + 16 * jb < last16 ? at + 16 * jb : last16) + (lane & 15);
      return base[pick_batch<0, NB>(dlt, jb) + tj];
    } else {
      const int t = at < last16 ? at : last16;
      const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base + t), 0,
                                                          4 * (cap - t), kBufferFlags);
      return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, 4 * lane, 0, 0));
    }
  };
  // positional keys: lane (t, gk) takes dims 8 gk .. + 7 and 32 + 8 gk .. + 7
  // of position t (16-byte loads; the capacity is a multiple of 16)
  const uint16_t* rp = nullptr;
  if constexpr (kRope)
    rp = static_cast<const uint16_t*>(a.k_new) +
         (static_cast<int64_t>(b) * (a.new_f16 ? 1 : a.n_kv_heads) + (a.new_f16 ? 0 : g)) *
             a.capacity * kRopeDim;
  auto load_k = [&](int at) {
    s.ks = load_scale(kn, at);
    s.vs = load_scale(vn, at);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int t = at + 16 * i < last16 ? at + 16 * i : last16;
      load_records(kc, dlt[i], t, s.kw[i]);
      if constexpr (kRope) {
        const u32x4_t* src =
            reinterpret_cast<const u32x4_t*>(rp + static_cast<int64_t>(t + col) * kRopeDim);
        s.rk[i][0] = src[grp];
        s.rk[i][1] = src[4 + grp];
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // value windows: lane (u, gk) takes, of records 4 gk + r, the dword that
  // holds its 8 codes (see window_pairs), straight in the products' layout
  constexpr int kLast = kRB - 4;   // the last dword of a record
  const int uoff = kBits * col < kLast ? kBits * col : kLast;
  const uint32_t vsh = static_cast<uint32_t>(8 * (kBits * col - uoff));
  const int voff = 4 * grp * kRB + uoff;
  auto load_v = [&](int at) {
    // (opaque here: the records' offsets then stay in the instructions instead
    // of three registers set before the loop)
    int vo = voff;
    asm volatile("" : "+v"(vo));
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int t = at + 16 * i < last16 ? at + 16 * i : last16;
      const int n = kPaged || cap - t > 16 ? 16 : cap - t;
      const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<uint8_t*>(vc + (dlt[i] + t) * kRB), 0, n * kRB, kBufferFlags);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        s.vw[i][r] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, vo + r * kRB, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  if constexpr (kPaged) load_pages(p);
  page_deltas(p, dlt);
  load_k(p);
  load_v(p);

  // ---- while the loads fly: the rotated query as operands in LDS ----------
  if (tid < kRotThreads) {
    // (opaque, like tid: the product is not held in a register between spans)
    float qscale = a.qscale;
    asm volatile("" : "+s"(qscale));
    const f32x4_t y = rotate_forward(qv, ql, qr, qblk, kInvSqrtDim * qscale);
    // the positional part, scaled like the scores, shares the head's operand
    // scale
    const f32x4_t yr = qrv * qscale;
    float amx = fmaxf(fmaxf(fabsf(y[0]), fabsf(y[1])), fmaxf(fabsf(y[2]), fabsf(y[3])));
    if constexpr (kRope)
      amx = fmaxf(amx,
                  fmaxf(fmaxf(fabsf(yr[0]), fabsf(yr[1])), fmaxf(fabsf(yr[2]), fabsf(yr[3]))));
    const float am = group32_max(amx);
    int qexp = 0;
    if (am > 0.f) {
      int e = 0;
      frexpf(am, &e);   // am < 2^e
      qexp = 14 - e;
      qexp = qexp > 100 ? 100 : (qexp < -100 ? -100 : qexp);
    }
    const float qup = ldexpf(1.0f, qexp);
    // fp16 hi and lo parts of a pair, as operand dwords
    auto split_pair = [&](float x0, float x1, uint32_t& hi, uint32_t& lo) {
      const _Float16 h0 = static_cast<_Float16>(x0), h1 = static_cast<_Float16>(x1);
      const _Float16 l0 = static_cast<_Float16>(x0 - static_cast<float>(h0));
      const _Float16 l1 = static_cast<_Float16>(x1 - static_cast<float>(h1));
      hi = static_cast<uint32_t>(__builtin_bit_cast(uint16_t, h0)) |
           (static_cast<uint32_t>(__builtin_bit_cast(uint16_t, h1)) << 16);
      lo = static_cast<uint32_t>(__builtin_bit_cast(uint16_t, l0)) |
           (static_cast<uint32_t>(__builtin_bit_cast(uint16_t, l1)) << 16);
    };
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      split_pair(y[2 * j] * qup, y[2 * j + 1] * qup, sm.qop[0][qh][2 * qblk + j],
                 sm.qop[1][qh][2 * qblk + j]);
      if constexpr (kRope) {
        if (qblk < 16)
          split_pair(yr[2 * j] * qup, yr[2 * j + 1] * qup, sm.qop_r[0][qh][2 * qblk + j],
                     sm.qop_r[1][qh][2 * qblk + j]);
      }
    }
    if (qblk == 0) sm.qexp[qh] = qexp;
    if (kAppend && append) sm.new_q[qh][qblk] = y;
  }
  lds_barrier();   // lut, qop, qexp
  if constexpr (kAppend) {
    if (append && wave >= kWaves - 2) {
      // (a chain of dependent instructions: ahead of the other waves')
      __builtin_amdgcn_s_setprio(3);
      const NewToken tok = new_token<kPaged>(a, g, b);
      compress_new_token(sm, a, kWaves - 1 - wave, g, b, lane, tok.rec, tok.written && vg == 0);
      if (g == 0 && vg == 0 && wave == kWaves - 1 && lane == 0) note_new_token(a, b, tok.written);
      __builtin_amdgcn_s_setprio(0);
    }
  }
  u32x4_t qb[4];
#pragma unroll
  for (int kb = 0; kb < 4; ++kb)
    qb[kb] = *reinterpret_cast<const u32x4_t*>(&sm.qop[col >> 3][col & 7][16 * grp + 4 * kb]);
  u32x4_t qbr[2];
  if constexpr (kRope) {
#pragma unroll
    for (int m = 0; m < 2; ++m)
      qbr[m] = *reinterpret_cast<const u32x4_t*>(&sm.qop_r[col >> 3][col & 7][16 * m + 4 * grp]);
  }
  const float qdown = ldexpf(1.0f, -sm.qexp[col & 7]);
  s.m = -INFINITY;
  s.l = 0.f;
  s.unit = kMinScaleBits;
#pragma unroll
  for (int nb = 0; nb < 4; ++nb) s.o[nb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  SpanStage& st = sm.stage[wave];
  // full chunks, the next one's loads (clamped: past the end they repeat the
  // last batch) issued from inside; then the rest
  while (left >= 16 * NB) {
    p += 16 * NB;
    left -= 16 * NB;
    if constexpr (kPaged)
      if (p - page_t == 64 * 16) load_pages(p);
    span_chunk<true, kBits, kRope>(
        s, st, qb, qbr, sm.lut, lane, col, grp, 16 * NB, vsh, qdown,
        [&] {
          page_deltas(p, dlt);
          load_k(p);
        },
        [&] { load_v(p); });
  }
  if (left > 0)
    span_chunk<false, kBits, kRope>(
        s, st, qb, qbr, sm.lut, lane, col, grp, left, vsh, qdown, [] {}, [] {});

  // ---- merge the 8 waves in LDS, as in attend_split -------------------------
  const float l = cols_sum(s.l + xor_lane<8>(s.l));
  lds_barrier();   // every wave is done with its staging area
  const float oscale = __builtin_bit_cast(float, s.unit) * (1.0f / 16384.0f);
#pragma unroll
  for (int r = 0; r < 4; ++r)
    sm.wave_o[wave][r][lane] = f32x4_t{s.o[0][r], s.o[1][r], s.o[2][r], s.o[3][r]} * oscale;
  if (lane < kHeads) {
    sm.wave_ml[wave][0][lane] = s.m * qdown;   // log2 units
    sm.wave_ml[wave][1][lane] = l;
  }
  lds_barrier();   // wave_o, wave_ml
  if (tid >= kRotThreads) return;
  const int mh = qh, md = 4 * qblk;
  float M = -INFINITY;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) M = fmaxf(M, sm.wave_ml[w][0][mh]);
  const int o_r = mh & 3, o_lane = (md >> 3) + 16 * ((mh >> 2) & 1), o_nb = (md & 7) >> 1;
  float L = 0.f;
  f32x4_t O = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const float mw = sm.wave_ml[w][0][mh];
    const float c = (mw == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mw - M);
    L += c * sm.wave_ml[w][1][mh];
    const f32x2_t s0 = *reinterpret_cast<const f32x2_t*>(
        reinterpret_cast<const float*>(&sm.wave_o[w][o_r][o_lane]) + o_nb);
    const f32x2_t s1 = *reinterpret_cast<const f32x2_t*>(
        reinterpret_cast<const float*>(&sm.wave_o[w][o_r][o_lane + 32]) + o_nb);
    O += c * f32x4_t{s0[0], s1[0], s0[1], s1[1]};
  }
  if (a1 > a0) {
    float* pp = part + mh * kPart;
    if (qblk == 0) {
      pp[0] = M;
      pp[1] = L;
    }
    *reinterpret_cast<f32x4_t*>(pp + 2 + md) = O;
  }
  if constexpr (kAppend) {
    if (append)
      publish_new_token<kBits>(sm, sm.new_q[qh][qblk], new_token<kPaged>(a, g, b), part_new, qh,
                               qblk);
  }
}

// The kernel: gridDim.x persistent workgroups, workgroup w taking run w (see
// SpanLine).  Partial slots: the span of run w in row r (rows counted over
// all sequences) writes slot w + r, which grows by at least one from span to
// span; a fused step's new-token partials follow the n_splits slots per row
// that the workspace has for splits.
//
// Short lines (only the kernel knows the lengths, the launch a bound of them)
// take the fixed splits of decode_g8_kernel, of split_len positions: a span's
// start and end, and the new token beside too few batches to hide it, cost
// more than equal runs gain.  Rows sized for 32768 positions, batch of 64 x 2
// rows, runs / splits: steps at 100 positions 19.8 / 14.0 us, at 1000 22.5 /
// 16.4, decode at 1000 15.2 / 13.2.  Where the line is drawn (kShortBatches),
// mean over nine shapes of rows, pages and bits: decode of 4 batches per wave
// 19.3 / 19.1, of 5 21.0 / 22.3; steps of 8 32.9 / 31.7, of 10 35.5 / 36.3.
// kSplits false (rows of any length, which those cannot load): always runs.
//
// by_rows (workspaces of one slot per row, i.e. short sequences): the
// workgroups take whole rows w, w + gridDim.x, ... instead, row r in slot r.
//
// kRope: 32 more registers of positional keys per wave, so one workgroup per
// CU.
template <bool kAppend, bool kPaged, int kBits, bool kRope, bool kSplits>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(kRope ? 2 : 4)))
void decode_span_kernel(
    const float* __restrict__ q, uint8_t* __restrict__ k_codes, float* __restrict__ k_norms,
    uint8_t* __restrict__ v_codes, float* __restrict__ v_norms,
    const int32_t* __restrict__ seq_lens, const float* __restrict__ quats,
    float* __restrict__ partials, int64_t capacity, int max_seq_len, int n_kv_heads,
    int n_splits, int split_len, float qscale, CodebookB<kBits> cb,
    const void* __restrict__ k_new, const void* __restrict__ v_new, int new_f16,
    int32_t* __restrict__ status, PageTable pages, int group, int batch,
    int32_t* __restrict__ lens0, int by_rows_arg) {
  const bool by_rows = !kSplits && by_rows_arg != 0;
  // (out is written by grids of one split only)
  const G8Args<kBits> a{q,        k_codes, k_norms, v_codes,  v_norms,     seq_lens,
                        quats,    partials, partials, capacity, max_seq_len, n_kv_heads,
                        n_splits, split_len, qscale, cb,      k_new,       v_new,
                        new_f16,  status,  pages,   group,    batch,       nullptr};
  static_assert(!kRope || (!kAppend && !kPaged && kBits == 3), "decode of 3-bit rows");
  // the LDS of a span or of a fixed split (the pair table first in both)
  constexpr size_t kSplitLds = kSplits ? sizeof(G8Smem<kBits, kRope, false>) : 0;
  constexpr size_t kLds =
      sizeof(SpanSmem<kBits, kRope>) > kSplitLds ? sizeof(SpanSmem<kBits, kRope>) : kSplitLds;
  __shared__ __attribute__((aligned(16))) char lds[kLds];
  auto& sm = *reinterpret_cast<SpanSmem<kBits, kRope>*>(lds);
  const int vshift = group > kHeads ? 1 : 0;
  const int n_rows = n_kv_heads << vshift;
  const int wg = static_cast<int>(blockIdx.x), n_wg = static_cast<int>(gridDim.x);
  const int lane = threadIdx.x & 63;
  build_pair_table(sm, cb, threadIdx.x);   // before the first span's barriers
  int b = wg / n_rows, y = wg - b * n_rows;   // the current row: sequence, row in it
  int start = 0, x = 0, x1 = 0;   // where b's rows start on the line, the run's rest x .. x1
  int len = 0;                    // b's clamped length
  bool splits = false;            // a short line
  int len0 = -1;
  if (!by_rows) {
    const SpanRun run =
        span_run<kAppend, kSplits>(seq_lens, batch, n_rows, max_seq_len, n_wg, lane, wg);
    splits = run.splits;
    len0 = run.first;
    x = run.x;
    x1 = run.x1;
    b = run.seq;
    start = run.start;
    len = run.len;
  }
  // for the merge: the clamped lengths as they are now (its workgroups of row 0
  // advance seq_lens), the sign bit set on short lines
  if (wg == 0) {
    const int flag = splits ? static_cast<int>(0x80000000u) : 0;
    if (len0 >= 0) {
      if (threadIdx.x < batch) lens0[threadIdx.x] = len0 | flag;   // (at most 64 of wave 0)
    } else {
      for (int i = threadIdx.x; i < batch; i += kThreads)
        lens0[i] = span_length(seq_lens[i], max_seq_len) | flag;
    }
  }
  if constexpr (kSplits) {
    if (__builtin_expect(splits, 1)) {
      wide_items<kMaxBatches, kAppend, kPaged, kBits, kRope>(
          *reinterpret_cast<G8Smem<kBits, kRope, false>*>(lds), a, group, n_rows, vshift, false,
          len0);
      return;
    }
  }
  if (by_rows) {
    if (b >= batch) return;
    len = span_length(seq_lens[b], max_seq_len);
  } else {
    if (x >= x1) return;
    y = (x - start) / span_width(len);
  }
  for (bool first = true;;) {
    const int width = span_width(len);   // of each row of this sequence
    const int r = b * n_rows + y;
    // the row's part in this run: batches a0 .. a1 - 1, its new token or not
    int a0 = 0, a1 = (len + 15) >> 4, e = 0;
    bool append = kAppend;
    if (!by_rows) {
      const int row0 = start + y * width;
      const int at0 = row0 + width - a1;
      e = x1 < row0 + width ? x1 : row0 + width;
      append = kAppend && x == row0;
      // (a run that ends before the row's positions has none of them)
      a0 = x > at0 ? x - at0 : 0;
      a1 = e > at0 ? e - at0 : 0;
    }
    if (append || a1 > a0) {
      if (!first) lds_barrier();   // the previous span is done with the LDS
      attend_span<kAppend, kPaged, kBits, kRope>(
          sm, a, group, y >> vshift, y & vshift, b, a0, a1, len,
          partials + (static_cast<int64_t>(by_rows ? 0 : wg) + r) * (kHeads * kPart), append,
          partials + (static_cast<int64_t>(batch) * n_rows * n_splits + r) * (kHeads * kPart));
      first = false;
    }
    if (by_rows) {
      b = (r + n_wg) / n_rows;
      y = r + n_wg - b * n_rows;
      if (b >= batch) return;
      len = span_length(seq_lens[b], max_seq_len);
    } else {
      x = e;
      if (x >= x1) return;
      if (++y == n_rows) {
        start += n_rows * width;
        y = 0;
        ++b;
        len = span_length(seq_lens[b], max_seq_len);
      }
    }
  }
}

// Merge of the spans of each row and the new token's partial, the inverse
// rotation and (fused step) the advance of the lengths, as merge_g8_kernel;
// the rows' spans are found from the line.  kHpw query heads per workgroup:
// 8 for rows of few spans (two groups of threads share a head's spans), 1
// for rows of many (eight groups; sixteen took 0.3 us more on short lines).
// lens0: the lengths as the span kernel saw them (see there); on short lines
// they place the row's partials without the line.  workers: runs of the line,
// 0 with whole rows.
// Bound by its chain of loads (lengths, then partials): one workgroup per
// row instead of one per query head reads the lengths an eighth as often.
template <int kHpw>
constexpr int merge_threads = kHpw == 1 ? 256 : 512;
template <bool kAppend, int kHpw>
__global__ __launch_bounds__(merge_threads<kHpw>) void merge_span_kernel(
    const float* __restrict__ partials, const float* __restrict__ quats, float* __restrict__ out,
    int n_kv_heads, int n_splits, int32_t* __restrict__ seq_lens,
    const int32_t* __restrict__ lens0, int64_t capacity, int group, int workers, int max_seq_len,
    int batch, int split_len) {
  constexpr int kGroups = merge_threads<kHpw> / (32 * kHpw);   // groups of threads per head
  constexpr int kUnroll = 8;
  __shared__ __attribute__((aligned(16))) f32x4_t red_o[kGroups][kHpw][32];
  __shared__ float red_m[kGroups][kHpw], red_l[kGroups][kHpw];
  const int tid = threadIdx.x;
  const int vshift = group > kHeads ? 1 : 0;
  const int n_rows = n_kv_heads << vshift;
  // workgroups per row: one, or one for each of its heads
  const int per = kHpw == 1 ? (group < kHeads ? group : kHeads) : 1;
  const int y = static_cast<int>(blockIdx.x) / per;
  const int h0 = static_cast<int>(blockIdx.x) - y * per;
  const int b = blockIdx.y;
  const int g = y >> vshift, vg = y & vshift;
  const int nh = group - kHeads * vg < kHeads ? group - kHeads * vg : kHeads;
  if (h0 >= nh) return;
  const int dq = tid & 31, hj = (tid >> 5) % kHpw, sg = (tid >> 5) / kHpw;
  const int hh = h0 + hj;
  const int r = b * n_rows + y;
  int seq0 = 0;
  const f32x4_t* qg =
      reinterpret_cast<const f32x4_t*>(quats + static_cast<int64_t>(g) * kQuatFloats + 8 * dq);
  const f32x4_t ql = qg[0], qr = qg[1];
  const int word = lens0[b];
  const bool splits = word < 0;
  const int len = word & 0x7fffffff;
  const int nb = (len + 15) >> 4;
  // the row's spans: slots slot0 .. slot0 + n_spans - 1; its new token's slot
  int64_t slot0 = r;
  int64_t slot_new = static_cast<int64_t>(batch) * n_rows * n_splits + r;
  int n_spans = nb > 0 ? 1 : 0;
  if (__builtin_expect(splits, 1)) {   // a short line: as the fixed splits' kernel lays them out
    slot0 = static_cast<int64_t>(r) * (n_splits + (kAppend ? 1 : 0));
    slot_new = slot0 + n_splits;
    n_spans = (len + split_len - 1) / split_len;
  } else if (workers > 0) {
    int start = 0;
    const SpanLine line =
        span_line(lens0, batch, n_rows, max_seq_len, workers, tid & 63, b, &start);
    const int width = span_width(len);
    const int at0 = start + y * width + width - nb;
    const int w0 = at0 / line.run;
    if (nb > 0) n_spans = (at0 + nb - 1) / line.run - w0 + 1;
    slot0 += w0;
  }
  float written = 0.f;
  if (kAppend && y == 0 && h0 == 0 && tid == 0) {
    seq0 = seq_lens[b];
    written = partials[slot_new * (kHeads * kPart) + 1];
  }
  const int n_iter = n_spans + (kAppend ? 1 : 0);
  const float* base = partials + hh * kPart;
  // the new token counts if it was written (its l entry) and lies before
  // max_seq_len; a row is empty without positions and without it
  const bool new_near = kAppend && len < max_seq_len;
  bool any = n_spans > 0;
  float M = -INFINITY, L = 0.f;
  f32x4_t O = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int s0 = sg; s0 < n_iter; s0 += kGroups * kUnroll) {
    f32x2_t ml[kUnroll];
    f32x4_t ov[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int s = s0 + kGroups * u < n_iter ? s0 + kGroups * u : s0;
      const int64_t slot = s < n_spans ? slot0 + s : slot_new;
      const float* p = base + slot * (kHeads * kPart);
      ml[u] = *reinterpret_cast<const f32x2_t*>(p);   // (m, l)
      ov[u] = *reinterpret_cast<const f32x4_t*>(p + 2 + 4 * dq);
    }
    __builtin_amdgcn_sched_barrier(0);   // every load of the pass before the first use
    float Mn = M;
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int s = s0 + kGroups * u;
      const bool live = s < n_spans || (s < n_iter && new_near && ml[u][1] > 0.f);
      any |= live;
      ml[u][0] = live ? ml[u][0] : -INFINITY;
      ml[u][1] = live ? ml[u][1] : 0.f;
      ov[u] = live ? ov[u] : f32x4_t{0.f, 0.f, 0.f, 0.f};
      Mn = fmaxf(Mn, ml[u][0]);
    }
    const float cM = (M == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(M - Mn);
    L *= cM;
    O *= cM;
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      // (m = -inf: every score -inf, or NaN with l NaN, which the zero keeps)
      const float c = ml[u][0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[u][0] - Mn);
      L += c * ml[u][1];
      O += c * ov[u];
    }
    M = Mn;
  }
  red_o[sg][hj][dq] = O;
  if (dq == 0) {
    red_m[sg][hj] = M;
    red_l[sg][hj] = L;
  }
  lds_barrier();
  if (sg == 0 && hh < nh) {
    float Mt = red_m[0][hj];
#pragma unroll
    for (int j = 1; j < kGroups; ++j) Mt = fmaxf(Mt, red_m[j][hj]);
    f32x4_t o = f32x4_t{0.f, 0.f, 0.f, 0.f};
    float l = 0.f;
#pragma unroll
    for (int j = 0; j < kGroups; ++j) {
      const float mj = red_m[j][hj];
      const float c = (mj == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mj - Mt);
      o += c * red_o[j][hj][dq];
      l += c * red_l[j][hj];
    }
    // an empty sequence gives a zero row, anything else o / l, also where l is
    // NaN (without spans, this group of threads has seen the new token)
    const f32x4_t res =
        any ? rotate_inverse(o * (1.0f / l), ql, qr, dq) : f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int64_t hq = static_cast<int64_t>(b) * n_kv_heads * group +
                       static_cast<int64_t>(g) * group + kHeads * vg + hh;
    *reinterpret_cast<f32x4_t*>(out + hq * kDim + 4 * dq) = res;
  }
  if (kAppend && y == 0 && h0 == 0 && tid == 0 && seq0 >= 0 && seq0 < capacity && written > 0.f)
    seq_lens[b] = seq0 + 1;
}

}  // namespace

// How the span kernel runs a call.  Runs need a slot for every span (runs +
// rows - 1 of them) in the n_splits slots per row of the workspace, lengths
// that every wave can sum (at most kSpanMaxBatch) and a line of 32-bit
// length; with one slot per row the workgroups take whole rows.  At most
// `workgroups` of them (two per CU, one with positional keys).  false: neither
// is possible.
bool span_plan(int64_t batch, int64_t n_rows, int64_t n_splits, int64_t max_seq_len,
               int64_t workgroups, int64_t split_len, SpanPlan* plan) {
  const int64_t rows = batch * n_rows;
  if (rows * (n_splits + 1) > (int64_t{1} << 30)) return false;   // slots: 32-bit indices
  if (n_splits == 1) {
    *plan = SpanPlan{static_cast<int>(rows < workgroups ? rows : workgroups), true, 0};
    return true;
  }
  if (batch > kSpanMaxBatch ||
      rows * ((max_seq_len + 15) / 16 + kRowBatches) + workgroups > 0x3fffffff)
    return false;
  const int64_t most = rows * (n_splits - 1) + 1;
  *plan = SpanPlan{static_cast<int>(most < workgroups ? most : workgroups), false,
                   static_cast<int>(split_len)};
  return true;
}

hipError_t launch_decode_span(const SpanPlan& plan, int64_t n_splits, const float* q,
                              uint8_t* k_codes, float* k_norms, uint8_t* v_codes, float* v_norms,
                              int32_t* seq_lens, int64_t capacity, int64_t max_seq_len,
                              const float* quats, int64_t batch, int64_t n_kv_heads,
                              int64_t group, float scale, float* out, float* partials,
                              const StepAppend* append, const PageTable* pages, int bits,
                              hipStream_t stream, const iq_codebook_t* cb, const RopeKeys* rope) {
  const int64_t n_rows = n_kv_heads * ((group + kHeads - 1) / kHeads);
  const dim3 grid(static_cast<unsigned>(plan.workers)), block(kThreads);
  const float qscale = scale * kLog2e;
  // the positional split passes its arguments in the append's three
  const void* k_new = append ? append->k_new : (rope ? rope->k_rope : nullptr);
  const void* v_new = append ? append->v_new : (rope ? rope->q_rope : nullptr);
  const int new_f16 = append ? append->f16 : (rope ? rope->shared : 0);
  int32_t* status = append ? append->status : nullptr;
  const PageTable pt = pages ? *pages : PageTable{nullptr, 0, 4, 1};
  int32_t* const lens0 = reinterpret_cast<int32_t*>(
      reinterpret_cast<char*>(partials) + g8_partial_region_bytes(batch, n_rows, n_splits));
#define IQ_LAUNCH_SPAN(APP_, PAGED_, BITS_, ROPE_, SPLITS_)                                     \
  hipLaunchKernelGGL((decode_span_kernel<APP_, PAGED_, BITS_, ROPE_, SPLITS_>), grid, block, 0,  \
                     stream, q, k_codes, k_norms, v_codes, v_norms, seq_lens, quats, partials,  \
                     capacity, static_cast<int>(max_seq_len), static_cast<int>(n_kv_heads),     \
                     static_cast<int>(n_splits), plan.split_len, qscale,                        \
                     codebook_for<BITS_>(cb), k_new, v_new, new_f16, status, pt,                \
                     static_cast<int>(group), static_cast<int>(batch), lens0,                   \
                     plan.by_rows ? 1 : 0)
#define IQ_LAUNCH_SPAN_A(APP_)                      \
  if (plan.split_len == 0) {                        \
    IQ_LAUNCH_SPAN(APP_, false, 3, false, false);   \
  } else if (pages) {                               \
    IQ_LAUNCH_SPAN(APP_, true, 3, false, true);     \
  } else if (bits == 2) {                           \
    IQ_LAUNCH_SPAN(APP_, false, 2, false, true);    \
  } else if (bits == 4) {                           \
    IQ_LAUNCH_SPAN(APP_, false, 4, false, true);    \
  } else {                                          \
    IQ_LAUNCH_SPAN(APP_, false, 3, false, true);    \
  }
  if (plan.split_len == 0 && (pages || bits != 3 || rope)) return hipErrorInvalidValue;
  if (rope) {
    IQ_LAUNCH_SPAN(false, false, 3, true, true);
  } else if (append) {
    IQ_LAUNCH_SPAN_A(true)
  } else {
    IQ_LAUNCH_SPAN_A(false)
  }
#undef IQ_LAUNCH_SPAN_A
#undef IQ_LAUNCH_SPAN
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // Workgroups of a whole row for rows of on average at most 16 spans (one pass)
  // and more than 2 query heads; for 1 or 2 the other heads' share of their
  // loads is wasted (positional keys, 16 rows of one head, batch of 4, 12 us
  // short calls: 0.3 us).
  const bool few = (plan.by_rows || plan.workers <= 15 * batch * n_rows) && group > 2;
  const int runs = plan.by_rows ? 0 : plan.workers;
  const dim3 mgrid(
      static_cast<unsigned>(few ? n_rows : n_rows * (group < kHeads ? group : kHeads)),
      static_cast<unsigned>(batch));
#define IQ_LAUNCH_SPAN_MERGE(APP_, HPW_)                                                        \
  hipLaunchKernelGGL((merge_span_kernel<APP_, HPW_>), mgrid, dim3(merge_threads<HPW_>), 0,       \
                     stream, partials, quats, out, static_cast<int>(n_kv_heads),                \
                     static_cast<int>(n_splits), seq_lens, lens0, capacity,                     \
                     static_cast<int>(group), runs, static_cast<int>(max_seq_len),              \
                     static_cast<int>(batch), plan.split_len)
  if (append && few) {
    IQ_LAUNCH_SPAN_MERGE(true, 8);
  } else if (append) {
    IQ_LAUNCH_SPAN_MERGE(true, 1);
  } else if (few) {
    IQ_LAUNCH_SPAN_MERGE(false, 8);
  } else {
    IQ_LAUNCH_SPAN_MERGE(false, 1);
  }
#undef IQ_LAUNCH_SPAN_MERGE
  return hipGetLastError();
}

}  // namespace iq
