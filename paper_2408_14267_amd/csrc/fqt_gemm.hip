// The two binary contractions of the 1-bit FQT backward on gfx950, int8 MFMA engine
// (Section 5.3, SCQ; Appendix C, Alg. 1 binary products and dequantization, the
// {0,1} <-> {+-1} conversion and the Folder).
//
// Both products contract b-bit codes q (one byte each, written by the quantizer next to
// the bit planes) with signs s = +-1 held as signed bytes, so one v_mfma_i32_32x32x32_i8
// chain gives I = sum_j q_j s_j exactly in int32.  For b = 8 the codes do not fit a
// signed byte: the MFMA takes q - 128 and 128 * (sum of the signs it saw) is added back.
//   dX: the weight signs arrive expanded to +-1 bytes (fqt_pack_weight_signs), so the
//       inner loop is 16-byte buffer loads and MFMAs.  The zero-point term c = sum over
//       the valid taps of the per-(channel, tap) sign sums is summed per output in the
//       split form and, in the register-tile form, is one float16 (D <= 2048) or a few
//       float32 MFMAs of the sign sums against the 0/1 reach flags (exact either way).
//   dW: the X signs stay packed; each 16-bit piece is expanded in registers to +-1
//       bytes once and feeds up to four MFMAs (128 kept channels).  c = 2 popcount - len.
// The rescale S * I + Z' * c is one float32 step per output without contraction.
//
// MFMA layouts (32 x 32 outputs, 16 accumulators per lane): lane l feeds row (src0) and
// column (src1) l % 32; in the i8 form its 16 bytes are contraction positions
// 16 (l / 32) .. 16 (l / 32) + 15, in the f32 32x32x2 form its one value is position
// l / 32, in the f16 32x32x16 form its 8 values are 8 of the 16 positions (the same
// ones in both operands).  Lane l then holds column l % 32 at rows
// 8 (v / 4) + 4 (l / 32) + (v % 4).
//
// Operands are read through buffer resources: a lane whose row does not exist (padding
// tap, pruned slot, channel past the end) gets the offset BUF_NONE, past every buffer,
// and loads zeros without touching memory.  Every operand layout puts the 32-byte
// contraction chunks of consecutive MFMA rows next to each other (chunk-major codes,
// word-major X signs, chunk-major weight bytes), so one operand load of a wave reads
// about 1 KB of contiguous memory instead of one cache line per lane.
#include <algorithm>
#include <type_traits>

#include "fqt_internal.hpp"

namespace fqt {
namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// 16 sign bits (LSB first) -> 16 signed bytes, +1 for a set bit and -1 for a clear one
// (byte m of dword k holds bit 4k + m).  A nibble times 0x00408102 puts bit m at bit
// 8m + 1 without carries; per byte 2t + 0x7F is 0x7F or 0x81, and flipping bit 7 gives
// 0xFF (-1) or 0x01 (+1).
__device__ __forceinline__ v4i signs16(uint32_t bits) {
  v4i r;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t t2 = (((bits >> (4 * k)) & 0xFu) * 0x00408102u) & 0x02020202u;
    r[k] = int((t2 + 0x7F7F7F7Fu) ^ 0x80808080u);
  }
  return r;
}

__device__ __forceinline__ v4i bias128(v4i a) {
  const int m = int(0x80808080u);
  return v4i{a.x ^ m, a.y ^ m, a.z ^ m, a.w ^ m};
}

__device__ __forceinline__ v16i mfma_i8(v4i a, v4i b, v16i c) {
  return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
}

// Zero `count` elements of `esize` bytes starting at element `first` of `base`, by the
// `nthr` threads of a block: 16-byte stores where the run is 16-byte aligned, bytes of
// the ragged ends one element at a time.
__device__ void zero_run(void *base, size_t first, size_t count, int esize, int tid, int nthr,
                         bool stream) {
  char *p = static_cast<char *>(base) + first * esize;
  const size_t bytes = count * esize;
  const size_t head = (16 - (reinterpret_cast<uintptr_t>(p) & 15)) & 15;
  const size_t lead = head < bytes ? head : bytes;
  const size_t nvec = (bytes - lead) / 16;
  for (size_t e = tid; e * esize < lead; e += nthr) {
    if (esize == 4) reinterpret_cast<uint32_t *>(p)[e] = 0u;
    else reinterpret_cast<uint16_t *>(p)[e] = 0;
  }
  uint4 *v = reinterpret_cast<uint4 *>(p + lead);
  if (stream) {
    for (size_t e = tid; e < nvec; e += nthr) {
      stream_fence();
      __builtin_nontemporal_store(u32x4{0u, 0u, 0u, 0u}, reinterpret_cast<u32x4 *>(v + e));
      stream_fence();
    }
  } else {
    for (size_t e = tid; e < nvec; e += nthr) v[e] = make_uint4(0u, 0u, 0u, 0u);
  }
  char *tail = p + lead + nvec * 16;
  const size_t rest = bytes - lead - nvec * 16;
  for (size_t e = tid; e * esize < rest; e += nthr) {
    if (esize == 4) reinterpret_cast<uint32_t *>(tail)[e] = 0u;
    else reinterpret_cast<uint16_t *>(tail)[e] = 0;
  }
}

// ----------------------------------------------------------------------------- dW

struct DwArgs {
  const uint8_t *codes;          // PCQ codes [2*Wr][D][32], chunk-major
  const int32_t *kept, *count;   // [D], [1]
  const float *scale, *offset;   // [D]
  const float2 *slot_sz;         // [D] (scale, offset) by kept slot, or null (read via kept)
  const uint64_t *xsign;         // [Wr][K], word-major
  float *dW;                     // [D][K]
  int32_t *I_out;                // [D][K] or null
  int32_t *part;                 // [S][D][Kp] partial sums of each split (slots < count)
  int32_t *partT;                // [S][Kp] set bits of each split of each sign line
  uint32_t D, K, Kp, R, Rp, Wr, ktiles, kgroups, codes_bytes, xsign_bytes, S, wps;
  uint32_t wpw;                  // in-block reduction form: words of the contraction per wave
  FastDiv divS, divKg, divQ;    // divQ: Kp / 4
  FastDiv divKt;                 // ktiles
};

constexpr int DW_WAVES = 4;                 // column tiles per block, one per wave
constexpr int DW_THREADS = DW_WAVES * 64;
constexpr int DW_PREF = 4;                  // 64-bit words of the contraction per batch

// One batch of a wave's operands: PREF words of its sign column and the two 32-byte
// code chunks of each word.
template <int PREF>
struct DwBatch {
  uint64_t word[PREF];
  v4i A[PREF][2];
};
template <int PREF>
__device__ __forceinline__ void dw_issue(const DwArgs &a, __amdgpu_buffer_rsrc_t crs,
                                         __amdgpu_buffer_rsrc_t xrs, uint32_t aoff,
                                         uint32_t boff, uint32_t c0, uint32_t w_end,
                                         DwBatch<PREF> &b) {
  const uint32_t chunk_bytes = a.D * 32;      // one 32-position chunk of every PCQ row
#pragma unroll
  for (int u = 0; u < PREF; ++u) {
    const uint32_t c = c0 + u < w_end ? c0 + u : c0;   // past the end: word c0 again
    b.word[u] = load8(xrs, boff, c * a.K * 8);
#pragma unroll
    for (int h = 0; h < 2; ++h) b.A[u][h] = load16(crs, aoff, (2 * c + h) * chunk_bytes);
  }
}
template <bool B8, int PREF>
__device__ __forceinline__ void dw_consume(const DwBatch<PREF> &b, uint32_t c0, uint32_t w_end,
                                           int g, v16i &acc, uint32_t &tpart) {
#pragma unroll
  for (int u = 0; u < PREF; ++u) {
    if (c0 + u >= w_end) break;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t bits = uint32_t(b.word[u] >> (32 * h + 16 * g)) & 0xFFFFu;
      tpart += __popc(bits);
      acc = mfma_i8(B8 ? bias128(b.A[u][h]) : b.A[u][h], signs16(bits), acc);
    }
  }
}

// The contraction of one wave's 32x32 tile over the words [c_first, w_end) of its split,
// double-buffered: the loads of batch i + 1 issue before the products of batch i (a
// sched_barrier keeps the compiler from sinking them), so a long contraction costs one
// exposed memory latency.
template <bool B8, int PREF = DW_PREF>
__device__ __forceinline__ void dw_accumulate(const DwArgs &a, __amdgpu_buffer_rsrc_t crs,
                                              __amdgpu_buffer_rsrc_t xrs, uint32_t aoff,
                                              uint32_t boff, uint32_t c_first, uint32_t w_end,
                                              int g, v16i &acc, uint32_t &tpart) {
  if (c_first >= w_end) return;
  DwBatch<PREF> b0, b1;
  uint32_t c0 = c_first;
  dw_issue<PREF>(a, crs, xrs, aoff, boff, c0, w_end, b0);
  for (;;) {
    if (c0 + PREF < w_end) dw_issue<PREF>(a, crs, xrs, aoff, boff, c0 + PREF, w_end, b1);
    __builtin_amdgcn_sched_barrier(0);
    dw_consume<B8, PREF>(b0, c0, w_end, g, acc, tpart);
    c0 += PREF;
    if (c0 >= w_end) break;
    if (c0 + PREF < w_end) dw_issue<PREF>(a, crs, xrs, aoff, boff, c0 + PREF, w_end, b0);
    __builtin_amdgcn_sched_barrier(0);
    dw_consume<B8, PREF>(b1, c0, w_end, g, acc, tpart);
    c0 += PREF;
    if (c0 >= w_end) break;
  }
}
// Words per batch of the in-block reduction form (8 was measured slower at the 256 -> 256
// conv on 8x8 maps: the products launch it shares with the dX blocks lost occupancy).
constexpr int DW_KRED_PREF = 4;

// dW rows of the slot tile [j0, j0 + 32) of one wave's 32 columns written directly (one
// split, S = 1): I, T, the rescale S_d I + Z'_d (2T - N*Ho*Wo) (b = 8 adds back
// 128 (2T - Rp)), zero rows for pruned slots.  acc: the wave's tile (rows
// acc_row(v, g) of column lane % 32); T: set bits of this lane's column.
template <bool B8>
__device__ __forceinline__ void dw_write_direct(const DwArgs &a, uint32_t j0, uint32_t kc,
                                                int count, const v16i &acc, int T) {
  const int g = (threadIdx.x & 63) >> 5;
  if (kc >= a.K) return;
  // The rows' kept ids, scales and offsets first, all loads together (after a row's dW
  // store the next row's loads could not move ahead of it).
  uint32_t dv[16];
  float2 szv[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const uint32_t j = j0 + uint32_t(acc_row(v, g));
    dv[v] = j < a.D ? uint32_t(a.kept[j]) : 0u;
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const uint32_t j = j0 + uint32_t(acc_row(v, g));
    szv[v] = make_float2(0.0f, 0.0f);
    if (int(j) < count)
      szv[v] = a.slot_sz ? a.slot_sz[j] : make_float2(a.scale[dv[v]], a.offset[dv[v]]);
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const uint32_t j = j0 + uint32_t(acc_row(v, g));
    if (j >= a.D) continue;
    const size_t d = dv[v];
    int I = 0;
    float out = 0.0f;
    if (int(j) < count) {
      I = acc[v] + (B8 ? 128 * (2 * T - int(a.Rp)) : 0);
      out = rescale(szv[v].x, I, szv[v].y, float(2 * T - int(a.R)));
    }
    a.dW[d * a.K + kc] = out;
    if (a.I_out) a.I_out[d * a.K + kc] = I;
  }
}

// Split-R partial products.  Grid: S splits x ceil(ceil(K/32) / 4) column groups x
// ceil(D/32) slot tiles over the slot capacity, the split index fastest (consecutive
// blocks land on different XCDs, so each XCD reads its own slices of the codes and of the
// signs) and the slot tile slowest.  Wave w of a block computes the 32x32 MFMA tile (slot
// tile, column tile 4 * group + w) over the words [s * wps, (s + 1) * wps) of the
// contraction over N*Ho*Wo: the four waves read the same code rows (one fetch from L2)
// and their own sign columns, and each writes its tile and the set-bit counts of its
// columns to the split's slice.  No LDS, no barrier.
// DIRECT (S = 1): the wave writes dW itself, and slot tiles past the kept channels zero
// their rows; otherwise those blocks exit at once and the finish pass writes dW.
template <bool B8, bool DIRECT>
__device__ __forceinline__ void dw_part_body(const DwArgs &a, uint32_t bid) {
  const int lane = threadIdx.x & 63;
  const uint32_t wave = wave_id();
  const int i = lane & 31, g = lane >> 5;
  const int count = *a.count;
  const uint32_t rest = fdiv(bid, a.divS);
  const uint32_t sp = bid - rest * a.S;
  const uint32_t rt = fdiv(rest, a.divKg);
  const uint32_t kt = (rest - rt * a.kgroups) * DW_WAVES + wave;
  const uint32_t j0 = rt * 32;
  if (kt >= a.ktiles) return;                   // past the columns
  const uint32_t kc = kt * 32 + i;
  if (int(j0) >= count) {                       // past the kept channels
    if (DIRECT) dw_write_direct<B8>(a, j0, kc, count, v16i{0}, 0);
    return;
  }

  const __amdgpu_buffer_rsrc_t crs = buffer_of(a.codes, a.codes_bytes);
  const __amdgpu_buffer_rsrc_t xrs = buffer_of(a.xsign, a.xsign_bytes);
  const uint32_t j = j0 + i;
  const uint32_t aoff = int(j) < count ? j * 32 + 16 * g : BUF_NONE;
  const bool b_ok = kc < a.K;
  const uint32_t boff = b_ok ? kc * 8 : BUF_NONE;
  const uint32_t w_end = min(a.Wr, (sp + 1) * a.wps);
  v16i acc = v16i{0};
  uint32_t tpart = 0;
  dw_accumulate<B8>(a, crs, xrs, aoff, boff, sp * a.wps, w_end, g, acc, tpart);

  // Set bits of column kc in this split: lanes i and i + 32 counted the two halves of
  // every 32-bit piece.
  const uint32_t T = tpart + lane_xor<32>(tpart);
  if (DIRECT) {
    dw_write_direct<B8>(a, j0, kc, count, acc, int(T));
    return;
  }
  if (!b_ok) return;
  if (rt == 0 && g == 0) a.partT[size_t(sp) * a.Kp + kc] = int32_t(T);
  int32_t *out = a.part + (size_t(sp) * a.D + j0) * a.Kp + kc;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int row = acc_row(v, g);
    if (int(j0) + row < count) out[size_t(row) * a.Kp] = acc[v];
  }
}

// dW with the contraction split over the four waves of a block and reduced in LDS (no
// partial sums leave the workgroup, no finish pass).  Grid: ceil(D/32) slot tiles x
// ceil(K/32) column tiles over the slot capacity, column tiles fastest (a column tile keeps
// its XCD across slot tiles when the number of column tiles is a multiple of eight, so its
// sign words are fetched into one L2).  Wave w contracts the 32 x 32 tile over the words
// [w wpw, (w + 1) wpw) of N*Ho*Wo; the four partial tiles and set-bit counts meet in LDS,
// and wave w finishes accumulator registers 4w .. 4w + 3 (slot rows 8w + 4g + u): the sum
// over the waves, the b = 8 bias term, the rescale and the dW stores.  Slot tiles past the
// kept channels write their rows of zeros.
struct DwRedLds {
  int32_t red[DW_WAVES][16][64];
  uint32_t tred[DW_WAVES][32];
};
template <bool B8>
__device__ __forceinline__ void dw_kred_body(const DwArgs &a, uint32_t bid, DwRedLds &sm) {
  const int lane = threadIdx.x & 63;
  const uint32_t wave = wave_id();
  const int i = lane & 31, g = lane >> 5;
  const int count = *a.count;
  const uint32_t rt = fdiv(bid, a.divKt);
  const uint32_t kt = bid - rt * a.ktiles;
  const uint32_t j0 = rt * 32, kc = kt * 32 + uint32_t(i);
  const bool live = int(j0) < count;            // uniform over the block
  if (live) {
    const __amdgpu_buffer_rsrc_t crs = buffer_of(a.codes, a.codes_bytes);
    const __amdgpu_buffer_rsrc_t xrs = buffer_of(a.xsign, a.xsign_bytes);
    const uint32_t j = j0 + uint32_t(i);
    const uint32_t aoff = int(j) < count ? j * 32 + 16 * g : BUF_NONE;
    const uint32_t boff = kc < a.K ? kc * 8 : BUF_NONE;
    const uint32_t cb = wave * a.wpw;
    const uint32_t ce = min(a.Wr, cb + a.wpw);
    v16i acc = v16i{0};
    uint32_t tpart = 0;
    dw_accumulate<B8, DW_KRED_PREF>(a, crs, xrs, aoff, boff, cb, ce, g, acc, tpart);
    const uint32_t T = tpart + lane_xor<32>(tpart);
#pragma unroll
    for (int v = 0; v < 16; ++v) sm.red[wave][v][lane] = acc[v];
    if (g == 0) sm.tred[wave][i] = T;
  }
  __syncthreads();
  int T = 0;
  if (live) T = int(sm.tred[0][i] + sm.tred[1][i] + sm.tred[2][i] + sm.tred[3][i]);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int v = 4 * int(wave) + u;
    const uint32_t j = j0 + uint32_t(acc_row(v, g));
    if (j >= a.D) continue;
    const size_t d = size_t(a.kept[j]);
    int I = 0;
    float out = 0.0f;
    if (int(j) < count) {
      I = sm.red[0][v][lane] + sm.red[1][v][lane] + sm.red[2][v][lane] + sm.red[3][v][lane];
      if (B8) I += 128 * (2 * T - int(a.Rp));
      const float2 sz = a.slot_sz ? a.slot_sz[j] : make_float2(a.scale[d], a.offset[d]);
      out = rescale(sz.x, I, sz.y, float(2 * T - int(a.R)));
    }
    if (kc < a.K) {
      a.dW[d * a.K + kc] = out;
      if (a.I_out) a.I_out[d * a.K + kc] = I;
    }
  }
}

// Large dW outputs in one split (DIRECT): each wave holds a (32 RT) x (32 CT) block of
// the output in RT x CT MFMA tiles, and a block's four waves take four adjacent column
// blocks of the same slots (the code rows come from L2 once).  Grid: ceil(D / (32 RT))
// slot blocks x ceil(K / (128 CT)) column groups, slots slowest.
// Here the X signs enter the MFMA as 0/1 bytes b (three VALU operations per four signs,
// shared by the row tiles) instead of +-1, and the signed sum comes back per output as
// sum q s = 2 sum q b - sum q (s = 2b - 1; b = 0 on the zero tail of the last word, where
// q = 0 too).  The code sums sum q of the rows are taken from the A fragments with
// v_dot4_u32_u8 (four per fragment, shared by the column tiles).  For b = 8 the codes
// enter as q - 128: sum q b = acc + 128 T.  The words of the contraction stream through a
// ring of ST register batches.
// Shapes (row tiles RT, column tiles CT, ring depth ST): long contractions take 2 x 4
// tiles and a four-word ring at two waves per SIMD; short ones (a few words, where the
// dW stores dominate) 2 x 2 tiles and two words at the occupancy the registers allow.
constexpr int DWB_LONG_WORDS = 8;     // contractions of at least this many words: long form
template <int RT, int CT, bool FP4 = false>
struct DwBigBatch {
  uint64_t word[CT];                      // FP4: the half-wave's 32 positions
  v4i A[FP4 ? 1 : 2][RT];                 // [half][row tile]
};
template <int RT, int CT, bool FP4>
__device__ __forceinline__ void dwb_issue(const DwArgs &a, __amdgpu_buffer_rsrc_t crs,
                                          __amdgpu_buffer_rsrc_t xrs, const uint32_t (&aoff)[RT],
                                          const uint32_t (&boff)[CT], uint32_t c,
                                          DwBigBatch<RT, CT, FP4> &b) {
  // Word offsets as scalars (kept out of any vector induction variable).
  const uint32_t xs = __builtin_amdgcn_readfirstlane(c * a.K * 8);
  const uint32_t cs0 = __builtin_amdgcn_readfirstlane((FP4 ? c : 2 * c) * a.D * 32);
  const uint32_t cs1 = __builtin_amdgcn_readfirstlane((2 * c + 1) * a.D * 32);
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
    b.word[ct] = FP4 ? uint32_t(__builtin_amdgcn_raw_buffer_load_b32(xrs, boff[ct], xs, 0))
                     : load8(xrs, boff[ct], xs);
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    b.A[0][rt] = load16(crs, aoff[rt], cs0);
    if constexpr (!FP4) b.A[1][rt] = load16(crs, aoff[rt], cs1);
  }
}
// FP4: +-1 nibbles from 32 sign bits in the codes' order (dword q: positions 4 n + q, the bit
// moved to the sign of a nibble 0x2), one fp4 MFMA per tile and word.
template <int RT, int CT>
__device__ __forceinline__ void dwb_consume4(const DwBigBatch<RT, CT, true> &b, uint32_t c88,
                                             v16f (&acc)[RT][CT], uint32_t (&tcnt)[CT]) {
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    const uint32_t n = ~uint32_t(b.word[ct]);
    tcnt[ct] += __popc(uint32_t(b.word[ct]));
    v4i B;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      B[q] = int(__builtin_amdgcn_bitop3_b32(n << (3 - q), c88, 0x22222222u, 0xEA));
    const v8i B8v{B.x, B.y, B.z, B.w, 0, 0, 0, 0};
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const v4i A = b.A[0][rt];
      acc[rt][ct] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
          v8i{A.x, A.y, A.z, A.w, 0, 0, 0, 0}, B8v, acc[rt][ct], 4, 4, 0, 127, 0, 127);
    }
  }
}
// Four sign bits of `half` from bit `off` (LSB first) as four 0/1 bytes: a nibble times
// 0x00204081 puts bit m at bit 8m (the cross terms land on other bits, without carries)
// and the mask keeps those.
__device__ __forceinline__ int bits01x4(uint32_t half, uint32_t off) {
  return int((__builtin_amdgcn_ubfe(half, off, 4) * 0x00204081u) & 0x01010101u);
}
template <bool B8, int RT, int CT>
__device__ __forceinline__ void dwb_consume(const DwBigBatch<RT, CT> &b, const uint32_t (&off)[4],
                                            v16i (&acc)[RT][CT], uint32_t (&tcnt)[CT],
                                            uint32_t (&qsum)[RT]) {
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
    tcnt[ct] += __popc(uint32_t(b.word[ct])) + __popc(uint32_t(b.word[ct] >> 32));
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    // For b = 8 the sums are taken of the biased bytes q - 128 (signed), the only form
    // kept in registers; the epilogue adds 128 per position back.
    v4i A[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      A[rt] = B8 ? bias128(b.A[h][rt]) : b.A[h][rt];
#pragma unroll
      for (int k = 0; k < 4; ++k)
        qsum[rt] = B8 ? uint32_t(__builtin_amdgcn_sdot4(A[rt][k], 0x01010101, int(qsum[rt]), false))
                      : __builtin_amdgcn_udot4(uint32_t(A[rt][k]), 0x01010101u, qsum[rt], false);
    }
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const uint32_t half = uint32_t(b.word[ct] >> (32 * h));
      const v4i B = v4i{bits01x4(half, off[0]), bits01x4(half, off[1]), bits01x4(half, off[2]),
                        bits01x4(half, off[3])};
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[rt][ct] = mfma_i8(A[rt], B, acc[rt][ct]);
    }
  }
}
// SPLIT: the same tiles over the word slice [s wps, (s + 1) wps) of a split-R product,
// writing the slice's partial sums (in the split kernel's form, sum over the slice of
// A_r s_r with A_r the MFMA code byte: 2 sum A b - sum A) and its set-bit counts for the
// finish pass.  Grid: S slices (fastest) x slot blocks x column groups.
template <bool B8, int RT, int CT, int ST, bool SPLIT = false, bool STREAM = false, bool FP4 = false>
__device__ __forceinline__ void dw_big_body(const DwArgs &a, uint32_t bid) {
  const int lane = threadIdx.x & 63;
  const uint32_t wave = wave_id();
  const int i = lane & 31, g = lane >> 5;
  const int count = *a.count;
  const uint32_t kgroups = (a.K + DW_WAVES * 32 * CT - 1) / (DW_WAVES * 32 * CT);
  uint32_t sp = 0;
  if (SPLIT) {
    const uint32_t rest = fdiv(bid, a.divS);
    sp = bid - rest * a.S;
    bid = rest;
  }
  const uint32_t cb = SPLIT ? sp * a.wps : 0u;
  const uint32_t ce = SPLIT ? min(a.Wr, cb + a.wps) : a.Wr;
  const uint32_t rb = bid / kgroups;
  const uint32_t j0 = rb * (32 * RT);
  const uint32_t k0 = ((bid - rb * kgroups) * DW_WAVES + wave) * (32 * CT);
  if (k0 >= a.K) return;
  std::conditional_t<FP4, v16f, v16i> acc[RT][CT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = std::conditional_t<FP4, v16f, v16i>{0};
  uint32_t tcnt[CT], qsum[RT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) tcnt[ct] = 0u;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) qsum[rt] = 0u;
  if (int(j0) < count && ce > cb) {
    const __amdgpu_buffer_rsrc_t crs = buffer_of(a.codes, a.codes_bytes);
    const __amdgpu_buffer_rsrc_t xrs = buffer_of(a.xsign, a.xsign_bytes);
    uint32_t aoff[RT], boff[CT], off[4];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const uint32_t j = j0 + 32 * rt + i;
      aoff[rt] = int(j) < count ? j * 32 + 16 * g : BUF_NONE;
    }
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const uint32_t kc = k0 + 32 * ct + i;
      boff[ct] = kc < a.K ? kc * 8 + (FP4 ? 4 * g : 0) : BUF_NONE;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) off[k] = uint32_t(16 * g + 4 * k);
    // A ring of ST words: word c + ST is requested as soon as word c has
    // been used, so ST - 1 words are in flight during each word's products.  Every
    // step issues the same loads (a word past the end re-reads the last one), so the
    // waits count exactly.
    DwBigBatch<RT, CT, FP4> bs[ST];
    uint32_t c88 = 0x88888888u;           // (in a vector register: an instruction takes one scalar)
    asm("" : "+v"(c88));
    const uint32_t last = ce - 1;
#pragma unroll
    for (int u = 0; u < ST; ++u) dwb_issue(a, crs, xrs, aoff, boff, min(cb + uint32_t(u), last), bs[u]);
    for (uint32_t c = cb; c < ce; c += ST) {
#pragma unroll
      for (int u = 0; u < ST; ++u) {
        if (c + u >= ce) break;
        if constexpr (FP4) dwb_consume4<RT, CT>(bs[u], c88, acc, tcnt);
        else dwb_consume<B8, RT, CT>(bs[u], off, acc, tcnt, qsum);
        __builtin_amdgcn_sched_barrier(0);
        dwb_issue(a, crs, xrs, aoff, boff, min(c + u + ST, last), bs[u]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  if constexpr (FP4)                      // each half-wave counted its own positions
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) tcnt[ct] += lane_xor<32>(tcnt[ct]);
  // Lane i (and i + 32) holds half of the code sum of row i of each row tile; the
  // accumulator rows of a lane are acc_row(v, g), fetched from their lanes.
  if (SPLIT) {
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const uint32_t kc = k0 + 32 * ct + i;
      if (rb == 0 && g == 0 && kc < a.K) a.partT[size_t(sp) * a.Kp + kc] = int32_t(tcnt[ct]);
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int qrow = int(qsum[rt] + lane_xor<32>(qsum[rt]));   // sum of A over the slice
      int qv[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) qv[v] = __shfl(qrow, acc_row(v, g));
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const uint32_t kc = k0 + 32 * ct + i;
        if (kc >= a.K) continue;
        int32_t *out = a.part + (size_t(sp) * a.D + j0 + 32 * rt) * a.Kp + kc;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int row = acc_row(v, g);
          if (int(j0) + 32 * rt + row < count) out[size_t(row) * a.Kp] = 2 * int(acc[rt][ct][v]) - qv[v];
        }
      }
    }
    return;
  }
  // The tiles go out through a row-major LDS copy per wave, two column tiles (64 columns) at a
  // time, consecutive lanes storing consecutive 16-byte pieces: 256 bytes of each kept row,
  // whole lines (pieces of two lanes per row and tile reached 3.1 TB/s at 25088 -> 4096, batch
  // 64).  Misaligned rows, columns past K and the integer debug output take element stores.
  if constexpr (!SPLIT) {
    if (!a.I_out) {
      constexpr int SC = 64, SP = SC + 4;     // staged columns, and their pitch in floats
      static_assert(CT % 2 == 0, "pairs of column tiles");
      __shared__ __align__(16) float stage[DW_WAVES][32 * SP];
      float *st = stage[wave];
      const bool vec = (a.K & 3) == 0 && (reinterpret_cast<uintptr_t>(a.dW) & 15) == 0;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const int qrow = int(qsum[rt] + lane_xor<32>(qsum[rt])) + (B8 ? 128 * int(a.Rp) : 0);
        int qv[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) qv[v] = __shfl(qrow, acc_row(v, g));
        const uint32_t jt = j0 + 32 * rt;
        // The rows' scales and offsets and this lane's store rows, loaded once per row tile,
        // all at once (inside the column-tile loop they would follow each tile's dW stores,
        // which the compiler cannot move them across: a dependent round trip per tile).
        float2 szv[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const uint32_t j = jt + uint32_t(acc_row(v, g));
          szv[v] = make_float2(0.0f, 0.0f);
          if (int(j) < count)
            szv[v] = a.slot_sz ? a.slot_sz[j] : make_float2(a.scale[a.kept[j]], a.offset[a.kept[j]]);
        }
        uint32_t drow[8];                     // row 4 k + lane / 16 of the tile
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const uint32_t j = jt + 4 * k + uint32_t(lane >> 4);
          drow[k] = j < a.D ? uint32_t(a.kept[j]) : 0;
        }
#pragma unroll
        for (int cp = 0; cp < CT; cp += 2) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int T = int(tcnt[cp + h]);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
              const uint32_t j = jt + uint32_t(acc_row(v, g));
              float out = 0.0f;
              if (int(j) < count) {
                const int I = FP4 ? int(acc[rt][cp + h][v])
                                  : 2 * (int(acc[rt][cp + h][v]) + (B8 ? 128 * T : 0)) - qv[v];
                out = rescale(szv[v].x, I, szv[v].y, float(2 * T - int(a.R)));
              }
              st[acc_row(v, g) * SP + 32 * h + i] = out;
            }
          }
          __builtin_amdgcn_wave_barrier();    // LDS operations of a wave run in order
          const uint32_t col = k0 + 32 * cp + 4 * uint32_t(lane & 15);
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const int row = 4 * k + (lane >> 4);
            if (jt + row >= a.D || col >= a.K) continue;
            const u32x4 f = *reinterpret_cast<const u32x4 *>(st + row * SP + 4 * (lane & 15));
            float *dst = a.dW + size_t(drow[k]) * a.K + col;
            if (vec) {
              if constexpr (STREAM) __builtin_nontemporal_store(f, reinterpret_cast<u32x4 *>(dst));
              else *reinterpret_cast<u32x4 *>(dst) = f;
            } else {
              dst[0] = __uint_as_float(f[0]);
              if (col + 1 < a.K) dst[1] = __uint_as_float(f[1]);
              if (col + 2 < a.K) dst[2] = __uint_as_float(f[2]);
              if (col + 3 < a.K) dst[3] = __uint_as_float(f[3]);
            }
          }
          __builtin_amdgcn_wave_barrier();    // the next tiles' copy waits for these reads
        }
      }
      return;
    }
  }
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    // Sum of the codes of row i of the tile (b = 8: of q - 128 over all Rp positions).
    const int qrow = int(qsum[rt] + lane_xor<32>(qsum[rt])) + (B8 ? 128 * int(a.Rp) : 0);
    int qv[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) qv[v] = __shfl(qrow, acc_row(v, g));
    const uint32_t jt = j0 + 32 * rt;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const uint32_t kc = k0 + 32 * ct + i;
      if (kc >= a.K) continue;
      const int T = int(tcnt[ct]);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const uint32_t j = jt + uint32_t(acc_row(v, g));
        if (j >= a.D) continue;
        const size_t d = size_t(a.kept[j]);
        int I = 0;
        float out = 0.0f;
        if (int(j) < count) {
          const float2 sz = a.slot_sz ? a.slot_sz[j] : make_float2(a.scale[d], a.offset[d]);
          I = FP4 ? int(acc[rt][ct][v]) : 2 * (int(acc[rt][ct][v]) + (B8 ? 128 * T : 0)) - qv[v];
          out = rescale(sz.x, I, sz.y, float(2 * T - int(a.R)));
        }
        a.dW[d * a.K + kc] = out;
        if (a.I_out) a.I_out[d * a.K + kc] = I;
      }
    }
  }
}
// Blocks of the big form with RT row tiles and CT column tiles per wave.
uint32_t dw_big_blocks(uint32_t D, uint32_t K, int rt, int ct) {
  return ((D + 32 * rt - 1) / (32 * rt)) * ((K + DW_WAVES * 32 * ct - 1) / (DW_WAVES * 32 * ct));
}

// Split-R partials in the big form (long slices of the contraction, wide outputs): two row
// tiles per wave, or one when the kept channels are expected to fit 32 rows (a second
// row tile would multiply zeros).  A four-word ring (163 registers for two row tiles, 96
// for one) was measured 2-5 % faster than two words on VGG-16's layers at 224.
template <bool B8, int RT>
__global__ __launch_bounds__(DW_THREADS) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_mfma_dw_split(DwArgs a) {
  dw_big_body<B8, RT, 2, 4, true>(a, blockIdx.x);
}
uint32_t dw_split_blocks(const DwArgs &a, int rt) {
  return a.S * dw_big_blocks(a.D, a.K, rt, 2);
}

// Long contractions: two waves per SIMD (the accumulators and the word ring fit 256
// registers).
template <bool B8, bool STREAM>
__global__ __launch_bounds__(DW_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mfma_dw_big(DwArgs a) {
  dw_big_body<B8, 2, 4, 4, false, STREAM>(a, blockIdx.x);
}
// The same from nibble codes (b <= 2, the layer backward): 8 expansion operations per 64
// positions of a column instead of 24, half the matrix steps and code bytes.
template <bool STREAM>
__global__ __launch_bounds__(DW_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mfma_dw_big4(DwArgs a) {
  dw_big_body<false, 2, 4, 4, false, STREAM, true>(a, blockIdx.x);
}
// Short contractions: three waves per SIMD, for the stores.
template <bool B8, bool STREAM>
__global__ __launch_bounds__(DW_THREADS) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_mfma_dw_short(DwArgs a) {
  dw_big_body<B8, 2, 2, 2, false, STREAM>(a, blockIdx.x);
}

template <bool B8, bool DIRECT>
__global__ __launch_bounds__(DW_THREADS) void k_mfma_dw_part(DwArgs a) {
  dw_part_body<B8, DIRECT>(a, blockIdx.x);
}

template <bool B8>
__global__ __launch_bounds__(DW_THREADS) void k_mfma_dw_kred(DwArgs a) {
  __shared__ DwRedLds sm;
  dw_kred_body<B8>(a, blockIdx.x, sm);
}

// dW from the split partials: one thread per 4 columns (slot, k .. k + 3) of the slot
// capacity, reading 16 bytes of each partial row.  A kept slot sums its S partials,
// I = sum (+ 128 (2T - Rp) for b = 8, whose codes entered as q - 128 against every sign
// including the zero tail of the last word) and writes S_d * I + Z'_d * (2T - N*Ho*Wo) to
// row d = kept[slot]; a pruned slot zeroes its row.
template <bool B8>
__global__ __launch_bounds__(256) void k_dw_finish(DwArgs a) {
  const uint32_t e = blockIdx.x * 256 + threadIdx.x;
  const uint32_t qrow = a.Kp / 4;
  if (e >= a.D * qrow) return;
  const uint32_t slot = fdiv(e, a.divQ), k = 4 * (e - slot * qrow);
  if (k >= a.K) return;
  const int count = *a.count;
  const size_t d = size_t(a.kept[slot]);
  int I[4] = {0, 0, 0, 0};
  float out[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if (int(slot) < count) {
    int4 acc = make_int4(0, 0, 0, 0), T4 = make_int4(0, 0, 0, 0);
    // Eight slices' loads issue together (a slice past S re-reads the last one and is not
    // added), so the sum costs one memory latency per eight slices.
    constexpr uint32_t U = 8;
    for (uint32_t s0 = 0; s0 < a.S; s0 += U) {
      int4 v[U], t4[U];
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t s = min(s0 + u, a.S - 1);
        v[u] = *reinterpret_cast<const int4 *>(a.part + (size_t(s) * a.D + slot) * a.Kp + k);
        t4[u] = *reinterpret_cast<const int4 *>(a.partT + size_t(s) * a.Kp + k);
      }
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const int m = s0 + u < a.S ? 1 : 0;
        acc.x += m * v[u].x; acc.y += m * v[u].y; acc.z += m * v[u].z; acc.w += m * v[u].w;
        T4.x += m * t4[u].x; T4.y += m * t4[u].y; T4.z += m * t4[u].z; T4.w += m * t4[u].w;
      }
    }
    const int T[4] = {T4.x, T4.y, T4.z, T4.w};
    I[0] = acc.x; I[1] = acc.y; I[2] = acc.z; I[3] = acc.w;
    const float2 sz = a.slot_sz ? a.slot_sz[slot] : make_float2(a.scale[d], a.offset[d]);
    const float Sd = sz.x, Zd = sz.y;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (B8) I[u] += 128 * (2 * T[u] - int(a.Rp));
      out[u] = rescale(Sd, I[u], Zd, float(2 * T[u] - int(a.R)));
    }
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    if (k + u >= a.K) break;
    a.dW[d * a.K + k + u] = out[u];
    if (a.I_out) a.I_out[d * a.K + k + u] = I[u];
  }
}

// The same for many splits: one block per (slot, 64 columns); thread t sums every 16th
// split of column quad t % 16 from split t / 16, and the 16 partial sums of each quad
// meet in LDS.
constexpr int DWF_CHUNKS = 16;
template <bool B8>
__global__ __launch_bounds__(256) void k_dw_finish_wide(DwArgs a) {
  __shared__ int4 red[DWF_CHUNKS][16], tred[DWF_CHUNKS][16];
  const int t = threadIdx.x, quad = t & 15, chunk = t >> 4;
  const uint32_t qblocks = a.Kp / 64 + (a.Kp % 64 ? 1 : 0);
  const uint32_t slot = blockIdx.x / qblocks;
  const uint32_t k = (blockIdx.x - slot * qblocks) * 64 + 4 * quad;
  const int count = *a.count;
  const bool live = int(slot) < count && k < a.Kp;
  int4 acc = make_int4(0, 0, 0, 0), T4 = make_int4(0, 0, 0, 0);
  if (live) {
    // Four of this chunk's slices load together (a slice past S re-reads the last one and
    // is not added).
    constexpr uint32_t U = 4;
    for (uint32_t s0 = chunk; s0 < a.S; s0 += U * DWF_CHUNKS) {
      int4 v[U], t4[U];
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t s = min(s0 + u * DWF_CHUNKS, a.S - 1);
        v[u] = *reinterpret_cast<const int4 *>(a.part + (size_t(s) * a.D + slot) * a.Kp + k);
        t4[u] = *reinterpret_cast<const int4 *>(a.partT + size_t(s) * a.Kp + k);
      }
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const int m = s0 + u * DWF_CHUNKS < a.S ? 1 : 0;
        acc.x += m * v[u].x; acc.y += m * v[u].y; acc.z += m * v[u].z; acc.w += m * v[u].w;
        T4.x += m * t4[u].x; T4.y += m * t4[u].y; T4.z += m * t4[u].z; T4.w += m * t4[u].w;
      }
    }
  }
  red[chunk][quad] = acc;
  tred[chunk][quad] = T4;
  __syncthreads();
  if (chunk != 0 || k >= a.K) return;
#pragma unroll
  for (int c = 1; c < DWF_CHUNKS; ++c) {
    const int4 v = red[c][quad], t4 = tred[c][quad];
    acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    T4.x += t4.x; T4.y += t4.y; T4.z += t4.z; T4.w += t4.w;
  }
  const size_t d = size_t(a.kept[slot]);
  int I[4] = {0, 0, 0, 0};
  float out[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if (live) {
    const int T[4] = {T4.x, T4.y, T4.z, T4.w};
    I[0] = acc.x; I[1] = acc.y; I[2] = acc.z; I[3] = acc.w;
    const float2 sz = a.slot_sz ? a.slot_sz[slot] : make_float2(a.scale[d], a.offset[d]);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (B8) I[u] += 128 * (2 * T[u] - int(a.Rp));
      out[u] = rescale(sz.x, I[u], sz.y, float(2 * T[u] - int(a.R)));
    }
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    if (k + u >= a.K) break;
    a.dW[d * a.K + k + u] = out[u];
    if (a.I_out) a.I_out[d * a.K + k + u] = I[u];
  }
}
// Splits above which the finish takes a block per (slot, 64 columns).
constexpr uint32_t DWF_WIDE = 32;

// ----------------------------------------------------------------------------- dX

struct DxArgs {
  const uint8_t *codes;          // PSQ codes [Dp/32][N*Ho*Wo][32], chunk-major
  const int32_t *kept, *count;   // [N], [1]
  const float *scale, *offset;   // [N]
  const float2 *slot_sz;         // [N] (scale, offset) by kept slot, or null (read via kept)
  const int8_t *wsb;             // sign(W) bytes [Dp/32][kh*kw][C][32]: +-1, 0 past D
  const int32_t *wlsum;          // [C*kh*kw] sum over d of the signs of each line
  void *dX;                      // [N][C][H][W]
  int32_t *I_out;
  int dx_t;
  uint32_t N, C, H, W, HW, Ho, Wo, P, R, Dp, ctiles, CHW, taps, nch;   // nch = ceil(D / 32)
  uint32_t codes_bytes, wsb_bytes;
  int kh, kw, sh, sw, ph, pw;
  FastDiv divHW, divW, divKw, divNch, divCt, divSh, divSw;
  uint32_t nblocks;              // blocks of the dX grid (compute tiles + zero pool)
  uint32_t zpieces;              // pieces of DX_ZCHUNK elements per pruned sample
  uint32_t wide;                 // DxForm
  uint32_t vec;                  // register tiles: pieces of 4 pixels (HW % 4 == 0, aligned dX and X, no I_out)
  uint32_t D;
  uint32_t cblocks;              // register-tile forms: channel blocks of 32 CT channels
  FastDiv divCb;
  uint32_t stream;               // dX by non-temporal stores (STREAM_BYTES)
  const float *ste;              // training: X; dX (float32) is 0 where |X| <= 1 does not hold
};

// The straight-through estimator's mask of element o.
__device__ __forceinline__ bool ste_pass(const DxArgs &a, size_t o) {
  return !a.ste || __builtin_fabsf(a.ste[o]) <= 1.0f;
}

// The forms of the dX product: the contraction of a 32 x 32 tile split over four waves, or
// register tiles (one channel tile per wave, two, two with the channels along the lanes).
enum DxForm : uint32_t { DX_SPLIT = 0, DX_CT1 = 1, DX_CT2 = 2, DX_LIN = 3 };
constexpr int DX_MAX_TAPS = 64;
constexpr uint32_t DX_ZCHUNK = 65536;    // elements of a pruned sample one block zeroes
constexpr int DX_WAVES = 4;
constexpr int DX_THREADS = DX_WAVES * 64;
// Tiles (channel tiles fastest, then pixel tiles) of one XCD run: 16 split-form tiles of
// 32 x 32, 32 register-form tiles of 256 pixels x 32 CT channels.
constexpr uint32_t DX_XCD_RUN = 16, DXW_XCD_RUN = 32;

// NB: contraction steps (tap, 32 bytes of D) a wave loads at once, sized on the host so
// that the common shapes take one batch: the loads of a wave then cost one memory latency.
// Grid: one block per 32x32 tile of (channel, row m = (kept slot, h, w)) over the capacity
// N*H*W rows, plus a pool of extra blocks.  Blocks of the first ceil(count*H*W/32) row
// tiles compute; all later blocks zero the pruned samples of dX (each a contiguous run of
// C*H*W elements) in pieces of DX_ZCHUNK elements.
// A computing block is one 32x32 MFMA tile with the sign operand as src0 (rows =
// channels) so output lanes run along pixels.  Its four waves take every fourth
// contraction step (tap, 32 bytes of D).  For tap (i, j) a pixel (h, w) reads the code row
// of the output pixel (ho, wo) with ho*sh - ph + i = h and wo*sw - pw + j = w, or nothing;
// the byte offset of every (tap, pixel) row is tabulated once per block, next to the sign
// sums of the block's channels per tap.  The four partial tiles meet in LDS and wave w
// finishes accumulator registers 4w .. 4w + 3 (channel rows 8w + 4g + u): their integer
// sums, the zero-point term c = sum of the channel's sign sums over the taps that reach
// the pixel (exact integers), the rescale and the stores.
struct alignas(16) DxLds {
  uint32_t rowoff[DX_MAX_TAPS][32];     // 32 * code row, BUF_NONE if none
  int32_t wl[DX_MAX_TAPS][32];          // sign sum of line (channel c0 + k, tap), 0 past C
  int32_t red[DX_WAVES][16][64];        // partial tiles of the four waves
  int32_t pix_out[32];                  // NCHW offset of (sample, pixel) minus channel
  float pix_s[32], pix_z[32];
};

// Zeroing of the pruned samples by the blocks of the zero pool: task t of
// (N - count) * zpieces is piece t % zpieces of pruned slot t / zpieces.
__device__ __forceinline__ void dx_zero_pool(const DxArgs &a, uint32_t zb, uint32_t nz,
                                             int count) {
  const int t = threadIdx.x;
  const uint32_t tasks = (a.N - uint32_t(count)) * a.zpieces;
  for (uint32_t task = zb; task < tasks; task += nz) {
    const uint32_t slot = task / a.zpieces, piece = task - slot * a.zpieces;
    const size_t n = size_t(a.kept[uint32_t(count) + slot]);
    const size_t first = size_t(piece) * DX_ZCHUNK;
    const size_t len = min(size_t(DX_ZCHUNK), size_t(a.CHW) - first);
    zero_run(a.dX, n * a.CHW + first, len, a.dx_t == FQT_BF16 ? 2 : 4, t, DX_THREADS, a.stream);
    if (a.I_out) zero_run(a.I_out, n * a.CHW + first, len, 4, t, DX_THREADS, false);
  }
}

// The code-row offsets of a block's BP pixel rows m0 .. m0 + BP - 1 over the taps:
// rowoff[tap][p] = 32 * (code row of the output pixel that pixel m0 + p meets through the
// tap), BUF_NONE where the tap falls between strides or outside dY, or past the live rows.
// Thread t decodes pixel p = t % BP once and walks the taps t / BP, t / BP + NT / BP, ...
// (a pixel's taps differ only in the tap's (i, j)).
template <uint32_t BP, int NT>
__device__ __forceinline__ void dx_row_table(const DxArgs &a, uint32_t m0, uint32_t live_rows,
                                             uint32_t (*rowoff)[BP]) {
  static_assert(NT % BP == 0, "whole pixel sets per pass");
  constexpr uint32_t STEP = NT / BP;
  const uint32_t p = uint32_t(threadIdx.x) % BP;
  const uint32_t m = m0 + p;
  const bool live = m < live_rows;
  uint32_t slot = 0, h = 0, w = 0;
  if (live) {
    slot = fdiv(m, a.divHW);
    const uint32_t pix = m - slot * a.HW;
    h = fdiv(pix, a.divW);
    w = pix - h * a.W;
  }
  uint32_t tap = uint32_t(threadIdx.x) / BP;
  uint32_t ti = fdiv(tap, a.divKw), tj = tap - ti * uint32_t(a.kw);
  for (; tap < a.taps; tap += STEP) {
    uint32_t off = BUF_NONE;
    const int th = int(h) + a.ph - int(ti), tw = int(w) + a.pw - int(tj);
    if (live && th >= 0 && tw >= 0) {
      const uint32_t ho = fdiv(uint32_t(th), a.divSh), wo = fdiv(uint32_t(tw), a.divSw);
      if (ho * uint32_t(a.sh) == uint32_t(th) && wo * uint32_t(a.sw) == uint32_t(tw) &&
          ho < a.Ho && wo < a.Wo)
        off = (slot * a.P + ho * a.Wo + wo) * 32;
    }
    rowoff[tap][p] = off;
    tj += STEP;
    while (tj >= uint32_t(a.kw)) {
      tj -= uint32_t(a.kw);
      ++ti;
    }
  }
}

template <bool B8, int NB>
__device__ __forceinline__ void dx_body(const DxArgs &a, uint32_t bid, DxLds &sm) {
  bid = xcd_tile<DX_XCD_RUN>(bid, a.nblocks);
  const int t = threadIdx.x, lane = t & 63;
  const uint32_t wave = wave_id();
  const int i = lane & 31, g = lane >> 5;
  const int count = *a.count;
  // Loads that do not depend on the count issue with it: the pixel parameters and the
  // line sign sums this block needs were it a computing block (indices clamped into the
  // arrays for the zeroing blocks past the capacity tiles).
  const uint32_t mt = fdiv(bid, a.divCt);
  const uint32_t m0 = mt * 32, c0 = (bid - mt * a.ctiles) * 32;
  const int taps = int(a.taps);
  int kn = 0;
  float2 sz = make_float2(0.0f, 0.0f);
  uint32_t pslot = 0, ppix = 0;
  if (t < 32) {
    const uint32_t m = min(m0 + uint32_t(t), a.N * a.HW - 1);
    pslot = fdiv(m, a.divHW);
    ppix = m - pslot * a.HW;
    kn = a.kept[pslot];
    if (a.slot_sz) sz = a.slot_sz[pslot];
  }
  constexpr int WLT = DX_MAX_TAPS * 32 / DX_THREADS;   // sign sums per thread, at most
  int wlv[WLT];
#pragma unroll
  for (int k = 0; k < WLT; ++k) {
    const int e = t + k * DX_THREADS, p = e & 31, tap = e >> 5;
    const uint32_t ch = c0 + uint32_t(p);
    wlv[k] = (e < 32 * taps && ch < a.C) ? a.wlsum[ch * a.taps + uint32_t(tap)] : 0;
  }
  const uint32_t live_rows = uint32_t(count) * a.HW;
  const uint32_t live_blocks = ((live_rows + 31) / 32) * a.ctiles;

  if (bid >= live_blocks) {      // zero the pruned samples, a piece of one per block
    dx_zero_pool(a, bid - live_blocks, a.nblocks - live_blocks, count);
    return;
  }

  if (t < 32) {
    const bool live = m0 + uint32_t(t) < live_rows;
    if (!a.slot_sz && live) sz = make_float2(a.scale[kn], a.offset[kn]);
    sm.pix_out[t] = live ? int(uint32_t(kn) * a.CHW + ppix) : -1;
    sm.pix_s[t] = live ? sz.x : 0.0f;
    sm.pix_z[t] = live ? sz.y : 0.0f;
  }
#pragma unroll
  for (int k = 0; k < WLT; ++k) {
    const int e = t + k * DX_THREADS;
    if (e < 32 * taps) sm.wl[e >> 5][e & 31] = wlv[k];
  }
  dx_row_table<32, DX_THREADS>(a, m0, live_rows, sm.rowoff);
  __syncthreads();

  // Training: the mask of this lane's four outputs, loaded ahead of the contraction.
  const int r0 = 8 * int(wave) + 4 * g;   // channel rows r0 .. r0 + 3 of this lane
  const int off = sm.pix_out[i];
  bool pass[4] = {true, true, true, true};
  if (a.ste && off >= 0) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t cc = min(c0 + uint32_t(r0 + u), a.C - 1);
      pass[u] = ste_pass(a, size_t(off) + size_t(cc) * a.HW);
    }
  }

  // This lane: A row = channel c0 + i, B column = pixel m0 + i.
  const uint32_t ch = c0 + i;
  const uint32_t abase = ch < a.C ? ch * 32 + 16 * g : BUF_NONE;
  const __amdgpu_buffer_rsrc_t ars = buffer_of(a.wsb, a.wsb_bytes);
  const __amdgpu_buffer_rsrc_t brs = buffer_of(a.codes, a.codes_bytes);
  const uint32_t steps = a.taps * a.nch;
  v16i acc = {0};
  for (uint32_t s0 = wave; s0 < steps; s0 += DX_WAVES * NB) {
    // All NB steps' loads issue before the first product (one memory latency per batch);
    // a step past the end reads zeros through its A operand and adds nothing.
    v4i A[NB], B[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const uint32_t st0 = s0 + u * DX_WAVES;
      const bool live = st0 < steps;
      const uint32_t st = live ? st0 : 0;
      const uint32_t tap = fdiv(st, a.divNch);
      const uint32_t kc = st - tap * a.nch;
      A[u] = load16(ars, live ? abase : BUF_NONE, (kc * a.taps + tap) * a.C * 32);
      B[u] = load16(brs, sm.rowoff[tap][i] + 16 * g, kc * a.R * 32);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < NB; ++u) acc = mfma_i8(A[u], B8 ? bias128(B[u]) : B[u], acc);
  }

#pragma unroll
  for (int v = 0; v < 16; ++v) sm.red[wave][v][lane] = acc[v];
  __syncthreads();
  if (off < 0) return;                    // rows past the count belong to the zero blocks
  const float S = sm.pix_s[i], Z = sm.pix_z[i];
  int I[4], c[4] = {0, 0, 0, 0}, lt[4] = {0, 0, 0, 0};
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int v = 4 * int(wave) + u;
    I[u] = sm.red[0][v][lane] + sm.red[1][v][lane] + sm.red[2][v][lane] + sm.red[3][v][lane];
  }
  for (int tap = 0; tap < taps; ++tap) {
    const bool reach = sm.rowoff[tap][i] != BUF_NONE;
    const int4 w4 = *reinterpret_cast<const int4 *>(&sm.wl[tap][r0]);
    c[0] += reach ? w4.x : 0; c[1] += reach ? w4.y : 0;
    c[2] += reach ? w4.z : 0; c[3] += reach ? w4.w : 0;
    if (B8) { lt[0] += w4.x; lt[1] += w4.y; lt[2] += w4.z; lt[3] += w4.w; }
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const uint32_t cc = c0 + uint32_t(r0 + u);
    if (cc >= a.C) continue;
    const int Iu = I[u] + (B8 ? 128 * lt[u] : 0);
    const float out = pass[u] ? rescale(S, Iu, Z, float(c[u])) : 0.0f;
    const size_t o = size_t(off) + size_t(cc) * a.HW;
    if (a.dx_t == FQT_BF16) static_cast<uint16_t *>(a.dX)[o] = f32_to_bf16(out);
    else static_cast<float *>(a.dX)[o] = out;
    if (a.I_out) a.I_out[o] = Iu;
  }
}

// Large layers: register tiles.  A wave holds DXT_RT pixel tiles x CT channel tiles of 32 x 32 and
// runs their whole contraction (no split over the waves, no reduction), so each loaded sign
// fragment feeds DXT_RT MFMAs and each code fragment CT of them; a block's four waves take
// consecutive pixels of the same channels.  Steps run over the taps of a 32-byte chunk before
// the next chunk, so that the taps' rows of codes come from the L1.  A wave tabulates its pixels'
// code rows in LDS, tap by tap, a lane per pixel (found in the loop from the pixel, with
// divisions under a stride, they took the VALU longer than the products take the matrix cores:
// 512 -> 512 on 28 x 28, b = 2: 67 us of the launch against 54; 4 -> 223, 3 x 3 / 2 on 147 x 147,
// b = 3: 80 against 50).  Batches of DXT_NB steps are double-buffered.
//   FP4: codes and signs as e2m1 nibbles (b <= 2; half the bytes and half the steps), sums in
//        float32, exact below 2^24.
//   LIN: one pixel per sample and one tap, no padding (every sample is reached): codes feed the
//        MFMA's rows, so that output lanes run along the channels, as dX does.
constexpr int DXT_RT = 2;                            // pixel tiles per wave
constexpr int DXT_NB = 2;                            // contraction steps per load batch
constexpr uint32_t DXT_BP = DX_WAVES * DXT_RT * 32;  // pixel rows per block
constexpr int DXT_PITCH = 32 * DXT_RT + 4;           // staged floats per channel
struct alignas(16) DxTileLds {
  uint32_t lds[DX_WAVES][32 * DXT_PITCH];            // code rows [tap][pixel], then the output tile
  int32_t pix_out[DXT_BP];                           // offset of each pixel in dX, -1 past the live rows
  float2 pix_sz[DXT_BP];                             // its sample's scale and offset
  uint64_t reach[DXT_BP];                            // the taps that meet an output pixel
};
constexpr int DXT_TAPS = 32;                         // taps tabulated at once
static_assert(DXT_TAPS * 32 * DXT_RT <= 32 * DXT_PITCH && 32 * DXT_RT == 64, "code rows in the tile's place");

// Stores of one wave's 32 channels x 64 pixels from their LDS copy [channel][pixel]: pieces of
// 4 pixels of one channel (HW % 4 == 0: of one sample), consecutive lanes on consecutive
// pixels.
__device__ __forceinline__ void dx_store_tile(const DxArgs &a, const int32_t *pix, const uint32_t *st,
                                              uint32_t c0, int lane) {
  constexpr int PIECES = 4 * DXT_RT, QROW = 8 * DXT_RT;   // pieces per lane, per channel row
  const int off = pix[4 * (lane % QROW)];
  if (off < 0) return;
  auto put = [&](auto store) {
#pragma unroll
    for (int k = 0; k < PIECES; ++k) {
      const uint32_t row = uint32_t(lane / QROW + (64 / QROW) * k);
      if (c0 + row >= a.C) continue;
      const size_t o = size_t(off) + size_t(c0 + row) * a.HW;
      const uint4 q = *reinterpret_cast<const uint4 *>(st + row * DXT_PITCH + 4 * (lane % QROW));
      float4 f = make_float4(__uint_as_float(q.x), __uint_as_float(q.y), __uint_as_float(q.z),
                             __uint_as_float(q.w));
      if (a.ste) {
        const float4 x = *reinterpret_cast<const float4 *>(a.ste + o);
        f.x = __builtin_fabsf(x.x) <= 1.0f ? f.x : 0.0f;
        f.y = __builtin_fabsf(x.y) <= 1.0f ? f.y : 0.0f;
        f.z = __builtin_fabsf(x.z) <= 1.0f ? f.z : 0.0f;
        f.w = __builtin_fabsf(x.w) <= 1.0f ? f.w : 0.0f;
      }
      if (a.dx_t == FQT_BF16)
        store(reinterpret_cast<u32x2 *>(static_cast<uint16_t *>(a.dX) + o),
              u32x2{f32_to_bf16(f.x) | (uint32_t(f32_to_bf16(f.y)) << 16),
                    f32_to_bf16(f.z) | (uint32_t(f32_to_bf16(f.w)) << 16)});
      else
        store(reinterpret_cast<u32x4 *>(static_cast<float *>(a.dX) + o),
              u32x4{__float_as_uint(f.x), __float_as_uint(f.y), __float_as_uint(f.z),
                    __float_as_uint(f.w)});
    }
  };
  if (a.stream)
    put([](auto *p, auto v) { stream_fence(); __builtin_nontemporal_store(v, p); stream_fence(); });
  else put([](auto *p, auto v) { *p = v; });
}

// A pixel's or a tap's remainders under the strides as one word: a tap's are below DX_MAX_TAPS (as
// are kh and kw), so a pixel's may be clamped to it.
__device__ __forceinline__ uint32_t tap_rem(uint32_t h, uint32_t w) { return h << 16 | w; }

template <bool FP4, bool B8, int CT, bool LIN>
__device__ __forceinline__ void dx_body_tiles(const DxArgs &a, uint32_t bid, DxTileLds &sm) {
  using Acc = std::conditional_t<FP4, v16f, v16i>;
  bid = xcd_tile<DXW_XCD_RUN>(bid, a.nblocks);
  const int t = threadIdx.x, lane = t & 63;
  const uint32_t wave = wave_id();
  const int i = lane & 31, g = lane >> 5;
  const int count = *a.count;
  const uint32_t mt = fdiv(bid, a.divCb);
  const uint32_t m0 = mt * DXT_BP + wave * (32 * DXT_RT), c0 = (bid - mt * a.cblocks) * (CT * 32);
  const uint32_t live_rows = uint32_t(count) * a.HW;
  const uint32_t live_blocks = ((live_rows + DXT_BP - 1) / DXT_BP) * a.cblocks;
  if (bid >= live_blocks) {
    dx_zero_pool(a, bid - live_blocks, a.nblocks - live_blocks, count);
    return;
  }
  if (m0 >= live_rows) return;                   // (no barrier below: each wave has its own LDS)
  int32_t *pix = sm.pix_out + wave * (32 * DXT_RT);
  float2 *psz = sm.pix_sz + wave * (32 * DXT_RT);
  uint64_t *reach = sm.reach + wave * (32 * DXT_RT);
  uint32_t *lds = sm.lds[wave];
  // Lane l's own pixel m0 + l: position under tap (0, 0) divided by the strides (quotients, and both
  // remainders in one word), first code row.
  const uint32_t m = m0 + uint32_t(lane), mm = min(m, live_rows - 1);
  const uint32_t slot = fdiv(mm, a.divHW), p = mm - slot * a.HW;
  const uint32_t h = fdiv(p, a.divW), w = p - h * a.W, n = uint32_t(a.kept[slot]);
  const uint32_t hq = fdiv(h + uint32_t(a.ph), a.divSh), wq = fdiv(w + uint32_t(a.pw), a.divSw);
  const uint32_t rem = tap_rem(min(h + uint32_t(a.ph) - hq * uint32_t(a.sh), uint32_t(DX_MAX_TAPS)),
                               min(w + uint32_t(a.pw) - wq * uint32_t(a.sw), uint32_t(DX_MAX_TAPS)));
  const uint32_t first = slot * a.P;
  pix[lane] = m < live_rows ? int(n * a.CHW + p) : -1;
  psz[lane] = a.slot_sz ? a.slot_sz[slot] : make_float2(a.scale[n], a.offset[n]);
  uint32_t abase[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    const uint32_t ch = c0 + uint32_t(32 * ct + i);
    abase[ct] = ch < a.C ? ch * 32 + 16 * g : BUF_NONE;
  }
  const __amdgpu_buffer_rsrc_t ars = buffer_of(a.wsb, a.wsb_bytes);
  const __amdgpu_buffer_rsrc_t brs = buffer_of(a.codes, a.codes_bytes);
  const uint32_t wstride = a.C * 32;
  Acc acc[DXT_RT][CT];
#pragma unroll
  for (int rt = 0; rt < DXT_RT; ++rt)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = Acc{0};
  // The sign sums of 16 taps of this lane's channels (an operand of the zero-point term below),
  // loaded ahead of the contraction.
  const bool few = a.taps <= 16 && a.D <= 2048;  // one f16 MFMA per tile
  auto line_sum = [&](uint32_t ch, uint32_t tap) {
    return tap < a.taps && ch < a.C ? a.wlsum[ch * a.taps + tap] : 0;
  };
  f16x8 wsum[LIN ? 1 : CT];
  if (!LIN && few) {
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int k = 0; k < 8; ++k)
        wsum[ct][k] = _Float16(float(line_sum(c0 + uint32_t(32 * ct + i), 8 * g + k)));
  }
  struct Batch {
    v4i A[DXT_NB][CT], B[DXT_NB][DXT_RT];
  };
  auto consume = [&](const Batch &q) {
#pragma unroll
    for (int u = 0; u < DXT_NB; ++u)
#pragma unroll
      for (int rt = 0; rt < DXT_RT; ++rt) {
        const v4i b = B8 ? bias128(q.B[u][rt]) : q.B[u][rt];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          const v4i x = LIN ? b : q.A[u][ct], y = LIN ? q.A[u][ct] : b;
          if constexpr (FP4)
            acc[rt][ct] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                as_v8(x), as_v8(y), acc[rt][ct], 4, 4, 0, 127, 0, 127);
          else acc[rt][ct] = mfma_i8(x, y, acc[rt][ct]);
        }
      }
    __builtin_amdgcn_sched_barrier(0);
  };
  // Taps in groups of DXT_TAPS: each lane tabulates its pixel's code rows (BUF_NONE where the tap meets
  // no output pixel, and a bit of the reach mask where it does), then the group's steps run.
  uint64_t mask = 0;
  int tj = 0;
  uint32_t tq = 0, tr = 0, uq = 0, ur = 0;       // tap (ti, tj): ti = sh tq + tr, tj = sw uq + ur
  for (uint32_t g0 = 0; g0 < a.taps; g0 += DXT_TAPS) {
    const uint32_t nt = min(a.taps - g0, uint32_t(DXT_TAPS)), steps = nt * a.nch;
    if constexpr (!LIN) {
      __builtin_amdgcn_wave_barrier();           // (LDS operations of a wave run in order)
      for (uint32_t t = 0; t < nt; ++t) {
        const uint32_t ho = hq - tq, wo = wq - uq;
        const bool ok = rem == tap_rem(tr, ur) && ho < a.Ho && wo < a.Wo;
        lds[64 * t + lane] = ok ? (first + ho * a.Wo + wo) * 32 : BUF_NONE;
        mask |= uint64_t(ok ? 1 : 0) << (g0 + t);
        ++tj;
        ++ur;
        if (ur == uint32_t(a.sw)) {
          ur = 0;
          ++uq;
        }
        if (tj == a.kw) {
          tj = 0;
          uq = ur = 0;
          ++tr;
          if (tr == uint32_t(a.sh)) {
            tr = 0;
            ++tq;
          }
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
    // The code rows of a batch of steps, read a batch ahead of their loads; (kc, t) the step's
    // chunk and tap.
    uint32_t row[DXT_NB][DXT_RT], t = 0, kc = 0, tn = 0;
    auto rows = [&]() {
#pragma unroll
      for (int u = 0; u < DXT_NB; ++u) {
#pragma unroll
        for (int rt = 0; rt < DXT_RT; ++rt) row[u][rt] = lds[64 * tn + 32 * rt + i] + 16 * g;
        ++tn;
        tn = tn == nt ? 0 : tn;
      }
    };
    if constexpr (LIN) {
#pragma unroll
      for (int rt = 0; rt < DXT_RT; ++rt)
#pragma unroll
        for (int u = 0; u < DXT_NB; ++u)
          row[u][rt] = fdiv(min(m0 + 32 * rt + uint32_t(i), live_rows - 1), a.divHW) * 32 + 16 * g;
    } else {
      rows();
    }
    // The loads of a batch of steps (a step past the end multiplies by zero signs).
    auto issue = [&](uint32_t s0, Batch &b) {
#pragma unroll
      for (int u = 0; u < DXT_NB; ++u) {
        const bool live = s0 + u < steps;
        const uint32_t kl = min(kc, a.nch - 1), ws = (kl * a.taps + g0 + t) * wstride;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) b.A[u][ct] = load16(ars, live ? abase[ct] : BUF_NONE, ws);
#pragma unroll
        for (int rt = 0; rt < DXT_RT; ++rt) b.B[u][rt] = load16(brs, row[u][rt], kl * a.R * 32);
        ++t;
        kc += t == nt ? 1 : 0;
        t = t == nt ? 0 : t;
      }
      if constexpr (!LIN) rows();
      __builtin_amdgcn_sched_barrier(0);
    };
    // Two batches in turn: one loads behind the other's products.  Nibbles: no load under a condition
    // in the loop, whose waits would cover both batches (512 -> 512 on 28 x 28, b = 2: 59 us of the
    // launch against 53); with bytes the copies behind the loop spill (64 -> 64 on 56 x 56, b = 3: 44
    // against 30).
    Batch b0, b1;
    issue(0, b0);
    if constexpr (FP4) {
      uint32_t s0 = 0;
      for (; s0 + 2 * DXT_NB < steps; s0 += 2 * DXT_NB) {
        issue(s0 + DXT_NB, b1);
        consume(b0);
        issue(s0 + 2 * DXT_NB, b0);
        consume(b1);
      }
      if (s0 + DXT_NB < steps) {
        issue(s0 + DXT_NB, b1);
        consume(b0);
        consume(b1);
      } else {
        consume(b0);
      }
    } else {
      for (uint32_t s0 = 0;;) {
        if (s0 + DXT_NB < steps) issue(s0 + DXT_NB, b1);
        consume(b0);
        s0 += DXT_NB;
        if (s0 >= steps) break;
        if (s0 + DXT_NB < steps) issue(s0 + DXT_NB, b0);
        consume(b1);
        s0 += DXT_NB;
        if (s0 >= steps) break;
      }
    }
  }

  if constexpr (LIN) {
    // Columns are channels, rows the pixels (samples): the zero-point term is the channel's
    // line sum.
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const uint32_t cc = c0 + uint32_t(32 * ct + i);
      if (cc >= a.C) continue;
      const int wl = a.wlsum[cc];
#pragma unroll
      for (int rt = 0; rt < DXT_RT; ++rt)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int row = 32 * rt + acc_row(v, g), o0 = pix[row];
          if (o0 < 0) continue;
          const size_t o = size_t(o0) + cc;
          const int I = int(acc[rt][ct][v]) + (B8 ? 128 * wl : 0);
          const float out = ste_pass(a, o) ? rescale(psz[row].x, I, psz[row].y, float(wl)) : 0.0f;
          if (a.dx_t == FQT_BF16) static_cast<uint16_t *>(a.dX)[o] = f32_to_bf16(out);
          else static_cast<float *>(a.dX)[o] = out;
          if (a.I_out) a.I_out[o] = I;
        }
    }
    return;
  }
  __builtin_amdgcn_wave_barrier();        // the tile's copy takes the place of the code rows
  reach[lane] = mask;
  __builtin_amdgcn_wave_barrier();
  uint64_t rmask[DXT_RT];
#pragma unroll
  for (int rt = 0; rt < DXT_RT; ++rt) rmask[rt] = reach[32 * rt + i];
  auto reaches = [&](int rt, uint32_t tap) { return ((rmask[rt] >> tap) & 1u) != 0; };
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    const uint32_t ch = c0 + uint32_t(32 * ct + i);
    // b = 8: the sum of the signs of channel i over the taps (half-wave g sums every second one); the
    // accumulators fetch their rows' sums from the lanes (a walk of the taps per accumulator took
    // longer than the products: 64 -> 64, 5 x 5 on 56 x 56, batch 64: 131 us of the launch against 46).
    int wtot = 0;
    if constexpr (B8) {
      for (uint32_t tap = uint32_t(g); tap < a.taps; tap += 2) wtot += line_sum(ch, tap);
      wtot += int(lane_xor<32>(uint32_t(wtot)));
    }
#pragma unroll
    for (int rt = 0; rt < DXT_RT; ++rt) {
      // Zero-point term of each output, c = sum over the taps that reach the pixel of the
      // channel's line sign sum: the product [channel][tap] x [tap][pixel] of the sign sums and
      // the 0/1 reach flags in the accumulator layout of the tile.  Exact: with D <= 2048 every
      // sign sum is a float16 integer and 16 taps go into one f16 MFMA (lane half g holds taps
      // 8 g .. 8 g + 7); else two taps per float32 MFMA.
      v16f cz = v16f{0};
      if (few) {
        f16x8 rb;
#pragma unroll
        for (int k = 0; k < 8; ++k) rb[k] = reaches(rt, 8 * g + k) ? _Float16(1.0f) : _Float16(0.0f);
        cz = __builtin_amdgcn_mfma_f32_32x32x16_f16(wsum[ct], rb, cz, 0, 0, 0);
      } else if (a.D <= 2048) {
        for (uint32_t tb = 0; tb < a.taps; tb += 16) {
          f16x8 wa, rb;
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            wa[k] = _Float16(float(line_sum(ch, tb + 8 * g + k)));
            rb[k] = tb + 8 * g + k < a.taps && reaches(rt, tb + 8 * g + k) ? _Float16(1.0f) : _Float16(0.0f);
          }
          cz = __builtin_amdgcn_mfma_f32_32x32x16_f16(wa, rb, cz, 0, 0, 0);
        }
      } else {
        for (uint32_t j = 0; 2 * j < a.taps; ++j)
          cz = __builtin_amdgcn_mfma_f32_32x32x2f32(float(line_sum(ch, 2 * j + g)),
                                                    2 * j + g < a.taps && reaches(rt, 2 * j + g) ? 1.0f : 0.0f,
                                                    cz, 0, 0, 0);
      }
      const float S = psz[32 * rt + i].x, Z = psz[32 * rt + i].y;
      const int off = pix[32 * rt + i];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = acc_row(v, g);
        const uint32_t cc = c0 + uint32_t(32 * ct + row);
        const int I = int(acc[rt][ct][v]) + (B8 ? 128 * __shfl(wtot, row) : 0);
        float out = rescale(S, I, Z, cz[v]);
        if (a.vec) {
          lds[row * DXT_PITCH + 32 * rt + i] = __float_as_uint(out);
        } else if (off >= 0 && cc < a.C) {
          const size_t o = size_t(off) + size_t(cc) * a.HW;
          out = ste_pass(a, o) ? out : 0.0f;
          if (a.dx_t == FQT_BF16) static_cast<uint16_t *>(a.dX)[o] = f32_to_bf16(out);
          else static_cast<float *>(a.dX)[o] = out;
          if (a.I_out) a.I_out[o] = I;
        }
      }
    }
    if (a.vec) {
      __builtin_amdgcn_wave_barrier();    // LDS operations of a wave run in order
      dx_store_tile(a, pix, lds, c0 + uint32_t(32 * ct), lane);
      __builtin_amdgcn_wave_barrier();    // the next tile's copy waits for these reads
    }
  }
}

// Linear layers of at most DXR_ROWS rows with large W (dx_rows_form): the product is bound by reading W, so W is
// read once, as it is (no byte copy of its signs).  A block takes 64 channels, its waves every
// DXR_WAVES-th chunk of 32 output channels d; lane (i = lane % 32, g = lane / 32) loads channels
// 2 i, 2 i + 1 of rows d = 16 g .. 16 g + 15 (256 contiguous bytes per row) and packs their
// signs to the 16 bytes it feeds as column i of two MFMA tiles (even and odd channels).  The
// codes' rows are the MFMA's rows, so that output lanes run along the channels.  Line sums of
// the signs come from v_dot4 on the same bytes.  Rows of pruned samples are zeroed.
struct DxRowsArgs {
  const void *w;                 // [D][C]
  const uint8_t *codes;          // PSQ codes [Dp/32][N][32]
  const int32_t *kept, *count;
  const float2 *slot_sz;
  void *dX;                      // [N][C]
  const float *ste;
  int dx_t;
  uint32_t N, C, D, chunks, codes_bytes;   // chunks = ceil(D / 32)
};
constexpr int DXR_WAVES = 8, DXR_THREADS = 64 * DXR_WAVES;
constexpr uint32_t DXR_ROWS = 128;

template <bool B8, int NT, int WDT>
__global__ __launch_bounds__(DXR_THREADS) void k_dx_rows(DxRowsArgs a) {
  constexpr int ES = WDT == FQT_BF16 ? 2 : 4;
  __shared__ int32_t red[DXR_WAVES][2][16][64];
  const int lane = threadIdx.x & 63, i = lane & 31, g = lane >> 5;
  const uint32_t wave = wave_id();
  const int count = *a.count;
  const uint32_t c0 = blockIdx.x * 64, c = c0 + 2 * uint32_t(i);      // (C is even)
  const __amdgpu_buffer_rsrc_t crs = buffer_of(a.codes, a.codes_bytes);
  uint32_t aoff[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const uint32_t j = 32 * t + uint32_t(i);
    aoff[t] = int(j) < count ? j * 32 + 16 * g : BUF_NONE;
  }
  const uint32_t live = (uint32_t(count) + 31) / 32;                  // row tiles in use
  v16i acc[NT][2];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t][0] = acc[t][1] = v16i{0};
  int csum[2] = {0, 0};
  constexpr bool TWO = NT <= 2;                // two register sets of loads, where they fit
  uint64_t wv[TWO ? 2 : 1][16];
  auto issue = [&](uint32_t ch, uint64_t (&v)[16]) {
    const uint32_t d = ch * 32, rows = min(32u, a.D - d);
    const __amdgpu_buffer_rsrc_t wrs =
        buffer_of(static_cast<const char *>(a.w) + size_t(d) * a.C * ES, rows * a.C * ES);
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      const uint32_t off = c < a.C && uint32_t(16 * g + m) < rows
                               ? (uint32_t(16 * g + m) * a.C + c) * ES : BUF_NONE;
      if (ES == 4) v[m] = load8(wrs, off, 0);
      else v[m] = uint64_t(__builtin_amdgcn_raw_buffer_load_b32(wrs, off, 0, 0));
    }
  };
  auto consume = [&](uint32_t ch, uint64_t (&v)[16], v4i (&A)[NT]) {
    v4i b[2];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint32_t lo = 0, hi = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint64_t w = v[4 * q + e];
        const float x = __uint_as_float(ES == 4 ? uint32_t(w) : uint32_t(w) << 16);
        const float y = __uint_as_float(ES == 4 ? uint32_t(w >> 32) : uint32_t(w) & 0xFFFF0000u);
        lo |= x > 0.0f ? 0x01u << (8 * e) : 0xFFu << (8 * e);
        hi |= y > 0.0f ? 0x01u << (8 * e) : 0xFFu << (8 * e);
      }
      b[0][q] = int(lo);
      b[1][q] = int(hi);
      csum[0] = __builtin_amdgcn_sdot4(int(lo), 0x01010101, csum[0], false);
      csum[1] = __builtin_amdgcn_sdot4(int(hi), 0x01010101, csum[1], false);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (uint32_t(t) >= live) break;
      const v4i q = B8 ? bias128(A[t]) : A[t];
      acc[t][0] = mfma_i8(q, b[0], acc[t][0]);
      acc[t][1] = mfma_i8(q, b[1], acc[t][1]);
    }
  };
  auto codes = [&](uint32_t ch, v4i (&A)[NT]) {
#pragma unroll
    for (int t = 0; t < NT; ++t) A[t] = load16(crs, aoff[t], ch * a.N * 32);
  };
  if (wave < a.chunks) {
    if constexpr (TWO) {
      // Double-buffered: chunk k + 1's loads issue before chunk k's products (past the end,
      // the last chunk again).
      const uint32_t last = wave + (a.chunks - 1 - wave) / DXR_WAVES * DXR_WAVES;
      v4i Aa[NT], Ab[NT];
      uint32_t ch = wave;
      issue(ch, wv[0]);
      codes(ch, Aa);
      for (;;) {
        issue(min(ch + DXR_WAVES, last), wv[1]);
        codes(min(ch + DXR_WAVES, last), Ab);
        __builtin_amdgcn_sched_barrier(0);
        consume(ch, wv[0], Aa);
        ch += DXR_WAVES;
        if (ch >= a.chunks) break;
        issue(min(ch + DXR_WAVES, last), wv[0]);
        codes(min(ch + DXR_WAVES, last), Aa);
        __builtin_amdgcn_sched_barrier(0);
        consume(ch, wv[1], Ab);
        ch += DXR_WAVES;
        if (ch >= a.chunks) break;
      }
    } else {
      for (uint32_t ch = wave; ch < a.chunks; ch += DXR_WAVES) {
        v4i A[NT];
        issue(ch, wv[0]);
        codes(ch, A);
        __builtin_amdgcn_sched_barrier(0);
        consume(ch, wv[0], A);
      }
    }
  }
  // Line sums over the half-waves and the waves; rows of the last chunk past D counted as -1.
  __shared__ int32_t cs[DXR_WAVES][2][32];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int v = csum[h] + int(lane_xor<32>(uint32_t(csum[h])));
    if (g == 0) cs[wave][h][i] = v;
  }
  __syncthreads();
  int call[2] = {0, 0};
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int w = 0; w < DXR_WAVES; ++w) call[h] += cs[w][h][i];
  const int pad = int(a.chunks * 32 - a.D);
  auto store2 = [&](size_t o, float x, float y) {       // channels c, c + 1 of row o / C
    if (a.ste) {
      x = __builtin_fabsf(a.ste[o]) <= 1.0f ? x : 0.0f;
      y = __builtin_fabsf(a.ste[o + 1]) <= 1.0f ? y : 0.0f;
    }
    if (a.dx_t == FQT_BF16) {
      uint16_t *d = static_cast<uint16_t *>(a.dX) + o;
      if ((reinterpret_cast<uintptr_t>(d) & 3) == 0) {
        *reinterpret_cast<uint32_t *>(d) = f32_to_bf16(x) | (uint32_t(f32_to_bf16(y)) << 16);
      } else {
        d[0] = f32_to_bf16(x);
        d[1] = f32_to_bf16(y);
      }
    } else {
      float *d = static_cast<float *>(a.dX) + o;
      if ((reinterpret_cast<uintptr_t>(d) & 7) == 0) {
        *reinterpret_cast<float2 *>(d) = make_float2(x, y);
      } else {
        d[0] = x;
        d[1] = y;
      }
    }
  };
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (uint32_t(t) >= live) break;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int v = 0; v < 16; ++v) red[wave][h][v][lane] = acc[t][h][v];
    __syncthreads();
    // Wave w finishes accumulators 2 w, 2 w + 1 of both tiles.
#pragma unroll
    for (int u = 0; u < 16 / DXR_WAVES; ++u) {
      const int v = (16 / DXR_WAVES) * int(wave) + u;
      const uint32_t j = 32 * t + uint32_t(acc_row(v, g));
      int I[2] = {0, 0};
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int w = 0; w < DXR_WAVES; ++w) I[h] += red[w][h][v][lane];
      if (int(j) < count && c < a.C) {
        const float2 sz = a.slot_sz[j];
        const float x = rescale(sz.x, I[0] + (B8 ? 128 * call[0] : 0), sz.y, float(call[0] + pad));
        const float y = rescale(sz.x, I[1] + (B8 ? 128 * call[1] : 0), sz.y, float(call[1] + pad));
        store2(size_t(a.kept[j]) * a.C + c, x, y);
      }
    }
    __syncthreads();
  }
  for (uint32_t j = uint32_t(count) + 2 * wave + uint32_t(g); j < a.N; j += 2 * DXR_WAVES)
    if (c < a.C) store2(size_t(a.kept[j]) * a.C + c, 0.0f, 0.0f);
}

// WT: a DxForm.
template <int WT>
using DxLdsOf = std::conditional_t<WT != 0, DxTileLds, DxLds>;
template <bool FP4, bool B8, int NB, int WT>
__device__ __forceinline__ void dx_form_body(const DxArgs &a, uint32_t bid, DxLdsOf<WT> &sm) {
  if constexpr (WT == DX_SPLIT) dx_body<B8, NB>(a, bid, sm);
  else dx_body_tiles<FP4, B8, WT == DX_CT1 ? 1 : 2, WT == DX_LIN>(a, bid, sm);
}

// The two-channel-tile forms are held to three waves per SIMD (two batches of loads in flight;
// at four the epilogue spills), the one-channel-tile form to four.
template <bool B8, int NB, int WT>
__global__ __launch_bounds__(DX_THREADS) __attribute__((amdgpu_waves_per_eu(WT == DX_SPLIT ? 1 : WT == DX_CT1 ? 4 : 3)))
void k_mfma_dx(DxArgs a) {
  __shared__ DxLdsOf<WT> sm;
  dx_form_body<false, B8, NB, WT>(a, blockIdx.x, sm);
}

// How the dW blocks of the products launch run: split-R partials summed by a finish pass
// (PARTS), one split writing dW itself (DIRECT), or the contraction split over a block's
// waves and reduced in LDS (KRED).
enum DwForm { DWF_PARTS = 0, DWF_DIRECT = 1, DWF_KRED = 2 };

// Training: dgamma of DG_CH channels per block, the sum of their partial sums [parts][D] (in
// float64: the partial sums are what rounds), DG_ROWS rows side by side: these blocks are the launch's
// last, and a long walk down the rows ends it late (3 -> 32 on 20 x 20, 1000 rows: layer 82 us with four
// rows side by side, 76 with sixteen; 16 -> 64 on 16 x 16, 1024 rows 87.5 and 82.4).
struct DgArgs {
  const float *part;
  float *out;
  uint32_t parts, D;
};
constexpr uint32_t DG_CH = 16, DG_ROWS = DX_THREADS / DG_CH;    // channels per block, rows side by side
__device__ __forceinline__ void dgamma_body(const DgArgs &a, uint32_t bid, double (*sm)[DG_CH]) {
  const uint32_t c = threadIdx.x % DG_CH, row = threadIdx.x / DG_CH, d = bid * DG_CH + c;
  double s = 0.0;
  if (d < a.D) {
#pragma unroll 8
    for (uint32_t p = row; p < a.parts; p += DG_ROWS) s += double(a.part[size_t(p) * a.D + d]);
  }
  sm[row][c] = s;
  __syncthreads();
  if (row || d >= a.D) return;
#pragma unroll
  for (uint32_t r = 1; r < DG_ROWS; ++r) s += sm[r][c];
  a.out[d] = float(s);
}

// Both products in one launch (the layer backward): blocks [0, nfront) are the dW blocks of the
// slot tiles that pruning is expected to keep, the next dxa.nblocks dX blocks, then the other
// dW blocks up to ndw in all (they mostly write zero rows: 1728 of them ahead of the dX blocks
// held those back, 22.0 against 16.5 us for the launch, 512 -> 512 on 7x7 maps), and those past
// them sum dgamma; all share one LDS allocation.
template <int WT>
union ProductsLds {
  DxLdsOf<WT> dx;
  DwRedLds dw;
  double dg[DG_ROWS][DG_CH];
};
// TR: a training step (the straight-through mask, dgamma's blocks); a template parameter because
// the tests alone cost small layers a microsecond (256 -> 256 on 2x2 maps, N = 128: layer 23.3 us
// with them, 22.3 without).
template <bool B8, int NB, int DWF, int WT, bool FP4, bool TR>
__global__ __launch_bounds__(DX_THREADS) __attribute__((amdgpu_waves_per_eu(WT == DX_SPLIT ? 1 : WT == DX_CT1 ? 4 : 3)))
void k_products(DxArgs dxa, DwArgs dwa, uint32_t nfront, uint32_t ndw, DgArgs dg) {
  __shared__ ProductsLds<WT> sm;
  const uint32_t b = blockIdx.x;
  if constexpr (!TR) dxa.ste = nullptr;
  if constexpr (!TR && DWF == DWF_DIRECT) {     // (never reordered)
    if (b < ndw) dw_part_body<B8, true>(dwa, b);
    else dx_form_body<FP4, B8, NB, WT>(dxa, b - ndw, sm.dx);
    return;
  }
  if (b >= nfront && b - nfront < dxa.nblocks) {
    dx_form_body<FP4, B8, NB, WT>(dxa, b - nfront, sm.dx);
    return;
  }
  const uint32_t wb = b < nfront ? b : b - dxa.nblocks;
  if (TR && wb >= ndw) dgamma_body(dg, wb - ndw, sm.dg);
  else if constexpr (DWF == DWF_KRED) dw_kred_body<B8>(dwa, wb, sm.dw);
  else dw_part_body<B8, DWF == DWF_DIRECT>(dwa, wb);
}

}  // namespace

// Splits of the dW contraction over N*Ho*Wo: enough 32x32 wave tiles of the expected
// kept channels (all of them without AGP, about D / b with it) to give about 1024 waves
// while every split keeps at least 16 words (1024 positions), and at most 256 words per
// split (about 64 in the long split form, below), within at most DW_MAX_SPLITS splits,
// 128 MB of partials and one batch of words per split.
constexpr int64_t DW_TARGET_WAVES = 1024;
constexpr int64_t DW_MIN_WORDS = 16;
constexpr int64_t DW_MAX_WORDS = 256;
constexpr int64_t DW_MAX_SPLITS = 4096;
constexpr int64_t DW_MAX_PART_BYTES = int64_t(128) << 20;
constexpr int64_t DW_SPLIT_WORDS = 64;
constexpr int64_t DW_SPLIT_MIN = 768;         // contraction words of the split form, at least
int gemm_dw_splits(const Layer &L, const fqt_quant_cfg &cfg) {
  const int64_t dkeep =
      cfg.agp_mode == FQT_AGP_OFF ? L.D : std::max<int64_t>(1, (L.D + cfg.bits - 1) / cfg.bits);
  const int64_t tiles = ((dkeep + 31) / 32) * ((L.K + 31) / 32);
  int64_t S = std::max(std::min((DW_TARGET_WAVES + tiles - 1) / tiles,
                                (L.Wr + DW_MIN_WORDS - 1) / DW_MIN_WORDS),
                       (L.Wr + DW_MAX_WORDS - 1) / DW_MAX_WORDS);
  const int64_t kp = ((L.K + 31) / 32) * 32;
  const int64_t part_cap = std::max<int64_t>(1, DW_MAX_PART_BYTES / (L.D * kp * 4));
  S = std::min(S, part_cap);
  S = std::min(S, DW_MAX_SPLITS);
  S = std::min(S, (L.Wr + DW_PREF - 1) / DW_PREF);
  // Long contractions in the split form (their own launch: at least DW_SPLIT_MIN words,
  // slices of at least 16): slices of about DW_SPLIT_WORDS words, so that each wave's chain
  // of loads is short, while the many-split finish keeps at most 4 splits per block of its
  // D x ceil(Kp / 64) blocks (its reduction over the splits is serial per thread).
  if (S > 1 && L.Wr >= DW_SPLIT_MIN && (L.Wr + S - 1) / S >= 16) {
    int64_t Sb = std::min((L.Wr + DW_SPLIT_WORDS - 1) / DW_SPLIT_WORDS,
                          4 * L.D * ((kp + 63) / 64));
    Sb = std::min(std::min(Sb, part_cap), DW_MAX_SPLITS);
    S = std::max(S, Sb);
  }
  return int(std::max<int64_t>(S, 1));
}

// Contractions of at most this many words that would need split-R partials run in the
// in-block reduction form instead (four waves of at most 64 words each).
constexpr int64_t DW_KRED_MAX_WORDS = 256;
bool dw_kred_form(const Layer &L, int64_t S) { return S > 1 && L.Wr <= DW_KRED_MAX_WORDS; }

// dW workspace: partials [S][D][Kp] and set-bit counts [S][Kp] (Kp = K rounded up to 32);
// none when one split or the in-block reduction writes dW directly.
static size_t dw_kp(const Layer &L) { return size_t((L.K + 31) / 32) * 32; }
size_t gemm_dw_ws_bytes(const Layer &L, const fqt_quant_cfg &cfg) {
  const size_t S = size_t(gemm_dw_splits(L, cfg));
  if (S == 1 || dw_kred_form(L, int64_t(S))) return 256;
  return align256(S * size_t(L.D) * dw_kp(L) * 4) + align256(S * dw_kp(L) * 4);
}

namespace {

DwArgs make_dw_args(const Layer &L, const fqt_quant_cfg &cfg, const fqt_qgrad &q,
                    const uint64_t *xsign, float *dW, int32_t *I_out, void *ws) {
  const uint32_t ktiles = uint32_t((L.K + 31) / 32);
  const uint32_t S = uint32_t(gemm_dw_splits(L, cfg));
  DwArgs a;
  a.codes = q.pcq_codes; a.kept = q.pcq_kept; a.count = q.pcq_count;
  a.scale = q.pcq_scale; a.offset = q.pcq_offset; a.slot_sz = nullptr; a.xsign = xsign;
  a.dW = dW; a.I_out = I_out;
  a.part = S > 1 ? static_cast<int32_t *>(ws) : nullptr;
  a.partT = S > 1 ? reinterpret_cast<int32_t *>(static_cast<char *>(ws) +
                                                align256(size_t(S) * L.D * dw_kp(L) * 4))
                  : nullptr;
  a.D = uint32_t(L.D); a.K = uint32_t(L.K); a.Kp = uint32_t(dw_kp(L)); a.R = uint32_t(L.R);
  a.Rp = uint32_t(L.Wr * 64); a.Wr = uint32_t(L.Wr); a.ktiles = ktiles;
  a.codes_bytes = uint32_t(L.D * L.Wr * 64);
  a.xsign_bytes = uint32_t(L.Wr * L.K * 8);
  a.kgroups = (ktiles + DW_WAVES - 1) / DW_WAVES;
  a.S = S; a.wps = uint32_t((L.Wr + S - 1) / S);
  a.wpw = uint32_t((L.Wr + DW_WAVES - 1) / DW_WAVES);
  a.divS = make_fastdiv(S); a.divKg = make_fastdiv(a.kgroups); a.divQ = make_fastdiv(uint32_t(dw_kp(L) / 4));
  a.divKt = make_fastdiv(ktiles);
  return a;
}
// Blocks of the in-block reduction form: every (slot tile, column tile) of the capacity.
uint32_t dw_kred_blocks(const Layer &L, const DwArgs &a) {
  return a.ktiles * uint32_t((L.D + 31) / 32);
}
// Split-R partial blocks over the slot capacity: S x ceil(ceil(K/32) / 4) x ceil(D/32).
uint32_t dw_part_blocks(const Layer &L, const DwArgs &a) {
  return a.S * a.kgroups * uint32_t((L.D + 31) / 32);
}

// Register tiles where the samples expected to be kept (all, or about N / b under AGP) give enough
// waves, the more the longer the contraction: with few, the chip idles through a wave's whole
// contraction, which the split form spreads over four.  Time of the launch in register tiles over
// that in the split form, by waves (1 x 1 to 7 x 7 layers, strided ones among them, b = 1, 2, 3, 4
// and 8, 100 cases): 256 waves 1.1 - 2.8; about 400 with up to 18 steps 0.8 - 0.96, with 36 and
// more 1.1 - 1.5; 512 with 9, 18 and 36 steps 0.96, 0.77, 0.9; 784 0.67 - 0.82; 1568 and more
// 0.44 - 0.94.  Where the dW blocks share the launch (fewer than DW_SPLIT_MIN words) they run at the
// register tiles' occupancy too: 400 to 512 waves 1.1 - 1.25, 784 and 894 with byte codes 1.04 and 1.1,
// with nibbles 0.77 - 0.92, 1568 0.7 - 0.94.
// Linear layers: blocks of pruned samples count too, sixteen times as many in the split form and all
// of its time at b = 8, so a wave of the capacity weighs a fifth of a live one.  Layer time in register
// tiles over that in the split form (118 layers, C = 512 .. 8192, D = 64 .. 2048), by 4 live + capacity: up to
// 2000 0.98 - 1.28, 2000 - 3000 0.96 - 1.14 (median 1.0), 3000 - 4000 0.88 - 1.01, more 0.76 - 1.03.
uint32_t dx_form(const Layer &L, const fqt_quant_cfg &cfg) {
  const int64_t live =
      cfg.agp_mode == FQT_AGP_OFF ? L.N : std::max<int64_t>(1, (L.N + cfg.bits - 1) / cfg.bits);
  const int64_t ctiles = (L.C + 31) / 32, chunk = cfg.bits <= 2 ? 64 : 32;
  const int64_t steps = int64_t(L.kh) * L.kw * ((L.D + chunk - 1) / chunk);
  const int64_t waves = (live * L.HW + 32 * DXT_RT - 1) / (32 * DXT_RT) * ((ctiles + 1) / 2);
  // (padding puts output pixels where the one tap does not reach the map, and a stride may leave
  // only such pixels: those need the reach flags of the other forms)
  const bool lin = L.HW == 1 && L.kh * L.kw == 1 && L.ph == 0 && L.pw == 0;
  const int64_t all = (L.N * L.HW + 32 * DXT_RT - 1) / (32 * DXT_RT) * ((ctiles + 1) / 2);
  const int64_t need = L.Wr < DW_SPLIT_MIN ? (cfg.bits <= 2 ? 640 : 1024)
                                           : std::min<int64_t>(640, 300 + 5 * steps);
  if (lin ? 4 * waves + all < 3000 : waves < need) return DX_SPLIT;
  return lin ? DX_LIN : ctiles > 1 ? DX_CT2 : DX_CT1;
}

DxArgs make_dx_args(const Layer &L, const fqt_quant_cfg &cfg, const fqt_qgrad &q, const int8_t *wsb,
                    const int32_t *wlsum, void *dX, int32_t *I_out) {
  DxArgs a;
  a.codes = q.psq_codes; a.kept = q.psq_kept; a.count = q.psq_count;
  a.scale = q.psq_scale; a.offset = q.psq_offset; a.slot_sz = nullptr; a.wsb = wsb;
  a.wlsum = wlsum; a.ste = nullptr;
  a.stream = size_t(L.N) * L.C * L.HW * (L.dx_t == FQT_BF16 ? 2 : 4) >= STREAM_BYTES ? 1u : 0u;
  a.dX = dX; a.I_out = I_out; a.dx_t = L.dx_t;
  a.N = uint32_t(L.N); a.C = uint32_t(L.C); a.H = uint32_t(L.H); a.W = uint32_t(L.W);
  a.HW = uint32_t(L.HW); a.Ho = uint32_t(L.Ho); a.Wo = uint32_t(L.Wo); a.P = uint32_t(L.P);
  a.R = uint32_t(L.R); a.Dp = uint32_t(L.Wd * 64);
  a.ctiles = uint32_t((L.C + 31) / 32);
  a.CHW = uint32_t(L.C * L.HW);
  a.taps = uint32_t(L.kh * L.kw);
  a.nch = uint32_t((L.D + 31) / 32);     // (a chunk past D would be all zeros)
  a.codes_bytes = uint32_t(L.R * L.Wd * 64);
  a.wsb_bytes = uint32_t(L.K * L.Wd * 64);
  a.kh = L.kh; a.kw = L.kw; a.sh = L.sh; a.sw = L.sw; a.ph = L.ph; a.pw = L.pw;
  a.divHW = make_fastdiv(uint32_t(L.HW)); a.divW = make_fastdiv(uint32_t(L.W));
  a.divKw = make_fastdiv(uint32_t(L.kw)); a.divNch = make_fastdiv(a.nch);
  a.divCt = make_fastdiv(a.ctiles);
  a.divSh = make_fastdiv(uint32_t(L.sh)); a.divSw = make_fastdiv(uint32_t(L.sw));
  // Capacity tiles plus a pool of blocks that only zero pruned samples, a piece of at most
  // DX_ZCHUNK elements each: whatever the device-side count, at least
  // min(2048, N * pieces) blocks are left for the zeroing.
  a.zpieces = uint32_t((int64_t(a.CHW) + DX_ZCHUNK - 1) / DX_ZCHUNK);
  a.D = uint32_t(L.D);
  a.wide = dx_form(L, cfg);
  const uint32_t ct = a.wide == DX_CT1 ? 1 : 2;
  a.cblocks = a.wide ? (a.ctiles + ct - 1) / ct : a.ctiles;
  const size_t es = L.dx_t == FQT_BF16 ? 2 : 4;
  a.vec = L.HW % 4 == 0 && aligned(dX, 4 * es) && !I_out ? 1u : 0u;
  a.divCb = make_fastdiv(a.cblocks);
  const int64_t rows = a.wide ? DXT_BP : 32;
  a.nblocks = uint32_t(((L.N * L.HW + rows - 1) / rows) * a.cblocks +
                       std::min<int64_t>(2048, L.N * int64_t(a.zpieces)));
  return a;
}
// Contraction steps of one dX wave, rounded to the instantiated batch depths (10 steps
// per batch still leaves four resident blocks per CU; 18 steps in one batch was measured
// slower at the 256 -> 256 conv on 8x8 maps).
int dx_batch(const DxArgs &a) {
  const uint32_t per_wave = a.wide ? a.taps * a.nch : (a.taps * a.nch + DX_WAVES - 1) / DX_WAVES;
  return per_wave <= 4 ? 4 : per_wave <= 8 ? 8 : 10;
}

// One split (contractions of at most DW_PREF words always are) and at least 1024 waves of 64 x 64:
// the 2 x 2-tile form.
bool dw_big_tiles(const Layer &L) { return ((L.D + 63) / 64) * ((L.K + 63) / 64) >= 1024; }
bool dw_big(const Layer &L, const DwArgs &a) { return a.S == 1 && dw_big_tiles(L); }

// Split-R products over long contractions (N*Ho*Wo of DW_SPLIT_MIN words and more, slices
// of 16 words and more): the partials in the big form's wave tiles, in a launch of their
// own.  Shorter ones stay in the products launch, where their partial blocks overlap the dX
// blocks.
bool dw_split_big(const Layer &L, const DwArgs &a) {
  return a.S > 1 && L.Wr >= DW_SPLIT_MIN && a.wps >= 16;
}
// Row tiles of the split form: one when the expected kept channels (D, or D / b with AGP)
// fit 32 rows.
int dw_split_rt(const Layer &L, const fqt_quant_cfg &cfg) {
  const int64_t dkeep =
      cfg.agp_mode == FQT_AGP_OFF ? L.D : (L.D + cfg.bits - 1) / std::max(cfg.bits, 1);
  return dkeep <= 32 ? 1 : 2;
}
template <bool B8>
void launch_dw_split(const DwArgs &a, int rt, hipStream_t s) {
  if (rt == 1)
    hipLaunchKernelGGL((k_mfma_dw_split<B8, 1>), dim3(dw_split_blocks(a, 1)), dim3(DW_THREADS), 0,
                       s, a);
  else
    hipLaunchKernelGGL((k_mfma_dw_split<B8, 2>), dim3(dw_split_blocks(a, 2)), dim3(DW_THREADS), 0,
                       s, a);
}

template <bool B8>
void launch_dw_big(const DwArgs &a, bool fp4, hipStream_t s) {
  auto go = [&]<bool STREAM>() {
    if (!B8 && fp4)
      hipLaunchKernelGGL(k_mfma_dw_big4<STREAM>, dim3(dw_big_blocks(a.D, a.K, 2, 4)),
                         dim3(DW_THREADS), 0, s, a);
    else if (a.Wr >= uint32_t(DWB_LONG_WORDS))
      hipLaunchKernelGGL((k_mfma_dw_big<B8, STREAM>), dim3(dw_big_blocks(a.D, a.K, 2, 4)),
                         dim3(DW_THREADS), 0, s, a);
    else
      hipLaunchKernelGGL((k_mfma_dw_short<B8, STREAM>), dim3(dw_big_blocks(a.D, a.K, 2, 2)),
                         dim3(DW_THREADS), 0, s, a);
  };
  if (size_t(a.D) * a.K * 4 >= STREAM_BYTES) go.template operator()<true>();
  else go.template operator()<false>();
}

template <bool B8>
void launch_dw_finish(const Layer &L, const DwArgs &a, hipStream_t s) {
  if (a.S > DWF_WIDE) {
    const uint32_t qblocks = uint32_t((dw_kp(L) + 63) / 64);
    hipLaunchKernelGGL(k_dw_finish_wide<B8>, dim3(unsigned(L.D) * qblocks), dim3(256), 0, s, a);
  } else {
    const dim3 fgrid(unsigned((L.D * (dw_kp(L) / 4) + 255) / 256));
    hipLaunchKernelGGL(k_dw_finish<B8>, fgrid, dim3(256), 0, s, a);
  }
}

}  // namespace

// Nibble PCQ codes for dW: codes of at most 3, the long one-split form, sums below 2^24.
bool dw_fp4_form(const Layer &L, const fqt_quant_cfg &cfg) {
  if (cfg.bits > 2 || L.Wr < DWB_LONG_WORDS || ((1 << cfg.bits) - 1) * L.R >= (int64_t(1) << 24))
    return false;
  DwArgs a;
  a.S = uint32_t(gemm_dw_splits(L, cfg));
  return dw_big(L, a);
}

// Nibble codes and signs for dX: codes of at most 3, register tiles, sums below 2^24.
bool dx_fp4_form(const Layer &L, const fqt_quant_cfg &cfg) {
  return cfg.bits <= 2 && dx_form(L, cfg) != DX_SPLIT &&
         ((1 << cfg.bits) - 1) * L.D * L.kh * L.kw < (int64_t(1) << 24);
}

// The linear layers k_dx_rows takes: few rows; dW in a launch of its own (else the packed form's dX
// shares the dW blocks' launch and packing W hides beside the selection: layer time 1.06 - 1.36 of
// the packed form's for N = 1 .. 128, C = 1024 .. 25088); enough blocks of 64 channels (float32 W,
// D = 512 .. 4096: C = 1024 1.07 - 1.15, 2048 0.96 - 1.14, 4096 0.92 - 1.02 up to 64 rows and
// 0.99 - 1.09 above, 8192 0.85 - 1.04, 16384 0.77 - 0.98); pairs of channels on 4-byte addresses,
// 32 rows of W in one buffer.
bool dx_rows_form(const Layer &L, const void *W) {
  const int64_t es = L.w_t == FQT_BF16 ? 2 : 4;
  return L.kind == FQT_LINEAR && L.N <= int64_t(DXR_ROWS) && L.C >= (L.N <= 64 ? 4096 : 8192) &&
         dw_big_tiles(L) && L.C % 2 == 0 && aligned(W, 4) && 32 * L.C * es < (int64_t(1) << 31);
}

int launch_gemm_dw(const Layer &L, const fqt_quant_cfg &cfg, const fqt_qgrad &q,
                   const uint64_t *xsign, float *dW, int32_t *I_out, void *ws, hipStream_t s) {
  const DwArgs a = make_dw_args(L, cfg, q, xsign, dW, I_out, ws);
  const dim3 grid(dw_part_blocks(L, a));
  auto go = [&]<bool B8>() {
    if (dw_big(L, a)) {
      launch_dw_big<B8>(a, false, s);
    } else if (dw_kred_form(L, a.S) && !dw_split_big(L, a)) {
      hipLaunchKernelGGL(k_mfma_dw_kred<B8>, dim3(dw_kred_blocks(L, a)), dim3(DW_THREADS), 0, s,
                         a);
    } else if (dw_split_big(L, a)) {
      launch_dw_split<B8>(a, dw_split_rt(L, cfg), s);
      launch_dw_finish<B8>(L, a, s);
    } else if (a.S == 1) {
      hipLaunchKernelGGL((k_mfma_dw_part<B8, true>), grid, dim3(DW_THREADS), 0, s, a);
    } else {
      hipLaunchKernelGGL((k_mfma_dw_part<B8, false>), grid, dim3(DW_THREADS), 0, s, a);
      launch_dw_finish<B8>(L, a, s);
    }
  };
  if (cfg.bits == 8) go.template operator()<true>();
  else go.template operator()<false>();
  return last_launch_status();
}

int launch_gemm_dx(const Layer &L, const fqt_quant_cfg &cfg, const fqt_qgrad &q,
                   const int8_t *wsb, const int32_t *wlsum, void *dX, int32_t *I_out,
                   hipStream_t s) {
  if (L.kh * L.kw > DX_MAX_TAPS) return FQT_E_SHAPE;
  const DxArgs a = make_dx_args(L, cfg, q, wsb, wlsum, dX, I_out);
  const dim3 grid(a.nblocks);
  const int nb = dx_batch(a);
  auto go = [&]<bool B8, int WT>() {
    if constexpr (WT != 0)      // the register-tile forms batch DXT_NB steps themselves
      hipLaunchKernelGGL((k_mfma_dx<B8, 4, WT>), grid, dim3(DX_THREADS), 0, s, a);
    else if (nb == 4) hipLaunchKernelGGL((k_mfma_dx<B8, 4, 0>), grid, dim3(DX_THREADS), 0, s, a);
    else if (nb == 8) hipLaunchKernelGGL((k_mfma_dx<B8, 8, 0>), grid, dim3(DX_THREADS), 0, s, a);
    else hipLaunchKernelGGL((k_mfma_dx<B8, 10, 0>), grid, dim3(DX_THREADS), 0, s, a);
  };
  auto go2 = [&]<bool B8>() {
    if (a.wide == DX_LIN) go.template operator()<B8, DX_LIN>();
    else if (a.wide == DX_CT2) go.template operator()<B8, DX_CT2>();
    else if (a.wide == DX_CT1) go.template operator()<B8, DX_CT1>();
    else go.template operator()<B8, DX_SPLIT>();
  };
  if (cfg.bits == 8) go2.template operator()<true>();
  else go2.template operator()<false>();
  return last_launch_status();
}

// Whether the dW blocks past the channels expected to be kept, which only write zeros, follow the dX
// blocks of the products launch: in the in-block reduction, where they are many beside the dX tiles
// expected to be live, the more the longer the live dW blocks' contractions run on beside them.
// Else their zeros go out first, under those contractions.  Layer time with them last over that with
// them first (194 layers, 3 x 3 and 1 x 1, b = 3, 4, 8): up to 64 words, 700 zeroing blocks and two per
// live dX tile 0.80 - 0.96 (two layers of 256 channels 1.02 and 1.07), fewer per tile 0.99 - 1.08, fewer
// blocks 0.96 - 1.10; 74 to 135 words, six per tile 0.87 - 0.98, five (also of 172 words) 1.00 - 1.02,
// fewer 0.96 - 1.21; split-R partials 0.97 - 1.21.  Beside register tiles, by live waves (50 layers):
// one and a half per wave and more 0.91 - 1.01, 1.1 - 1.4 0.94 - 1.06, fewer 0.90 - 1.08.
bool dw_zeros_last(const Layer &L, const fqt_quant_cfg &cfg, uint32_t zeroing, bool wide) {
  constexpr int64_t FEW_WORDS = 64, MIN_BLOCKS = 700;
  const int64_t live = (L.N + cfg.bits - 1) / cfg.bits, ctiles = (L.C + 31) / 32;
  if (wide)
    return 2 * int64_t(zeroing) >= 3 * ((live * L.HW + 32 * DXT_RT - 1) / (32 * DXT_RT) * ((ctiles + 1) / 2));
  const int64_t tiles = (live * L.HW + 31) / 32 * ctiles;
  return zeroing >= MIN_BLOCKS && zeroing >= (L.Wr <= FEW_WORDS ? 2 : 6) * tiles;
}

int launch_products(const Layer &L, const fqt_quant_cfg &cfg, const fqt_qgrad &q,
                    const uint64_t *xsign, const int8_t *wsb, const int32_t *wlsum, void *dX,
                    float *dW, void *dw_ws, const float2 *sslot, const float2 *cslot,
                    hipStream_t s, const TrainJob *train, const TapsPlan *taps, char *arena,
                    const void *wrows, bool fp4, bool dw4) {
  if (L.kh * L.kw > DX_MAX_TAPS || (wrows && fp4)) return FQT_E_SHAPE;
  DwArgs dwa = make_dw_args(L, cfg, q, xsign, dW, nullptr, dw_ws);
  DxArgs dxa = make_dx_args(L, cfg, q, wsb, wlsum, dX, nullptr);
  dwa.slot_sz = cslot;
  dxa.slot_sz = sslot;
  // A large one-split dW runs as its own launch in the 2 x 2-tile form; the products
  // launch then holds only dX blocks.
  // Long split-R contractions likewise run their partials as their own launch.
  if (dw4) dwa.codes_bytes /= 2;
  const bool big = taps || dw_big(L, dwa);
  const bool split_big = !big && dw_split_big(L, dwa);
  const bool kred = !big && !split_big && dw_kred_form(L, dwa.S);
  if (taps) {
    const int st = launch_dw_taps(L, cfg, *taps, q, arena, cslot, dW, s);
    if (st != FQT_OK) return st;
  } else if (big) {
    if (cfg.bits == 8) launch_dw_big<true>(dwa, false, s);
    else launch_dw_big<false>(dwa, dw4, s);
  } else if (split_big) {
    if (cfg.bits == 8) launch_dw_split<true>(dwa, dw_split_rt(L, cfg), s);
    else launch_dw_split<false>(dwa, dw_split_rt(L, cfg), s);
  }
  const uint32_t ndw = (big || split_big) ? 0u
                      : kred ? dw_kred_blocks(L, dwa) : dw_part_blocks(L, dwa);
  if (wrows) {
    DxRowsArgs r;
    r.w = wrows; r.codes = q.psq_codes; r.kept = q.psq_kept; r.count = q.psq_count;
    r.slot_sz = sslot; r.dX = dX; r.ste = train ? train->X : nullptr; r.dx_t = L.dx_t;
    r.N = uint32_t(L.N); r.C = uint32_t(L.C); r.D = uint32_t(L.D);
    r.chunks = uint32_t((L.D + 31) / 32); r.codes_bytes = dxa.codes_bytes;
    const dim3 rgrid(unsigned((L.C + 63) / 64));
    auto go = [&]<bool B8, int WDT>() {
      if (L.N <= 32) hipLaunchKernelGGL((k_dx_rows<B8, 1, WDT>), rgrid, dim3(DXR_THREADS), 0, s, r);
      else if (L.N <= 64)
        hipLaunchKernelGGL((k_dx_rows<B8, 2, WDT>), rgrid, dim3(DXR_THREADS), 0, s, r);
      else hipLaunchKernelGGL((k_dx_rows<B8, 4, WDT>), rgrid, dim3(DXR_THREADS), 0, s, r);
    };
    dispatch_dtype(L.w_t, [&]<int WDT>() {
      if (cfg.bits == 8) go.template operator()<true, WDT>();
      else go.template operator()<false, WDT>();
    });
    if (last_launch_status() != FQT_OK) return FQT_E_HIP;
    dxa.nblocks = 0;                      // the products launch holds what is left
    if (ndw == 0 && !train) return FQT_OK;
  }
  DgArgs dg{};
  if (fp4) {                              // nibble operands: half the chunks and bytes
    dxa.nch = uint32_t((L.D + 63) / 64);
    dxa.divNch = make_fastdiv(dxa.nch);
    dxa.codes_bytes /= 2;
    dxa.wsb_bytes /= 2;
  }
  if (train) {
    if (!aligned(train->X, 16)) dxa.vec = 0;
    dxa.ste = train->X;
    dg = DgArgs{train->part, train->dgamma, train->parts, uint32_t(L.D)};
  }
  // (the slot tile is the slowest index of the dW blocks)
  const uint32_t stiles = uint32_t((L.D + 31) / 32);
  const uint32_t keep = uint32_t(
      cfg.agp_mode == FQT_AGP_OFF ? stiles : ((L.D + cfg.bits - 1) / cfg.bits + 31) / 32);
  uint32_t nfront = ndw / stiles * keep;
  if (!kred || !dw_zeros_last(L, cfg, ndw - nfront, dxa.wide != DX_SPLIT)) nfront = ndw;
  const dim3 grid(ndw + dxa.nblocks + (train ? unsigned((L.D + DG_CH - 1) / DG_CH) : 0u));
  const int nb = dx_batch(dxa);
  auto go_tr = [&]<bool B8, int DWF, int WT, bool TR>() {
    if constexpr (WT != 0) {
      if constexpr (!B8)
        if (fp4) {
          hipLaunchKernelGGL((k_products<B8, 4, DWF, WT, true, TR>), grid, dim3(DX_THREADS), 0, s, dxa,
                             dwa, nfront, ndw, dg);
          if (DWF == DWF_PARTS) launch_dw_finish<B8>(L, dwa, s);
          return;
        }
      hipLaunchKernelGGL((k_products<B8, 4, DWF, WT, false, TR>), grid, dim3(DX_THREADS), 0, s, dxa,
                         dwa, nfront, ndw, dg);
    } else if (nb == 4)
      hipLaunchKernelGGL((k_products<B8, 4, DWF, 0, false, TR>), grid, dim3(DX_THREADS), 0, s, dxa, dwa,
                         nfront, ndw, dg);
    else if (nb == 8)
      hipLaunchKernelGGL((k_products<B8, 8, DWF, 0, false, TR>), grid, dim3(DX_THREADS), 0, s, dxa, dwa,
                         nfront, ndw, dg);
    else
      hipLaunchKernelGGL((k_products<B8, 10, DWF, 0, false, TR>), grid, dim3(DX_THREADS), 0, s, dxa, dwa,
                         nfront, ndw, dg);
    if (DWF == DWF_PARTS) launch_dw_finish<B8>(L, dwa, s);
  };
  auto go = [&]<bool B8, int DWF, int WT>() {
    if (train) go_tr.template operator()<B8, DWF, WT, true>();
    else go_tr.template operator()<B8, DWF, WT, false>();
  };
  auto go2 = [&]<bool B8, int DWF>() {
    if (dxa.wide == DX_LIN) go.template operator()<B8, DWF, DX_LIN>();
    else if (dxa.wide == DX_CT2) go.template operator()<B8, DWF, DX_CT2>();
    else if (dxa.wide == DX_CT1) go.template operator()<B8, DWF, DX_CT1>();
    else go.template operator()<B8, DWF, DX_SPLIT>();
  };
  auto go3 = [&]<bool B8>() {
    // With the dW product in its own launch the products launch has no dW blocks: the big
    // form (one split) needs no finish, the split_big partials do.
    if (split_big) go2.template operator()<B8, DWF_PARTS>();
    else if (big || dwa.S == 1) go2.template operator()<B8, DWF_DIRECT>();
    else if (kred) go2.template operator()<B8, DWF_KRED>();
    else go2.template operator()<B8, DWF_PARTS>();
  };
  if (cfg.bits == 8) go3.template operator()<true>();
  else go3.template operator()<false>();
  return last_launch_status();
}

}  // namespace fqt
