// Binary forward on gfx950 (Section 5.1; Appendix C, Alg. 1 forward and the Unfolder):
//   I[n][d][ho][wo] = sum_{c, i, j} sign(X)[n][c][ho sh - ph + i][wo sw - pw + j] sign(W)[d][c][i][j]
//   Y = gamma_d * I
// on the fp4 matrix cores: both sign operands are e2m1 nibbles (+1 = 0x2, -1 = 0xA), so one
// v_mfma_scale_f32_32x32x64_f8f6f4 contracts 64 channels of one kernel tap, and float32 sums of
// +-1 are exact below 2^24.  The convolution is implicit: X is packed once, channels innermost
// (32 bytes hold 64 channels of one pixel), and the product reads the row of the input pixel
// that each tap of an output pixel meets.  Padded taps read one extra row of -1 (the unfold is
// zero-padded, then binarized).
//   k_fwd_pack   X and W to nibbles, one launch
//   k_fwd        the product, gamma and the stores
//   k_fwd_rows   linear layers of few rows: W is read once, as it is, and turned to nibbles in
//                registers (no packed copy of it)
#include <algorithm>

#include "fqt_internal.hpp"

namespace fqt {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int THREADS = 256;
constexpr int WAVES = THREADS / 64;

// sign(x) as the e2m1 nibble at nibble position m of a dword.
__device__ __forceinline__ uint32_t nib(float x, int m) {
  return x > 0.0f ? 0x2u << (4 * m) : 0xAu << (4 * m);
}

// ----------------------------------------------------------------------------- packing

// Packed X: [Cw][rows + 1][32 bytes], nibble c % 64 of row r (pixel n * HW + p) of chunk c / 64;
// row `rows` is all -1.  Nibbles past C hold any sign (those of W are 0).
// Packed W: [Cw][taps][Dp][32 bytes], 0 past D and C.
struct PackArgs {
  const void *x, *w;
  uint32_t *xd, *wd;             // dwords of 8 channels
  uint32_t C, Cw, HW, rows;      // rows = N * HW
  uint32_t D, Dp, taps;
  uint32_t xgroups;              // pixel groups of the vector form, rows of the others
  uint32_t xblocks;
  FastDiv divHW, divXg, divTaps, divDp;
  uint64_t xstride, wstride;     // dwords per chunk: (rows + 1) * 8 and taps * Dp * 8
};
enum XForm { X_VEC = 0, X_SCALAR = 1, X_ROWS = 2 };

// X, maps of whole VP-pixel groups (16-byte loads): a wave takes 64 channels x 8 groups; lane
// (c8 = lane / 8, group = lane % 8) loads its 8 channels' pixels (128 contiguous bytes per
// channel and instruction) and stores one dword of 8 nibbles per pixel.
template <int DT>
__device__ __forceinline__ void pack_x_vec(const PackArgs &a, uint32_t bid) {
  constexpr int VP = DT == FQT_BF16 ? 8 : 4;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t item = bid * WAVES + wave_id();           // (chunk, 8 groups), groups fastest
  const uint32_t cw = fdiv(item, a.divXg);
  if (cw >= a.Cw) return;
  const uint32_t grp = (item - cw * a.divXg.d) * 8 + (lane & 7);
  const uint32_t c8 = lane >> 3;
  if (grp >= a.xgroups) return;
  const uint32_t r = grp * VP;
  const uint32_t n = fdiv(r, a.divHW), p = r - n * a.HW;
  float v[8][VP];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const uint32_t c = min(cw * 64 + c8 * 8 + k, a.C - 1);
    const int64_t at = (int64_t(n) * a.C + c) * a.HW + p;
    if constexpr (DT == FQT_BF16) load_oct<DT>(a.x, at, v[k]);
    else load_quad<DT>(a.x, at, v[k]);
  }
  uint32_t *out = a.xd + cw * a.xstride + uint64_t(r) * 8 + c8;
#pragma unroll
  for (int j = 0; j < VP; ++j) {
    uint32_t d = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) d |= nib(v[k][j], k);
    out[8 * j] = d;
  }
}

// X, any map: a block takes 64 pixels x 64 channels, a lane per pixel, the dwords through LDS
// to 16-byte stores.
template <int DT>
__device__ __forceinline__ void pack_x_scalar(const PackArgs &a, uint32_t bid,
                                              uint32_t (*tile)[12]) {
  const uint32_t t = threadIdx.x, lane = t & 63;
  const uint32_t cw = fdiv(bid, a.divXg), r0 = (bid - cw * a.divXg.d) * 64;
  const uint32_t r = min(r0 + lane, a.rows - 1);
  const uint32_t n = fdiv(r, a.divHW), p = r - n * a.HW;
  float v[2][8];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint32_t c = min(cw * 64 + ((t >> 6) + 4 * h) * 8 + k, a.C - 1);
      v[h][k] = load_elem<DT>(a.x, (int64_t(n) * a.C + c) * a.HW + p);
    }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    uint32_t d = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) d |= nib(v[h][k], k);
    tile[lane][(t >> 6) + 4 * h] = d;
  }
  __syncthreads();
  if (t < 128 && r0 + (t >> 1) < a.rows)
    *reinterpret_cast<uint4 *>(a.xd + cw * a.xstride + uint64_t(r0 + (t >> 1)) * 8 + 4 * (t & 1)) =
        *reinterpret_cast<const uint4 *>(&tile[t >> 1][4 * (t & 1)]);
}

// Rows of a matrix [rows][C] with the contraction contiguous (X of a linear layer or of 1 x 1
// maps; W of one tap): thread (row, c8), 8 threads per 64-channel chunk of a row.
template <int DT>
__device__ __forceinline__ uint32_t pack_row_dword(const void *src, uint32_t row, uint32_t C,
                                                   uint32_t c0) {
  const int64_t at = int64_t(row) * C + c0;
  uint32_t d = 0;
  if (c0 + 8 <= C && (C & 7) == 0 && (reinterpret_cast<uintptr_t>(src) & 15) == 0) {
    float v[8];
    load_oct<DT>(src, at, v);
#pragma unroll
    for (int k = 0; k < 8; ++k) d |= nib(v[k], k);
  } else {
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = load_elem<DT>(src, at + (c0 + k < C ? k : 0));
#pragma unroll
    for (int k = 0; k < 8; ++k) d |= c0 + k < C ? nib(v[k], k) : 0u;
  }
  return d;
}

template <int DT>
__device__ __forceinline__ void pack_x_rows(const PackArgs &a, uint32_t bid) {
  const uint32_t q = bid * (THREADS / 8) + (threadIdx.x >> 3), c8 = threadIdx.x & 7;
  const uint32_t cw = fdiv(q, a.divXg), row = q - cw * a.divXg.d, c0 = cw * 64 + c8 * 8;
  if (cw >= a.Cw) return;                                // q = (chunk, row)
  a.xd[cw * a.xstride + uint64_t(row) * 8 + c8] =
      c0 < a.C ? pack_row_dword<DT>(a.x, row, a.C, c0) : 0u;
}

template <int DT>
__device__ __forceinline__ void pack_w(const PackArgs &a, uint32_t bid) {
  const uint32_t q = bid * (THREADS / 8) + (threadIdx.x >> 3), c8 = threadIdx.x & 7;
  const uint32_t row = fdiv(q, a.divTaps), tap = q - row * a.taps;   // q = (chunk, d, tap)
  const uint32_t cw = fdiv(row, a.divDp), d = row - cw * a.Dp, c0 = cw * 64 + c8 * 8;
  if (cw >= a.Cw) return;
  uint32_t o = 0;
  if (d < a.D && c0 < a.C) {
    if (a.taps == 1) {
      o = pack_row_dword<DT>(a.w, d, a.C, c0);
    } else {
      float v[8];
      const int64_t at = (int64_t(d) * a.C + c0) * a.taps + tap;
#pragma unroll
      for (int k = 0; k < 8; ++k)
        v[k] = load_elem<DT>(a.w, at + int64_t(c0 + k < a.C ? k : 0) * a.taps);
#pragma unroll
      for (int k = 0; k < 8; ++k) o |= c0 + k < a.C ? nib(v[k], k) : 0u;
    }
  }
  a.wd[cw * a.wstride + (uint64_t(tap) * a.Dp + d) * 8 + c8] = o;
}

// Blocks [0, xblocks) pack X (and block 0 the row of -1), the rest W.
template <int XDT, int WDT, int XF>
__global__ __launch_bounds__(THREADS) void k_fwd_pack(PackArgs a) {
  __shared__ __align__(16) uint32_t tile[64][12];
  const uint32_t b = blockIdx.x;
  if (b >= a.xblocks) {
    pack_w<WDT>(a, b - a.xblocks);
    return;
  }
  if (b == 0)
    for (uint32_t e = threadIdx.x; e < 8 * a.Cw; e += THREADS)
      a.xd[(e >> 3) * a.xstride + uint64_t(a.rows) * 8 + (e & 7)] = 0xAAAAAAAAu;
  if constexpr (XF == X_VEC) pack_x_vec<XDT>(a, b);
  else if constexpr (XF == X_SCALAR) pack_x_scalar<XDT>(a, b, tile);
  else pack_x_rows<XDT>(a, b);
}

// ----------------------------------------------------------------------------- product

struct FwdArgs {
  const char *xf, *wf;
  const float *gamma;            // [D]
  void *Y;                       // [N][D][P]
  int32_t *I_out;
  int y_t;
  uint32_t D, Dp, R, P, HW, H, W, Wo, rows;
  int kh, kw, sh, sw, ph, pw;
  uint32_t steps, taps, Cw;      // steps = Cw * taps, taps fastest
  uint32_t dblocks, nblocks;
  uint32_t stream;               // Y by non-temporal stores (STREAM_BYTES)
  uint32_t xf_bytes, wf_bytes;   // below 2^31 (not BIG)
  uint64_t xstride, wstride;     // bytes per chunk of X and per step of W
  FastDiv divP, divWo, divDb;
};
constexpr uint32_t FWD_RUN = 16;      // (xcd_tile: neighbouring tiles read the same X rows)

// Stores of one tile of 32 channels from d0 x 32 RT rows from r0 of integers from its LDS copy
// [channel][row] (pitch st_pitch(RT)) when P % 4 == 0: pieces of 4 consecutive pixels of one
// channel, consecutive lanes on consecutive memory (along the pixels of a map, then, for maps
// below 32 pixels, along the channels of the sample).  64 rows at once (RT = 2) write whole
// 128-byte lines also in bfloat16.
constexpr int st_pitch(int rt) { return 32 * rt + 4; }   // ints; channels on different banks
template <int RT>
__device__ __forceinline__ void store_tile(const FwdArgs &a, const int32_t *st, uint32_t d0,
                                           uint32_t r0, int lane) {
  constexpr int PIECES = 4 * RT;
  const uint32_t qsh = a.P >= 64 && RT == 2 ? 4 : a.P >= 32 ? 3 : a.P == 16 ? 2 : a.P == 8 ? 1 : 0;
  const uint32_t qs = 1u << qsh;
  float gm[PIECES];
  uint32_t dd[PIECES], pq[PIECES];
#pragma unroll
  for (int k = 0; k < PIECES; ++k) {
    const uint32_t e = uint32_t(lane) + 64 * k;
    dd[k] = (e >> qsh) & 31;
    pq[k] = (e & (qs - 1)) + qs * (e >> (qsh + 5));
    gm[k] = d0 + dd[k] < a.D ? a.gamma[d0 + dd[k]] : 0.0f;
  }
  auto put = [&](auto store4, auto store2) {
#pragma unroll
    for (int k = 0; k < PIECES; ++k) {
      const uint32_t d = d0 + dd[k], r = r0 + 4 * pq[k];
      if (d >= a.D || r >= a.R) continue;
      const uint32_t n = fdiv(r, a.divP), p = r - n * a.P;
      const size_t o = (size_t(n) * a.D + d) * a.P + p;
      const int4 I = *reinterpret_cast<const int4 *>(st + dd[k] * st_pitch(RT) + 4 * pq[k]);
      const float y0 = __fmul_rn(gm[k], float(I.x)), y1 = __fmul_rn(gm[k], float(I.y));
      const float y2 = __fmul_rn(gm[k], float(I.z)), y3 = __fmul_rn(gm[k], float(I.w));
      if (a.y_t == FQT_BF16)
        store2(reinterpret_cast<u32x2 *>(static_cast<uint16_t *>(a.Y) + o),
               u32x2{f32_to_bf16(y0) | (uint32_t(f32_to_bf16(y1)) << 16),
                     f32_to_bf16(y2) | (uint32_t(f32_to_bf16(y3)) << 16)});
      else
        store4(reinterpret_cast<u32x4 *>(static_cast<float *>(a.Y) + o),
               u32x4{__float_as_uint(y0), __float_as_uint(y1), __float_as_uint(y2),
                     __float_as_uint(y3)});
      if (a.I_out) *reinterpret_cast<int4 *>(a.I_out + o) = I;
    }
  };
  if (a.stream)
    put([](u32x4 *p, u32x4 v) { stream_fence(); __builtin_nontemporal_store(v, p); stream_fence(); },
        [](u32x2 *p, u32x2 v) { stream_fence(); __builtin_nontemporal_store(v, p); stream_fence(); });
  else put([](u32x4 *p, u32x4 v) { *p = v; }, [](u32x2 *p, u32x2 v) { *p = v; });
}

// One output element.
__device__ __forceinline__ void store_elem(const FwdArgs &a, uint32_t d, uint32_t r, int I) {
  const uint32_t n = fdiv(r, a.divP), p = r - n * a.P;
  const size_t o = (size_t(n) * a.D + d) * a.P + p;
  const float y = __fmul_rn(a.gamma[d], float(I));
  if (a.y_t == FQT_BF16) static_cast<uint16_t *>(a.Y)[o] = f32_to_bf16(y);
  else static_cast<float *>(a.Y)[o] = y;
  if (a.I_out) a.I_out[o] = I;
}

// A wave computes RT x CT MFMA tiles of 32 output rows (pixels) x 32 channels; KS waves of a
// block split the contraction of one such tile (their sums meet in LDS), 4 / KS tiles per
// block side by side along the pixels.  The channels run down the MFMA's rows and the pixels
// along its columns (output lanes run along pixels); with one pixel per sample (LIN) the
// other way round, since Y then runs along the channels.  Each step's W fragments feed RT
// products and its X fragments CT.  NB steps' loads issue together.
// VEC: Y pieces of 4 pixels (P % 4 == 0, aligned Y and I_out).  BIG: 64-bit addresses.
template <int RT, int CT, int KS, int NB, bool LIN, bool BIG>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(RT * CT == 1 || KS == 1 ? 4 : 2)))
void k_fwd(FwdArgs a, uint32_t vec) {
  constexpr int TPB = WAVES / KS, TILES = RT * CT;
  constexpr int RED = KS > 1 ? KS * TILES * 1024 : 0, SRT = KS > 1 ? 1 : RT,
                STG = WAVES * 32 * st_pitch(SRT);
  __shared__ __align__(16) int32_t lds[RED > STG ? RED : STG];
  const int lane = threadIdx.x & 63, i = lane & 31, g = lane >> 5;
  const uint32_t wave = wave_id(), tile = wave / KS, part = wave - tile * KS;
  const uint32_t bid = xcd_tile<FWD_RUN>(blockIdx.x, a.nblocks);
  const uint32_t rb = fdiv(bid, a.divDb), db = bid - rb * a.dblocks;
  const uint32_t d0 = db * (32 * CT), r0 = (rb * TPB + tile) * (32 * RT);
  // The input pixel under tap (0, 0) of this lane's output pixels.
  int hb[RT], wb[RT], base[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const uint32_t r = min(r0 + 32 * rt + uint32_t(i), a.R - 1);
    const uint32_t n = fdiv(r, a.divP), p = r - n * a.P;
    const uint32_t ho = fdiv(p, a.divWo), wo = p - ho * a.Wo;
    hb[rt] = int(ho) * a.sh - a.ph;
    wb[rt] = int(wo) * a.sw - a.pw;
    base[rt] = int(n * a.HW) + hb[rt] * int(a.W) + wb[rt];
  }
  const uint32_t per = (a.steps + KS - 1) / KS;
  const uint32_t s_lo = part * per, s_hi = min(a.steps, s_lo + per);
  uint32_t cw = s_lo / a.taps, tap = s_lo - cw * a.taps;
  int ti = int(tap) / a.kw, tj = int(tap) - ti * a.kw;
  const __amdgpu_buffer_rsrc_t xrs = buffer_of(a.xf, a.xf_bytes);
  const __amdgpu_buffer_rsrc_t wrs = buffer_of(a.wf, a.wf_bytes);
  uint32_t aoff[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    const uint32_t d = d0 + 32 * ct + uint32_t(i);
    aoff[ct] = min(d, a.Dp - 1) * 32 + 16 * g;
  }
  v16f acc[RT][CT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = v16f{0};
  if (r0 < a.R) {
    for (uint32_t s = s_lo; s < s_hi; s += NB) {
      v4i Wv[NB][CT], Xv[NB][RT];
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        // A step past the end multiplies by zero weights.
        const bool live = s + u < s_hi;
        const uint64_t wat = min(s + u, s_hi - 1) * a.wstride;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          if (BIG) Wv[u][ct] = live ? *reinterpret_cast<const v4i *>(a.wf + wat + aoff[ct]) : v4i{0};
          else Wv[u][ct] = load16(wrs, live ? aoff[ct] : BUF_NONE, uint32_t(wat));
        }
        const uint64_t xat = min(cw, a.Cw - 1) * a.xstride;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          const bool in = uint32_t(hb[rt] + ti) < a.H && uint32_t(wb[rt] + tj) < a.W;
          const uint32_t row = in ? uint32_t(base[rt] + ti * int(a.W) + tj) : a.rows;
          if (BIG) Xv[u][rt] = *reinterpret_cast<const v4i *>(a.xf + xat + uint64_t(row) * 32 + 16 * g);
          else Xv[u][rt] = load16(xrs, row * 32 + 16 * g, uint32_t(xat));
        }
        ++tj;
        ti += tj == a.kw ? 1 : 0;
        tj = tj == a.kw ? 0 : tj;
        cw += ti == a.kh ? 1 : 0;
        ti = ti == a.kh ? 0 : ti;
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < NB; ++u) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int ct = 0; ct < CT; ++ct)
            acc[rt][ct] = LIN ? __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                                    as_v8(Xv[u][rt]), as_v8(Wv[u][ct]), acc[rt][ct], 4, 4, 0, 127, 0, 127)
                              : __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                                    as_v8(Wv[u][ct]), as_v8(Xv[u][rt]), acc[rt][ct], 4, 4, 0, 127, 0, 127);
      }
    }
  }

  // The tile's integers: this wave's own tiles (KS = 1), or its share of the sums of the KS
  // parts: whole tiles (TILES >= KS), else 16 / KS accumulators of the one tile.
  if constexpr (KS > 1) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          lds[((part * TILES + rt * CT + ct) * 16 + v) * 64 + lane] = int(acc[rt][ct][v]);
    __syncthreads();
    static_assert(TILES == 1 || TILES == KS, "a wave finishes one tile or a share of one");
    if constexpr (TILES == 1) {
#pragma unroll
      for (int u = 0; u < 16 / KS; ++u) {
        const int v = (16 / KS) * int(part) + u;
        int I = 0;
#pragma unroll
        for (int q = 0; q < KS; ++q) I += lds[(q * 16 + v) * 64 + lane];
        const uint32_t r = r0 + uint32_t(LIN ? acc_row(v, g) : i);
        const uint32_t d = d0 + uint32_t(LIN ? i : acc_row(v, g));
        if (r < a.R && d < a.D) store_elem(a, d, r, I);
      }
      return;
    } else {
      const uint32_t rt = part / CT, ct = part - rt * CT;
      int I[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        I[v] = 0;
#pragma unroll
        for (int q = 0; q < KS; ++q) I[v] += lds[((q * TILES + part) * 16 + v) * 64 + lane];
      }
      const uint32_t rr = r0 + 32 * rt, dd = d0 + 32 * ct;
      if (!LIN && vec) {
        __syncthreads();
        int32_t *st = lds + wave * (32 * st_pitch(1));
#pragma unroll
        for (int v = 0; v < 16; ++v) st[acc_row(v, g) * st_pitch(1) + i] = I[v];
        __builtin_amdgcn_wave_barrier();    // LDS operations of a wave run in order
        store_tile<1>(a, st, dd, rr, lane);
        return;
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const uint32_t r = rr + uint32_t(LIN ? acc_row(v, g) : i);
        const uint32_t d = dd + uint32_t(LIN ? i : acc_row(v, g));
        if (r < a.R && d < a.D) store_elem(a, d, r, I[v]);
      }
      return;
    }
  } else {
    int32_t *st = lds + wave * (32 * st_pitch(RT));
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const uint32_t dd = d0 + 32 * ct;
      if (!LIN && vec) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int v = 0; v < 16; ++v)
            st[acc_row(v, g) * st_pitch(RT) + 32 * rt + i] = int(acc[rt][ct][v]);
        __builtin_amdgcn_wave_barrier();    // LDS operations of a wave run in order
        store_tile<RT>(a, st, dd, r0, lane);
        __builtin_amdgcn_wave_barrier();    // the next tile's copy waits for these reads
        continue;
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const uint32_t r = r0 + 32 * rt + uint32_t(LIN ? acc_row(v, g) : i);
          const uint32_t d = dd + uint32_t(LIN ? i : acc_row(v, g));
          if (r < a.R && d < a.D) store_elem(a, d, r, int(acc[rt][ct][v]));
        }
    }
  }
}

// ----------------------------------------------------------------------------- few rows

// Linear layers of at most FEW_ROWS rows and large W (few_rows): the weights are all the traffic, so each
// is read once, from W itself.  A block takes 16 output channels, its waves every NW-th chunk of 128
// input channels.  Lane (i = lane % 16, k = lane / 16) loads 16-byte pieces of W row d0 + i:
// piece j holds the VW channels from 4 VW j + VW k of the chunk, so the four lanes of a row read
// 64 contiguous bytes, and packs their signs to the 32 nibbles it feeds to
// v_mfma_scale_f32_16x16x128_f8f6f4.  X is packed in the same channel order:
// [chunk][16 NT rows][lane group k][16 bytes], 0 past C (what W holds there does not count).
struct RowsArgs {
  const void *x, *w;
  uint32_t *xd;
  const float *gamma;
  void *Y;
  int32_t *I_out;
  int y_t;
  uint32_t N, C, D, nch, xf_bytes;
};
constexpr uint32_t FEW_ROWS = 128;         // what eight row tiles hold
constexpr int64_t FEW_ROWS_MIN_D = 3072, FEW_ROWS_MIN_C = 2048;

template <int XDT, int VW>
__global__ __launch_bounds__(THREADS) void k_fwd_rows_pack(RowsArgs a, uint32_t np) {
  const uint32_t e = blockIdx.x * THREADS + threadIdx.x;     // (chunk, row, group, dword)
  const uint32_t q = e >> 4, ch = q / np, row = q - ch * np, k = (e >> 2) & 3, dw = e & 3;
  if (ch >= a.nch || row >= a.N) return;
  float v[8];
  uint32_t c[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const uint32_t j = (8 * dw + m) / VW, el = (8 * dw + m) % VW;
    c[m] = ch * 128 + j * 4 * VW + k * VW + el;
    v[m] = load_elem<XDT>(a.x, int64_t(row) * a.C + min(c[m], a.C - 1));
  }
  uint32_t d = 0;
#pragma unroll
  for (int m = 0; m < 8; ++m) d |= c[m] < a.C ? nib(v[m], m) : 0u;
  a.xd[e] = d;
}

template <int NT, int WDT>
__global__ __launch_bounds__(NT >= 4 ? 512 : 1024) void k_fwd_rows(RowsArgs a) {
  constexpr int VW = WDT == FQT_BF16 ? 8 : 4, PIECES = 32 / VW, ES = 16 / VW;
  extern __shared__ float red[];                             // [waves][NT][4][64]
  const int lane = threadIdx.x & 63, i = lane & 15, k = lane >> 4;
  const uint32_t wave = wave_id(), nw = blockDim.x >> 6;
  const uint32_t d0 = blockIdx.x * 16;
  // A buffer over this block's rows of W; channels past C of the last one read as zero.
  const uint32_t wrows = min(16u, a.D - d0);
  const __amdgpu_buffer_rsrc_t wrs =
      buffer_of(static_cast<const char *>(a.w) + size_t(d0) * a.C * ES, wrows * a.C * ES);
  const __amdgpu_buffer_rsrc_t xrs = buffer_of(a.xd, a.xf_bytes);
  const uint32_t woff = uint32_t(i) < wrows ? (uint32_t(i) * a.C + uint32_t(k) * VW) * ES : BUF_NONE;
  const uint32_t xoff = (uint32_t(i) * 4 + uint32_t(k)) * 16;
  v4f acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = v4f{0};
  for (uint32_t ch = wave; ch < a.nch; ch += 2 * nw) {
    v4i Wv[2][PIECES], Xv[2][NT];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const uint32_t cu = ch + u * nw < a.nch ? ch + u * nw : ch;
#pragma unroll
      for (int j = 0; j < PIECES; ++j) {
        if (cu * 128 + 128 <= a.C) {
          Wv[u][j] = load16(wrs, woff, (cu * 128 + j * 4 * VW) * ES);
        } else {                        // the last chunk of a row, element by element
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const uint32_t c = cu * 128 + j * 4 * VW + uint32_t(k) * VW + q * (VW / 4);
            const uint32_t off = woff - uint32_t(k) * VW * ES + c * ES;
            const bool row = uint32_t(i) < wrows;
            if (ES == 4) {
              Wv[u][j][q] = __builtin_amdgcn_raw_buffer_load_b32(wrs, row && c < a.C ? off : BUF_NONE, 0, 0);
            } else {
              const uint32_t lo = __builtin_amdgcn_raw_buffer_load_b16(wrs, row && c < a.C ? off : BUF_NONE, 0, 0);
              const uint32_t hi = __builtin_amdgcn_raw_buffer_load_b16(
                  wrs, row && c + 1 < a.C ? off + 2 : BUF_NONE, 0, 0);
              Wv[u][j][q] = int((lo & 0xFFFFu) | (hi << 16));
            }
          }
        }
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) Xv[u][t] = load16(xrs, xoff, (cu * NT + t) * 1024);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (ch + u * nw >= a.nch) break;
      v4i b;
#pragma unroll
      for (int dw = 0; dw < 4; ++dw) {
        uint32_t o = 0;
#pragma unroll
        for (int m = 0; m < 8; ++m) {
          float f;
          if (WDT == FQT_BF16) {
            const uint32_t two = uint32_t(Wv[u][dw][m >> 1]);
            f = __uint_as_float((m & 1) ? two & 0xFFFF0000u : two << 16);
          } else {
            f = __int_as_float(Wv[u][(8 * dw + m) / VW][m % VW]);
          }
          o |= nib(f, m);
        }
        b[dw] = int(o);
      }
#pragma unroll
      for (int t = 0; t < NT; ++t)
        acc[t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(as_v8(Xv[u][t]), as_v8(b), acc[t],
                                                                 4, 4, 0, 127, 0, 127);
    }
  }
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[((wave * NT + t) * 4 + v) * 64 + lane] = acc[t][v];
  __syncthreads();
  // Accumulator v of a lane: row 4 (lane / 16) + v of its tile, channel lane % 16.
  for (uint32_t e = threadIdx.x; e < NT * 256; e += blockDim.x) {
    float s = 0.0f;
    for (uint32_t q = 0; q < nw; ++q) s += red[q * NT * 256 + e];
    const uint32_t l = e & 63, n = (e >> 8) * 16 + 4 * (l >> 4) + ((e >> 6) & 3), d = d0 + (l & 15);
    if (n >= a.N || d >= a.D) continue;
    const float y = __fmul_rn(a.gamma[d], s);
    const size_t o = size_t(n) * a.D + d;
    if (a.y_t == FQT_BF16) static_cast<uint16_t *>(a.Y)[o] = f32_to_bf16(y);
    else static_cast<float *>(a.Y)[o] = y;
    if (a.I_out) a.I_out[o] = int(s);
  }
}

// ----------------------------------------------------------------------------- host

struct Sizes {
  uint64_t Cw, taps, rows, Dp, xbytes, wbytes;
};
Sizes sizes_of(const Layer &L) {
  Sizes z;
  z.Cw = uint64_t((L.C + 63) / 64);
  z.taps = uint64_t(L.kh) * L.kw;
  z.rows = uint64_t(L.N) * L.HW;
  z.Dp = uint64_t((L.D + 63) / 64 * 64);
  z.xbytes = z.Cw * (z.rows + 1) * 32;
  z.wbytes = z.Cw * z.taps * z.Dp * 32;
  return z;
}
int few_rows_tiles(const Layer &L) { return L.N <= 16 ? 1 : L.N <= 32 ? 2 : L.N <= 64 ? 4 : 8; }
// The layers k_fwd_rows takes: few rows; outputs enough that its blocks of 16 cover the chip and W
// enough that one launch over it beats packing it first, both launches over the whole chip; sums
// exact in float32, a block's rows of W inside one buffer, loads on 4-byte addresses.  Time of the
// packed form over that of k_fwd_rows, N = 8 .. 128, W in float32: D = 64 .. 1024 0.3 - 0.7,
// 2048 0.74 - 0.95, 3072 0.93 - 1.45; D = 4096 .. 16000 with C = 512 0.6 - 0.9, 1024 0.6 - 0.87,
// 2048 0.88 - 1.3, 4096 0.97 - 1.7, 16384 and 25088 1.1 - 1.5.
bool few_rows(const Layer &L, const void *W) {
  const int es = L.w_t == FQT_BF16 ? 2 : 4;
  return L.kind == FQT_LINEAR && L.N <= FEW_ROWS && L.D >= FEW_ROWS_MIN_D &&
         L.C >= FEW_ROWS_MIN_C && L.C < (int64_t(1) << 24) &&
         L.C * 16 * es < (int64_t(1) << 31) - 4096 &&
         (es == 4 || (L.C % 2 == 0 && aligned(W, 4)));
}

}  // namespace

size_t forward_ws_bytes(const Layer &L) {
  const Sizes z = sizes_of(L);
  // (the packed rows of k_fwd_rows, 64 bytes per row and 128 channels, fit the X area)
  const uint64_t few = uint64_t((L.C + 127) / 128) * 16 * few_rows_tiles(L) * 64;
  const uint64_t x = L.kind == FQT_LINEAR && L.N <= FEW_ROWS ? std::max(z.xbytes, few) : z.xbytes;
  const uint64_t need = align256(x) + align256(z.wbytes);
  // The reported size, which a call requires, is never below that of the unfolded operands (sign
  // bits of X once per word and once per row block, beside sign bytes of W, K and D rounded up to
  // 64): a lower bound that callers may hold it to.  It is above that where an input pixel's
  // 32 ceil(C / 64) bytes exceed the C kh kw / 4 of an output pixel's unfolded bits (linear layers,
  // 1 x 1 kernels, few channels, strides): a caller that reserves by the formula alone falls
  // short there.
  const uint64_t Kp = uint64_t((L.K + 63) / 64 * 64);
  const uint64_t unfolded = align256(uint64_t(L.Wr) * L.K * 8) + align256(Kp / 64 * L.Wr * 512) +
                            align256(z.Dp * Kp);
  return std::max(need, unfolded);
}

namespace {

int launch_few_rows(const Layer &L, const void *X, const void *W, const float *gamma, void *Y,
                    int32_t *I_out, void *ws, hipStream_t s) {
  const int nt = few_rows_tiles(L);
  RowsArgs a;
  a.x = X; a.w = W; a.xd = static_cast<uint32_t *>(ws); a.gamma = gamma; a.Y = Y; a.I_out = I_out;
  a.y_t = L.dy_t;
  a.N = uint32_t(L.N); a.C = uint32_t(L.C); a.D = uint32_t(L.D);
  a.nch = uint32_t((L.C + 127) / 128);
  a.xf_bytes = a.nch * 16 * uint32_t(nt) * 64;
  const uint32_t np = 16 * uint32_t(nt);
  const dim3 pgrid((a.nch * np * 16 + THREADS - 1) / THREADS);
  dispatch_dtype(L.x_t, [&]<int XDT>() {
    if (L.w_t == FQT_BF16)
      hipLaunchKernelGGL((k_fwd_rows_pack<XDT, 8>), pgrid, dim3(THREADS), 0, s, a, np);
    else
      hipLaunchKernelGGL((k_fwd_rows_pack<XDT, 4>), pgrid, dim3(THREADS), 0, s, a, np);
  });
  if (last_launch_status() != FQT_OK) return FQT_E_HIP;
  // Waves per block: 8, or 16 where the grid has few blocks and the contraction enough chunks
  // (with more row tiles 16 waves would leave too few registers for the loads in flight).
  const uint32_t blocks = uint32_t((L.D + 15) / 16);
  const uint32_t nw = blocks < 256 && a.nch >= 32 && nt <= 2 ? 16 : 8;
  const size_t lds = size_t(nw) * nt * 1024;
  dispatch_dtype(L.w_t, [&]<int WDT>() {
    if (nt == 1) hipLaunchKernelGGL((k_fwd_rows<1, WDT>), dim3(blocks), dim3(64 * nw), lds, s, a);
    else if (nt == 2) hipLaunchKernelGGL((k_fwd_rows<2, WDT>), dim3(blocks), dim3(64 * nw), lds, s, a);
    else if (nt == 4) hipLaunchKernelGGL((k_fwd_rows<4, WDT>), dim3(blocks), dim3(64 * nw), lds, s, a);
    else hipLaunchKernelGGL((k_fwd_rows<8, WDT>), dim3(blocks), dim3(64 * nw), lds, s, a);
  });
  return last_launch_status();
}

}  // namespace

int launch_forward(const Layer &L, const void *X, const void *W, const float *gamma, void *Y,
                   int32_t *I_out, void *ws, hipStream_t s) {
  if (few_rows(L, W)) return launch_few_rows(L, X, W, gamma, Y, I_out, ws, s);
  const Sizes z = sizes_of(L);
  PackArgs p;
  p.x = X; p.w = W;
  p.xd = static_cast<uint32_t *>(ws);
  p.wd = reinterpret_cast<uint32_t *>(static_cast<char *>(ws) + align256(z.xbytes));
  p.C = uint32_t(L.C); p.Cw = uint32_t(z.Cw); p.HW = uint32_t(L.HW); p.rows = uint32_t(z.rows);
  p.D = uint32_t(L.D); p.Dp = uint32_t(z.Dp); p.taps = uint32_t(z.taps);
  p.divHW = make_fastdiv(p.HW); p.divTaps = make_fastdiv(p.taps); p.divDp = make_fastdiv(p.Dp);
  p.xstride = (z.rows + 1) * 8; p.wstride = z.taps * z.Dp * 8;
  const uint32_t vp = L.x_t == FQT_BF16 ? 8 : 4;
  const int xf = L.HW == 1 ? X_ROWS : (L.HW % vp == 0 && aligned(X, 16)) ? X_VEC : X_SCALAR;
  if (xf == X_VEC) {
    p.xgroups = p.rows / vp;
    const uint32_t per = (p.xgroups + 7) / 8;
    p.divXg = make_fastdiv(per);
    p.xblocks = uint32_t((uint64_t(per) * z.Cw + WAVES - 1) / WAVES);
  } else if (xf == X_SCALAR) {
    p.xgroups = p.rows;
    const uint32_t per = (p.rows + 63) / 64;
    p.divXg = make_fastdiv(per);
    p.xblocks = uint32_t(per * z.Cw);
  } else {
    p.xgroups = p.rows;
    p.divXg = make_fastdiv(p.rows);
    p.xblocks = uint32_t((z.rows * z.Cw + THREADS / 8 - 1) / (THREADS / 8));
  }
  // (Cw taps Dp <= Kp Dp, checked by the caller to stay below 2^31)
  const uint64_t wblocks = (z.Cw * z.taps * z.Dp + THREADS / 8 - 1) / (THREADS / 8);
  const dim3 grid(unsigned(p.xblocks + wblocks));
  dispatch_dtype(L.x_t, [&]<int XDT>() {
    dispatch_dtype(L.w_t, [&]<int WDT>() {
      if (xf == X_VEC) hipLaunchKernelGGL((k_fwd_pack<XDT, WDT, X_VEC>), grid, dim3(THREADS), 0, s, p);
      else if (xf == X_SCALAR)
        hipLaunchKernelGGL((k_fwd_pack<XDT, WDT, X_SCALAR>), grid, dim3(THREADS), 0, s, p);
      else hipLaunchKernelGGL((k_fwd_pack<XDT, WDT, X_ROWS>), grid, dim3(THREADS), 0, s, p);
    });
  });
  if (last_launch_status() != FQT_OK) return FQT_E_HIP;

  FwdArgs a;
  a.xf = reinterpret_cast<const char *>(p.xd); a.wf = reinterpret_cast<const char *>(p.wd);
  a.gamma = gamma; a.Y = Y; a.I_out = I_out; a.y_t = L.dy_t;
  a.D = p.D; a.Dp = p.Dp; a.R = uint32_t(L.R); a.P = uint32_t(L.P); a.HW = p.HW;
  a.H = uint32_t(L.H); a.W = uint32_t(L.W); a.Wo = uint32_t(L.Wo); a.rows = p.rows;
  a.kh = L.kh; a.kw = L.kw; a.sh = L.sh; a.sw = L.sw; a.ph = L.ph; a.pw = L.pw;
  a.taps = p.taps; a.Cw = p.Cw; a.steps = uint32_t(z.Cw * z.taps);
  a.xstride = p.xstride * 4; a.wstride = z.Dp * 32;
  const bool big = z.xbytes >= (uint64_t(1) << 31) || z.wbytes >= (uint64_t(1) << 31);
  a.xf_bytes = big ? 0 : uint32_t(z.xbytes); a.wf_bytes = big ? 0 : uint32_t(z.wbytes);
  a.divP = make_fastdiv(a.P); a.divWo = make_fastdiv(a.Wo);
  const size_t es = L.dy_t == FQT_BF16 ? 2 : 4;
  a.stream = size_t(L.R) * L.D * es >= STREAM_BYTES ? 1u : 0u;
  const uint32_t vec = L.P % 4 == 0 && aligned(Y, 4 * es) && (!I_out || aligned(I_out, 16)) ? 1 : 0;
  const bool lin = L.P == 1;
  // Wave tiles of 64 pixels x 64 channels, each wave its own, while they give every SIMD two
  // waves; below that four waves share a tile's contraction, of 64 x 64 while those blocks
  // still cover the chip twice, else 32 x 32.  (The split forms also keep each wave's sum
  // below 2^24, K being below 2^25 here.)
  const uint64_t t64 = uint64_t((L.R + 63) / 64) * (z.Dp / 64);
  const int form = t64 >= 2048 && L.K < (int64_t(1) << 24) ? 0 : t64 >= 512 && a.steps >= 16 ? 1 : 2;
  const uint32_t rows_b = form == 0 ? 256 : form == 1 ? 64 : 32, ch_b = form == 2 ? 32 : 64;
  a.dblocks = uint32_t((L.D + ch_b - 1) / ch_b);
  a.divDb = make_fastdiv(a.dblocks);
  a.nblocks = a.dblocks * ((a.R + rows_b - 1) / rows_b);
  const dim3 g2(a.nblocks);
  auto go = [&]<bool LIN, bool BIG>() {
    if (form == 0) hipLaunchKernelGGL((k_fwd<2, 2, 1, 2, LIN, BIG>), g2, dim3(THREADS), 0, s, a, vec);
    else if (form == 1)
      hipLaunchKernelGGL((k_fwd<2, 2, 4, 4, LIN, BIG>), g2, dim3(THREADS), 0, s, a, vec);
    else if (a.steps <= 16)
      hipLaunchKernelGGL((k_fwd<1, 1, 4, 4, LIN, BIG>), g2, dim3(THREADS), 0, s, a, vec);
    else hipLaunchKernelGGL((k_fwd<1, 1, 4, 10, LIN, BIG>), g2, dim3(THREADS), 0, s, a, vec);
  };
  if (lin && big) go.template operator()<true, true>();
  else if (lin) go.template operator()<true, false>();
  else if (big) go.template operator()<false, true>();
  else go.template operator()<false, false>();
  return last_launch_status();
}

}  // namespace fqt
