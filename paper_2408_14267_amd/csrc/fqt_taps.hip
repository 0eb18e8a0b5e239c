// The dW product of 3 x 3, stride-1, pad-1 convolutions over long contractions, with the nine
// taps of an input channel taken from one string of sign bits (Section 5.3, SCQ; Appendix C,
// Alg. 1 and the Unfolder):
//   I[d][c][i][j] = sum_r q[d][r] s[c][r + (i - 1) W + (j - 1)],   s = -1 off the image.
// The im2col of X's signs holds every bit nine times: at 64 -> 64 on 224 x 224 (batch 64) it
// was 231 MB written and 470 read, the largest traffic of the layer.  Here the signs are
// packed once, dword-major (dword m of channel c, positions 32 m .. 32 m + 31, at m C + c, so
// that 32 channels' dwords are one line), and a wave forms a tap's bits with one funnel
// shift, the same for all its lanes (they differ in the channel), and one AND with the
// row's and the column's mask of the image.
//
// Two operand formats of the PCQ codes, chosen so that expanding sign bits to MFMA operands
// costs the least (the VALU, not the matrix cores, bounds an expansion in position order):
//   b <= 2  e2m1 nibbles (0, 1, 2, 3 are exact), v_mfma_scale_f32_32x32x64_f8f6f4: dword j of
//           a half-wave holds positions p % 4 = j of its 32, so that +-1 is bit p moved to a
//           nibble's sign: one shift and one and-or for 8 positions.  Sums are exact in
//           float32 below 2^24.
//   b >= 3  bytes, v_mfma_i32_32x32x32_i8: byte n of dword j of half-wave g is position
//           8 n + 4 g + j, so that the 0/1 byte is one shift and one AND for 4 positions;
//           sum q s = 2 sum q b - sum q, the code sums by v_dot4.
#include <algorithm>
#include <numeric>

#include "fqt_internal.hpp"

namespace fqt {
namespace {

typedef int v3i __attribute__((ext_vector_type(3)));

struct TapsArgs {
  const uint8_t *codes;          // PCQ codes in the formats above
  const int32_t *kept, *count;
  const float2 *slot_sz;         // (scale, offset) by kept slot
  const uint32_t *plane;         // sign dwords, `halo` rows before and after the layer's
  const uint4 *masks;            // [3][per + 1]: bits of kernel row i's three taps inside the image
  float *dW;
  int32_t *part, *partT;         // [S][D][9 Cp], [S][9 Cp], column tap * Cp + c
  uint32_t C, Cp, D, R, Rp, Wr, S, wps, per, cblks, halo;
  uint32_t codes_bytes, plane_bytes, mstep;   // mstep = 2 KS mod per
  int k[3];                      // per kernel row: dword and bit of position r + (i - 1) W - 1
  uint32_t sh[3];
  FastDiv divS, divCb;
};

constexpr int KS = 4;                         // waves that share a kernel row's contraction
constexpr int TAP_WAVES = 3 * KS, TAP_THREADS = 64 * TAP_WAVES;
constexpr int SLOTS = 64;                     // kept channels per block: two MFMA row tiles

// One word (64 positions) of a wave's operands.
template <bool FP4>
struct Word {
  static constexpr int H = FP4 ? 1 : 2;       // MFMA steps per word
  v4i A[H][2];
  uint32_t d[FP4 ? 3 : 4];
  v3i m[H];                                   // masks of taps j = 0, 1, 2
};

// Grid: S slices (fastest: with S a multiple of eight each XCD keeps its slices' codes and
// signs in its own L2) x channel blocks of 32 x slot blocks of 64.  Wave (row i = wave % 3,
// share = wave / 3) takes the three taps of kernel row i over every fourth word of the slice;
// the shares of a row meet in LDS.
template <bool FP4, bool B8>
__global__ __launch_bounds__(TAP_THREADS) __attribute__((amdgpu_waves_per_eu(3, 3))) void
k_dw_taps(TapsArgs a) {
  constexpr int H = Word<FP4>::H, ST = FP4 ? 3 : 2;
  using Acc = std::conditional_t<FP4, v16f, v16i>;
  __shared__ int32_t red[TAP_WAVES][16][64];
  const int lane = threadIdx.x & 63, i32 = lane & 31, g = lane >> 5;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t share = wave / 3, row = wave - 3 * share;
  const int count = *a.count;
  const uint32_t rest = fdiv(blockIdx.x, a.divS), sl = blockIdx.x - rest * a.S;
  const uint32_t pair = fdiv(rest, a.divCb), cb = rest - pair * a.cblks;
  const uint32_t j0 = pair * SLOTS, c = cb * 32 + uint32_t(i32);
  if (int(j0) >= count) return;
  // The second row tile holds kept channels.
  const bool two = __builtin_amdgcn_readfirstlane(int(j0) + 32 < count ? 1 : 0);
  const __amdgpu_buffer_rsrc_t crs = buffer_of(a.codes, a.codes_bytes);
  const __amdgpu_buffer_rsrc_t prs = buffer_of(a.plane - size_t(a.halo) * a.C, a.plane_bytes);
  const __amdgpu_buffer_rsrc_t mrs = buffer_of(a.masks + row * (a.per + 1), (a.per + 1) * 16);
  uint32_t aoff[2];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    const uint32_t j = j0 + 32 * rt + uint32_t(i32);
    aoff[rt] = int(j) < count ? j * 32 + 16 * g : BUF_NONE;
  }
  const int k = row == 0 ? a.k[0] : row == 1 ? a.k[1] : a.k[2];
  const uint32_t sh = row == 0 ? a.sh[0] : row == 1 ? a.sh[1] : a.sh[2];
  const uint32_t poff =
      c < a.C ? (uint32_t(int(a.halo) + k + (FP4 ? g : 0)) * a.C + c) * 4 : BUF_NONE;
  const uint32_t w0 = sl * a.wps + share, w_end = min(a.Wr, (sl + 1) * a.wps);
  const uint32_t tail = a.Rp - a.R;           // positions of the last word past R

  Acc acc[2][3];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
#pragma unroll
    for (int j = 0; j < 3; ++j) acc[rt][j] = Acc{0};
  uint32_t zeros[3] = {0, 0, 0}, qsum[2] = {0, 0}, words = 0;
  uint32_t m0 = (2 * w0) % a.per;             // mask entry of the next word to be issued
  uint32_t c88 = 0x88888888u;                 // (in a vector register: an instruction takes one scalar)
  asm("" : "+v"(c88));

  auto issue = [&](uint32_t w, Word<FP4> &b) {
    const uint32_t cs = __builtin_amdgcn_readfirstlane(w * H * a.D * 32);
    const uint32_t ps = __builtin_amdgcn_readfirstlane(2 * w * a.C * 4);
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) b.A[h][rt] = load16(crs, aoff[rt], cs + h * a.D * 32);
#pragma unroll
    for (int q = 0; q < (FP4 ? 3 : 4); ++q)
      b.d[q] = __builtin_amdgcn_raw_buffer_load_b32(prs, poff, ps + q * a.C * 4, 0);
    // (the entry after the last repeats the first)
    const uint32_t ms = __builtin_amdgcn_readfirstlane(m0 * 16);
#pragma unroll
    for (int h = 0; h < H; ++h)         // (three dwords: a fourth, unused, would make its register
                                        //  free while the load is in flight, and a use wait for it)
      b.m[h] = __builtin_bit_cast(v3i, __builtin_amdgcn_raw_buffer_load_b96(mrs, FP4 ? g * 16 : 0,
                                                                           ms + 16 * h, 0));
    m0 += a.mstep;
    m0 -= m0 >= a.per ? a.per : 0;
  };
  auto consume = [&](uint32_t w, Word<FP4> &b) {
    ++words;
    uint32_t y[3];                            // bits sh .. sh + 95 of the dwords
#pragma unroll
    for (int q = 0; q < H + 1; ++q) y[q] = __builtin_amdgcn_alignbit(b.d[q + 1], b.d[q], sh);
#pragma unroll
    for (int h = 0; h < H; ++h) {
      if (w == a.Wr - 1 && tail) {            // positions past R count as clear bits
        const int keep = 64 - int(tail) - 32 * (FP4 ? g : h);
        const int km = keep >= 32 ? -1 : keep > 0 ? int((1u << keep) - 1) : 0;
        b.m[h] = v3i{b.m[h].x & km, b.m[h].y & km, b.m[h].z & km};
      }
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
        if constexpr (!FP4) {
          if (B8) {
            const int m = int(0x80808080u);
            b.A[h][rt] = v4i{b.A[h][rt].x ^ m, b.A[h][rt].y ^ m, b.A[h][rt].z ^ m, b.A[h][rt].w ^ m};
          }
#pragma unroll
          for (int q = 0; q < 4; ++q)
            qsum[rt] = B8 ? uint32_t(__builtin_amdgcn_sdot4(b.A[h][rt][q], 0x01010101, int(qsum[rt]), false))
                          : __builtin_amdgcn_udot4(uint32_t(b.A[h][rt][q]), 0x01010101u, qsum[rt], false);
        }
      }
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const uint32_t x = j == 0 ? y[h] : __builtin_amdgcn_alignbit(y[h + 1], y[h], j);
        const uint32_t n = ~(x & uint32_t(b.m[h][j]));   // set: sign -1
        zeros[j] += __popc(n);
        if constexpr (FP4) {
          // Bits 3, 7, ... of n << (3 - q) over 0x2 in every nibble: (a & b) | c.
          v4i B;
#pragma unroll
          for (int q = 0; q < 4; ++q)
            B[q] = int(__builtin_amdgcn_bitop3_b32(n << (3 - q), c88, 0x22222222u, 0xEA));
          acc[0][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as_v8(b.A[h][0]), as_v8(B),
                                                                     acc[0][j], 4, 4, 0, 127, 0, 127);
          if (two)
            acc[1][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as_v8(b.A[h][1]), as_v8(B),
                                                                       acc[1][j], 4, 4, 0, 127, 0, 127);
        } else {
          const uint32_t t = ~n >> (4 * g);
          const v4i B = v4i{int(t & 0x01010101u), int((t >> 1) & 0x01010101u),
                            int((t >> 2) & 0x01010101u), int((t >> 3) & 0x01010101u)};
          acc[0][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(b.A[h][0], B, acc[0][j], 0, 0, 0);
          if (two) acc[1][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(b.A[h][1], B, acc[1][j], 0, 0, 0);
        }
      }
    }
  };
  if (w0 < w_end) {
    // A ring of ST words, each word's loads issued ST - 1 words ahead (a word past the end
    // repeats the last one and is not used).
    Word<FP4> ring[ST];
    const uint32_t last = w0 + (w_end - 1 - w0) / KS * KS;
#pragma unroll
    for (int u = 0; u < ST; ++u) {
      issue(min(w0 + KS * u, last), ring[u]);
      __builtin_amdgcn_sched_barrier(0);        // in ring order, so that the waits count exactly
    }
    for (uint32_t w = w0; w < w_end; w += KS * ST) {
#pragma unroll
      for (int u = 0; u < ST; ++u) {
        if (w + KS * u >= w_end) break;
        consume(w + KS * u, ring[u]);
        __builtin_amdgcn_sched_barrier(0);
        issue(min(w + KS * (u + ST), last), ring[u]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // The slice's sums in the split form's convention (sum of A s, A the MFMA's code byte).
  const uint32_t KT = 9 * a.Cp;
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    if (rt == 1 && !two) break;
    int qv[16];
    if constexpr (!FP4) {
      const int qrow = int(qsum[rt] + lane_xor<32>(qsum[rt]));
#pragma unroll
      for (int v = 0; v < 16; ++v) qv[v] = __shfl(qrow, acc_row(v, g));
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        if constexpr (FP4) red[wave][v][lane] = int(acc[rt][j][v]);
        else red[wave][v][lane] = 2 * acc[rt][j][v] - qv[v];
      }
      __syncthreads();
      int32_t *out = a.part + (size_t(sl) * a.D + j0 + 32 * rt) * KT + (3 * row + j) * a.Cp + c;
#pragma unroll
      for (int u = 0; u < 16 / KS; ++u) {
        const int v = (16 / KS) * int(share) + u, r = acc_row(v, g);
        int s = 0;
#pragma unroll
        for (int q = 0; q < KS; ++q) s += red[3 * q + row][v][lane];
        if (int(j0) + 32 * rt + r < count) out[size_t(r) * KT] = s;
      }
      __syncthreads();
    }
  }
  if (pair) return;
  // Set bits of each column (FP4: the half-waves saw a half word each).
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    uint32_t z = zeros[j];
    if (FP4) z += lane_xor<32>(z);
    if (g == 0) red[wave][j][i32] = int(64 * words - z);
  }
  __syncthreads();
  if (share == 0 && g == 0)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      int s = 0;
#pragma unroll
      for (int q = 0; q < KS; ++q) s += red[3 * q + row][j][i32];
      a.partT[size_t(sl) * KT + (3 * row + j) * a.Cp + c] = s;
    }
}

// dW from the slices: a block takes one slot and 64 channels (576 outputs, contiguous in dW);
// thread (chunk, quad) sums every fourth slice of 4 channels of one tap, U slices' loads
// together; the chunks and the order of the taps meet in LDS.
constexpr int FIN_QUADS = 9 * 16, FIN_CHUNKS = 4, FIN_THREADS = FIN_QUADS * FIN_CHUNKS;
template <bool B8, uint32_t U>
__global__ __launch_bounds__(FIN_THREADS) void k_dw_taps_finish(TapsArgs a) {
  __shared__ int4 red[FIN_CHUNKS][FIN_QUADS], tred[FIN_CHUNKS][FIN_QUADS];
  __shared__ float out[64 * 9];
  const uint32_t t = threadIdx.x, chunk = t / FIN_QUADS, quad = t - chunk * FIN_QUADS;
  const uint32_t cg = (a.C + 63) / 64, slot = blockIdx.x / cg, c0 = (blockIdx.x - slot * cg) * 64;
  const uint32_t tap = quad / 16, c = 4 * (quad & 15);
  const bool live = int(slot) < *a.count;
  const uint32_t KT = 9 * a.Cp;
  const size_t d = size_t(a.kept[slot]);
  const uint32_t outs = min(64u, a.C - c0) * 9;
  float *dst = a.dW + (d * a.C + c0) * 9;
  if (!live) {
    if (t < outs) dst[t] = 0.0f;
    return;
  }
  int4 acc = make_int4(0, 0, 0, 0), T = make_int4(0, 0, 0, 0);
  if (c0 + c < a.Cp) {
    const uint32_t col = tap * a.Cp + c0 + c;
    for (uint32_t s0 = chunk; s0 < a.S; s0 += U * FIN_CHUNKS) {
      int4 v[U], tv[U];
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t s = min(s0 + u * FIN_CHUNKS, a.S - 1);
        v[u] = *reinterpret_cast<const int4 *>(a.part + (size_t(s) * a.D + slot) * KT + col);
        tv[u] = *reinterpret_cast<const int4 *>(a.partT + size_t(s) * KT + col);
      }
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const int m = s0 + u * FIN_CHUNKS < a.S ? 1 : 0;
        acc.x += m * v[u].x; acc.y += m * v[u].y; acc.z += m * v[u].z; acc.w += m * v[u].w;
        T.x += m * tv[u].x; T.y += m * tv[u].y; T.z += m * tv[u].z; T.w += m * tv[u].w;
      }
    }
  }
  red[chunk][quad] = acc;
  tred[chunk][quad] = T;
  __syncthreads();
  if (chunk == 0) {
#pragma unroll
    for (int q = 1; q < FIN_CHUNKS; ++q) {
      const int4 v = red[q][quad], tv = tred[q][quad];
      acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
      T.x += tv.x; T.y += tv.y; T.z += tv.z; T.w += tv.w;
    }
    const int I[4] = {acc.x, acc.y, acc.z, acc.w}, Tq[4] = {T.x, T.y, T.z, T.w};
    const float2 sz = a.slot_sz[slot];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int Iu = I[u] + (B8 ? 128 * (2 * Tq[u] - int(a.Rp)) : 0);
      out[(c + u) * 9 + tap] = __fadd_rn(__fmul_rn(sz.x, float(Iu)),
                                         __fmul_rn(sz.y, float(2 * Tq[u] - int(a.R))));
    }
  }
  __syncthreads();
  if (t < outs) dst[t] = out[t];
}

}  // namespace

// The layers that take this form: 3 x 3, stride 1, pad 1, maps of whole quads, at least
// TAPS_MIN_WORDS words of contraction (below, the products launch reduces the contraction in its
// blocks beside the dX blocks), both group sets in one-workgroup selections (whose launch
// packs the signs).  Slices: enough for TAPS_BLOCKS blocks of the expected kept channels, of at
// least 16 words, and no more than fit `arena` bytes.
constexpr int64_t TAPS_MIN_WORDS = 768, TAPS_BLOCKS = 256;
// Few channels leave most of a 32-channel tile empty, and their unfolded signs are small: 64 maps of
// 224 x 224 in bf16, D = 64, C = 3: 316 us by taps against 291 by the unfold, 8: 319 / 323, 16: 337 /
// 361, 24: 324 / 390; 128 maps of 56 x 56 in float32, 3: 88 / 66, 16: 83 / 79, 24: 85 / 83, 32: 87 / 91.
constexpr int64_t TAPS_MIN_C = 24;
bool taps_plan(const Layer &L, const fqt_quant_cfg &cfg, size_t arena, TapsPlan *p) {
  if (L.kind != FQT_CONV2D || L.kh != 3 || L.kw != 3 || L.sh != 1 || L.sw != 1 || L.ph != 1 ||
      L.pw != 1 || L.P % 4 || L.Wr < TAPS_MIN_WORDS || L.N > 1024 || L.D > 1024 ||
      L.C < TAPS_MIN_C)
    return false;
  const int64_t dkeep =
      cfg.agp_mode == FQT_AGP_OFF ? L.D : std::max<int64_t>(1, (L.D + cfg.bits - 1) / cfg.bits);
  const int64_t cblks = (L.C + 31) / 32;
  const int64_t blocks = cblks * ((dkeep + SLOTS - 1) / SLOTS);
  p->fmt = cfg.bits <= 2 ? PCQ_TAPS4 : PCQ_TAPS8;
  p->Cp = uint32_t(cblks * 32);
  p->per = uint32_t(L.P / std::gcd(L.P, int64_t(32)));
  p->halo = uint32_t(L.W / 32 + 4);
  const size_t row = size_t(L.C) * 4;
  p->plane_bytes = (size_t(2 * L.Wr) + 2 * p->halo) * row;
  p->mask_at = align256(p->plane_bytes);
  p->part_at = p->mask_at + align256(3 * (size_t(p->per) + 1) * 16);
  const size_t slice = (size_t(L.D) + 1) * 9 * p->Cp * 4;
  if (p->plane_bytes >= (size_t(1) << 31) || p->part_at + slice + 512 > arena) return false;
  int64_t S = std::min((TAPS_BLOCKS + blocks - 1) / blocks, L.Wr / 16);
  S = std::min<int64_t>(S, (int64_t(128) << 20) / int64_t(slice));
  S = std::min<int64_t>(S, int64_t((arena - p->part_at - 512) / slice));
  if (S > 8) S = S / 8 * 8;
  p->S = uint32_t(std::max<int64_t>(S, 1));
  p->wps = uint32_t((L.Wr + p->S - 1) / p->S);
  p->partT_at = p->part_at + align256(size_t(p->S) * L.D * 9 * p->Cp * 4);
  // Float32 sums of a slice's codes (b <= 2, at most 3) are exact below 2^24.
  return p->fmt != PCQ_TAPS4 || int64_t(p->wps) * 64 * 3 < (int64_t(1) << 24);
}

int launch_dw_taps(const Layer &L, const fqt_quant_cfg &cfg, const TapsPlan &p,
                   const fqt_qgrad &q, char *arena, const float2 *slot_sz, float *dW,
                   hipStream_t s) {
  TapsArgs a;
  a.codes = q.pcq_codes; a.kept = q.pcq_kept; a.count = q.pcq_count; a.slot_sz = slot_sz;
  a.plane = reinterpret_cast<const uint32_t *>(arena) + size_t(p.halo) * L.C;
  a.masks = reinterpret_cast<const uint4 *>(arena + p.mask_at);
  a.dW = dW;
  a.part = reinterpret_cast<int32_t *>(arena + p.part_at);
  a.partT = reinterpret_cast<int32_t *>(arena + p.partT_at);
  a.C = uint32_t(L.C); a.Cp = p.Cp; a.D = uint32_t(L.D); a.R = uint32_t(L.R);
  a.Rp = uint32_t(L.Wr * 64); a.Wr = uint32_t(L.Wr); a.S = p.S; a.wps = p.wps; a.per = p.per;
  a.cblks = p.Cp / 32; a.halo = p.halo;
  a.codes_bytes = uint32_t(L.D * L.Wr * (p.fmt == PCQ_TAPS4 ? 32 : 64));
  a.plane_bytes = uint32_t(p.plane_bytes);
  for (int i = 0; i < 3; ++i) {
    const int64_t o = int64_t(i - 1) * L.W - 1;
    a.k[i] = int(o >= 0 ? o / 32 : -((-o + 31) / 32));
    a.sh[i] = uint32_t(o - int64_t(a.k[i]) * 32);
  }
  a.divS = make_fastdiv(a.S); a.divCb = make_fastdiv(a.cblks); a.mstep = 2 * KS % a.per;
  const dim3 grid(a.S * a.cblks * unsigned((L.D + SLOTS - 1) / SLOTS));
  if (p.fmt == PCQ_TAPS4)
    hipLaunchKernelGGL((k_dw_taps<true, false>), grid, dim3(TAP_THREADS), 0, s, a);
  else if (cfg.bits == 8)
    hipLaunchKernelGGL((k_dw_taps<false, true>), grid, dim3(TAP_THREADS), 0, s, a);
  else hipLaunchKernelGGL((k_dw_taps<false, false>), grid, dim3(TAP_THREADS), 0, s, a);
  if (last_launch_status() != FQT_OK) return FQT_E_HIP;
  const dim3 fgrid(unsigned(L.D) * unsigned((L.C + 63) / 64));
  auto finish = [&]<bool B8>() {
    if (p.S <= FIN_CHUNKS)
      hipLaunchKernelGGL((k_dw_taps_finish<B8, 1>), fgrid, dim3(FIN_THREADS), 0, s, a);
    else if (p.S <= 2 * FIN_CHUNKS)
      hipLaunchKernelGGL((k_dw_taps_finish<B8, 2>), fgrid, dim3(FIN_THREADS), 0, s, a);
    else hipLaunchKernelGGL((k_dw_taps_finish<B8, 8>), fgrid, dim3(FIN_THREADS), 0, s, a);
  };
  if (cfg.bits == 8) finish.template operator()<true>();
  else finish.template operator()<false>();
  return last_launch_status();
}

}  // namespace fqt
