// Device code of the frozen-weight 3x3 convolution (stride 1) by minimal filtering F(2x2, 3x3) (Winograd; Lavin and Gray,
// "Fast Algorithms for Convolutional Neural Networks") on the bf16 matrix cores, fp32 operands split three ways
// (conv_split_kernel.h): Z = A^T [ sum over channels (G w G^T) . (B^T d B) ] A per 2x2 output tile and its 4x4 window d, sixteen
// products a channel where the direct form has 36.  G w G^T is formed in fp64 and split at upload (conv_wino.hip).
//
// Accuracy.  An accumulator's running sum is rounded 6 times per 16 channels (the direct kernel's 54 times), which outweighs
// what the transforms add (B^T d B in fp32; 1.75 times the error of a sum passes into z).  rms error of z against fp64, aligned direct
// kernel -> this one: 64 -> 128 channels at 16x16 3.5e-7 -> 1.9e-7, 64 at 56x56 3.5e-7 -> 1.8e-7, 512 at 4x4 3.2e-7 -> 2.2e-7; the
// fp32 MFMA kernel 3.0e-7, 3.0e-7, 2.7e-7.  The stacked rows' sums in two levels are below that (1.3e-7 at 67 channels, 1.9e-7 here) and
// stay on the maps they serve.  These are weights and maps as a teacher has them.  B^T d B and G w G^T mix a window's pixels and a
// filter's taps, so an output's error is relative to the window's largest pixel times the filter's largest tap, not to each
// product: 2^-24 of 64 (11 + 6 channels / 16) times that, summed over the channels, at most (two roundings of v <= 4 pixels are 2 of its units, the
// products left out 4, the output transform 5; an output's nine positions weigh 64 pixels x taps).  An output that meets a pixel far above
// the others only where the tap is far below the others has that error, where the direct kernel's is of its own products.  Weights
// that are zero for the most part are left to the direct kernel (tiles_suit, pbkd_runtime.hip).
//
// A workgroup has 64 output channels x 64 tiles x 16 positions of accumulators: 4 waves, a SIMD each, with all 512 registers,
// 256 of them accumulators.  Wave i holds row i of the transformed tile, so its products need rows a and b of a window only and
// half the output transform happens in its registers.  Per chunk of 16 channels a wave issues 96 MFMAs (3 072 cycles) and, one
// slice behind each, everything else: window values from LDS (fp32, BatchNorm and ReLU applied when they were put there), B^T d B,
// the split into pieces, the weights of the position after this one (each wave its own, straight from memory: 98 KB a chunk and
// workgroup), the values of the chunk after next and their way into LDS.  With 256 registers and two waves a SIMD nothing could
// be fetched far enough ahead (5 200 to 5 700 cycles a chunk).  Persistent, as conv_split_kernel.h.
//
// Bound by power as much as by issue: 4 400 cycles a chunk and 14 000 a tile's end at 1.6 to 1.75 GHz (the direct kernel: 1.9).
// Whole calls, direct -> this, one box: 256 channels at 56x56, batch 32, 562 -> 377 us; 512 at 28x28 614 -> 400; 64 at 224x224
// 692 -> 570; 480 -> 272 at 36x36, batch 67, 1735 -> 651 (the direct kernel's power-of-two tiles are a third empty there).
#pragma once
#include <hip/hip_ext.h>
#include <utility>

#include "conv_rows_kernel.h"

namespace pbkd {

template <int... I, class F>
__device__ __forceinline__ void static_for_each(std::integer_sequence<int, I...>, F &&f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
  static_for_each(std::make_integer_sequence<int, N>{}, f);
}

template <int SR, bool BN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void conv_wino_kernel(ConvArgs p) {
  constexpr int CAP = kWinoPositions, QP = CAP * 16, PP = QP / 2, COPY = 4 * QP;
  constexpr int EP = 68;                                   // floats of an exchange row
  extern __shared__ float smem[];
  char *const Ss = reinterpret_cast<char *>(smem);                                 // [2][4 quads][positions][4 channels]
  float *const Ex = reinterpret_cast<float *>(Ss + 2 * COPY);                      // [4 waves][2][32 channels][EP]
  SplitTile *const tiles = reinterpret_cast<SplitTile *>(Ex + kWinoExchangeFloats);
  uintx2 *const places = reinterpret_cast<uintx2 *>(tiles + kSplitMaxTiles);       // [64]: a finished tile's 2x2 tiles, see leave
  typedef float f4 __attribute__((ext_vector_type(4)));
  typedef float f2 __attribute__((ext_vector_type(2)));
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));           // row of the transformed tile; quad of channels this wave stages
  const int lane = threadIdx.x & 63, l31 = lane & 31, lh = lane >> 5;
  const int TW = p.g.TW, TH = p.g.TH, SH = p.g.SH, Th = (SH - 2) >> 1;
  const int IW = p.g.IW, IWS = p.g.IWS;
  const int HW = p.H * p.W, nchunks = p.g.nchunks;

  // ---- this workgroup's tiles
  const int G = gridDim.x;
  const int items = p.g.n_ptiles * p.g.mtiles * p.g.ksplit;
  const int first = xcd_contiguous(blockIdx.x, G);
  const int n_mine = (items - first + G - 1) / G;
  if ((int)threadIdx.x < n_mine) {
    const int L = first + (int)threadIdx.x * G;
    SplitTile d;
    d.pt = L % p.g.n_ptiles;
    const int r = L / p.g.n_ptiles;
    d.mt = r % p.g.mtiles;
    d.kz = r / p.g.mtiles;
    d.x0 = (d.pt % p.g.tiles_x) * TW;
    const int R = (d.pt / p.g.tiles_x) * TH;
    d.n0 = R / Th;
    d.y0 = R - d.n0 * Th;
    d.kb = d.kz * p.g.kchunks;
    d.nk = (nchunks - d.kb < p.g.kchunks) ? nchunks - d.kb : p.g.kchunks;
    tiles[threadIdx.x] = d;
  }
  __syncthreads();

  const unsigned mSH = ((1u << 20) + SH - 1) / SH, mTh = ((1u << 16) + Th - 1) / Th;
  auto div_Th = [&](int v) __attribute__((always_inline)) { return Th >= 64 ? (int)(v >= Th) : (int)(((unsigned)v * mTh) >> 16); };
  auto div_SH = [&](int v) __attribute__((always_inline)) { return SH >= 130 ? (int)(v >= SH) : (int)(((unsigned)v * mSH) >> 20); };

  // ---- staging: this thread's positions
  const __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float *>(p.in), 0, (int)((unsigned)p.N * p.Cin * HW * sizeof(float)), 0x00020000);
  unsigned loff[SR / 2];                                   // 16-byte units from a quad's start, of positions 2 k and (16 bits up) 2 k + 1
  const float rIW = 1.f / (float)IW;
#pragma unroll
  for (int sl = 0; sl < SR; ++sl) {
    const int q = lane + 64 * sl, r = (int)(((float)q + 0.5f) * rIW), c = q - r * IW;
    const unsigned at = q < p.g.PLd ? (c & 1) * (CAP / 2) + r * IWS + (c >> 1) : CAP - 1;
    if (sl & 1) loff[sl >> 1] |= at << 16;
    else loff[sl >> 1] = at;
  }
  unsigned goff[SR], there = 0;                            // byte offsets of channel 0; bit sl: the position is inside an image
  auto enter = [&](const SplitTile &d) __attribute__((always_inline)) {
    int q = lane;
    asm volatile("" : "+v"(q));                            // (rows and columns are worked out anew: as registers they would cost a spill)
    there = 0;
#pragma unroll
    for (int sl = 0; sl < SR; ++sl, q += 64) {
      const int r = (int)(((float)q + 0.5f) * rIW), c = q - r * IW;
      const int V = 2 * d.y0 + r, di = div_SH(V), n = d.n0 + di, y = V - di * SH - 1, x = 2 * d.x0 - 1 + c;
      const bool ok = (q < p.g.PLd) & (n < p.N) & ((unsigned)y < (unsigned)p.H) & ((unsigned)x < (unsigned)p.W);
      there |= (unsigned)ok << sl;
      goff[sl] = ok ? ((unsigned)n * p.Cin * HW + (unsigned)(y * p.W + x)) * 4u : 0u;
    }
  };
  typedef float Floats4 __attribute__((ext_vector_type(4), aligned(4)));
  typedef const Floats4 __attribute__((address_space(4))) *ConstFloats4;
  typedef const float __attribute__((address_space(4))) *ConstFloats;
  const ConstFloats cscale = (ConstFloats)(p.in_scale), cshift = (ConstFloats)(p.in_shift);
  const unsigned HWb = (unsigned)HW * 4u;
  float sv[SR][4], psh[4];
  Floats4 psc, nsc, nsh;               // scale and shift of the values that are put, and of those on their way
  unsigned sthere = 0, soff = 0;
  auto fetch_begin = [&](int k) __attribute__((always_inline)) {
    const int c = (k * 16 < p.Cin - 16 ? k * 16 : p.Cin - 16) + 4 * w;             // this wave's quad of chunk k
    soff = (unsigned)c * HWb;
    if constexpr (BN) nsc = *(ConstFloats4)(cscale + c), nsh = *(ConstFloats4)(cshift + c);
    sthere = there;
  };
  auto fetch = [&](int n) __attribute__((always_inline)) {           // value n of 4 SR
    sv[n / 4][n % 4] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rin, goff[n / 4], soff + (n % 4) * HWb, 0));
  };
  auto put_bn = [&]() __attribute__((always_inline)) {
    if constexpr (BN) {
      psc = nsc;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        psh[e] = nsh[e];
        asm("" : "+v"(psh[e]));        // (an fma takes one scalar operand)
      }
    }
  };
  // BatchNorm + ReLU of the producing layer; zeros outside the image: med3(x * scale + shift, 0, most), with most = infinity inside
  // and 0 outside; where there is no BatchNorm, x's bits and a mask (a med3 would make an infinity of a NaN)
  auto put = [&](int copy, int sl) __attribute__((always_inline)) {
    const unsigned inside = (unsigned)__builtin_amdgcn_sbfe((int)sthere, sl, 1);
    const float most = __builtin_bit_cast(float, inside & 0x7f800000u);
    f4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      o[e] = BN ? __builtin_amdgcn_fmed3f(fmaf(sv[sl][e], psc[e], psh[e]), 0.f, most)
                : __builtin_bit_cast(float, __builtin_bit_cast(unsigned, sv[sl][e]) & inside);
    const unsigned lo16 = sl & 1 ? loff[sl >> 1] >> 16 : loff[sl >> 1] & 0xffffu;
    *reinterpret_cast<f4 *>(Ss + (copy * COPY + w * QP) + lo16 * 16) = o;
  };
  // A chunk's slots (one per MFMA).  Loads return in order, so what is fetched behind a phase's weights is waited for with the next
  // phase's: values set out behind them, one a slot (a burst holds up the wave), and go into LDS some 40 slots later, up to slot
  // 33 of the next chunk, where the barrier is.
  struct Slots {
    static constexpr int load(int n) { return n < 12 ? 36 + n : n < 28 ? 44 + n : 52 + n; }                     // 36 .. 47, 56 .. 71, 80 ..
    static constexpr int put(int sl) { return SR == 6 ? (sl < 3 ? 84 + 4 * sl : 90 + 6 * sl) : sl < 3 ? 80 + 4 * sl : sl < 7 ? 88 + 4 * sl : 110 + 2 * sl; }
  };
  static_assert(Slots::load(4 * SR - 1) < 96 && Slots::put(SR - 1) < 96 + 34, "staging does not fit a chunk's slots");

  // ---- multiplying side: operand row l31 of block mt is tile 32 mt + l31 of the workgroup's 64
  const float rTW = 1.f / (float)TW;
  auto tile_at = [&](int t, int &ty, int &tx) __attribute__((always_inline)) {
    ty = (int)(((float)t + 0.5f) * rTW);
    tx = t - ty * TW;
  };
  int tyx = 0;                                             // 16 bits each: row and column of tiles l31 and 32 + l31
#pragma unroll
  for (int mt = 0; mt < 2; ++mt) {
    int ty, tx;
    tile_at(32 * mt + l31, ty, tx);
    tyx |= (ty < TH ? ty << 8 | tx : 0) << (16 * mt);
  }
  const int ra = w == 0 ? 0 : w == 2 ? 2 : 1, rb = w == 3 ? 3 : w == 2 ? 1 : 2;
  const float vs = w == 1 ? 1.f : -1.f;
  const int ab = (rb - ra) * IWS * 16;
  auto window = [&](const SplitTile &d, int mt) __attribute__((always_inline)) {       // row a of the tile's window, in copy 0
    const int ty = tyx >> (16 * mt + 8) & 255, tx = tyx >> (16 * mt) & 255, di = div_Th(d.y0 + ty);
    return ((2 * (ty + di) + ra) * IWS + tx) * 16 + lh * (2 * QP);
  };
  int adr[2], adrb[2], nadr[2];                            // rows a and b in the copy that is read next; row a of the next tile
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float *>(p.wpk), 0, (int)((unsigned)p.g.mtiles * nchunks * (unsigned)kWinoChunkBytes), 0x00020000);
  const unsigned aoff[3] = {(unsigned)lane * 16u, (unsigned)lane * 16u + 4096u, (unsigned)lane * 16u + 8192u};
  uintx4 wt[2][2][3];                                      // [position & 1][channel block][piece]
  auto load_w = [&](int j, int no, int pc, unsigned wk) __attribute__((always_inline)) {       // wk: byte offset of the chunk's weights of this row
const int at = (j & 1) * 6 + no * 3 + pc;              // in KB, from the first of its two positions
    wt[j & 1][no][pc] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(rw, aoff[at / 4] + (at % 4) * 1024, j < 2 ? wk : wk + 12288u, 0));
  };
  sfloatx16 acc[4][2][2];                                  // [position][tile block][channel block]
  auto mul = [&](const uintx4 &x, const uintx4 &v, sfloatx16 &c) __attribute__((always_inline)) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, v), c, 0, 0, 0);
  };
  // A chunk is four phases, one position j of the row each, of 24 MFMAs (four accumulators in turn: with two, each MFMA waited
  // for the one before the last).  Beside each MFMA goes a slice of other work: the next phase's operand is formed, and per half
  // phase one column of the window (of one tile block) is combined from its two rows, those of the next chunk from half 3 on.
  f4 raw[2];                                               // rows a and b
  f4 t[4][2][2];                                           // [column][tile block][quad]
  uintx4 x[2][2][3];                                       // [phase & 1][tile block][piece]
  constexpr int kCol[8] = {1, 3, 3, 0, 2, 0, 2, 1}, kBlk[8] = {1, 0, 1, 0, 0, 1, 1, 0};       // combined in half h
  auto read = [&](int h, int qd) __attribute__((always_inline)) {
    const int c = kCol[h], mt = kBlk[h], o = (c & 1) * PP + (c >> 1) * 16 + qd * QP;
    raw[0] = *reinterpret_cast<const f4 *>(Ss + adr[mt] + o);
    raw[1] = *reinterpret_cast<const f4 *>(Ss + adrb[mt] + o);
  };
  auto combine = [&](int h, int qd) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 4; ++e) t[kCol[h]][kBlk[h]][qd][e] = fmaf(vs, raw[1][e], raw[0][e]);
  };
  // The pieces of an activation are cut off (the leading 8 bits, the next 8, the rest: exact as well), not rounded: that takes no
  // v_cvt_pk_bf16_f32, which issues in 8 cycles where other vector instructions take 5 (8 behind the one they depend on:
  // hence the order here).  What is left out of the products is then 2^-26 rms of them instead of 2^-27.
  float v[4], u[4];
  unsigned top = 0xffff0000u;
  asm("" : "+s"(top));
  auto cut = [&](float f) __attribute__((always_inline)) { return __builtin_bit_cast(float, __builtin_bit_cast(unsigned, f) & top); };
  auto pair = [](float a, float b) __attribute__((always_inline)) {       // the leading halves of both
    return __builtin_amdgcn_perm(__builtin_bit_cast(unsigned, b), __builtin_bit_cast(unsigned, a), 0x07060302u);
  };
  auto form = [&](int j, int mt, int qd, int part) __attribute__((always_inline)) {      // a sixth of the work on a quad
    uintx4(&X)[3] = x[j & 1][mt];
    if (part == 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        v[e] = j == 0 ? t[0][mt][qd][e] - t[2][mt][qd][e] : j == 1 ? t[1][mt][qd][e] + t[2][mt][qd][e]
               : j == 2 ? t[2][mt][qd][e] - t[1][mt][qd][e] : t[1][mt][qd][e] - t[3][mt][qd][e];
      u[0] = cut(v[0]), u[1] = cut(v[1]);
    } else if (part == 1) {
      u[2] = cut(v[2]), u[3] = cut(v[3]);
      X[0][2 * qd] = pair(v[0], v[1]);
      v[0] -= u[0], v[1] -= u[1];
    } else if (part == 2) {
      X[0][2 * qd + 1] = pair(v[2], v[3]);
      v[2] -= u[2], v[3] -= u[3];
      u[0] = cut(v[0]), u[1] = cut(v[1]);
    } else if (part == 3) {
      u[2] = cut(v[2]), u[3] = cut(v[3]);
      X[1][2 * qd] = pair(v[0], v[1]);
      v[0] -= u[0], v[1] -= u[1];
    } else if (part == 4) {
      X[1][2 * qd + 1] = pair(v[2], v[3]);
      v[2] -= u[2], v[3] -= u[3];
      X[2][2 * qd] = pair(v[0], v[1]);
    } else {
      X[2][2 * qd + 1] = pair(v[2], v[3]);
    }
  };
  // hook(i): what else is done in the slots i of a chunk (one per MFMA)
  auto multiply = [&](auto fresh, unsigned wnow, unsigned wnext, auto &&hook) __attribute__((always_inline)) {
    constexpr bool FRESH = decltype(fresh)::value;         // a tile's first chunk: the accumulators start here (and its second position's weights are there)
    static_for<96>([&](auto slot) __attribute__((always_inline)) {
      constexpr int i = decltype(slot)::value, j = i / 24, m = i % 24, k = m / 4, mt = m >> 1 & 1, no = m & 1;
      constexpr int g = m / 6, part = m % 6, h = i / 12, s = i % 12;
      constexpr int PX[6] = {2, 1, 0, 1, 0, 0}, PW[6] = {0, 1, 2, 0, 1, 0};
      if constexpr (FRESH && k == 0) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][mt][no][r] = 0.f;
      }
      mul(x[j & 1][mt][PX[k]], wt[j & 1][no][PW[k]], acc[j][mt][no]);
      form((j + 1) & 3, g >> 1, g & 1, part);
      if constexpr (part == 5) combine(h, g & 1);
      if constexpr (s == 5) read(h, 1);
      if constexpr (s == 11) read((h + 1) & 7, 0);
      if constexpr (m >= 2 && m < 8 && !(FRESH && j == 0)) load_w((j + 1) & 3, (m - 2) / 3, (m - 2) % 3, j < 3 ? wnow : wnext);
      hook(slot);
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // ---- a finished tile: back through the output transform
  const int HWo = p.Ho * p.Wo;
  const __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc(
      p.g.ksplit > 1 ? p.split_out : p.out, 0, (int)((unsigned)p.g.ksplit * p.N * p.Cout * HWo * sizeof(float)), 0x00020000);
  constexpr unsigned kNowhere = kPastBuffer - 15u;
  const int vw = (TW % 2 == 0 && p.Wo % 4 == 0) ? 4 : p.Wo % 2 == 0 ? 2 : 1;
  // where tile t of the workgroup's 64 lies
  struct Where {
    int n, y, x;                       // image, first row and column
    bool ok;
  };
  auto where = [&](const SplitTile &d, int t) __attribute__((always_inline)) {
    int ty, tx;
    tile_at(t, ty, tx);
    const int di = div_Th(d.y0 + ty);
    Where v;
    v.n = d.n0 + di;
    v.y = 2 * (d.y0 + ty - di * Th);
    v.x = 2 * (d.x0 + tx);
    v.ok = ty < TH && v.n < p.N && v.x < p.Wo;
    return v;
  };
  auto leave = [&](const SplitTile &d, unsigned wnext) __attribute__((always_inline)) {     // wnext: the next tile's weights
    const bool stats = p.stat_partial && p.g.ksplit == 1;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                          // (as in enter)
    const int oc = tid >> 3, pr = tid & 7, l31 = tid & 31, lh = tid >> 5 & 1, lane = tid & 63;
    // places: byte offset of the 2x2 tile's first pixel in channel 0; bit 0: exists, 1: its second column does, 2: its second row
    if (tid < 64) {
      const Where v = where(d, tid);
      const unsigned pix = ((unsigned)(d.kz * p.N + v.n) * (unsigned)(p.Cout * HWo) + (unsigned)(v.y * p.Wo + v.x)) * 4u;
      places[tid] = uintx2{pix, v.ok ? 1u | (v.x + 1 < p.Wo ? 2u : 0u) | (v.y + 1 < p.Ho ? 4u : 0u) : 0u};
    }
    // the next tile's second position's weights, ahead of the stores: loads behind them are waited for with them
#pragma unroll
    for (int i = 0; i < 6; ++i) load_w(1, i / 3, i % 3, wnext);
#pragma unroll
    for (int no = 0; no < 2; ++no) {
      const int o = d.mt * 64 + no * 32 + oc;
      const unsigned ob = o < p.Cout ? (unsigned)o * (unsigned)HWo * 4u : kNowhere, row = (unsigned)p.Wo * 4u;
      float *const ex = Ex + (2 * w * 32 + l31) * EP + 4 * lh;
      if (no == 1) __syncthreads();                        // (the first half has been read)
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
#pragma unroll
        for (int j = 0; j < 4; ++j) asm volatile("" : "+a"(acc[j][mt][no])::"memory");     // (not fetched from the accumulation registers before here)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          f4 y0, y1;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float m0 = acc[0][mt][no][4 * g + r], m1 = acc[1][mt][no][4 * g + r], m2 = acc[2][mt][no][4 * g + r], m3 = acc[3][mt][no][4 * g + r];
            y0[r] = m0 + m1 + m2;
            y1[r] = m1 - m2 - m3;
          }
          *reinterpret_cast<f4 *>(ex + 32 * mt + 8 * g) = y0;
          *reinterpret_cast<f4 *>(ex + 32 * EP + 32 * mt + 8 * g) = y1;
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __syncthreads();
      float *const rd = Ex + oc * EP + 2 * pr;             // this thread's pairs of 2x2 tiles: 2 (pr + 8 k) and the next
      float z[4][8];                                       // [pair][tile, row, column]
      uintx4 pl[4];
      bool whole = true;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        pl[k] = *reinterpret_cast<const uintx4 *>(places + 2 * (pr + 8 * k));
        whole = whole && (pl[k][1] & pl[k][3]) == 7;
      }
      whole = __all(whole);
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          f2 Y[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) Y[i] = *reinterpret_cast<const f2 *>(rd + 16 * k + (2 * i + c) * 32 * EP);
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            z[k][4 * i + c] = Y[0][i] + Y[1][i] + Y[2][i];
            z[k][4 * i + 2 + c] = Y[1][i] - Y[2][i] - Y[3][i];
          }
        }
      // sums about the channel's first pixel
      float pv, s1[2], s2[2], cnt;
      auto sums = [&]() __attribute__((always_inline)) {
        pv = __shfl(z[0][0], lane & 56, 64);
        s1[0] = s1[1] = s2[0] = s2[1] = cnt = 0.f;
        if (whole) {
#pragma unroll
          for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int v = 0; v < 8; ++v) {
              const float dv = z[k][v] - pv;
              s1[v & 1] += dv;
              s2[v & 1] = fmaf(dv, dv, s2[v & 1]);
            }
          cnt = 32.f;
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int v = 0; v < 8; ++v) {
              const unsigned need = 1u | (v & 1 ? 2u : 0u) | (v & 2 ? 4u : 0u);
              const bool there = (pl[k][v < 4 ? 1 : 3] & need) == need;
              const float dv = there ? z[k][v] - pv : 0.f;
              s1[v & 1] += dv;
              s2[v & 1] = fmaf(dv, dv, s2[v & 1]);
              cnt += there ? 1.f : 0.f;
            }
        }
      };
      sums();
      if (__any(!(fabsf(s1[0] + s1[1]) < __builtin_inff()))) {       // infinities, or numbers too large for the pieces: fp32 products
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
          for (int v = 0; v < 8; ++v) rd[16 * k + (v >> 1) * (32 * EP) + (v & 1)] = z[k][v];         // (in the thread's own slots)
#pragma unroll 1
        for (int i = 0; i < 32; ++i) {
          const int k = i >> 3, v = i & 7;
          const Where at = where(d, 2 * (pr + 8 * k) + (v >> 2));
          const int y = at.y + (v >> 1 & 1), x = at.x + (v & 1);
          float *const zp = rd + 16 * k + (v >> 1) * (32 * EP) + (v & 1);
          if (!(fabsf(*zp) < __builtin_inff()) && o < p.Cout && at.ok && y < p.Ho && x < p.Wo)
            *zp = plain_conv_sum(p, o, at.n, y, x, d.kb * 16, (d.kb + d.nk) * 16 < p.Cin ? (d.kb + d.nk) * 16 : p.Cin);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
          for (int v = 0; v < 8; ++v) z[k][v] = rd[16 * k + (v >> 1) * (32 * EP) + (v & 1)];
        sums();
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (vw == 4) {
          const unsigned off = (ob != kNowhere && pl[k][1]) ? pl[k][0] + ob : kNowhere;
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            const f4 v = {z[k][2 * r], z[k][2 * r + 1], z[k][4 + 2 * r], z[k][5 + 2 * r]};
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uintx4, v), rout, r == 0 ? off : (off != kNowhere && (pl[k][1] & 4)) ? off + row : kNowhere, 0, 0);
          }
        } else {
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const unsigned off = (ob != kNowhere && pl[k][2 * i + 1]) ? pl[k][2 * i] + ob : kNowhere;
#pragma unroll
            for (int r = 0; r < 2; ++r) {
              const bool rok = off != kNowhere && (!r || (pl[k][2 * i + 1] & 4));
              const float v0 = z[k][4 * i + 2 * r], v1 = z[k][4 * i + 2 * r + 1];
              if (vw == 2) {
                const f2 v = {v0, v1};
                __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uintx2, v), rout, rok ? off + r * row : kNowhere, 0, 0);
              } else {
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v0), rout, rok ? off + r * row : kNowhere, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v1), rout, rok && (pl[k][2 * i + 1] & 2) ? off + r * row + 4u : kNowhere, 0, 0);
              }
            }
          }
        }
      }
      if (stats) {
        StatPart sp;
        auto sum8 = [](float q) {
          q += dpp_mov<0xB1>(q);       // quad_perm [1,0,3,2]
          q += dpp_mov<0x4E>(q);       // quad_perm [2,3,0,1]
          q += dpp_mov<0x141>(q);      // row_half_mirror
          return q;
        };
        sp.pivot = pv;
        sp.s1 = sum8(s1[0] + s1[1]);
        sp.s2 = sum8(s2[0] + s2[1]);
        sp.n = sum8(cnt);
        if (pr == 0 && o < p.Cout) stat_store(p.stat_partial, (size_t)o * p.g.n_ptiles + d.pt, sp);
      }
    }
  };

  // ---- the walk: chunk after chunk through all tiles.  Chunk c+1 is put into LDS, in two halves, while chunk c is multiplied;
  // the one barrier of a chunk stands where it has been read by all.
  int ft = 0, fk, fend;                                    // the fetching side: tile, chunk, past its last chunk
  {
    const SplitTile d = uniform_tile(tiles[0]);
    enter(d);
    fk = d.kb, fend = d.kb + d.nk;
  }
  auto advance = [&]() __attribute__((always_inline)) {    // past the end the last chunk is loaded again, and dropped
    if (fk + 1 < fend) {
      ++fk;
    } else if (ft + 1 < n_mine) {
      const SplitTile d = uniform_tile(tiles[++ft]);
      enter(d);
      fk = d.kb, fend = d.kb + d.nk;
    }
  };
  auto tile_weights = [&](const SplitTile &d) __attribute__((always_inline)) {
    return (unsigned)(d.mt * nchunks + d.kb) * (unsigned)kWinoChunkBytes + (unsigned)(w * (kWinoChunkBytes / 4));
  };
  int tn = 0, copy = 0;                                    // the multiplying side: tile; the copy its chunk is in
  SplitTile md = uniform_tile(tiles[0]);
#pragma unroll
  for (int mt = 0; mt < 2; ++mt) adr[mt] = window(md, mt), adrb[mt] = adr[mt] + ab;
  unsigned wnow = tile_weights(md);
  fetch_begin(fk);
#pragma unroll
  for (int n = 0; n < 4 * SR; ++n) fetch(n);
#pragma unroll
  for (int i = 0; i < 12; ++i) load_w(i / 6, i % 6 / 3, i % 3, wnow);
  put_bn();
#pragma unroll
  for (int sl = 0; sl < SR; ++sl) put(0, sl);
  advance();
  fetch_begin(fk);
#pragma unroll
  for (int n = 0; n < 4 * SR; ++n) fetch(n);
  put_bn();
#pragma unroll
  for (int sl = 0; sl < SR; ++sl)
    if (Slots::put(sl) < 96) put(1, sl);
  advance();
  __syncthreads();
#pragma unroll
  for (int h = 3; h < 8; ++h)
#pragma unroll
    for (int qd = 0; qd < 2; ++qd) read(h, qd), combine(h, qd);
#pragma unroll
  for (int g = 0; g < 4; ++g)
#pragma unroll
    for (int part = 0; part < 6; ++part) form(0, g >> 1, g & 1, part);
  read(0, 0);
  auto step = [&](auto fresh, bool last) __attribute__((always_inline)) {
    const unsigned wnext = !last ? wnow + (unsigned)kWinoChunkBytes : tn + 1 < n_mine ? tile_weights(uniform_tile(tiles[tn + 1])) : wnow;
    multiply(fresh, wnow, wnext, [&](auto slot) __attribute__((always_inline)) {
      constexpr int i = decltype(slot)::value;
      static_for<SR>([&](auto sl_) __attribute__((always_inline)) {
        constexpr int sl = decltype(sl_)::value, ps = Slots::put(sl);
        if constexpr (i == ps % 96) put(ps < 96 ? copy : 1 - copy, sl);
      });
      if constexpr (i == 34) {
        __syncthreads();
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
          adr[mt] = (last ? nadr[mt] : adr[mt] - copy * COPY) + (1 - copy) * COPY;
          adrb[mt] = adr[mt] + ab;
        }
      }
      if constexpr (i == 35) fetch_begin(fk);
      static_for<4 * SR>([&](auto n) __attribute__((always_inline)) {
        if constexpr (i == Slots::load(decltype(n)::value)) fetch(decltype(n)::value);
      });
      if constexpr (i == Slots::put(0) - 1) put_bn();
    });
    // (what is for the next chunk only is used here: else the compiler moves its computation behind the branches that follow,
    // out of the MFMAs' shadow)
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
#pragma unroll
      for (int pc = 0; pc < 3; ++pc) asm volatile("" : "+v"(x[0][mt][pc]));
#pragma unroll
      for (int qd = 0; qd < 2; ++qd) {
        asm volatile("" : "+v"(t[2][mt][qd]));
        if (mt == 0) asm volatile("" : "+v"(t[1][mt][qd]));
      }
    }
    wnow = wnext;
    copy = 1 - copy;
  };
  for (;;) {
    {
      const SplitTile d = uniform_tile(tiles[tn + 1 < n_mine ? tn + 1 : tn]);
      nadr[0] = window(d, 0), nadr[1] = window(d, 1);
    }
    step(std::true_type{}, md.nk == 1);
    advance();
    for (int c = md.nk - 1; c > 0; --c) {
      step(std::false_type{}, c == 1);
      advance();
    }
    leave(md, wnow);
    if (++tn == n_mine) break;
    md = uniform_tile(tiles[tn]);
  }
}

}  // namespace pbkd
