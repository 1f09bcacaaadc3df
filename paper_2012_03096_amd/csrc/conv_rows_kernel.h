// Device code of the split 3x3 convolution for maps of any width and any alignment (arithmetic, pipeline and MFMA side:
// conv_split_kernel.h).  It differs in what a tile is and in how the activations arrive.
//
// A tile is TH output rows x TW output columns, neither a power of two, out of the STACK of all images' rows: row R of
// the stack is row R % Ho of image R / Ho, so a tile runs on from one image into the next and only the last tile of the
// whole batch is part empty.  The input side of the stack keeps every image's zero rows: an image takes
// SH = stride (Ho - 1) + 3 staged rows (input rows -1 .. ), output row y of image n reads stack rows n SH + stride y + 0..2,
// and a tile stages the contiguous stack rows its own rows span.  14x14 maps: 18 rows x 14 columns, 252 of a 256-pixel
// tile's columns used, where a power-of-two tile of whole images uses 196; 27x23 maps: 5 x 23 of 128 (90 %) for 61 %.
//
// A loader thread owns staged positions and loads their eight channels of a chunk itself, 4 bytes each, straight into
// registers a stage ahead of the split: any alignment, no raw copy in LDS (whole 16-byte groups need a width that is a
// multiple of 4).  The channel goes into the scalar offset, so a load costs no vector instruction beyond itself.  The weights
// go from memory into the MFMA waves' operand registers, and a finished tile leaves through LDS and the loader waves.
//
// Infinities, and numbers past bfloat16's largest, make every sum that holds one a NaN (their pieces are none).  Sums that are
// NaN are formed again in fp32 from the operands themselves (plain_conv_sum): an infinity, a number, or a NaN, as fp32
// products have it.
//
// Sums are in two levels (a chunk's products from zero, then one addition to the running sum), for accuracy: rms error of z
// against fp64 at 67 channels on 27x23 maps 3.0e-7 for the fp32 MFMA kernel, 3.6e-7 with one running sum, 1.3e-7 so; at 512 on
// 14x14 8.3e-7, 5.0e-7, 1.5e-7.  That costs 4 % of the time.
//
// Bound by the MFMA waves' stage, on maps of one round of tiles by start-up and last stores, on 224x224 maps by the loads.
// Measured against the fp32-MFMA kernel that unaligned maps ran before, forward of two layers: 512 channels at 14x14,
// batch 32, 571 -> 314 us; 128 at 27x23, batch 77, 474 -> 197; 64 there 141 -> 74; 256 at 10x10, batch 128, 692 -> 187.
#pragma once
#include <type_traits>

#include "conv_split_kernel.h"

namespace pbkd {

// output channel o at row y, column x of image n in fp32 multiply-adds over the input channels [c0, c1)
__device__ __forceinline__ float plain_conv_sum(const ConvArgs &p, int o, int n, int y, int x, int c0, int c1) {
  float s = 0.f;
#pragma unroll 1
  for (int c = c0; c < c1 && s == s; ++c) {
    const float *in = p.in + ((size_t)n * p.Cin + c) * p.H * p.W, *w = p.w_canon + ((size_t)o * p.Cin + c) * 9;
    const float sc = p.in_scale ? p.in_scale[c] : 1.f, sh = p.in_scale ? p.in_shift[c] : 0.f;
#pragma unroll 1
    for (int t = 0; t < 9; ++t) {
      const int yy = p.stride * y - 1 + t / 3, xx = p.stride * x - 1 + t % 3;
      float v = 0.f;
      if (yy >= 0 && yy < p.H && xx >= 0 && xx < p.W) {
        v = fmaf(in[(size_t)yy * p.W + xx], sc, sh);
        if (p.in_scale) v = fmaxf(v, 0.f);                 // (ReLU; without one a NaN stays a NaN)
      }
      s = fmaf(w[t], v, s);
    }
  }
  return s;
}

template <int WGM, int MB, int NB, int BSLOTS, bool VEC>
__global__ __launch_bounds__(512) void conv_rows_kernel(ConvArgs p) {
  constexpr int WGN = 4 / WGM;
  constexpr int BM = WGM * MB * 32;     // output channels per workgroup
  constexpr int WN = NB * 32;           // pixels per wave
  constexpr int A_STRIDE = conv_split_a_stride(BM);
  extern __shared__ float smem[];
  constexpr int BN = WGN * WN;          // pixels per workgroup
  constexpr int CAP = conv_rows_positions(BSLOTS);         // staged positions a plane has room for; the last is never read
  constexpr int PLANE = CAP * 16, COPY = 3 * PLANE;        // bytes of a piece's plane, of a copy of all pieces
  constexpr int OROW = BN + 4;                             // floats of a channel's row of the finished tile
  char *const Ss = reinterpret_cast<char *>(smem);         // [2][3 pieces][CAP][8 channels of bf16]
  float *const Os = reinterpret_cast<float *>(Ss + 2 * COPY);                      // [BM][OROW]: a finished tile
  StatPart *const red = reinterpret_cast<StatPart *>(Os + BM * OROW);              // [WGN][BM]
  SplitTile *const tiles = reinterpret_cast<SplitTile *>(red + WGN * BM);          // [kSplitMaxTiles]

  const bool loader = threadIdx.x >= 256;
  const int tid = threadIdx.x & 255, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WGM, wn = wave / WGM;
  const int l31 = lane & 31, lh = lane >> 5;
  const int TW = p.g.TW, TH = p.g.TH, SH = p.g.SH;
  const int IW = p.g.IW, IWS = p.g.IWS;
  const int s = p.stride;
  const int HWo = p.Ho * p.Wo;
  const int HW = p.H * p.W;
  const int nchunks = p.g.nchunks;

  // ---- this workgroup's tiles (y0 and n0: row and image of the tile's first stack row)
  const int G = gridDim.x;
  const int items = p.g.n_ptiles * p.g.mtiles * p.g.ksplit;
  const int first = xcd_contiguous(blockIdx.x, G);
  const int n_mine = (items - first + G - 1) / G;          // the host launches G <= items, and G*kSplitMaxTiles >= items
  if ((int)threadIdx.x < n_mine) {
    const int L = first + (int)threadIdx.x * G;
    SplitTile d;
    d.pt = L % p.g.n_ptiles;
    const int r = L / p.g.n_ptiles;
    d.mt = r % p.g.mtiles;
    d.kz = r / p.g.mtiles;
    d.x0 = (d.pt % p.g.tiles_x) * TW;
    const int R = (d.pt / p.g.tiles_x) * TH;
    d.n0 = R / p.Ho;
    d.y0 = R - d.n0 * p.Ho;
    d.kb = d.kz * p.g.kchunks;
    d.nk = (nchunks - d.kb < p.g.kchunks) ? nchunks - d.kb : p.g.kchunks;
    tiles[threadIdx.x] = d;
  }
  __syncthreads();
  int TC = 0;                                              // chunks in all of this workgroup's tiles
  for (int t = 0; t < n_mine; ++t) TC += tiles[t].nk;
  TC = __builtin_amdgcn_readfirstlane(TC);

  if (loader) {
    // ------------------------------------------------------------------ loader waves: loads, split; statistics' last step and stores
    const __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(p.in), 0, (int)((unsigned)p.N * p.Cin * HW * sizeof(float)), 0x00020000);
    // the staged positions this thread loads and splits: row and column in the tile do not depend on the tile
    int srow[BSLOTS], scol[BSLOTS], loff[BSLOTS];          // row -1: no such position (it works on the spare one)
#pragma unroll
    for (int sl = 0; sl < BSLOTS; ++sl) {
      const int q = tid + 256 * sl;
      const bool in_tile = q < p.g.PLd;
      const int r = q / IW;
      srow[sl] = in_tile ? r : -1;
      scol[sl] = q - r * IW;
      loff[sl] = (in_tile ? r * IWS + scol[sl] : CAP - 1) * 16;
    }
    // where the positions' values are: byte offset in the tensor of channel 0, and whether there is one (halo positions
    // outside the image are zeros: they load the tensor's first value and are clamped to zero, so every load is in bounds)
    unsigned goff[BSLOTS];
    float hi[BSLOTS];                   // what a position's value is clamped to from above: zero where there is none
    auto enter = [&](const SplitTile &d) __attribute__((always_inline)) {
#pragma unroll
      for (int sl = 0; sl < BSLOTS; ++sl) {
        const int V = d.n0 * SH + d.y0 * s + srow[sl];
        const int n = V / SH, y = V - n * SH - 1, x = d.x0 * s - 1 + scol[sl];
        const bool ok = srow[sl] >= 0 && n < p.N && y >= 0 && y < p.H && x >= 0 && x < p.W;
        hi[sl] = ok ? __builtin_inff() : 0.f;
        goff[sl] = ok ? ((unsigned)n * p.Cin * HW + (unsigned)(y * p.W + x)) * 4u : 0u;
      }
    };
    // A chunk's first channel: a ragged last chunk reaches back to the last eight channels, with zero weights for those
    // the chunk before has had (Cin > 8: the host checks).
    auto first_channel = [&](int k) __attribute__((always_inline)) { return k * 8 < p.Cin - 8 ? k * 8 : p.Cin - 8; };
    const unsigned HWb = (unsigned)HW * 4u;
    auto fetch = [&](int c0, float (&v)[BSLOTS][8]) __attribute__((always_inline)) {
      unsigned soff = (unsigned)c0 * HWb;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
#pragma unroll
        for (int sl = 0; sl < BSLOTS; ++sl)
          v[sl][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rin, goff[sl], soff, 0));
        soff += HWb;
      }
    };
    // the producing layer's scale and shift for a chunk's channels, through the scalar cache (the constant address
    // space: an earlier kernel wrote them): two loads of eight
    const bool bn = p.in_scale != nullptr;
    const float lo = bn ? 0.f : -__builtin_inff();             // ReLU only where there is a BatchNorm to apply
    typedef float Floats8 __attribute__((ext_vector_type(8), aligned(4)));
    typedef const Floats8 __attribute__((address_space(4))) *ConstFloats8;
    typedef const float __attribute__((address_space(4))) *ConstFloats;
    const ConstFloats cscale = (ConstFloats)(p.in_scale), cshift = (ConstFloats)(p.in_shift);
    struct Bn {
      Floats8 sc, sh;
    };
    auto fetch_bn = [&](int c0) __attribute__((always_inline)) {
      Bn v;
      if (bn) {
        v.sc = *(ConstFloats8)(cscale + c0), v.sh = *(ConstFloats8)(cshift + c0);
      } else {
        v.sc = 1.f, v.sh = 0.f;
      }
      return v;
    };
    auto split = [&](const float (&raw)[BSLOTS][8], const float (&most)[BSLOTS], const Bn &v, int rc) __attribute__((always_inline)) {
      char *Sd = Ss + rc * COPY;
      float shv[8];                     // an fma takes one scalar operand: the shifts in vector registers
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        shv[e] = v.sh[e];
        asm("" : "+v"(shv[e]));
      }
#pragma unroll
      for (int sl = 0; sl < BSLOTS; ++sl) {
        uintx4 pp[3];
        const float least = most[sl] > 0.f ? lo : 0.f;
#pragma unroll
        for (int t = 0; t < 4; ++t) {              // channels 2t, 2t+1
          float x[2];
#pragma unroll
          for (int e = 0; e < 2; ++e)              // BatchNorm, then ReLU and the halo's zeros in one step
            x[e] = __builtin_amdgcn_fmed3f(fmaf(raw[sl][2 * t + e], v.sc[2 * t + e], shv[2 * t + e]), least, most[sl]);
          unsigned q[3];
          split3_bf16(x[0], x[1], q);
#pragma unroll
          for (int pc = 0; pc < 3; ++pc) pp[pc][t] = q[pc];
        }
#pragma unroll
        for (int pc = 0; pc < 3; ++pc) *reinterpret_cast<uintx4 *>(Sd + loff[sl] + pc * PLANE) = pp[pc];
      }
    };
    // Stage i splits chunk i-1, then issues the loads of chunk i+1's activations into the registers it has just emptied: they
    // stay in flight across the barrier and have the whole next stage to arrive.  Two sets take turns: set c & 1 holds chunk c.
    struct Held {
      float v[BSLOTS][8];
      float hi[BSLOTS];
      int c0;                           // first channel
    };
    Held held[2];
    int lt = 0, lc = 0;                 // tile and chunk of the fetching side
    SplitTile ld = uniform_tile(tiles[0]);
    enter(ld);
    auto fetch_next = [&](Held &h) __attribute__((always_inline)) {
      h.c0 = first_channel(ld.kb + lc);
      fetch(h.c0, h.v);
#pragma unroll
      for (int sl = 0; sl < BSLOTS; ++sl) h.hi[sl] = hi[sl];
      if (++lc == ld.nk) {
        if (lt + 1 < n_mine) {
          lc = 0;
          ld = uniform_tile(tiles[++lt]);
          enter(ld);
        } else {
          --lc;                         // past the end the last chunk is loaded again, and dropped
        }
      }
    };
    // A finished tile lies in Os from the stage after its last chunk until the next tile's end.  The loader waves finish its
    // statistics and store it, a quarter a stage where the next tile has the stages for it, beside their own work: by the MFMA
    // waves, stores and sums took 20 000 cycles a tile in which nothing multiplied (a quarter of a 32-chunk tile's time).
    // VEC (rows start on 16-byte boundaries): a thread stores four pixels of a channel, else one, for every CSTEP-th channel.
    // (Stores that are always issued, past the buffer where there is nothing to store, would keep the count of younger
    // operations fixed that a wait for a load allows for; measured level with VEC and 20 % slower without.)
    constexpr int CSTEP = (VEC ? 1024 : 256) / BN, PASSES = BM / CSTEP, PQ = PASSES / 4;
    const int opx = VEC ? 4 * (tid & (BN / 4 - 1)) : tid & (BN - 1);
    const int oc0 = VEC ? tid / (BN / 4) : tid / BN;
    const int orow = opx / TW, ocol = opx - orow * TW;
    const __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc(
        p.g.ksplit > 1 ? p.split_out : p.out, 0, (int)((unsigned)p.g.ksplit * p.N * p.Cout * HWo * sizeof(float)), 0x00020000);
    constexpr unsigned kNowhere = kPastBuffer - 15u;           // (the host keeps the buffer's end below it)
    int quarter = 4, at_once = 1;                              // quarters stored of the finished tile, and how many a stage
    int och = 0;                                               // this thread's first channel
    unsigned ooff = kNowhere;
    auto finish_tile = [&](int t, int stages) __attribute__((always_inline)) {     // stages: until the next tile's end overwrites Os
      const SplitTile d = uniform_tile(tiles[t]);
      const int rr = d.y0 + orow, di = rr / p.Ho, y = rr - di * p.Ho, n = d.n0 + di;
      och = d.mt * BM + oc0;
      ooff = (orow < TH && n < p.N && d.x0 + ocol < p.Wo)
                 ? ((unsigned)((d.kz * p.N + n) * p.Cout + och) * (unsigned)HWo + (unsigned)(y * p.Wo + d.x0 + ocol)) * 4u
                 : kNowhere;
      quarter = 0;
      at_once = stages >= 4 ? 1 : 4;
      if (p.stat_partial && p.g.ksplit == 1) {
        // the MFMA waves' partials, re-expressed about the first one's pivot and added
        for (int e = tid; e < BM; e += 256) {
          const int o = d.mt * BM + e;
          if (o < p.Cout) {
            StatPart v = red[e];
#pragma unroll
            for (int w = 1; w < WGN; ++w) stat_rebase_add(v, red[w * BM + e]);
            stat_store(p.stat_partial, (size_t)o * p.g.n_ptiles + d.pt, v);
          }
        }
      }
    };
    auto store_quarter = [&]() __attribute__((always_inline)) {
      const unsigned step = (unsigned)(CSTEP * HWo) * 4u;
      const int first = quarter * PQ;
      const float *src = Os + (oc0 + first * CSTEP) * OROW + opx;
      const bool some = ooff != kNowhere;
#pragma unroll
      for (int k = 0; k < PQ; ++k) {
        const unsigned off = (some && och + (first + k) * CSTEP < p.Cout) ? ooff + (unsigned)(first + k) * step : kNowhere;
        if constexpr (VEC) {
          __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const uintx4 *>(src + k * CSTEP * OROW), rout, off, 0, 0);
        } else {
          const float v = src[k * CSTEP * OROW];
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rout, off, 0, 0);
        }
      }
      ++quarter;
    };
    // the multiplying side's tile, and its chunks left (it is at chunk i-2 in stage i)
    int ft = 0, left = ld.nk + 1;
    int ended = -1;                     // the tile that ended in the stage before this one
    fetch_next(held[0]);                // stage 0
    fetch_next(held[1]);
    Bn now = fetch_bn(held[0].c0);
    auto load_stage = [&](int odd, Held &h, const Held &other) __attribute__((always_inline)) {       // odd: chunk i-1's parity
      const Bn next = fetch_bn(other.c0);                              // chunk i's scale and shift
      split(h.v, h.hi, now, odd);
      if (ended >= 0) {
        finish_tile(ended, left - 1);
        ended = -1;
      }
      if (--left == 0) {
        ended = ft;
        if (++ft < n_mine) left = __builtin_amdgcn_readfirstlane(tiles[ft].nk);
      }
      fetch_next(h);
      for (int k = 0; k < at_once && quarter < 4; ++k) store_quarter();
      now = next;
      __syncthreads();
    };
    __syncthreads();
    // Stages 1 .. TC in pairs.  With an odd TC the last pair's second half is stage TC + 1, in which the MFMA waves multiply
    // the last chunk: what it splits (the last chunk again) goes where they do not read.  (An exit between the two halves
    // costs more: the compiler then waits in the first for loads that are a stage old at most.)
    for (int i = 1; i <= TC; i += 2) {
      load_stage(0, held[0], held[1]);
      load_stage(1, held[1], held[0]);
    }
    if (!(TC & 1)) __syncthreads();     // stage TC + 1 (the tile before the last, of two chunks at least each, is stored)
    finish_tile(n_mine - 1, 1);
    while (quarter < 4) store_quarter();
  } else {
    // ------------------------------------------------------------------ MFMA waves
    sfloatx16 acc[MB][NB];
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
    // The pixels are the MFMA's rows and the channels its columns, so that a lane's accumulators are 16 pixels per block of
    // ONE channel and the statistics need no step across lanes (but one between the half-waves).  As operand row, lane l31 of
    // block nb supplies pixel wn*WN + nb*32 + l31: its row and column in the tile, and per tile its place in the staged
    // positions for every tap pair (tap 2j+h of this half-wave; in the last step both half-waves read tap 8).
    int prow[NB], pcol[NB], padr[NB][5];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int pn = wn * WN + nb * 32 + l31;
      prow[nb] = pn / TW;
      pcol[nb] = pn - prow[nb] * TW;
    }
    unsigned valid[NB];                 // bit l31: pixel l31 of the block exists (the same in all lanes)
    auto enter = [&](const SplitTile &d) __attribute__((always_inline)) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int r = d.y0 + prow[nb], di = r / p.Ho, y = r - di * p.Ho;
        const bool ok = prow[nb] < TH && d.n0 + di < p.N && d.x0 + pcol[nb] < p.Wo;
        valid[nb] = (unsigned)__ballot(ok);
        // (a row without a pixel repeats the tile's first one: the statistics' pivot is always a value of the tile)
        const int at = ok ? (di * SH + s * (y - d.y0)) * IWS + s * pcol[nb] : 0;
#pragma unroll
        for (int j = 0; j < 5; ++j) {
          const int tap = (2 * j + lh < 9) ? 2 * j + lh : 8;
          padr[nb][j] = (at + (tap / 3) * IWS + (tap % 3)) * 16;
        }
      }
    };
    // The weights come straight from memory (the L1 and L2 hold them) into operand registers: a register set per tap pair,
    // refilled for the next pass as soon as the pair's MFMAs are issued, so a load has a whole pass to arrive.  Through LDS
    // they would double its reads, and LDS gives 64 bytes a cycle: 512 cycles a tap pair for 384 of MFMAs.
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(p.wpk), 0, (int)((unsigned)p.g.mtiles * nchunks * A_STRIDE), 0x00020000);
    const unsigned aoff = (unsigned)(lh * BM + wm * (MB * 32) + l31) * 16u;
    // Channel blocks are multiplied MG at a time, so that a pass over the chunk has 32 registers of sums at most beside acc.
    constexpr int MG = NB == 1 ? MB : 1, PASSES = MB / MG;
    uintx4 a[5][3][MG];
    auto load_a = [&](int j, int g, unsigned wk) __attribute__((always_inline)) {        // wk: byte offset of the chunk's weights
#pragma unroll
      for (int pc = 0; pc < 3; ++pc)
#pragma unroll
        for (int m = 0; m < MG; ++m)
          a[j][pc][m] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(rw, aoff + (g * MG + m) * 512, wk + (unsigned)((pc * 5 + j) * BM * 32), 0));
    };
    auto mul = [&](const uintx4 &w, const uintx4 &x, sfloatx16 &c) __attribute__((always_inline)) {
      c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, w), c, 0, 0, 0);
    };

    // One pipeline stage of the MFMA waves: multiplies the chunk whose planes are in copy mc; wnow and wnext: its weights and the
    // next chunk's.  A chunk's 27 products are summed from zero and added to acc once, so that the roundings that happen
    // at the size of the whole sum are one per eight channels instead of 27.  Small products come first: what
    // w0x0 rounds away is then the only loss at a chunk's own size, and an activation piece's registers fall free three
    // products before the next tap pair needs them.  The ninth tap's pairing of pieces is conv_split_kernel.h's.
    auto stage = [&](auto copy, unsigned wnow, unsigned wnext) __attribute__((always_inline)) {
      const char *Sb = Ss + decltype(copy)::value * COPY;
      uintx4 bv[3][NB];
      auto fill_b = [&](int pc, int j) __attribute__((always_inline)) {
        // operand slot pc is piece pc, but for the ninth tap, where the half-waves read two different pieces of it
        const int plane = (j < 4 ? pc : kSplitLastX[pc][0] + lh * (kSplitLastX[pc][1] - kSplitLastX[pc][0])) * PLANE;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) bv[pc][nb] = *reinterpret_cast<const uintx4 *>(Sb + padr[nb][j] + plane);
      };
      fill_b(2, 0); fill_b(1, 0); fill_b(0, 0);
#pragma unroll
      for (int g = 0; g < PASSES; ++g) {
        sfloatx16 sum[MG][NB];
#pragma unroll
        for (int m = 0; m < MG; ++m)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r) sum[m][nb][r] = 0.f;
#pragma unroll
        for (int j = 0; j < 5; ++j) {
          __builtin_amdgcn_sched_barrier(0);
          constexpr int PA[6] = {0, 0, 1, 2, 1, 0}, PB[6] = {2, 1, 1, 0, 0, 0}, PL4[3] = {2, 1, 0};
          const bool more = j + 1 < 5 || g + 1 < PASSES;
          const int jn = j + 1 < 5 ? j + 1 : 0;
#pragma unroll
          for (int q = 0; q < (j < 4 ? 6 : 3); ++q) {
            const int qa = j < 4 ? PA[q] : PL4[q], qb = j < 4 ? PB[q] : PL4[q];
#pragma unroll
            for (int m = 0; m < MG; ++m)
#pragma unroll
              for (int nb = 0; nb < NB; ++nb) mul(a[j][qa][m], bv[qb][nb], sum[m][nb]);
            __builtin_amdgcn_sched_barrier(0);
            // the next tap pair's pieces, into the registers that have just fallen free
            if (more && (j == 4 || q == 0 || q == 2 || q == 5)) fill_b(j == 4 ? qb : PB[q], jn);
          }
          if (g + 1 < PASSES) load_a(j, g + 1, wnow);
          else load_a(j, 0, wnext);
        }
#pragma unroll
        for (int m = 0; m < MG; ++m)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) acc[g * MG + m][nb] += sum[m][nb];
      }
    };
    // The multiplying side leaves a tile: statistics partials into red, the tile into Os, accumulators cleared.  Accumulator
    // register r of lane l holds pixel 8*(r/4) + 4*(l/32) + r%4 of the block, channel l%32.
    auto leave = [&](const SplitTile &d) __attribute__((always_inline)) {
      const bool stats = p.stat_partial && p.g.ksplit == 1;
      const int ch = wm * (MB * 32) + l31;            // this lane's channel of the tile, block 0
      unsigned mask[NB];                              // bit 8q + e: register 4q + e holds a pixel that exists
      bool all = true;
      float cnt = 0.f;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        mask[nb] = valid[nb] >> (4 * lh);
        all = all && valid[nb] == 0xffffffffu;
        cnt += (float)__popc(mask[nb] & 0x0f0f0f0fu);
      }
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        float *const dst = Os + (ch + mb * 32) * OROW + wn * WN + 4 * lh;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            typedef float f4 __attribute__((ext_vector_type(4)));
            const f4 v = {acc[mb][nb][4 * q], acc[mb][nb][4 * q + 1], acc[mb][nb][4 * q + 2], acc[mb][nb][4 * q + 3]};
            *reinterpret_cast<f4 *>(dst + nb * 32 + 8 * q) = v;
          }
        float odd = 0.f;                               // stays zero unless a value is no number, or infinite
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int r = 0; r < 16; ++r) odd = fmaf(acc[mb][nb][r], 0.f, odd);
        if (__any(odd != odd)) {                       // each lane's own values, where a loop can index them: in Os
          const int o = d.mt * BM + ch + mb * 32;
#pragma unroll 1
          for (int i = 0; i < 16 * NB; ++i) {
            const int px = 32 * (i / 16) + 8 * (i / 4 % 4) + i % 4, pn = wn * WN + 4 * lh + px;
            const int r = d.y0 + pn / TW, di = r / p.Ho, x = d.x0 + pn % TW;
            const bool ok = pn / TW < TH && d.n0 + di < p.N && x < p.Wo;        // (else the tile's first pixel, see enter)
            if (dst[px] != dst[px] && o < p.Cout)
              dst[px] = plain_conv_sum(p, o, ok ? d.n0 + di : d.n0, ok ? r - di * p.Ho : d.y0, ok ? x : d.x0, d.kb * 8,
                                       (d.kb + d.nk) * 8 < p.Cin ? (d.kb + d.nk) * 8 : p.Cin);
          }
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mb][nb][r] = dst[nb * 32 + 8 * (r / 4) + r % 4];
        }
        if (stats) {
          // sums about the wave's first pixel (register 0 of the lower half-wave); four chains of each
          const float pv = __shfl(acc[mb][0][0], l31, 64);
          float s1[4] = {0.f, 0.f, 0.f, 0.f}, s2[4] = {0.f, 0.f, 0.f, 0.f};
          if (all) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
              for (int r = 0; r < 16; ++r) {
                const float dv = acc[mb][nb][r] - pv;
                s1[r & 3] += dv;
                s2[r & 3] = fmaf(dv, dv, s2[r & 3]);
              }
          } else {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
              for (int r = 0; r < 16; ++r) {
                const float dv = (mask[nb] >> (8 * (r / 4) + r % 4) & 1u) ? acc[mb][nb][r] - pv : 0.f;
                s1[r & 3] += dv;
                s2[r & 3] = fmaf(dv, dv, s2[r & 3]);
              }
          }
          StatPart sp;
          sp.pivot = pv;
          sp.s1 = (s1[0] + s1[1]) + (s1[2] + s1[3]);
          sp.s2 = (s2[0] + s2[1]) + (s2[2] + s2[3]);
          sp.s1 += __shfl_xor(sp.s1, 32, 64);
          sp.s2 += __shfl_xor(sp.s2, 32, 64);
          sp.n = cnt + __shfl_xor(cnt, 32, 64);
          if (lh == 0) red[wn * BM + ch + mb * 32] = sp;
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[mb][nb][r] = 0.f;
      }
    };
    int mt = 0, mc = 0;
    SplitTile md = uniform_tile(tiles[0]);
    auto tile_weights = [&](int t) __attribute__((always_inline)) {              // byte offset of the first chunk's weights of tile t
      return (unsigned)__builtin_amdgcn_readfirstlane(tiles[t].mt * nchunks + tiles[t].kb) * (unsigned)A_STRIDE;
    };
    unsigned wnow = tile_weights(0), wtile = tile_weights(n_mine > 1 ? 1 : 0);       // this chunk's, the next tile's
    enter(md);
#pragma unroll
    for (int j = 0; j < 5; ++j) load_a(j, 0, wnow);
    __syncthreads();                              // stage 0: the loaders fetch chunk 0
    __syncthreads();                              // stage 1: ... and split it
    auto multiply = [&](auto copy) __attribute__((always_inline)) {              // stage i: multiplies chunk i-2, whose planes are in copy i & 1
      const bool last = mc + 1 == md.nk;
      const unsigned wnext = last ? wtile : wnow + (unsigned)A_STRIDE;
      stage(copy, wnow, wnext);
      wnow = wnext;
      ++mc;
      if (last) {
        leave(md);
        mc = 0;
        if (mt + 1 < n_mine) {
          md = uniform_tile(tiles[++mt]);
          wtile = tile_weights(mt + 1 < n_mine ? mt + 1 : mt);
          enter(md);
        }
      }
      __syncthreads();
    };
    for (int i = 2; i <= TC + 1; i += 2) {
      multiply(std::integral_constant<int, 0>{});
      if (i + 1 <= TC + 1) multiply(std::integral_constant<int, 1>{});
    }
  }
}

}  // namespace pbkd
