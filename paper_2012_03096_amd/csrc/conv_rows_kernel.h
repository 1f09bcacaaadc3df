// Device code of the bf16-split 3x3 convolution for maps of any width and any alignment (arithmetic, pipeline and MFMA
// side: conv_split_kernel.h).  It differs in what a tile is and in how the activations arrive.
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
// multiple of 4).  The channel goes into the scalar offset, so a load costs no vector instruction beyond itself.
// Bound by the MFMA stream and, on tiles of one round, by start-up and stores.  Measured against the fp32-MFMA kernel
// that these maps ran before: 512 -> 512 channels at 14x14, batch 32, 282 -> 134 us (220 TFLOP/s); 67 -> 100 and
// 100 -> 67 at 27x23, batch 77, 169 -> 59 us.
#pragma once
#include "conv_split_kernel.h"

namespace pbkd {

template <int WGM, int MB, int NB, int BSLOTS>
__global__ __launch_bounds__(512) void conv_rows_kernel(ConvArgs p) {
  constexpr int WGN = 4 / WGM;
  constexpr int BM = WGM * MB * 32;     // output channels per workgroup
  constexpr int WN = NB * 32;           // pixels per wave
  constexpr int A_STRIDE = conv_split_a_stride(BM);
  constexpr int NA = A_STRIDE / 4096;
  extern __shared__ float smem[];
  const int PL = p.g.PL + 1;                               // staged positions + one that is never read
  char *const As = reinterpret_cast<char *>(smem);         // [2][A_STRIDE]
  char *const Ss = As + 2 * A_STRIDE;                      // [2][PL][3 pieces][8 bf16]
  StatPart *const red = reinterpret_cast<StatPart *>(Ss + (size_t)2 * 3 * PL * 16);
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

  // After the barrier that follows a tile's end: the WGN MFMA waves' statistics partials (in red), re-expressed about the
  // first one's pivot and added.  The loader waves do it: they have nothing else to do while they wait for their copies.
  auto finish_stats = [&](const SplitTile &d) {
    if (p.stat_partial && p.g.ksplit == 1) {
      for (int e = tid; e < BM; e += 256) {
        const int o = d.mt * BM + e;
        if (o < p.Cout) {
          StatPart a = red[e];
#pragma unroll
          for (int w = 1; w < WGN; ++w) stat_rebase_add(a, red[w * BM + e]);
          stat_store(p.stat_partial, (size_t)o * p.g.n_ptiles + d.pt, a);
        }
      }
    }
  };

  if (loader) {
    // ------------------------------------------------------------------ loader waves: copies, split, and the statistics' last step
    const __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(p.in), 0, (int)((unsigned)p.N * p.Cin * HW * sizeof(float)), 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(p.wpk), 0, (int)((unsigned)p.g.mtiles * nchunks * A_STRIDE), 0x00020000);
    const unsigned aoff = (unsigned)(tid * 16);
    auto copy_a = [&](int mt, int k, int buf) {
      const unsigned wk = (unsigned)(((size_t)mt * nchunks + k) * A_STRIDE);
      char *Ad = As + buf * A_STRIDE + __builtin_amdgcn_readfirstlane(wave) * 1024;
#pragma unroll
      for (int i = 0; i < NA; ++i) load16_to_lds(rw, Ad + i * 4096, aoff, wk + (unsigned)(i * 4096));
    };
    // the staged positions this thread loads and splits: row and column in the tile do not depend on the tile
    int srow[BSLOTS], scol[BSLOTS], loff[BSLOTS];          // row -1: no such position (it works on the spare one)
#pragma unroll
    for (int sl = 0; sl < BSLOTS; ++sl) {
      const int q = tid + 256 * sl;
      const bool in_tile = q < p.g.PLd;
      const int r = q / IW;
      srow[sl] = in_tile ? r : -1;
      scol[sl] = q - r * IW;
      loff[sl] = in_tile ? r * IWS + scol[sl] : PL - 1;
    }
    // where the positions' values are: byte offset in the tensor of channel 0, and whether there is one (halo positions
    // outside the image are zeros: they load the tensor's first value and a select drops it, so every load is in bounds)
    unsigned goff[BSLOTS];
    bool gok[BSLOTS];
    auto enter = [&](const SplitTile &d) {
#pragma unroll
      for (int sl = 0; sl < BSLOTS; ++sl) {
        const int V = d.n0 * SH + d.y0 * s + srow[sl];
        const int n = V / SH, y = V - n * SH - 1, x = d.x0 * s - 1 + scol[sl];
        gok[sl] = srow[sl] >= 0 && n < p.N && y >= 0 && y < p.H && x >= 0 && x < p.W;
        goff[sl] = gok[sl] ? ((unsigned)n * p.Cin * HW + (unsigned)(y * p.W + x)) * 4u : 0u;
      }
    };
    // chunk k's values (a ragged last chunk's missing channels repeat the last one: their weights are zero)
    auto fetch = [&](int k, float (&v)[BSLOTS][8]) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        int c = k * 8 + e;
        if (c > p.Cin - 1) c = p.Cin - 1;
        const unsigned soff = (unsigned)c * (unsigned)HW * 4u;
#pragma unroll
        for (int sl = 0; sl < BSLOTS; ++sl)
          v[sl][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rin, goff[sl], soff, 0));
      }
    };
    const bool bn = (p.in_scale != nullptr);
    const float lo = bn ? 0.f : -__builtin_inff();             // ReLU only where there is a BatchNorm to apply
    // the producing layer's scale and shift for a chunk's channels, through the scalar cache (the constant address
    // space: an earlier kernel wrote them): two loads of eight for a whole chunk instead of sixteen vector loads
    typedef const float __attribute__((address_space(4))) *ConstFloats;
    const ConstFloats cscale = (ConstFloats)(p.in_scale), cshift = (ConstFloats)(p.in_shift);
    float sc[8], sh[8];
    auto fetch_bn = [&](int kc) {
#pragma unroll
      for (int e = 0; e < 8; ++e) sc[e] = 1.f, sh[e] = 0.f;
      if (bn) {
        if (kc * 8 + 8 <= p.Cin) {
          typedef float Floats8 __attribute__((ext_vector_type(8), aligned(4)));
          typedef const Floats8 __attribute__((address_space(4))) *ConstFloats8;
          const Floats8 a = *(ConstFloats8)(cscale + kc * 8), b = *(ConstFloats8)(cshift + kc * 8);
#pragma unroll
          for (int e = 0; e < 8; ++e) sc[e] = a[e], sh[e] = b[e];
        } else {                         // a ragged last chunk: its missing channels take the last one's (their weights are zero)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            int c = kc * 8 + e;
            if (c > p.Cin - 1) c = p.Cin - 1;
            sc[e] = cscale[c], sh[e] = cshift[c];
          }
        }
      }
    };
    auto split = [&](const float (&raw)[BSLOTS][8], const bool (&ok)[BSLOTS], int rc) {
      char *Sd = Ss + (size_t)rc * 3 * PL * 16;
#pragma unroll
      for (int sl = 0; sl < BSLOTS; ++sl) {
        uintx4 pp[3];
#pragma unroll
        for (int t = 0; t < 4; ++t) {              // channels 2t, 2t+1
          const float x0 = ok[sl] ? fmaxf(fmaf(raw[sl][2 * t], sc[2 * t], sh[2 * t]), lo) : 0.f;
          const float x1 = ok[sl] ? fmaxf(fmaf(raw[sl][2 * t + 1], sc[2 * t + 1], sh[2 * t + 1]), lo) : 0.f;
          unsigned q[3];
          split3_bf16(x0, x1, q);
#pragma unroll
          for (int pc = 0; pc < 3; ++pc) pp[pc][t] = q[pc];
        }
#pragma unroll
        for (int pc = 0; pc < 3; ++pc) *reinterpret_cast<uintx4 *>(Sd + loff[sl] * 48 + pc * 16) = pp[pc];
      }
    };
    // Stage i: fetches the activations of chunk i into registers and the weights of chunk i-1 into LDS and, while those
    // are on their way, splits chunk i-1.
    float cur[BSLOTS][8], nxt[BSLOTS][8];
    bool okc[BSLOTS];                   // the positions of the chunk in `cur` that exist
#pragma unroll
    for (int sl = 0; sl < BSLOTS; ++sl) {
      okc[sl] = false;
#pragma unroll
      for (int e = 0; e < 8; ++e) cur[sl][e] = nxt[sl][e] = 0.f;
    }
    int lt = 0, lc = 0, a_mt = 0, a_k = 0;
    SplitTile ld = uniform_tile(tiles[0]);
    enter(ld);
    int ft = 0, fc = 0;                 // the multiplying side's tile and chunk (it is at chunk i-2 in stage i)
    bool pending = false;
    SplitTile fd = ld, pd = ld;
    for (int i = 0; i <= TC + 1; ++i) {
      const bool splits = i >= 1 && i <= TC;
      if (splits) fetch_bn(a_k);
      if (splits) copy_a(a_mt, a_k, (i - 1) & 1);
      if (i < TC) fetch(ld.kb + lc, nxt);
      if (pending) {                    // the tile that ended in the stage before this one
        finish_stats(pd);
        pending = false;
      }
      if (splits) split(cur, okc, (i - 1) & 1);
      if (i >= 2) {
        if (++fc == fd.nk) {
          pd = fd;
          pending = true;
          fc = 0;
          if (ft + 1 < n_mine) fd = uniform_tile(tiles[++ft]);
        }
      }
      a_mt = ld.mt;
      a_k = ld.kb + lc;
#pragma unroll
      for (int sl = 0; sl < BSLOTS; ++sl) okc[sl] = gok[sl];
      if (i + 1 < TC) {
        if (++lc == ld.nk) {
          lc = 0;
          ld = uniform_tile(tiles[++lt]);
          enter(ld);
        }
      }
      __syncthreads();
#pragma unroll
      for (int sl = 0; sl < BSLOTS; ++sl)
#pragma unroll
        for (int e = 0; e < 8; ++e) cur[sl][e] = nxt[sl][e];
    }
    if (pending) finish_stats(pd);
  } else {
    // ------------------------------------------------------------------ MFMA waves
    sfloatx16 acc[MB][NB];
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
    // this lane's pixel columns: row and column in the tile, and (per tile) their place in the staged tile and the output
    int prow[NB], pcol[NB], pixoff[NB], py[NB], pimg[NB];
    bool pvalid[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int pn = wn * WN + nb * 32 + l31;
      prow[nb] = pn / TW;
      pcol[nb] = pn - prow[nb] * TW;
    }
    auto enter = [&](const SplitTile &d) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int r = d.y0 + prow[nb], di = r / p.Ho, y = r - di * p.Ho;
        pimg[nb] = d.n0 + di;
        py[nb] = y;
        pvalid[nb] = prow[nb] < TH && pimg[nb] < p.N && d.x0 + pcol[nb] < p.Wo;
        // (a column without a pixel repeats the tile's first one: the statistics' pivot is always a value of the tile)
        pixoff[nb] = pvalid[nb] ? (di * SH + s * (y - d.y0)) * IWS + s * pcol[nb] : 0;
      }
    };
    // tap 2j+h of this half-wave as an offset in the staged tile (in the last step both half-waves read tap 8)
    int toff[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      const int tap = (2 * j + lh < 9) ? 2 * j + lh : 8;
      toff[j] = (tap / 3) * IWS + (tap % 3);
    }
    const int arow = (wm * (MB * 32) + l31) * 16;      // byte offset of this lane's weight row within a [BM][8] slab

    // One pipeline stage of the MFMA waves: multiplies the chunk whose weights and bf16 planes are in copy mc.
    //
    // The six products of a tap pair run in the order (weight piece, activation piece) = 10 11 20 00 01 02.  Every
    // operand piece then falls free at least two products (eight MFMAs) before the next tap pair needs it again, so
    // the next tap pair's pieces are fetched into the same registers: no second set of operand registers.  The ninth
    // tap's three products (operand slot c with operand slot c) follow in the order 1 0 2, the order their operands
    // arrive in.  The fences keep the compiler from moving the LDS reads down to their first use.
    auto stage = [&](int mc) {
      const char *Ab = As + mc * A_STRIDE + arow;
      const char *Sb = Ss + (size_t)mc * 3 * PL * 16;
      auto lda = [&](int pc, int j, int mb) {
        return *reinterpret_cast<const uintx4 *>(Ab + ((pc * 5 + j) * 2 + lh) * (BM * 16) + mb * 512);
      };
      auto ldb = [&](int pc, int j, int nb) {
        // operand slot pc is piece pc, but for the ninth tap, where the half-waves read two different pieces of it
        const int piece = j < 4 ? pc : kSplitLastX[pc][0] + lh * (kSplitLastX[pc][1] - kSplitLastX[pc][0]);
        return *reinterpret_cast<const uintx4 *>(Sb + (pixoff[nb] + toff[j]) * 48 + piece * 16);
      };
      uintx4 av[3][MB], bv[3][NB];
      auto fill_a = [&](int pc, int j) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) av[pc][mb] = lda(pc, j, mb);
      };
      auto fill_b = [&](int pc, int j) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) bv[pc][nb] = ldb(pc, j, nb);
      };
      // tap pair 0, in the order of first use
      fill_a(1, 0); fill_b(0, 0); fill_b(1, 0); fill_a(2, 0); fill_a(0, 0); fill_b(2, 0);
#pragma unroll
      for (int j = 0; j < 5; ++j) {
        __builtin_amdgcn_sched_barrier(0);
        constexpr int PA[6] = {1, 1, 2, 0, 0, 0}, PB[6] = {0, 1, 0, 0, 1, 2}, PL4[3] = {1, 0, 2};
#pragma unroll
        for (int q = 0; q < (j < 4 ? 6 : 3); ++q) {
          const int qa = j < 4 ? PA[q] : PL4[q], qb = j < 4 ? PB[q] : PL4[q];
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
              acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av[qa][mb]),
                                                                    __builtin_bit_cast(bf16x8, bv[qb][nb]), acc[mb][nb], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          if (j + 1 < 5) {          // the next tap pair's pieces, into the registers that have just fallen free
            if (q == 1) fill_a(1, j + 1);
            if (q == 2) fill_a(2, j + 1);
            if (q == 3) fill_b(0, j + 1);
            if (q == 4) fill_b(1, j + 1);
            if (q == 5) { fill_a(0, j + 1); fill_b(2, j + 1); }
          }
        }
      }
    };
    // the multiplying side leaves a tile (conv_split_kernel.h)
    const __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc(
        p.g.ksplit > 1 ? p.split_out : p.out, 0, (int)((unsigned)p.g.ksplit * p.N * p.Cout * HWo * sizeof(float)), 0x00020000);
    auto leave = [&](const SplitTile &d) {
      const int m0 = d.mt * BM + wm * (MB * 32);      // first channel of this wave
      unsigned voff[NB];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        voff[nb] = (unsigned)(((d.kz * p.N + pimg[nb]) * p.Cout + 4 * lh) * HWo + py[nb] * p.Wo + d.x0 + pcol[nb]) * 4u;
      // per-channel statistics partial of this pixel tile (as in the fp32-MFMA kernel): every wave sums about the value
      // of its own first pixel column
      // (all of it on the vector ALU: the pivot through two lane reads, the half-wave sums through DPP with the
      // total arriving in the half-wave's upper 16 lanes; LDS permutes would make 64 dependent round trips of it)
      if (p.stat_partial && p.g.ksplit == 1) {
        float cnt = 0.f;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) cnt += pvalid[nb] ? 1.f : 0.f;
        cnt = half32_sum_upper(cnt);
        StatPart *const rw = red + wn * BM + wm * (MB * 32) + 4 * lh;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float a0 = acc[mb][0][r];
            const float p0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, a0), 0));
            const float p1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, a0), 32));
            const float pv = lh ? p1 : p0;
            float s1 = 0.f, s2 = 0.f;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
              const float dv = pvalid[nb] ? acc[mb][nb][r] - pv : 0.f;
              s1 += dv;
              s2 += dv * dv;
            }
            s1 = half32_sum_upper(s1);
            s2 = half32_sum_upper(s2);
            if (l31 == 16) {
              StatPart sp;
              sp.pivot = pv; sp.s1 = s1; sp.s2 = s2; sp.n = cnt;
              rw[mb * 32 + 8 * (r / 4) + (r % 4)] = sp;
            }
          }
      }
      const bool whole8 = (p.Cout & 7) == 0;          // then the eight channels of an accumulator row group exist or do not together
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int ou = m0 + mb * 32 + 8 * (r / 4) + (r % 4);     // wave-uniform part of the channel
          const unsigned soff = (unsigned)ou * (unsigned)HWo * 4u;
          const bool ch_ok = whole8 ? (ou < p.Cout) : (ou + 4 * lh < p.Cout);
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) {
            const float v = acc[mb][nb][r];       // (a bit cast applied to the vector element itself reads element 0)
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rout,
                                                  (pvalid[nb] && ch_ok) ? voff[nb] + soff : kPastBuffer, 0, 0);
          }
        }
#pragma unroll
      for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
    };
    int mt = 0, mc = 0;
    SplitTile md = uniform_tile(tiles[0]);
    enter(md);
    __syncthreads();                              // stage 0: the loaders fetch chunk 0
    __syncthreads();                              // stage 1: ... and split it
    for (int i = 2; i <= TC + 1; ++i) {           // stage i: multiplies chunk i-2
      stage(i & 1);
      if (++mc == md.nk) {
        leave(md);
        mc = 0;
        if (mt + 1 < n_mine) {
          md = uniform_tile(tiles[++mt]);
          enter(md);
        }
      }
      __syncthreads();
    }
  }
}

}  // namespace pbkd
