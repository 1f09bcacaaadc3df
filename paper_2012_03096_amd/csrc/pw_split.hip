// 1x1 convolution (the student's pointwise conv, its data gradient, the projection shortcut) with its fp32 products
// formed on the bf16 matrix cores from operands split three ways (split_bf16.h; the arithmetic and its error bound:
// conv_split_kernel.h).  z[n,o,p] = sum_c A[o,c] * in[n,c,p].
//
// An fp32 product costs six bf16 ones, 192 cycles of a SIMD per 32 x 32 outputs and 16 channels against 512 on the fp32
// matrix cores, and the kernels that did it there were bound by exactly that wherever there are 128 channels or more.
//
// Weights come pre-split (by the host at upload, by the update kernel after every step) in operand order: per (32 output
// channels, chunk of 16 input channels, piece) one kilobyte, lane l's 16 bytes being row l%32, channels 8*(l/32) .. +7.
// Activations go from memory straight into registers: lane (l%32, h = l/32) owns VW adjacent pixels and loads the eight
// channels 8h..8h+7 of a chunk for them, which after the split ARE the MFMA operand of those pixels: no LDS, no
// transposition.  MFMA e of the VW takes element e, so its column n is pixel VW*n + e.
//
// Infinities, and numbers past bfloat16's largest (3.39e38): the difference from the first piece is then no number, so every
// sum that holds such an operand comes out as a NaN.  Sums that are NaN are formed again in fp32 from the operands
// themselves (plain_sum), which makes of them what fp32 products make: an infinity, a number, or a NaN.
//
// Cin not a multiple of 16: the last chunk starts at channel Cin-16 and the weights of the channels it shares with the
// one before are zero there, so that every load is of a real channel.
#include "conv_mfma_kernel.h"
#include "split_bf16.h"

namespace pbkd {

namespace {
// chunks of weights per LDS stage of pw_split_kernel: 48 KB for 64 channels, three workgroups per compute unit
constexpr int kStage = 8;

template <int VW> struct PixVec;
template <> struct PixVec<1> {
  typedef float type;
  static __device__ __forceinline__ float load(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
  }
  static __device__ __forceinline__ float get(float v, int) { return v; }
  static __device__ __forceinline__ float make(const float *v) { return v[0]; }
  static __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t r, float v, unsigned voff, unsigned soff) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, voff, soff, 0);
  }
};
template <> struct PixVec<2> {
  typedef floatx2 type;
  static __device__ __forceinline__ floatx2 load(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    return __builtin_bit_cast(floatx2, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
  }
  static __device__ __forceinline__ float get(floatx2 v, int e) { return v[e]; }
  static __device__ __forceinline__ floatx2 make(const float *v) { return floatx2{v[0], v[1]}; }
  static __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t r, floatx2 v, unsigned voff, unsigned soff) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uintx2, v), r, voff, soff, 0);
  }
};
template <> struct PixVec<4> {
  typedef float type __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    return __builtin_bit_cast(type, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
  }
  static __device__ __forceinline__ float get(type v, int e) { return v[e]; }
  static __device__ __forceinline__ type make(const float *v) { return type{v[0], v[1], v[2], v[3]}; }
  static __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t r, type v, unsigned voff, unsigned soff) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uintx4, v), r, voff, soff, 0);
  }
};

// byte offset of channel 0 of the VW pixels from pixel g on in the input (P % VW == 0: they exist together; pixels past the
// last read the last ones, and are never stored)
template <int VW>
__device__ __forceinline__ unsigned input_offset(const PwArgs &p, long long g) {
  const int HWo = p.Ho * p.Wo;
  const long long P = (long long)p.N * HWo;
  if (g >= P) g = P - VW;
  const int n = (int)((unsigned)g / (unsigned)HWo), r = (int)((unsigned)g - (unsigned)n * (unsigned)HWo);   // P < 2^31
  int pix = r;
  if (VW == 1 && p.stride != 1) {
    const int i = r / p.Wo, j = r - i * p.Wo;
    pix = p.stride * (i * p.Win + j);
  }
  return ((unsigned)n * (unsigned)p.Cin * (unsigned)p.HWin + (unsigned)pix) * 4u;
}
// the same in the output; kPastBuffer for pixels that do not exist
template <int SV>
__device__ __forceinline__ unsigned output_offset(const PwArgs &p, long long g) {
  const int HWo = p.Ho * p.Wo;
  if (g >= (long long)p.N * HWo) return kPastBuffer;
  const int n = (int)((unsigned)g / (unsigned)HWo), r = (int)((unsigned)g - (unsigned)n * (unsigned)HWo);
  return ((unsigned)n * (unsigned)p.Cout * (unsigned)HWo + (unsigned)r) * 4u;
}

// the eight channels of a chunk for one of the lane's pixels -> the three operand pieces
template <int VW>
__device__ __forceinline__ void split_operand(const typename PixVec<VW>::type (&x)[8], int e, uintx4 (&b)[3]) {
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    unsigned q[3];
    split3_bf16(PixVec<VW>::get(x[2 * t], e), PixVec<VW>::get(x[2 * t + 1], e), q);
#pragma unroll
    for (int pc = 0; pc < 3; ++pc) b[pc][t] = q[pc];
  }
}

// the six products (activation piece, weight piece) = 20 10 11 02 01 00 of MB blocks of 32 channels, small ones first: what
// they round away is then below the last one's rounding.  Activations are the A operand: an accumulator's rows are pixels and its columns channels, so a lane holds pixels of ONE channel and takes
// its statistics without leaving its registers.
template <int MB>
__device__ __forceinline__ void six_products(const uintx4 (&w)[MB][3], const uintx4 (&x)[3], floatx16 (&acc)[MB]) {
  constexpr int PW[6] = {0, 0, 1, 2, 1, 0}, PX[6] = {2, 1, 1, 0, 0, 0};
#pragma unroll
  for (int q = 0; q < 6; ++q)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
      acc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x[PX[q]]), __builtin_bit_cast(bf16x8, w[mb][PW[q]]),
                                                        acc[mb], 0, 0, 0);
}

// One block of 32 channels as accumulated (register r of lane l: pixel row 8*(r/4) + 4*(l/32) + r%4, channel l%32; MFMA e
// of the VW holds pixels VW*row + e) -> LDS as [channel][32*VW pixels + 4].  The row length keeps 16-byte accesses of
// neighbouring channels in different banks.
template <int VW>
constexpr int kTileRow = 32 * VW + 4;
template <int VW, int MB>
__device__ __forceinline__ void transpose_to_lds(const floatx16 (&acc)[VW][MB], int mb, float *T, int l31, int lh) {
  typedef float f4 __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float v[4 * VW];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int e = 0; e < VW; ++e) v[r * VW + e] = acc[e][mb][4 * q + r];
    f4 *dst = reinterpret_cast<f4 *>(T + l31 * kTileRow<VW> + (8 * q + 4 * lh) * VW);
#pragma unroll
    for (int j = 0; j < VW; ++j) {
      const f4 t = {v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3]};
      dst[j] = t;
    }
  }
}

// one output value in fp32 multiply-adds (g: its pixel, of which there is one)
__device__ __forceinline__ float plain_sum(const PwArgs &p, int o, long long g) {
  const int HWo = p.Ho * p.Wo;
  const int n = (int)((unsigned)g / (unsigned)HWo), r = (int)((unsigned)g - (unsigned)n * (unsigned)HWo);
  const int i = r / p.Wo, j = r - i * p.Wo;
  const float *x = p.in + (size_t)n * p.Cin * p.HWin + (p.stride == 1 ? r : p.stride * (i * p.Win + j));
  const float *w = p.w + (size_t)o * p.w_row;
  float s = 0.f;
#pragma unroll 1
  for (int k = 0; k < p.Cin && s == s; ++k) s = fmaf(w[(size_t)k * p.w_col], x[(size_t)k * p.HWin], s);
  return s;
}

// sum over a group of GPR = 8 or 32 neighbouring lanes
template <int GPR>
__device__ __forceinline__ float group_sum(float v) {
  if (GPR == 32) return half32_sum(v);
  v += dpp_mov<0xB1>(v);
  v += dpp_mov<0x4E>(v);
  return v + dpp_mov<0x141>(v);
}
}  // namespace

// ---- many pixels: a workgroup owns 32*MB channels x 4 waves x 32*VW pixels.  The weights of up to kStage chunks are staged
// in LDS at a time; each wave then runs on its own, its activations two chunks ahead of the multiplication, the split of
// the next operand between the MFMAs of the current one.
// With one pixel per lane a stage's chunks (128 channels) are summed from zero and added to the running sum: long sums over few
// pixels were split four ways on the fp32 matrix cores, and one running sum leaves more error than that (rms against fp64
// at 433 -> 169 channels, 41x48, batch 7: 1.9e-7 then, 3.3e-7 with one sum, 1.7e-7 so; a sum every 32 channels 1.1e-7 but
// 28 us for 23).  One block of 32 channels, where sums from 128 channels on were split, can afford a sum every 32 channels
// (128 -> 24 at 32x34, batch 32: 1.2e-7 then, 1.7e-7 with one sum, 0.9e-7 so).  With two pixels a lane (many pixels: no sum was split) one running sum rounds 6 times per 16
// channels, fp32 multiply-adds 16 times.
template <int MB, int VW, int SV>
__global__ __launch_bounds__(256) void pw_split_kernel(PwArgs p) {
  constexpr int D = 2;                         // chunks of activations in flight
  constexpr int ST = kStage;
  typedef typename PixVec<VW>::type vec_t;
  extern __shared__ float smem[];
  StatPart *const red = reinterpret_cast<StatPart *>(smem);               // [4 waves][32*MB]
  char *const Ws = reinterpret_cast<char *>(red + 4 * 32 * MB);           // [MB][ST][3][1024]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l31 = lane & 31, lh = lane >> 5;
  // workgroup -> (pixel tile bxl, channel tile byl): the channel tiles of one pixel tile read the same activations, so
  // they are made neighbours on one die (channel tile fastest, a contiguous range of pixel tiles per die)
  const int lin = xcd_contiguous(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
  const int byl = lin % gridDim.y, bxl = lin / gridDim.y;
  const int HWo = p.Ho * p.Wo;
  const long long P = (long long)p.N * HWo;
  const int nch = p.nchunks;
  const long long g0 = ((long long)bxl * 4 + wave) * (32 * VW);           // this wave's first pixel

  const __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float *>(p.in), 0, (int)((unsigned)p.N * p.Cin * p.HWin * sizeof(float)), 0x00020000);
  const unsigned rowb = (unsigned)p.HWin * 4u;
  const unsigned voff = input_offset<VW>(p, g0 + VW * l31) + (unsigned)(8 * lh) * rowb;
  auto fetch = [&](int ch, vec_t (&x)[8]) {
    int k0 = ch * 16;
    if (k0 > p.Cin - 16) k0 = p.Cin - 16;      // the ragged last chunk; past the end: a real chunk, never multiplied
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = PixVec<VW>::load(rin, voff, (unsigned)(k0 + j) * rowb);
  };
  // weights: memory -> LDS directly, a kilobyte (one block of 32 channels, chunk and piece) per wave and instruction
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float *>(p.wpk), 0, (int)((unsigned)p.g.mtiles * MB * nch * 3072u), 0x00020000);
  auto stage_weights = [&](int s0, int ns) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const unsigned src = (unsigned)((byl * MB + mb) * nch + s0) * 3072u;
      char *dst = Ws + mb * (ST * 3072);
      for (int u = wave; u < ns * 3; u += 4) load16_to_lds(rw, dst + u * 1024, (unsigned)lane * 16u, src + (unsigned)u * 1024u);
    }
  };

  floatx16 acc[VW][MB];
#pragma unroll
  for (int e = 0; e < VW; ++e)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[e][mb][r] = 0.f;

  floatx16 sum[MB];                            // VW == 1: of this stage's chunks (MB == 1: of two chunks)
  auto clear_sum = [&]() {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) sum[mb][r] = 0.f;
  };
  auto add_sum = [&]() {
    if constexpr (VW == 1) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) acc[0][mb] += sum[mb];
      clear_sum();
    }
  };
  clear_sum();
  vec_t ring[D][8];
  uintx4 x[3];                                 // the operand multiplied next
  stage_weights(0, nch < ST ? nch : ST);       // ahead of the activations: loads complete in order
  fetch(0, ring[0]);
  fetch(1, ring[1]);
  auto weights = [&](int c, uintx4 (&w)[MB][3]) {
    const uintx4 *Wl = reinterpret_cast<const uintx4 *>(Ws + c * 3072) + lane;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int pc = 0; pc < 3; ++pc) w[mb][pc] = Wl[mb * (ST * 192) + pc * 64];
  };
  // multiplies the chunk in ring[d] (chunk ch overall, weights w) and fetches chunk ch + D into its place
  auto chunk = [&](int d, int ch, const uintx4 (&w)[MB][3]) {
#pragma unroll
    for (int e = 0; e < VW; ++e) {
      uintx4 nx[3];
      if (e + 1 < VW) split_operand<VW>(ring[d], e + 1, nx);
      else split_operand<VW>(ring[d ^ 1], 0, nx);
      if (e == (VW > 1 ? VW - 2 : 0)) fetch(ch + D, ring[d]);   // (its last pixel has just been split; with VW = 1 a chunk ago)
      six_products<MB>(w, x, VW == 1 ? sum : acc[e]);
#pragma unroll
      for (int q = 0; q < 6 * MB; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x002, 48 / (6 * MB), 0);    // and a share of the next operand's split
      }
#pragma unroll
      for (int pc = 0; pc < 3; ++pc) x[pc] = nx[pc];
    }
  };

  for (int s0 = 0; s0 < nch; s0 += ST) {
    const int ns = nch - s0 < ST ? nch - s0 : ST;
    if (s0 > 0) {
      __syncthreads();
      stage_weights(s0, ns);
    }
    __syncthreads();
    if (s0 == 0) split_operand<VW>(ring[0], 0, x);
    int c = 0;
    for (; c + 1 < ns; c += 2) {
      uintx4 w0[MB][3], w1[MB][3];
      weights(c, w0);
      weights(c + 1, w1);
      chunk(0, s0 + c, w0);
      chunk(1, s0 + c + 1, w1);
      if (MB == 1) add_sum();
    }
    if (c < ns) {                              // an odd number of chunks: only in the last stage
      uintx4 w0[MB][3];
      weights(c, w0);
      chunk(0, s0 + c, w0);
    }
    add_sum();
  }

  __syncthreads();                             // nobody reads the weights any more
  float *const T = reinterpret_cast<float *>(Ws) + wave * (32 * kTileRow<VW>);      // this wave's part of LDS from here on
  const int m0 = byl * (32 * MB);

  // ---- per-channel statistics partial over this wave's pixels: each lane sums about the first of its own values, the two
  // lanes of a channel and then the four waves are re-expressed about one pivot and added
  const bool whole = g0 + 32 * VW <= P;        // wave-uniform: every pixel of the wave exists
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    float odd = 0.f;                           // stays zero unless a value is no number, or infinite
#pragma unroll
    for (int e = 0; e < VW; ++e)
#pragma unroll
      for (int r = 0; r < 16; ++r) odd = fmaf(acc[e][mb][r], 0.f, odd);
    if (__any(odd != odd)) {
      // each lane's own values through LDS, where a loop can index them
      transpose_to_lds<VW, MB>(acc, mb, T, l31, lh);
      float *const own = T + l31 * kTileRow<VW> + 4 * VW * lh;
#pragma unroll 1
      for (int i = 0; i < 16 * VW; ++i) {
        const int px = 8 * VW * (i / (4 * VW)) + i % (4 * VW);
        const long long g = g0 + 4 * VW * lh + px;
        if (own[px] != own[px] && m0 + mb * 32 + l31 < p.Cout) own[px] = plain_sum(p, m0 + mb * 32 + l31, g < P ? g : P - 1);
      }
#pragma unroll
      for (int e = 0; e < VW; ++e)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[e][mb][r] = own[(8 * (r / 4) + r % 4) * VW + e];
    }
    if (p.stat_partial) {
      StatPart a;
      a.pivot = acc[0][mb][0];
      a.s1 = a.s2 = 0.f;
      a.n = 16.f * VW;
      if (whole) {
#pragma unroll
        for (int e = 0; e < VW; ++e)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float d = acc[e][mb][r] - a.pivot;
            a.s1 += d;
            a.s2 = fmaf(d, d, a.s2);
          }
      } else {
        const long long left = P - g0 - 4 * VW * lh;
        a.n = 0.f;
#pragma unroll
        for (int e = 0; e < VW; ++e)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const bool ok = VW * (8 * (r / 4) + r % 4) + e < left;
            const float d = ok ? acc[e][mb][r] - a.pivot : 0.f;
            a.s1 += d;
            a.s2 = fmaf(d, d, a.s2);
            a.n += ok ? 1.f : 0.f;
          }
      }
      StatPart b;
      b.pivot = __shfl_xor(a.pivot, 32, 64);
      b.s1 = __shfl_xor(a.s1, 32, 64);
      b.s2 = __shfl_xor(a.s2, 32, 64);
      b.n = __shfl_xor(a.n, 32, 64);
      stat_rebase_add(a, b);
      if (lh == 0) red[wave * (32 * MB) + mb * 32 + l31] = a;
    }
  }

  // ---- stores: each block of 32 channels through LDS (every wave in a part of its own) and out along the pixels, SV
  // pixels = 4*SV bytes a lane, through a buffer descriptor: what does not exist gets an offset past the buffer
  constexpr int GPR = 32 * VW / SV, RPI = 64 / GPR;       // lanes per row of pixels, rows per instruction
  const __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc(
      p.out, 0, (int)((unsigned)p.N * p.Cout * HWo * sizeof(float)), 0x00020000);
  const unsigned orow = (unsigned)HWo * 4u;
  const int grp = lane % GPR, row0 = lane / GPR;
  const unsigned ooff = output_offset<SV>(p, g0 + grp * SV);
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    transpose_to_lds<VW, MB>(acc, mb, T, l31, lh);
#pragma unroll
    for (int i = 0; i < 32 / RPI; ++i) {
      const int row = i * RPI + row0, o = m0 + mb * 32 + row;
      const typename PixVec<SV>::type v = *reinterpret_cast<const typename PixVec<SV>::type *>(T + row * kTileRow<VW> + grp * SV);
      PixVec<SV>::store(rout, v, (o < p.Cout && ooff != kPastBuffer) ? ooff + (unsigned)o * orow : kPastBuffer - 15u, 0);
    }
  }
  if (p.stat_partial) {
    __syncthreads();                           // the four waves' partials are there
    for (int i = tid; i < 32 * MB; i += 256) {
      const int o = m0 + i;
      if (o < p.Cout) {
        StatPart a = red[i];
#pragma unroll
        for (int w = 1; w < 4; ++w) stat_rebase_add(a, red[w * (32 * MB) + i]);
        stat_store(p.stat_partial, (size_t)o * gridDim.x + bxl, a);
      }
    }
  }
}

// ---- few pixels, many channels: a workgroup owns 32*MB channels x 32*VW pixels and its four waves take a quarter of the
// chunks each, weights and activations both straight from memory into registers (each is used by one wave only), two
// chunks ahead; the four partial tiles meet in LDS and are added in wave order.
template <int MB, int VW, int SV>
__global__ __launch_bounds__(256) void pw_split_kwaves_kernel(PwArgs p) {
  constexpr int D = 2;
  typedef typename PixVec<VW>::type vec_t;
  extern __shared__ float smem[];              // [4 waves][32*MB channels][kTileRow<VW>]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l31 = lane & 31, lh = lane >> 5;
  const int lin = xcd_contiguous(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
  const int byl = lin % gridDim.y, bxl = lin / gridDim.y;
  const int HWo = p.Ho * p.Wo;
  const long long P = (long long)p.N * HWo;
  const int nch = p.nchunks;
  const int per_wave = (nch + 3) / 4;
  const int c_begin = wave * per_wave;
  const int c_end = c_begin + per_wave < nch ? c_begin + per_wave : nch;
  const long long g0 = (long long)bxl * (32 * VW);

  const __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float *>(p.in), 0, (int)((unsigned)p.N * p.Cin * p.HWin * sizeof(float)), 0x00020000);
  const unsigned rowb = (unsigned)p.HWin * 4u;
  const unsigned voff = input_offset<VW>(p, g0 + VW * l31) + (unsigned)(8 * lh) * rowb;
  const uintx4 *const wsrc = reinterpret_cast<const uintx4 *>(p.wpk) + (size_t)byl * MB * nch * 192 + lane;
  auto fetch = [&](int ch, vec_t (&x)[8], uintx4 (&a)[MB][3]) {
    if (ch > nch - 1) ch = nch - 1;            // past the end: a real chunk, never multiplied
    int k0 = ch * 16;
    if (k0 > p.Cin - 16) k0 = p.Cin - 16;
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = PixVec<VW>::load(rin, voff, (unsigned)(k0 + j) * rowb);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int pc = 0; pc < 3; ++pc) a[mb][pc] = wsrc[((size_t)mb * nch + ch) * 192 + pc * 64];
  };

  floatx16 acc[VW][MB];
#pragma unroll
  for (int e = 0; e < VW; ++e)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[e][mb][r] = 0.f;

  vec_t rx[D][8];
  uintx4 ra[D][MB][3];
  fetch(c_begin, rx[0], ra[0]);
  fetch(c_begin + 1, rx[1], ra[1]);
  auto chunk = [&](int d, int ch) {
    uintx4 b[VW][3], a[MB][3];
#pragma unroll
    for (int e = 0; e < VW; ++e) split_operand<VW>(rx[d], e, b[e]);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int pc = 0; pc < 3; ++pc) a[mb][pc] = ra[d][mb][pc];
    fetch(ch + D, rx[d], ra[d]);
#pragma unroll
    for (int e = 0; e < VW; ++e) six_products<MB>(a, b[e], acc[e]);
  };
  int c = c_begin;
  for (; c + 1 < c_end; c += 2) {
    chunk(0, c);
    chunk(1, c + 1);
  }
  if (c < c_end) chunk(0, c);

#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
    transpose_to_lds<VW, MB>(acc, mb, smem + (wave * MB + mb) * (32 * kTileRow<VW>), l31, lh);
  __syncthreads();
  typedef typename PixVec<SV>::type svec_t;
  constexpr int GPR = 32 * VW / SV, RPI = 64 / GPR, RWV = 8 * MB;         // RWV: channel rows this wave finishes
  static_assert(RWV % RPI == 0, "whole instructions");
  const __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc(
      p.out, 0, (int)((unsigned)p.N * p.Cout * HWo * sizeof(float)), 0x00020000);
  const unsigned orow = (unsigned)HWo * 4u;
  const int grp = lane % GPR, row0 = lane / GPR;
  const unsigned ooff = output_offset<SV>(p, g0 + grp * SV);
  const bool valid = ooff != kPastBuffer;
  const float cnt = (float)(P - g0 < 32 * VW ? P - g0 : 32 * VW);
#pragma unroll
  for (int i = 0; i < RWV / RPI; ++i) {
    const int row = wave * RWV + i * RPI + row0, o = byl * (32 * MB) + row;
    float v[SV];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const svec_t t = *reinterpret_cast<const svec_t *>(smem + (w * 32 * MB + row) * kTileRow<VW> + grp * SV);
#pragma unroll
      for (int e = 0; e < SV; ++e) v[e] = w == 0 ? PixVec<SV>::get(t, e) : v[e] + PixVec<SV>::get(t, e);
    }
    bool number = true;
#pragma unroll
    for (int e = 0; e < SV; ++e) number = number && v[e] == v[e];
    if (!number && valid && o < p.Cout) {
#pragma unroll
      for (int e = 0; e < SV; ++e)
        if (v[e] != v[e]) v[e] = plain_sum(p, o, g0 + grp * SV + e);
    }
    PixVec<SV>::store(rout, PixVec<SV>::make(v), (valid && o < p.Cout) ? ooff + (unsigned)o * orow : kPastBuffer - 15u, 0);
    if (p.stat_partial) {                      // this wave holds the whole tile's pixels of the row, about its first
      StatPart a;
      a.pivot = __shfl(v[0], lane & ~(GPR - 1), 64);
      float s1 = 0.f, s2 = 0.f;
#pragma unroll
      for (int e = 0; e < SV; ++e) {
        const float d = valid ? v[e] - a.pivot : 0.f;
        s1 += d;
        s2 = fmaf(d, d, s2);
      }
      a.s1 = group_sum<GPR>(s1);
      a.s2 = group_sum<GPR>(s2);
      a.n = cnt;
      if (grp == 0 && o < p.Cout) stat_store(p.stat_partial, (size_t)o * gridDim.x + bxl, a);
    }
  }
}

// Variants kPwSplitFirst + i: i = 0..3 pw_split_kernel<MB, VW>, 4 and 5 pw_split_kwaves_kernel<MB, VW>
static const int kMB[6] = {2, 1, 2, 1, 2, 1}, kVW[6] = {1, 1, 2, 2, 1, 1};

bool pw_split_ok(int N, int Cin, int Cout, int HWin, int Ho, int Wo) {
  return Cin >= 16 && (unsigned long long)N * Cin * HWin * sizeof(float) < (1ull << 32) &&
         (unsigned long long)N * Cout * Ho * Wo * sizeof(float) < (1ull << 32) - 64 &&
         (unsigned long long)cdiv(Cout, 128) * 128 * cdiv(Cin, 16) * 16 * 6 < (1ull << 32);       // (weights, padded to the largest tile)
}

// Which tile.  Measured on MI355X (us, forward with statistics / data gradient, kernel events, which read about 3 us high;
// the first figure is the fp32 kernel this replaced):
//   64 -> 64, 224x224 x 32:    197/173    64 ch x 4 x 32 px 185/157    64 ch x 4 x 64 px 173/154
//   256 -> 256, 56x56 x 32:    168/157                       97/86                        91/81
//   64 -> 64, 32x32 x 128:     22.1/20.7                     19.0/16.1                    20.2/16.9
//   128 -> 128, 16x16 x 128:   22.1/20.2                     16.0/14.1                    15.8/14.5
//   512 -> 512, 14x14 x 32:    55.6/53.1                     30.8/29.1                    32.2/30.5
//   67 -> 100, 27x23 x 77:     28.6/27.0                     15.7/15.3
//   128 -> 256, 8x8 x 128:     16.4/13.4                     11.7/12.2    K over the waves, 64 ch x 32 px 12.4/10.0
//   512 -> 512, 4x4 x 128:     21.5/20.5                     21.8/20.7    14.2/13.3
//   512 -> 512, 2x2 x 128:     12.6/10.8                     23.1/20.7    11.2/10.7    32 ch x 32 px 9.9/9.4
// So: 64 x 4*64 pixels where that is four workgroups or more per compute unit (its wider rows reach HBM's rate), else
// 64 x 4*32 while every compute unit gets one (of 128 x 64 too: where it does not, sums from 128 channels on have always been
// in four parts), else K over the waves.  32 channels where there are no more of them (median of
// both directions from a kernel trace; fp32 kernel, 64 ch x 4 x 64 px, 32 ch x 4 x 64 px, 32 ch x 4 x 32 px):
//   16 -> 16, 112x112 x 32:    16.8   19.2   13.1   15.0
//   32 -> 32, 112x112 x 32:    24.0   26.2   20.1   21.5
//   32 -> 32, 32x32 x 128:      9.9           9.2    8.6
int pw_split_choice(long long P, int Cout, int HW, int stride) {
  auto wgs = [&](int i) {
    const long long px = (i < 4 ? 4ll : 1ll) * 32 * kVW[i];
    return (long long)cdiv(Cout, 32 * kMB[i]) * ((P + px - 1) / px);
  };
  if (wgs(2) >= 1024 && pw_split_fits(2, HW, stride)) return Cout > 32 ? 2 : 3;
  if (wgs(0) >= 256 && cdiv(Cout, 128) * ((P + 63) / 64) >= 256) return Cout > 32 ? 0 : 1;
  return Cout > 32 && wgs(4) >= 256 ? 4 : 5;
}

PwGeom pw_split_geom(int i, int N, int Cin, int Cout, int Ho, int Wo) {
  PwGeom g{};
  const long long P = (long long)N * Ho * Wo;
  g.variant = kPwSplitFirst + i;
  g.split = 1;
  g.K = Cin;
  g.bm = 32 * kMB[i];
  g.mtiles = cdiv(Cout, g.bm);
  g.nchunks = cdiv(Cin, 16);
  const long long px = (i < 4 ? 4ll : 1ll) * 32 * kVW[i];
  g.n_ptiles = (int)((P + px - 1) / px);
  const size_t tile = (size_t)4 * 32 * (32 * kVW[i] + 4) * sizeof(float);   // one block of 32 channels of each of four waves
  const size_t weights = (size_t)kMB[i] * kStage * 3072;
  g.lds_bytes = i < 4 ? (size_t)4 * g.bm * sizeof(StatPart) + (weights > tile ? weights : tile) : kMB[i] * tile;
  return g;
}

bool pw_split_fits(int i, int HW, int stride) { return i >= 0 && i < 6 && (kVW[i] == 1 || (stride == 1 && HW % kVW[i] == 0)); }

namespace {
// SV: pixels per store, four where rows of pixels allow it
template <int K, int MB, int VW, int SV>
hipError_t split_attr() {
  const void *f;
  if constexpr (K) f = reinterpret_cast<const void *>(&pw_split_kwaves_kernel<MB, VW, SV>);
  else f = reinterpret_cast<const void *>(&pw_split_kernel<MB, VW, SV>);
  return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, MAX_LDS);
}
template <int K, int MB, int VW>
hipError_t split_init() {
  hipError_t e = split_attr<K, MB, VW, 4>();
  if (e != hipSuccess) return e;
  return split_attr<K, MB, VW, VW>();
}
template <int K, int MB, int VW>
void split_go(const PwArgs &a, hipStream_t s) {
  const dim3 grid(a.g.n_ptiles, a.g.mtiles), block(256);
  if ((a.Ho * a.Wo) % 4 == 0) {
    if constexpr (K) hipLaunchKernelGGL((pw_split_kwaves_kernel<MB, VW, 4>), grid, block, a.g.lds_bytes, s, a);
    else hipLaunchKernelGGL((pw_split_kernel<MB, VW, 4>), grid, block, a.g.lds_bytes, s, a);
  } else {
    if constexpr (K) hipLaunchKernelGGL((pw_split_kwaves_kernel<MB, VW, VW>), grid, block, a.g.lds_bytes, s, a);
    else hipLaunchKernelGGL((pw_split_kernel<MB, VW, VW>), grid, block, a.g.lds_bytes, s, a);
  }
}
}  // namespace

hipError_t init_pw_split_attributes() {
  hipError_t e;
  if ((e = split_init<0, 2, 1>()) != hipSuccess) return e;
  if ((e = split_init<0, 1, 1>()) != hipSuccess) return e;
  if ((e = split_init<0, 2, 2>()) != hipSuccess) return e;
  if ((e = split_init<0, 1, 2>()) != hipSuccess) return e;
  if ((e = split_init<1, 2, 1>()) != hipSuccess) return e;
  return split_init<1, 1, 1>();
}

hipError_t launch_pw_split(const PwArgs &a, hipStream_t s) {
  const int i = a.g.variant - kPwSplitFirst;
  if (!a.w || !pw_split_fits(i, a.Ho * a.Wo, a.stride) || !pw_split_ok(a.N, a.Cin, a.Cout, a.HWin, a.Ho, a.Wo) || a.g.K != a.Cin ||
      a.nchunks != cdiv(a.Cin, 16) || (a.stride == 1 && a.HWin != a.Ho * a.Wo) ||
      ((a.stride != 1) && ((a.Ho - 1) * a.stride * a.Win + (a.Wo - 1) * a.stride >= a.HWin)) ||
      (unsigned long long)a.g.mtiles * (a.g.bm / 32) * a.nchunks * 3072 >= (1ull << 32) ||
      (reinterpret_cast<uintptr_t>(a.in) & 15) || (reinterpret_cast<uintptr_t>(a.out) & 15))
    return hipErrorInvalidValue;
  switch (i) {
    case 0: split_go<0, 2, 1>(a, s); break;
    case 1: split_go<0, 1, 1>(a, s); break;
    case 2: split_go<0, 2, 2>(a, s); break;
    case 3: split_go<0, 1, 2>(a, s); break;
    case 4: split_go<1, 2, 1>(a, s); break;
    default: split_go<1, 1, 1>(a, s); break;
  }
  return hipGetLastError();
}

}  // namespace pbkd
