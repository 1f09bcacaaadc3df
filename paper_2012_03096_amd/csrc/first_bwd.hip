// Backward pass across a block's full 3x3 first layer and the depthwise convolution behind it in one kernel (FirstBwdArgs):
// from du, the gradient of the depthwise output, and z, the first layer's output,
//   g[c,q]   = 1[b > 0] * sum_k D[c,k] * du[c, q - off_k],  b = BatchNorm(z)     (never written)
//   dD[c,k]  = sum_q relu(b)[c,q] * du[c, q - off_k]                             (depthwise weight gradient)
//   dbeta    = sum_q g,   dgamma = sum_q g * xhat
//   dW[c,j]  = sum_q dz[c,q] * x_j[q],   x_j the input under tap j, dz the BatchNorm backward of g, taken as the three sums
//              g * x_j, (z - mean) * x_j and x_j, which first_bwd_finish_kernel puts together once dbeta and dgamma are known.
// Apart (dw_bwd_fast_kernel, dw_bwd_finalize_kernel, wgrad_taps_bn_kernel) g is written and read and z read twice: 5 tensors of the
// layer's output for 2 here.
//
// A workgroup owns 32 channels and a contiguous range of patches of 4x4 pixels, eight a tile.  A thread has one channel and one patch of the
// tile: its 6x6 window of du, its 16 values of z, and the channel's eleven sums; thread rows 0 to 26 also fetch their tap's input.  g,
// z - mean and the taps go to LDS, a row of 128 pixels per channel and tap, and the waves multiply them on the fp32 matrix cores, each
// one product of half of the pixels.  The sums over positions are taken with relu(b) at the centre and du in the window, so z needs no
// halo.  The window's two edge columns come from the neighbouring lanes, at the tile's ends from the tile before and from du of the next
// one, which is fetched a tile ahead: a tile is one cache line wide, and two more lines a row for its edges cost 40 us of 307.
//
// What bounds it: memory, which two workgroups a compute unit (their registers) do not keep busy while they multiply.  64 channels at
// 224x224, batch 32, 3 input channels: 265 us and 8 for the finish, 0.84 GB (1.1 with the halo rows that
// leave L2 between two rows of tiles), for 234 + 6 + 189 us apart; without the products 205 us,
// without most of the arithmetic 255.  Slower: three workgroups a compute unit and nothing ahead 307, multiplying waves of their own
// beside four loading ones 310; no faster: the next window's loads ahead of the arithmetic 267, two accumulators 268.  On 36 drawn shapes,
// 1 to 124 images, 4x4 to 214x260, 32 to 64 channels, a step is 1.02 to 1.16 times as fast, 1.046 in the mean.
#include "pbkd_internal.h"

namespace pbkd {

namespace {
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
constexpr unsigned kPast = 0x80000000u;        // offsets from here on are past every buffer: they read zeros
constexpr int kPitch = 132;                    // floats from row to row in LDS: 16-byte reads of sixteen rows in different banks
constexpr int kTaps = 32;                      // tap columns (9 * Cin <= 32)
}  // namespace

// ONE: a workgroup has a single tile (up to 1024 tiles a group of 32 channels).  So few pixels were summed 32 at a time by the kernel apart, and
// g x_j, whose sum dbeta and dgamma cancel in part, is larger than dz x_j: a wave then keeps four sums of 16 pixels.  rms error of dW
// against 64 bits, of the root of its terms' squares, inputs around 1, apart / one sum of 64 / so: one image of 16x16, 64 channels 1.17, 1.31 and
// 1.13e-7; two of 32x32, 32 channels 1.37, 1.48 and 1.25e-7 (around 0 at one image of 16x16 1.28, 1.38 and 1.30e-7).  With more tiles one sum does.
template <bool ONE>
__global__ __launch_bounds__(256, 2) void first_bwd_kernel(FirstBwdArgs p) {
  __shared__ __attribute__((aligned(16))) float lds[3][32][kPitch];   // g, z - mean, taps
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l31 = lane & 31, lh = lane >> 5;
  const int lin = xcd_contiguous(blockIdx.x, gridDim.x);              // the channel groups of one range read the same input: neighbours on a die
  const int split = lin / p.geo.groups, grp = lin - split * p.geo.groups;
  const int pq = tid & 7, row = tid >> 3;                             // patch of the tile; channel of the group, and tap
  const int H = p.H, W = p.W, HW = H * W, C = p.C;
  const int c = 32 * grp + row, cc = c < C ? c : C - 1;               // (a row past the last channel repeats it, and is never stored)

  const unsigned sizez = (unsigned)p.N * C * HW * 4u, sizex = (unsigned)p.N * p.Cin * HW * 4u;
  auto buffer = [](const float *q, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(q), 0, (int)bytes, 0x00020000);
  };
  const __amdgpu_buffer_rsrc_t rdu = buffer(p.du, sizez), rz = buffer(p.z, sizez), rx = buffer(p.x, sizex);
  auto load4 = [](const __amdgpu_buffer_rsrc_t &r, unsigned off) { return __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0)); };

  // this thread's patch of a tile: image, group of four rows, quad of columns; and what a tile's eight patches move it by
  const int W4 = W >> 2, HG = (H + 3) >> 2, per = W4 * HG, T = ONE ? 1 : p.geo.tiles_per_split;
  const int dn = 8 / per, dr = 8 - dn * per, dy = dr / W4, dx = dr - dy * W4;
  struct At {
    int n, yg, xq;
  };
  const long long first = (long long)split * T * 8 + pq;
  auto patch = [&](long long e) {
    At a;
    a.n = (int)(e / per);
    const int r = (int)(e - (long long)a.n * per);
    a.yg = r / W4, a.xq = r - a.yg * W4;
    return a;
  };
  At ahead = patch(first), at = ahead;           // of the tile whose du is fetched next, and whose z and taps are

  // Addresses: where a row does not exist they are past the buffer.  Most tiles have all their rows, and skip the selection; nothing is
  // loaded under a condition, so the compiler can count the loads in flight.
  auto fetch_du = [&](int t, f4 (&d)[6]) {       // past the range's end: the next tile's first patch, the last one's right edge
    const int y0 = 4 * ahead.yg;
    const bool ok = ahead.n < p.N && (t < T || (t == T && pq == 0));
    unsigned off[6];
    off[0] = ((((unsigned)ahead.n * (unsigned)C + (unsigned)cc) * (unsigned)H + (unsigned)(y0 - 1)) * (unsigned)W + 4u * (unsigned)ahead.xq) * 4u;
#pragma unroll
    for (int r = 1; r < 6; ++r) off[r] = off[r - 1] + 4u * (unsigned)W;
    if (!__all(ok && y0 > 0 && y0 + 4 < H)) {
#pragma unroll
      for (int r = 0; r < 6; ++r) off[r] = ok && y0 + r > 0 && y0 + r <= H ? off[r] : kPast;
    }
#pragma unroll
    for (int r = 0; r < 6; ++r) d[r] = load4(rdu, off[r]);
    ahead.xq += dx;
    const bool cx = ahead.xq >= W4;
    ahead.xq -= cx ? W4 : 0;
    ahead.yg += dy + (cx ? 1 : 0);
    const bool cy = ahead.yg >= HG;
    ahead.yg -= cy ? HG : 0;
    ahead.n += dn + (cy ? 1 : 0);
  };

  const int tap = row % 9, cin = row / 9 < p.Cin ? row / 9 : p.Cin - 1;
  const bool has_tap = row < 9 * p.Cin;
  const int tdy = tap / 3 - 1, tdx = tap % 3 - 1;
  f4 z4[4], x4[4];
  int shift = 0, left = 0, right = 0;           // which way the taps' values move; the patch has a neighbour in its row
  unsigned rows = 0;                            // rows of the patch that exist
  auto fetch_zx = [&](int t) {
    const int y0 = 4 * at.yg, x = 4 * at.xq, xs = x + tdx;
    const bool ok = at.n < p.N && t < T;
    const bool tl = xs < 0, tr = xs + 4 > W;    // the load starts at the row's first / last group, and the values are moved over
    unsigned oz[4], ox[4];
    oz[0] = ((((unsigned)at.n * (unsigned)C + (unsigned)cc) * (unsigned)H + (unsigned)y0) * (unsigned)W + (unsigned)x) * 4u;
    ox[0] = ((((unsigned)at.n * (unsigned)p.Cin + (unsigned)cin) * (unsigned)H + (unsigned)(y0 + tdy)) * (unsigned)W + (unsigned)(tl ? 0 : tr ? W - 4 : xs)) * 4u;
    ox[0] = has_tap ? ox[0] : kPast;
#pragma unroll
    for (int i = 1; i < 4; ++i) oz[i] = oz[i - 1] + 4u * (unsigned)W, ox[i] = has_tap ? ox[i - 1] + 4u * (unsigned)W : kPast;
    rows = 15u;
    if (!__all(ok && y0 > 0 && y0 + 4 < H)) {
      rows = 0u;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool rok = ok && y0 + i < H;
        const int y = y0 + i + tdy;
        rows |= rok ? 1u << i : 0u;
        oz[i] = rok ? oz[i] : kPast;
        ox[i] = rok && y >= 0 && y < H ? ox[i] : kPast;
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) z4[i] = load4(rz, oz[i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) x4[i] = load4(rx, ox[i]);
    shift = tl ? 1 : tr ? 2 : 0, left = x > 0, right = x + 4 < W;
    at = ahead;                                 // (the du fetched last is the tile after this one)
  };

  float w[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) w[k] = p.D[cc * 9 + k];
  const float sc = p.scale[cc], sh = p.shift[cc], mean = p.mean[cc];
  float sum[11], colsum = 0.f;
#pragma unroll
  for (int k = 0; k < 11; ++k) sum[k] = 0.f;
  const int which = wave & 1, half = wave >> 1;            // this wave multiplies g or z - mean, of half of a tile's pixels
  constexpr int PARTS = ONE ? 4 : 1;
  floatx16 acc[PARTS];
#pragma unroll
  for (int i = 0; i < PARTS; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;

  // du of this tile and of the next, whose first column is the right edge of this one's last patch; and the tile before's last
  // column, in the lane that will have had it: the one of the range's first patch is loaded
  f4 d4[6], next[6];
  float before[6];
  {
    const At b = patch(first >= 8 ? first - 8 : 0);
    const bool ok = first >= 8 && pq == 7;
#pragma unroll
    for (int r = 0; r < 6; ++r) {
      const int y = 4 * b.yg - 1 + r;
      const unsigned off = ((((unsigned)b.n * (unsigned)C + (unsigned)cc) * (unsigned)H + (unsigned)y) * (unsigned)W + 4u * (unsigned)b.xq + 3u) * 4u;
      before[r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rdu, ok && b.n < p.N && y >= 0 && y < H ? off : kPast, 0, 0));
    }
  }
  fetch_du(0, d4);
  fetch_zx(0);
  fetch_du(1, next);
#pragma unroll 1
  for (int t = 0; t < T; ++t) {
    float d[6][6];
#pragma unroll
    for (int r = 0; r < 6; ++r) {
      const float l = dpp_mov<0x111>(d4[r][3]), lb = dpp_mov<0x129>(before[r]);      // row_shr:1; row_ror:9: lane 0 of eight receives lane 7
      const float h = dpp_mov<0x101>(d4[r][0]), hn = dpp_mov<0x127>(next[r][0]);     // row_shl:1; row_ror:7: lane 7 receives lane 0
      d[r][0] = pq == 0 ? lb : l;
      d[r][5] = pq == 7 ? hn : h;
#pragma unroll
      for (int j = 0; j < 4; ++j) d[r][1 + j] = d4[r][j];
    }
    const bool border = __any(!left || !right);
    if (border) {
#pragma unroll
      for (int r = 0; r < 6; ++r) d[r][0] = left ? d[r][0] : 0.f, d[r][5] = right ? d[r][5] : 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f4 v = x4[i];
        x4[i][0] = shift == 1 ? 0.f : shift == 2 ? v[1] : v[0];
        x4[i][1] = shift == 1 ? v[0] : shift == 2 ? v[2] : v[1];
        x4[i][2] = shift == 1 ? v[1] : shift == 2 ? v[3] : v[2];
        x4[i][3] = shift == 1 ? v[2] : shift == 2 ? 0.f : v[3];
      }
    }
    if (t) __syncthreads();                                // the tile before has been multiplied
    float cs = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      cs += (x4[i][0] + x4[i][1]) + (x4[i][2] + x4[i][3]);
      *reinterpret_cast<f4 *>(&lds[2][row][32 * i + 4 * pq]) = x4[i];
    }
    colsum += cs;
    __builtin_amdgcn_sched_barrier(0);
    float s[11];                                           // of this tile: sixteen terms each
#pragma unroll
    for (int k = 0; k < 11; ++k) s[k] = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool rok = rows >> i & 1u;
      const float scr = rok ? sc : 0.f, shr = rok ? sh : 0.f;          // a row that does not exist: b = 0
      f4 g4, c4;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float a = fmaxf(fmaf(z4[i][j], scr, shr), 0.f);
        float da = 0.f;
#pragma unroll
        for (int ky = 0; ky < 3; ++ky)
#pragma unroll
          for (int kx = 0; kx < 3; ++kx) {
            const float v = d[i + 2 - ky][j + 2 - kx];
            da += w[ky * 3 + kx] * v;
            s[ky * 3 + kx] += a * v;
          }
        const float g = a > 0.f ? da : 0.f;
        const float zc = z4[i][j] - mean;
        s[9] += g;
        s[10] += g * zc;
        g4[j] = g;
        c4[j] = zc;
      }
      *reinterpret_cast<f4 *>(&lds[0][row][32 * i + 4 * pq]) = g4;
      *reinterpret_cast<f4 *>(&lds[1][row][32 * i + 4 * pq]) = c4;
    }
#pragma unroll
    for (int k = 0; k < 11; ++k) sum[k] += s[k];
    __builtin_amdgcn_sched_barrier(0);
    if (!ONE) {
#pragma unroll
      for (int r = 0; r < 6; ++r) before[r] = d4[r][3], d4[r] = next[r];
      fetch_zx(t + 1);
      fetch_du(t + 2, next);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) {                          // its 64 pixels, eight at a time: four products of two
      const int px = 64 * half + 8 * q + 4 * lh;
      const f4 av = *reinterpret_cast<const f4 *>(&lds[which][l31][px]);
      const f4 xv = *reinterpret_cast<const f4 *>(&lds[2][l31][px]);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[q * PARTS / 8] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[e], xv[e], acc[q * PARTS / 8], 0, 0, 0);
    }
  }

  // ---- the channel's sums over the tile's eight patches, and the taps'
  auto over_patches = [](float v) {
    v += dpp_mov<0xB1>(v);                                 // quad_perm [1,0,3,2]
    v += dpp_mov<0x4E>(v);                                 // quad_perm [2,3,0,1]
    return v + dpp_mov<0x141>(v);                          // row_half_mirror
  };
#pragma unroll
  for (int k = 0; k < 11; ++k) {
    const float v = over_patches(sum[k]);
    if (pq == 0 && c < C) p.dw_partial[((size_t)split * C + c) * 11 + k] = v;
  }
  colsum = over_patches(colsum);
  if (grp == 0 && pq == 0) p.colsum[(size_t)split * kTaps + row] = colsum;

  // ---- the halves' products added: register r of lane l is row 8*(r/4) + 4*(l/32) + r%4, column l%32
  __syncthreads();
  float *const M = &lds[0][0][0];                          // [halves][2][32][32]: 16 KB
  if constexpr (ONE) acc[0] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
#pragma unroll
  for (int r = 0; r < 16; ++r) M[wave * 1024 + (8 * (r / 4) + 4 * lh + r % 4) * 32 + l31] = acc[0][r];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int e = tid + 256 * j, ch = (e >> 5) & 31, o = 32 * grp + ch;
    if (o < C) p.partial[(((size_t)split * C + o) * 2 + (e >> 10)) * kTaps + (e & 31)] = M[e] + M[2048 + e];
  }
}

// A workgroup per channel and half of the tap columns: the splits' partials in a fixed order in fp64, and dW from them.
__global__ __launch_bounds__(1024) void first_bwd_finish_kernel(FirstBwdArgs p) {
  __shared__ double red[32][64];
  const int tid = threadIdx.x, c = blockIdx.x, j0 = 16 * blockIdx.y, S = p.geo.splits, C = p.C;
  const int v = tid & 31, row = tid >> 5;                  // columns v: g and z - mean with sixteen taps each; and those taps' sums, dbeta, dgamma
  const float *const q = p.partial + ((size_t)c * 2 + (v >> 4)) * kTaps + j0 + (v & 15);
  const float *const r = v < 16 ? p.colsum + j0 + v : p.dw_partial + (size_t)c * 11 + (v < 18 ? 9 + (v & 1) : 9);
  const size_t sq = (size_t)C * 2 * kTaps, sr = v < 16 ? kTaps : (size_t)C * 11;
  double a = 0.0, b = 0.0;
  int t = row;
  for (; t + 3 * 32 < S; t += 4 * 32) {                    // eight loads in flight, summed in index order
    float x[4], y[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = q[(size_t)(t + 32 * i) * sq], y[i] = r[(size_t)(t + 32 * i) * sr];
#pragma unroll
    for (int i = 0; i < 4; ++i) a += (double)x[i], b += (double)y[i];
  }
  for (; t < S; t += 32) a += (double)q[(size_t)t * sq], b += (double)r[(size_t)t * sr];
  red[row][v] = a;
  red[row][32 + v] = b;
  __syncthreads();
#pragma unroll
  for (int k = 16; k >= 1; k >>= 1) {
    if (row < k) red[row][v] += red[row + k][v], red[row][32 + v] += red[row + k][32 + v];
    __syncthreads();
  }
  const double rstd = (double)p.rstd[c], sc = (double)p.scale[c], db = red[0][48], dg = red[0][49] * rstd;
  if (tid == 0 && blockIdx.y == 0) p.dbeta[c] = (float)db, p.dgamma[c] = (float)dg;
  const int j = j0 + tid;
  if (tid < 16 && j < 9 * p.Cin) {
    const double m = (double)p.N * (double)p.H * (double)p.W;
    p.dW[(size_t)c * (9 * p.Cin) + j] = (float)(sc * red[0][tid] - sc / m * (dg * rstd * red[0][16 + tid] + db * red[0][32 + tid]));
  }
}

// Splits: two rounds of two workgroups per compute unit.  What a wave sums in fp32 for dW is a shorter chain than in the kernel apart (1 600
// pixels at 224x224, batch 32, for 2 091).  The eleven sums of a channel are a longer one: a thread adds its 16 pixels of a tile, then the
// tiles' sums one after another (25 there; 99 with 2048 channels at 112x112, batch 16), where dw_bwd_fast_kernel sums 8 or 16 pixels, then
// a tree, then fp64.  It does not show: errors of dD, dgamma and dbeta against 64 bits are those of the kernels apart within 1 % at 1 to 99
// tiles, inputs around 0, 2 and 30, since they come from du's and z's; dW's are 0.56 to 1.00 of them from two tiles on.
FirstBwdGeom first_bwd_geom(int N, int C, int H, int W) {
  FirstBwdGeom g{};
  g.groups = cdiv(C, 32);
  const long long patches = (long long)N * cdiv(H, 4) * (W / 4);
  const int tiles = (int)((patches + 7) / 8);
  int want = 1024 / g.groups;
  if (want < 1) want = 1;
  g.tiles_per_split = cdiv(tiles, want);
  g.splits = cdiv(tiles, g.tiles_per_split);
  return g;
}

hipError_t launch_first_bwd(const FirstBwdArgs &a, hipStream_t s) {
  const unsigned long long HW = (unsigned long long)a.H * a.W;
  const FirstBwdGeom &g = a.geo;
  if (a.N < 1 || a.C < 1 || a.C > 65535 || a.Cin < 1 || 9 * a.Cin > kTaps || a.H < 1 || a.W < 4 || a.W % 4 || g.groups != cdiv(a.C, 32) ||
      g.splits < 1 || g.tiles_per_split < 1 || (long long)g.splits * g.tiles_per_split * 8 < (long long)a.N * cdiv(a.H, 4) * (a.W / 4) ||
      (long long)g.splits * g.groups > 0x7fffffffLL || a.N * (HW * a.C * sizeof(float)) > (1ull << 31) || a.N * (HW * a.Cin * sizeof(float)) > (1ull << 31))
    return hipErrorInvalidValue;
  if (!a.du || !a.D || !a.z || !a.x || !a.scale || !a.shift || !a.mean || !a.rstd || !a.dw_partial || !a.partial || !a.colsum || !a.dW || !a.dgamma ||
      !a.dbeta || ((reinterpret_cast<uintptr_t>(a.du) | reinterpret_cast<uintptr_t>(a.z) | reinterpret_cast<uintptr_t>(a.x)) & 15))
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(g.tiles_per_split == 1 ? first_bwd_kernel<true> : first_bwd_kernel<false>, dim3(g.splits * g.groups), dim3(256), 0, s, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(first_bwd_finish_kernel, dim3(a.C, cdiv(9 * a.Cin, 16)), dim3(1024), 0, s, a);
  return hipGetLastError();
}

}  // namespace pbkd
