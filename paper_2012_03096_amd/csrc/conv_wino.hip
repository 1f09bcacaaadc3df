// Frozen-weight 3x3 convolutions (stride 1) by F(2x2, 3x3) on the bf16 matrix cores (device code: conv_wino_kernel.h): weight
// image, geometry, launch.
#include <type_traits>

#include "conv_wino_kernel.h"

namespace pbkd {

namespace {
constexpr int kMaxLds = 160 * 1024;

// Canonical weights [Cout][Cin][9] -> G w G^T, in fp64, split into three bf16 pieces, in the multiplying waves' operand order.
// One thread per (lane of an operand, channel block, chunk, channel tile, position): bound by the latency of its scattered reads,
// so many threads that read the same taps (from cache) beat one that forms all 16 positions in turn (64 -> 64 channels 81 -> 10
// us, 128 -> 128 82 -> 11, 256 -> 256 83 -> 17, 512 -> 512 85 -> 52, where the cache's bandwidth is the bound).
__global__ __launch_bounds__(128) void conv_wino_pack_kernel(const float *w, uintx4 *out, int nchunks, int Cout, int Cin) {
  const int lane = threadIdx.x & 63, no = threadIdx.x >> 6, ch = blockIdx.x, mt = blockIdx.y;
  const int i = blockIdx.z >> 2, j = blockIdx.z & 3;
  const int o = mt * 64 + no * 32 + (lane & 31);
  const int c0 = (ch * 16 < Cin - 16 ? ch * 16 : Cin - 16) + 8 * (lane >> 5);
  uintx4 *const dst = out + ((size_t)mt * nchunks + ch) * (kWinoChunkBytes / 16) + (4 * i + j) * (6 * 64) + no * (3 * 64) + lane;
  uintx4 pp[3];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    unsigned q[3] = {0, 0, 0};
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int c = c0 + 2 * t + e;
      double u = 0;
      if (o < Cout && c >= ch * 16 && c < Cin) {
        const float *g = w + ((size_t)o * Cin + c) * 9;
        double r[3];
        for (int b = 0; b < 3; ++b)
          r[b] = i == 0 ? (double)g[b] : i == 3 ? (double)g[6 + b]
                 : 0.5 * ((double)g[b] + (double)g[6 + b] + (i == 1 ? (double)g[3 + b] : -(double)g[3 + b]));
        u = j == 0 ? r[0] : j == 3 ? r[2] : 0.5 * (r[0] + r[2] + (j == 1 ? r[1] : -r[1]));
      }
#pragma unroll
      for (int pc = 0; pc < 3; ++pc) {
        const unsigned b = pack_bf16_rn((float)u, 0.f) & 0xffffu;
        q[pc] |= b << (16 * e);
        u -= (double)__builtin_bit_cast(float, b << 16);
      }
    }
#pragma unroll
    for (int pc = 0; pc < 3; ++pc) pp[pc][t] = q[pc];
  }
#pragma unroll
  for (int pc = 0; pc < 3; ++pc) dst[pc * 64] = pp[pc];
}

template <int SR>
hipError_t attr() {
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&conv_wino_kernel<SR, false>), hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
  return e != hipSuccess ? e : hipFuncSetAttribute(reinterpret_cast<const void *>(&conv_wino_kernel<SR, true>), hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
}
template <int SR>
void go(const dim3 &grid, const ConvArgs &a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  void (*const kernel)(ConvArgs) = a.in_scale ? &conv_wino_kernel<SR, true> : &conv_wino_kernel<SR, false>;
  if (e0 && e1) hipExtLaunchKernelGGL(kernel, grid, dim3(256), (unsigned)a.g.lds_bytes, s, e0, e1, 0, a);
  else hipLaunchKernelGGL(kernel, grid, dim3(256), a.g.lds_bytes, s, a);
}
int staged(int PLd, int PL) {     // positions per thread, 0: too many
  for (int sr : {6, 10})
    if (PLd <= 64 * sr && 2 * PL < kWinoPositions - 1) return sr;
  return 0;
}
// extra passes of the 16-lane groups of a wave's 16-byte reads over the LDS banks, for a row pitch (in 16-byte units)
int conflicts(int tw, int th, int pitch) {
  int extra = 0;
  for (int b = 0; b < 64; b += 16) {
    int n[16] = {}, most = 0;
    for (int t = b; t < b + 16; ++t) {
      const int ty = t / tw < th ? t / tw : 0, tx = t / tw < th ? t % tw : 0, bank = (2 * ty * pitch + tx) & 15;
      if (++n[bank] > most) most = n[bank];
    }
    extra += most - 1;
  }
  return extra;
}
}  // namespace

// Every (columns per workgroup tile, K split) is priced: rounds of 256 workgroups x (chunks x 4 400 cycles + 14 000 for the way back
// through the output transform), start-up, and the kernel that adds up a K split (as for the stacked rows).
bool conv_wino_geom(int N, int Cin, int Cout, int Ho, int Wo, ConvGeom &best, double &best_cost) {
  if (Cin < 16) return false;
  const int Th = cdiv(Ho, 2), Tw = cdiv(Wo, 2);
  const long long rows = (long long)N * Th;
  const double out_bytes = 4.0 * N * Cout * Ho * Wo;
  best_cost = 0;
  int last = 0;
  for (int tx = cdiv(Tw, 64); tx <= Tw; ++tx) {
    const int tw = cdiv(Tw, tx);
    if (tw == last) continue;
    if (last && tw < 4) break;
    last = tw;
    ConvGeom g{};
    g.bm = 64;
    g.kc = 16;
    g.mtiles = cdiv(Cout, 64);
    g.nchunks = cdiv(Cin, 16);
    g.split = g.wino = true;
    g.TW = tw;
    g.tiles_x = cdiv(Tw, tw);
    g.SH = 2 * Th + 2;
    g.IW = 2 * tw + 2;
    // PL counts the positions of one column parity
    const auto staged_rows = [&](int th) {
      const int cross = th % Th == 0 ? th / Th - 1 : Th % th == 0 ? 0 : cdiv(th - 1, Th);
      return 2 * th + 2 + 2 * cross;
    };
    g.TH = 64 / tw;
    if (g.TH > rows) g.TH = (int)rows;
    g.IWS = tw + 1;
    while (g.TH > 1 && !staged(staged_rows(g.TH) * g.IW, staged_rows(g.TH) * g.IWS)) --g.TH;
    g.IH = staged_rows(g.TH);
    g.PLd = g.IH * g.IW;
    const int sr = staged(g.PLd, g.IH * g.IWS);
    if (!sr) continue;
    for (int pitch = tw + 2; pitch <= tw + 8 && staged(g.PLd, g.IH * pitch) == sr; ++pitch)
      if (conflicts(tw, g.TH, pitch) < conflicts(tw, g.TH, g.IWS)) g.IWS = pitch;
    g.PL = g.IH * g.IWS;
    g.lds_bytes = kWinoLdsBytes;
    const long long tr = (rows + g.TH - 1) / g.TH;
    if (tr * g.tiles_x * g.mtiles > 0x7ffffff) continue;
    g.n_ptiles = (int)(tr * g.tiles_x);
    g.tiles_y = (int)tr;
    g.tiles_n = 1;
    if (g.nchunks > 65535 || g.mtiles > 65535 || (unsigned long long)g.mtiles * g.nchunks * kWinoChunkBytes >= (1ull << 32)) continue;
    for (int want = 1; want <= 8; ++want) {
      g.kchunks = cdiv(g.nchunks, want);
      g.ksplit = cdiv(g.nchunks, g.kchunks);
      if (g.ksplit != want || (want > 1 && g.kchunks < 2)) continue;
      if (g.ksplit * out_bytes >= 4294967296.0 - 64) continue;
      g.nimg = want > 1 ? cdiv(64, Ho * Wo) : 1;
      g.stat_parts = want > 1 ? cdiv(N, g.nimg) : g.n_ptiles;
      const long long items = (long long)g.n_ptiles * g.mtiles * g.ksplit;
      const double cost = (double)((items + 255) / 256) * (g.kchunks * 4400.0 + 14000) + 8000 +
                          conv_ksplit_cycles(g, N, Cout, Ho, Wo);
      if (best_cost == 0 || cost < best_cost) best_cost = cost, best = g;
    }
  }
  return best_cost > 0;
}

double conv_split_cycles(const ConvGeom &g, int N, int Cout, int Ho, int Wo) {
  static const double kStage[4] = {4250, 4250, 2500, 1800}, kEnd[4] = {8600, 8600, 5000, 3500};       // per workgroup tile
  const long long items = (long long)g.n_ptiles * g.mtiles * g.ksplit;
  return (double)((items + 255) / 256) * (g.kchunks * kStage[g.tile] + kEnd[g.tile]) + 2 * kStage[g.tile] +
         conv_ksplit_cycles(g, N, Cout, Ho, Wo);
}

hipError_t launch_conv_wino_pack(const float *w, float *wpk, const ConvGeom &g, int Cout, int Cin, hipStream_t s) {
  if (!g.wino || Cin < 16 || g.nchunks > 65535 || g.mtiles > 65535) return hipErrorInvalidValue;
  hipLaunchKernelGGL(conv_wino_pack_kernel, dim3(g.nchunks, g.mtiles, 16), dim3(128), 0, s, w, reinterpret_cast<uintx4 *>(wpk), g.nchunks, Cout, Cin);
  return hipGetLastError();
}

hipError_t conv_wino_init() {
  hipError_t e;
  if ((e = attr<6>()) != hipSuccess) return e;
  return attr<10>();
}

hipError_t launch_conv_wino(const ConvArgs &a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const ConvGeom &g = a.g;
  const int Th = cdiv(a.Ho, 2), sr = staged(g.PLd, g.PL);
  if (a.stride != 1 || a.Cin < 16 || a.H != a.Ho || a.W != a.Wo || !a.w_canon || !sr || g.lds_bytes != kWinoLdsBytes) return hipErrorInvalidValue;
  if (g.SH != 2 * Th + 2 || g.IW != 2 * g.TW + 2 || g.TW < 1 || g.TH < 1 || g.TW * g.TH > 64 || g.PL < g.IH * g.IWS || g.IWS <= g.TW ||
      g.PLd != g.IH * g.IW || (long long)g.tiles_x * g.TW < cdiv(a.Wo, 2) ||
      (long long)(g.n_ptiles / g.tiles_x) * g.TH < (long long)a.N * Th || (unsigned long long)a.N * a.Cin * a.H * a.W * sizeof(float) >= (1ull << 32))
    return hipErrorInvalidValue;
  if (g.ksplit < 1 || g.kchunks < 1 || (long long)(g.ksplit - 1) * g.kchunks >= g.nchunks || (long long)g.ksplit * g.kchunks < g.nchunks ||
      g.nchunks != cdiv(a.Cin, 16) || g.mtiles != cdiv(a.Cout, 64) || (g.ksplit > 1 && !a.split_out))
    return hipErrorInvalidValue;
  if ((unsigned long long)g.ksplit * a.N * a.Cout * a.Ho * a.Wo * sizeof(float) >= (1ull << 32) - 64) return hipErrorInvalidValue;
  if ((unsigned long long)g.mtiles * g.nchunks * kWinoChunkBytes >= (1ull << 32)) return hipErrorInvalidValue;
  const long long items = (long long)g.n_ptiles * g.mtiles * g.ksplit;
  if (items < 1 || items > 0x7fffffffLL) return hipErrorInvalidValue;
  const dim3 grid((unsigned)conv_persistent_workgroups(items, a.beside));
  if (sr == 6) go<6>(grid, a, s, e0, e1);
  else go<10>(grid, a, s, e0, e1);
  return hipGetLastError();
}

}  // namespace pbkd
