// 3x3 convolution with frozen weights on the bf16 matrix cores, fp32 operands split three ways (device code and the
// arithmetic: conv_split_kernel.h).  Same workgroup tiles and pixel-tile geometry as the fp32-MFMA kernel, launched as
// a persistent grid; this file instantiates the tiles and launches.
#include <cstdlib>
#include <type_traits>

#include "conv_mfma_kernel.h"
#include "conv_rows_kernel.h"

namespace pbkd {

namespace {
template <int WGM, int MB, int NB>
struct SplitLaunch {
  template <int BSLOTS>
  static hipError_t attr() {
    for (const void *k : {reinterpret_cast<const void *>(&conv_rows_kernel<WGM, MB, NB, BSLOTS, false>),
                          reinterpret_cast<const void *>(&conv_rows_kernel<WGM, MB, NB, BSLOTS, true>)}) {
      const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, MAX_LDS);
      if (e != hipSuccess) return e;
    }
    return hipFuncSetAttribute(reinterpret_cast<const void *>(&conv_split_kernel<WGM, MB, NB, BSLOTS>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, MAX_LDS);
  }
  static hipError_t init() {
    hipError_t e;
    if ((e = attr<1>()) != hipSuccess) return e;
    if ((e = attr<2>()) != hipSuccess) return e;
    if constexpr (WGM * MB * NB >= 4) return hipSuccess;      // the two large tiles stop at two halo slots per thread
    else return attr<3>();
  }
  template <int BSLOTS>
  static void go(const dim3 &grid, const dim3 &block, const ConvArgs &a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    const bool vec = a.g.TW % 4 == 0 && a.Wo % 4 == 0;          // stacked rows: 16-byte stores
    void (*const kernel)(ConvArgs) =
        !a.g.rows ? &conv_split_kernel<WGM, MB, NB, BSLOTS>
        : vec       ? &conv_rows_kernel<WGM, MB, NB, BSLOTS, true>
                    : &conv_rows_kernel<WGM, MB, NB, BSLOTS, false>;
    if (e0 && e1)
      hipExtLaunchKernelGGL(kernel, grid, block, (unsigned)a.g.lds_bytes, s, e0, e1, 0, a);
    else
      hipLaunchKernelGGL(kernel, grid, block, a.g.lds_bytes, s, a);
  }
  static hipError_t launch(const ConvArgs &a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    const long long items = (long long)a.g.n_ptiles * a.g.mtiles * a.g.ksplit;
    if (items < 1 || items > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)conv_persistent_workgroups(items, Company{})), block(512);
    switch (conv_bslots_for(a.g.PLd)) {
      case 1: go<1>(grid, block, a, s, e0, e1); break;
      case 2: go<2>(grid, block, a, s, e0, e1); break;
      case 3:
        if constexpr (WGM * MB * NB >= 4) return hipErrorInvalidValue;
        else go<3>(grid, block, a, s, e0, e1);
        break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
};
// Canonical 3x3 weights [Cout][Cin][9] -> the LDS images of every (channel tile, chunk), see kSplitLastW.  One
// thread per output channel (of whole tiles: channels past Cout are zeros) and chunk; bound by its scattered reads, 72
// floats a thread: 512 -> 512 channels in about 10 us, where the host took 20 ms.
__global__ __launch_bounds__(256) void conv_split_pack_kernel(const float *w, uintx4 *out, int bm, int nchunks, int a_stride, int M,
                                                              int Cout, int Cin, bool reach_back) {
  const int m = blockIdx.x * 256 + threadIdx.x, ch = blockIdx.y;
  if (m >= M) return;
  const int c0 = reach_back && ch * 8 > Cin - 8 ? Cin - 8 : ch * 8;
  uintx4 *const dst = out + ((size_t)(m / bm) * nchunks + ch) * (a_stride / 16) + m % bm;
  for (int tap = 0; tap < 9; ++tap) {
    uintx4 pp[3];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      float v[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int c = c0 + 2 * t + e;
        v[e] = (m < Cout && c >= ch * 8 && c < Cin) ? w[((size_t)m * Cin + c) * 9 + tap] : 0.f;
      }
      unsigned q[3];
      split3_bf16(v[0], v[1], q);
#pragma unroll
      for (int pc = 0; pc < 3; ++pc) pp[pc][t] = q[pc];
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if (tap < 8) dst[(size_t)(c * 10 + tap) * bm] = pp[c];
      else
#pragma unroll
        for (int h = 0; h < 2; ++h) dst[(size_t)(c * 10 + 8 + h) * bm] = pp[kSplitLastW[c][h]];
    }
  }
}

}  // namespace

long long conv_persistent_workgroups(long long items, const Company &beside) {
  static const int units = [] {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 1) v = 256;
    return v;
  }();
  long long G = units;
  if (const char *env = std::getenv("PBKD_SPLIT_WGS")) {
    const int v = std::atoi(env);
    if (v >= 1 && v < G) G = v;
  } else if (beside.units < 16) {
    const long long most = (G * beside.units + 15) / 16, rounds = (items + most - 1) / most;
    if (4 * rounds <= beside.rounds * ((items + G - 1) / G)) G = (items + rounds - 1) / rounds;
  }
  if (items < G) G = items;
  if (G * kSplitMaxTiles < items) G = (items + kSplitMaxTiles - 1) / kSplitMaxTiles;
  return G;
}

hipError_t launch_conv_split_pack(const float *w, float *wpk, const ConvGeom &g, int Cout, int Cin, hipStream_t s) {
  if (g.wino) return launch_conv_wino_pack(w, wpk, g, Cout, Cin, s);
  if (!g.split || (g.rows && Cin < 9) || g.nchunks > 65535) return hipErrorInvalidValue;
  const int M = g.mtiles * g.bm;
  hipLaunchKernelGGL(conv_split_pack_kernel, dim3(cdiv(M, 256), g.nchunks), dim3(256), 0, s, w, reinterpret_cast<uintx4 *>(wpk),
                     g.bm, g.nchunks, conv_split_a_stride(g.bm), M, Cout, Cin, g.rows);
  return hipGetLastError();
}

hipError_t conv_split_init() {
  hipError_t e;
  if ((e = SplitLaunch<2, 2, 2>::init()) != hipSuccess) return e;
  if ((e = SplitLaunch<1, 2, 2>::init()) != hipSuccess) return e;
  if ((e = SplitLaunch<1, 2, 1>::init()) != hipSuccess) return e;
  return SplitLaunch<2, 1, 1>::init();
}

hipError_t launch_conv_split(const ConvArgs &a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (!a.g.split || a.g.lds_bytes > (size_t)MAX_LDS) return hipErrorInvalidValue;
  if (a.g.wino) return launch_conv_wino(a, s, e0, e1);
  if (!a.g.rows && (!conv_split_fits_width(a.g, a.H, a.W, a.stride) || a.g.raw_rounds > conv_split_rounds_max(conv_bslots_for(a.g.PLd)) ||
                    a.g.raw_w % 4 != 0))
    return hipErrorInvalidValue;
  if (a.g.rows && (a.Cin < 9 || !a.w_canon || a.g.nchunks - (a.g.ksplit - 1) * a.g.kchunks < 2 || a.g.PL >= conv_rows_positions(cdiv(a.g.PLd, 256)) || (unsigned long long)a.N * a.Cin * a.H * a.W * sizeof(float) >= (1ull << 32) || a.g.SH != a.stride * (a.Ho - 1) + 3 ||
                   a.g.IW != a.stride * (a.g.TW - 1) + 3 || (long long)a.g.tiles_x * a.g.TW < a.Wo ||
                   (long long)(a.g.n_ptiles / a.g.tiles_x) * a.g.TH < (long long)a.N * a.Ho || a.g.PL < a.g.IH * a.g.IWS))
    return hipErrorInvalidValue;
  if (a.g.ksplit < 1 || a.g.kchunks < 1 || (long long)(a.g.ksplit - 1) * a.g.kchunks >= a.g.nchunks ||
      (long long)a.g.ksplit * a.g.kchunks < a.g.nchunks || (a.g.ksplit > 1 && !a.split_out))
    return hipErrorInvalidValue;
  // the output (all K splits of it) and the weight image are addressed through buffer descriptors with 32-bit offsets
  if ((unsigned long long)a.g.ksplit * a.N * a.Cout * a.Ho * a.Wo * sizeof(float) >= (1ull << 32) - (a.g.rows ? 64 : 0)) return hipErrorInvalidValue;
  if ((unsigned long long)a.g.mtiles * a.g.nchunks * conv_split_a_stride(a.g.bm) >= (1ull << 32)) return hipErrorInvalidValue;
  switch (a.g.tile) {
    case 0: return SplitLaunch<2, 2, 2>::launch(a, s, e0, e1);
    case 1: return SplitLaunch<1, 2, 2>::launch(a, s, e0, e1);
    case 2: return SplitLaunch<1, 2, 1>::launch(a, s, e0, e1);
    case 3: return SplitLaunch<2, 1, 1>::launch(a, s, e0, e1);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace pbkd
