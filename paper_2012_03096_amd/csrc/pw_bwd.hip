// Backward pass of a pointwise convolution in one kernel, for at most 128 output channels: the gradient dz of its output is formed on
// load (from what the BatchNorm behind it, or the block's head, has), and goes into both products that need it,
//   dP[o,c] = sum_q dz[o,q] * u[c,q]      (weight gradient: K = pixels, split over the workgroups, partials as pw_wgrad_mfma.hip's)
//   du[c,q] = sum_o P[o,c] * dz[o,q]      (data gradient:   K = output channels)
// without ever being written.  Apart (BatchNorm backward or head kernel, pw_wgrad_kernel, pw_split_kernel) dz is written once and read
// twice; here g and z (or the target and z) and u are read once and du is written: 4 tensors for 7 inside a block, 3.25 for 6.25
// under a pooled head, and one launch for three.
//
// A workgroup owns 64 columns of dP (input channels), all of its rows, and a contiguous range of pixels, taken in chunks of 64 (32
// with more than 64 output channels).  Eight loader waves fetch two chunks ahead into registers, form dz, split dz and u into three
// bf16 pieces (split_bf16.h, by rounding) and write them to LDS, pixels along a row.  Four MFMA waves multiply: for
// dP both operands are rows of pixels, sixteen bytes a lane; for du the operand's k runs along the channels, across the rows, which
// is what the transposing LDS read (ds_read_b64_tr_b16: four rows of sixteen 2-byte values, a lane receives a column) is for.  P's
// pieces, packed for the data gradient (pw_split_pack_index), stay in registers.  Each MFMA wave has a quarter of dP and one 32 x 32
// tile of du: (channel block, pixel block), or, with more than 64 output channels, (channel block, half of the channels summed).  The
// tiles go to LDS, and the loader waves, which have the time, add the halves and store them a chunk later, where they read u.
//
// du is summed over 16 channels (32 with more than 64 output channels) from zero and these sums are added, as few pixels' are in
// pw_split.hip: with one running sum over all channels and dz's pieces cut off du's rms error is 1.92e-7 of the root of its terms' squares
// at 64 channels, 9x7 maps, batch 3, so it is 1.67e-7, and apart 1.67e-7 (128 channels, 16x16, batch 8: 1.92, 1.71 and 1.72e-7).  The
// additions cost 0.3 of 21 us at 128 channels, 16x16, batch 128, nothing at 64.
//
// What bounds it: memory where the map is large (64 -> 64 at 224x224, batch 32, pooled head, 1.34 GB: 264 us, 5.1 TB/s, for
// 169 + 187 + 149 us apart; 64 -> 128 at 16x16, batch 1024: 5.3 TB/s), else the first loads and the channel sums before any product
// (5 of 16 us at 64 -> 128, 16x16, batch 128, for 10 + 14 + 14 apart) and the loaders' issue: 2 500 cycles a chunk for the MFMA
// waves' 2 100.  us, apart -> here: 128 -> 128 at 16x16, batch 128, pooled head 35 -> 23; 67 -> 100 at 27x23, batch 77 44 -> 28.
// On 69 drawn shapes, 16 to 512 input and 16 to 128 output channels, a student's step is 0.998 to 1.28 times as fast, 1.11 in the mean.
//
// Infinities and numbers past bfloat16's largest: as in the two kernels apart, sums that are NaN are formed again in fp32 from dz as
// the loaders form it (dz_value).
#include "conv_mfma_kernel.h"
#include "split_bf16.h"

namespace pbkd {

namespace {
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));

constexpr int kThreads = 768;                                    // 4 waves multiply, 8 load
constexpr int bwd_px(int bm) { return bm == 64 ? 64 : 32; }      // pixels a chunk
constexpr int bwd_pitch(int bm) { return bm == 64 ? 144 : 96; }  // bytes from row to row of a plane: a row of pixels and padding that keeps
                                                                 // 16-byte reads of 8 rows and transposing reads of 4 in different banks
constexpr int bwd_copy(int bm) { return 3 * (bm + 64) * bwd_pitch(bm); }
constexpr int bwd_tile_row(int bm) { return bwd_px(bm) + 4; }    // floats from row to row of a finished tile of du
constexpr int bwd_tile(int bm) { return 64 * bwd_tile_row(bm); }
constexpr int bwd_exchange(int bm) { return 2 * (bm == 64 ? 1 : 2) * bwd_tile(bm) * (int)sizeof(float); }
constexpr size_t bwd_lds(int bm) { return 2 * (size_t)bwd_copy(bm) + bwd_exchange(bm) + 2 * 128 * sizeof(float) + 4 * sizeof(double); }
constexpr unsigned kPast = 0x80000000u;                          // offsets from here on are past every buffer: loads give zeros, stores nothing

// What a loader thread reads: a group of four pixels of one image (any map of four pixels or more; the last group of an image starts
// at H*W-4 and `dup` of its pixels belong to the group before), or under the pool a unit of two rows and four columns (W % 4 == 0, H even).
template <bool POOL>
struct Cursor {
  int n, a, b;                                                   // image; POOL: row pair, quad of columns; else a = 0, b = group
  int bn, ba;                                                    // how many b per a, a per image
  int dn, da, db;                                                // one chunk on
  __device__ __forceinline__ Cursor(const PwBwdArgs &p, long long first, int per_chunk) {
    bn = POOL ? p.W >> 2 : (p.H * p.W + 3) >> 2;
    ba = POOL ? p.H >> 1 : 1;
    const int per = bn * ba;
    n = (int)(first / per);
    const int r = (int)(first - (long long)n * per);
    a = r / bn, b = r - a * bn;
    dn = per_chunk / per;
    const int s = per_chunk - dn * per;
    da = s / bn, db = s - da * bn;
  }
  __device__ __forceinline__ void next() {
    b += db;
    const bool cb = b >= bn;
    b -= cb ? bn : 0;
    a += da + (cb ? 1 : 0);
    const bool ca = a >= ba;
    a -= ca ? ba : 0;
    n += dn + (ca ? 1 : 0);
  }
  // pixel of the map at which the group (the unit's first row) starts
  __device__ __forceinline__ int pixel(const PwBwdArgs &p) const {
    if (POOL) return 2 * a * p.W + 4 * b;
    const int last = p.H * p.W - 4;
    return 4 * b < last ? 4 * b : last;
  }
};

// sixteen lanes give the addresses of four rows of sixteen 2-byte values (four lanes a row); lane i of them receives column i
__device__ __forceinline__ uintx2 read_transposed(const char *q) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4 *lds4;
  return __builtin_bit_cast(uintx2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(const_cast<char *>(q))));
#else
  (void)q;
  return uintx2{0u, 0u};
#endif
}

// the per-channel values that dz is made of
struct RowConst {
  float sc, sh, scs, shs, mu, rs, f, db, dg;
};

__device__ __forceinline__ float bn_backward(const RowConst &k, float m, float g, float z) {
  return k.f * (m * g - k.db - ((z - k.mu) * k.rs) * k.dg);
}

// one value of dz, from memory (SRC as the kernel's)
template <int SRC, bool HS>
__device__ __forceinline__ float dz_value(const PwBwdArgs &p, const float *sums, int n, int o, int px) {
  const size_t HW = (size_t)p.H * p.W;
  const size_t at = ((size_t)n * p.Co + o) * HW + px;
  if (SRC == 0) return p.g[at];
  const float m = (float)p.N * (float)p.H * (float)p.W;
  RowConst k;
  k.mu = p.mean[o], k.rs = p.rstd[o], k.f = p.scale[o] / m, k.db = sums[2 * o], k.dg = sums[2 * o + 1];
  if (SRC == 1) return bn_backward(k, m, p.g[at], p.z[at]);
  k.sc = p.scale[o], k.sh = p.shift[o];
  k.scs = !HS || p.identity_skip ? 1.f : p.scale_s[o], k.shs = !HS || p.identity_skip ? 0.f : p.shift_s[o];
  auto act = [&](size_t i) {
    float b = fmaf(p.z[i], k.sc, k.sh);
    if (HS) b = b + fmaf(p.zs[i], k.scs, k.shs);
    return b;
  };
  float g;
  if (SRC == 2) {
    const float b = act(at);
    g = b > 0.f ? p.gscale * (fmaxf(b, 0.f) - p.t[at]) : 0.f;
  } else {
    const int y = px / p.W, x = px - y * p.W;
    const size_t w0 = ((size_t)n * p.Co + o) * HW + (size_t)(y & ~1) * p.W + (x & ~1);
    float pv = fmaxf(act(w0), 0.f);
    int best = 0;
    for (int q = 1; q < 4; ++q) {
      const float v = fmaxf(act(w0 + (size_t)(q >> 1) * p.W + (q & 1)), 0.f);
      if (v > pv) pv = v, best = q;
    }
    const float d = pv - p.t[(((size_t)n * p.Co + o) * (p.H / 2) + y / 2) * (p.W / 2) + x / 2];
    const float gk = pv > 0.f ? p.gscale * d : 0.f;
    g = best == 2 * (y & 1) + (x & 1) ? gk : 0.f;
  }
  return bn_backward(k, m, g, p.z[at]);
}
}  // namespace

// SRC: where dz comes from.  0: it is given (p.g).  1: BatchNorm backward of p.g with p.z.  2, 3: the block's head, without and with the
// 2x2 max-pool, from the target p.t, p.z and (HS) a second input p.zs.  The channel sums that 1 to 3 need are finished here from
// the partials of the kernel before, by every workgroup in the same order; the first one stores them.
template <int BM, int SRC, bool HS>
__global__ __launch_bounds__(kThreads) void pw_bwd_kernel(PwBwdArgs p) {
  constexpr bool POOL = SRC == 3;
  constexpr int PX = bwd_px(BM), PITCH = bwd_pitch(BM), PLANE = (BM + 64) * PITCH, COPY = bwd_copy(BM);
  constexpr int PER = POOL ? PX / 8 : PX / 4;                 // units or groups a chunk
  constexpr int VA = POOL ? 2 : 1;                            // vectors of four pixels a unit or group has
  constexpr int RS = 512 / PER;                               // rows that the loaders take at a time
  constexpr int NA = BM / RS;                                 // rows of dz a loader thread has
  constexpr bool HALF = POOL && BM == 128;                    // units of u are shared by two threads, a row each
  constexpr int VB = HALF ? 1 : VA;
  constexpr int NB = HALF ? 1 : 64 / RS;
  // Register sets: one is stashed, the others' chunks are on their way.  (Three at 64 rows do not quite fit 168 registers: seven are spilled
  // under a head without a pool, one inside a block.)
  constexpr int SETS = HS ? 2 : 3;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  constexpr int TILES = BM == 128 ? 2 : 1, TILE = bwd_tile(BM);
  float *const tiles = reinterpret_cast<float *>(lds + 2 * COPY);                     // finished tiles of du: [2 chunks][TILES][64 channels][pixels]
  float *const sums = reinterpret_cast<float *>(lds + 2 * COPY + bwd_exchange(BM));   // [Co][dbeta, dgamma]
  double *const loss = reinterpret_cast<double *>(sums + 2 * 128);                    // of the four MFMA waves

  const bool loader = threadIdx.x >= 256;
  const int tid = loader ? threadIdx.x - 256 : threadIdx.x, lane = tid & 63;
  const int lin = xcd_contiguous(blockIdx.x, gridDim.x);      // the column tiles of one range of pixels are neighbours on a die
  const int split = lin / p.geo.tiles_n, c0 = 64 * (lin - split * p.geo.tiles_n);
  const int HW = p.H * p.W;
  const int nch = p.geo.chunks_per_split;
  const long long first = (long long)split * nch * PER;       // first group or unit

  if (loader) {
    const int kq = tid % PER, r0 = tid / PER;
    const int rb0 = HALF ? tid / 8 : r0, half = HALF ? (tid / PER) & 1 : 0;
    unsigned offa[NA], offb[NB];
#pragma unroll
    for (int j = 0; j < NA; ++j) {
      const int row = r0 + RS * j;
      offa[j] = (unsigned)(row < p.Co ? row : p.Co - 1) * (unsigned)HW * 4u;     // a row past the last repeats it, and is never stored
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int row = c0 + rb0 + RS * j;
      offb[j] = (unsigned)(row < p.Ci ? row : p.Ci - 1) * (unsigned)HW * 4u;
    }
    const unsigned sizea = (unsigned)p.N * p.Co * HW * 4u;
    auto buffer = [](const float *q, unsigned bytes) {
      return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(q), 0, (int)(q ? bytes : 0u), 0x00020000);
    };
    const __amdgpu_buffer_rsrc_t rg = buffer(SRC < 2 ? p.g : p.t, POOL ? sizea / 4 : sizea);
    const __amdgpu_buffer_rsrc_t rz = buffer(p.z, sizea), rs = buffer(HS ? p.zs : nullptr, sizea);
    const __amdgpu_buffer_rsrc_t ru = buffer(p.u, (unsigned)p.N * p.Ci * HW * 4u);
    auto load4 = [](const __amdgpu_buffer_rsrc_t &r, unsigned off) { return __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0)); };

    Cursor<POOL> at(p, first + kq, PER);
    f4 vg[SETS][NA], vz[SETS][NA][VA], vs[SETS][NA][VA], vu[SETS][NB][VB];
    int vdup[SETS];
    auto fetch = [&](int s) {
      // nothing here is conditional: the compiler then knows how many loads are in flight.  (Past the workgroup's range the chunks are the
      // next one's, fetched for nothing: one or two, 50.9 MB read for 41.9 at 64 -> 128, 16x16, batch 128, four chunks a workgroup.)
      const bool ok = at.n < p.N;
      const int px = at.pixel(p);
      vdup[s] = POOL ? 0 : 4 * at.b - px;
      const unsigned ba = ok ? ((unsigned)at.n * (unsigned)p.Co * (unsigned)HW + (unsigned)px) * 4u : kPast;
      const unsigned bb = ok ? ((unsigned)at.n * (unsigned)p.Ci * (unsigned)HW + (unsigned)px) * 4u : kPast;
#pragma unroll
      for (int j = 0; j < NA; ++j) {
        if (SRC > 0) {
#pragma unroll
          for (int v = 0; v < VA; ++v) {
            vz[s][j][v] = load4(rz, ba + offa[j] + (unsigned)(v * p.W) * 4u);
            if (HS) vs[s][j][v] = load4(rs, ba + offa[j] + (unsigned)(v * p.W) * 4u);
          }
        }
        if (POOL) {                                       // two pooled values
          const unsigned bt = ok ? ((unsigned)at.n * (unsigned)p.Co * (unsigned)HW + (unsigned)(2 * at.a * p.W + 8 * at.b)) : kPast;
          const f2 t = __builtin_bit_cast(f2, __builtin_amdgcn_raw_buffer_load_b64(rg, (bt + offa[j] / 4), 0, 0));
          vg[s][j] = f4{t[0], t[1], 0.f, 0.f};
        } else {
          vg[s][j] = load4(rg, ba + offa[j]);
        }
      }
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int v = 0; v < VB; ++v) vu[s][j][v] = load4(ru, bb + offb[j] + (unsigned)((v + half) * p.W) * 4u);
      at.next();
    };

    const float m = (float)p.N * (float)p.H * (float)p.W;
    RowConst k[NA];
#pragma unroll
    for (int j = 0; j < NA; ++j) {
      const int row = r0 + RS * j, o = row < p.Co ? row : p.Co - 1;
      if (SRC > 0) {
        k[j].sc = p.scale[o], k[j].mu = p.mean[o], k[j].rs = p.rstd[o];
        k[j].f = k[j].sc / m;
        k[j].sh = SRC > 1 ? p.shift[o] : 0.f;
        k[j].scs = HS && !p.identity_skip ? p.scale_s[o] : 1.f;
        k[j].shs = HS && !p.identity_skip ? p.shift_s[o] : 0.f;
      }
    }
    __builtin_amdgcn_sched_barrier(0);                     // (loads complete in order: these few before the chunks')
#pragma unroll
    for (int i = 0; i < SETS - 1; ++i) fetch(i);
    __syncthreads();                                       // the channel sums are there
    if (SRC > 0) {
#pragma unroll
      for (int j = 0; j < NA; ++j) {
        const int row = r0 + RS * j, o = row < p.Co ? row : p.Co - 1;
        k[j].db = sums[2 * o], k[j].dg = sums[2 * o + 1];
      }
    }
    auto put = [&](char *row, const f4 &w) {
      unsigned q[2][3];
#pragma unroll
      for (int h = 0; h < 2; ++h) split3_bf16(w[2 * h], w[2 * h + 1], q[h]);
#pragma unroll
      for (int pc = 0; pc < 3; ++pc) *reinterpret_cast<uintx2 *>(row + pc * PLANE) = uintx2{q[0][pc], q[1][pc]};
    };
    auto stash = [&](int c, int s) {
      char *const copy = lds + (c & 1) * COPY;
#pragma unroll
      for (int j = 0; j < NA; ++j) {
        f4 w[VA];
        if (SRC == 0) {
          w[0] = vg[s][j];
        } else if (SRC == 1) {
#pragma unroll
          for (int e = 0; e < 4; ++e) w[0][e] = bn_backward(k[j], m, vg[s][j][e], vz[s][j][0][e]);
        } else {
          f4 b[VA];
#pragma unroll
          for (int v = 0; v < VA; ++v)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              b[v][e] = fmaf(vz[s][j][v][e], k[j].sc, k[j].sh);
              if (HS) b[v][e] += fmaf(vs[s][j][v][e], k[j].scs, k[j].shs);
            }
          if constexpr (SRC == 2) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float d = fmaxf(b[0][e], 0.f) - vg[s][j][e];
              const float g = b[0][e] > 0.f ? p.gscale * d : 0.f;
              w[0][e] = bn_backward(k[j], m, g, vz[s][j][0][e]);
            }
          } else {
#pragma unroll
            for (int wv = 0; wv < 2; ++wv) {
              // window order (row, col): (0,0) (0,1) (1,0) (1,1); strict '>': the first maximum wins
              float pv = fmaxf(b[0][2 * wv], 0.f);
              int best = 0;
#pragma unroll
              for (int q = 1; q < 4; ++q) {
                const float y = fmaxf(b[q >> 1][2 * wv + (q & 1)], 0.f);
                if (y > pv) pv = y, best = q;
              }
              const float d = pv - vg[s][j][wv];
              const float gk = pv > 0.f ? p.gscale * d : 0.f;
#pragma unroll
              for (int q = 0; q < 4; ++q)
                w[q >> 1][2 * wv + (q & 1)] = bn_backward(k[j], m, q == best ? gk : 0.f, vz[s][j][q >> 1][2 * wv + (q & 1)]);
            }
          }
        }
        if (!POOL && HW % 4) {                             // pixels that the group before has had
#pragma unroll
          for (int e = 0; e < 4; ++e) w[0][e] = e < vdup[s] ? 0.f : w[0][e];
        }
#pragma unroll
        for (int v = 0; v < VA; ++v) {
          put(copy + (r0 + RS * j) * PITCH + 8 * (v * PER + kq), w[v]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int v = 0; v < VB; ++v)
          put(copy + (BM + rb0 + RS * j) * PITCH + 8 * ((v + half) * PER + kq), vu[s][j][v]);
    };
    // du of the next chunk to store, from LDS to where this thread's part of u was
    Cursor<POOL> done(p, first + kq, PER);
    const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(p.du, 0, (int)((unsigned)p.N * p.Ci * HW * 4u), 0x00020000);
    auto store_du = [&](int c) {
      const bool ok = done.n < p.N;
      const int px = done.pixel(p), dup = POOL ? 0 : 4 * done.b - px;
      const unsigned bb = ok ? ((unsigned)done.n * (unsigned)p.Ci * (unsigned)HW + (unsigned)px) * 4u : kPast;
      const float *const T = tiles + (c & 1) * (TILES * TILE);
      float odd = 0.f;
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int v = 0; v < VB; ++v) {
          const float *const at4 = T + (rb0 + RS * j) * bwd_tile_row(BM) + 4 * ((v + half) * PER + kq);
          f4 d = *reinterpret_cast<const f4 *>(at4);
          if (TILES == 2) d += *reinterpret_cast<const f4 *>(at4 + TILE);
          const unsigned off = c0 + rb0 + RS * j < p.Ci ? bb + offb[j] + (unsigned)((v + half) * p.W) * 4u : kPast;
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uintx4, d), rd, dup ? kPast : off, 0, 0);
          if (!POOL && __any(dup)) {                       // an image's last group, some of whose pixels the one before has had
#pragma unroll
            for (int e = 1; e < 4; ++e)
              __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, (float)d[e]), rd, dup && e >= dup ? off + 4u * e : kPast, 0, 0);
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) odd = fmaf(d[e], 0.f, odd);
        }
      if (__any(odd != odd)) {
        // no numbers, or infinite: again in fp32, where this thread has just put them
        __threadfence();
#pragma unroll 1
        for (int i = 0; ok && i < NB * VB * 4; ++i) {
          const int e = i & 3, v = (i >> 2) % VB, ch = c0 + rb0 + RS * (i / (4 * VB));
          if (ch >= p.Ci || e < dup) continue;
          const int at_px = px + (v + half) * p.W + e;
          float *const q = p.du + ((size_t)done.n * p.Ci + ch) * HW + at_px;
          const float have = __builtin_nontemporal_load(q);
          if (have == have) continue;
          float s = 0.f;
#pragma unroll 1
          for (int o = 0; o < p.Co && s == s; ++o) s = fmaf(p.w[(size_t)o * p.Ci + ch], dz_value<SRC, HS>(p, sums, done.n, o, at_px), s);
          *q = s;
        }
      }
      done.next();
    };
    int c = 0;
    for (; c + SETS <= nch; c += SETS) {                   // (no way out in its middle: see pw_wgrad_mfma.hip)
#pragma unroll
      for (int i = 0; i < SETS; ++i) {
        fetch((i + SETS - 1) % SETS);
        __builtin_amdgcn_sched_barrier(0);
        stash(c + i, i);
        if (c + i >= 2) store_du(c + i - 2);
        __syncthreads();
      }
    }
#pragma unroll
    for (int i = 0; i < SETS - 1; ++i)
      if (c + i < nch) {
        stash(c + i, i);
        if (c + i >= 2) store_du(c + i - 2);
        __syncthreads();
      }
    if (nch >= 2) store_du(nch - 2);
    __syncthreads();
    store_du(nch - 1);
    return;
  }

  // ------------------------------------------------------------------ MFMA waves
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l31 = lane & 31, lh = lane >> 5;
  constexpr int MBW = BM / 64;                             // blocks of 32 rows of dP a wave has, 32 columns wide
  constexpr int DU_SUM = BM == 128 ? 2 : 1;                // chunks of channels whose sum is formed from zero
  constexpr bool KH = BM == 128;                           // du: waves 2 and 3 sum the upper half of the channels
  const int wm = wave & 1, wn = wave >> 1;
  const int cb = wave & 1, hi = wave >> 1;                 // du: block of 32 input channels; upper half of the channels, or of the pixels
  const int nk = (p.Co + 15) / 16;

  if (SRC > 0) {
    for (int e = tid; e < 2 * p.Co; e += 256) {            // one of the two sums of a channel each
      const int o = e >> 1, which = e & 1;
      float v;
      if (p.sum_partial) {
        const float *q = p.sum_partial + (size_t)o * p.sum_row + p.sum_at + which;
        const size_t step = (size_t)p.Co * p.sum_row;
        double t = 0.0;
#pragma unroll 1
        for (int i = 0; i < p.sum_parts; i += 16) {        // sixteen loads in flight whatever their number: a remainder loads one
          float x[16];                                     // after the other (33.5 -> 30.3 us at 100 -> 67, 27x23, batch 77: 47 parts)
#pragma unroll
          for (int j = 0; j < 16; ++j) x[j] = q[(size_t)(i + j < p.sum_parts ? i + j : p.sum_parts - 1) * step];
#pragma unroll
          for (int j = 0; j < 16; ++j) t += i + j < p.sum_parts ? (double)x[j] : 0.0;
        }
        v = (float)t;
        if (lin == 0) (which ? p.dgamma : p.dbeta)[o] = v;
      } else {
        v = (which ? p.dgamma : p.dbeta)[o];
      }
      sums[e] = v;
    }
    if (SRC > 1 && p.loss_out && lin == 0) {
      double l = 0.0;
      const int all = p.sum_parts * p.Co;
#pragma unroll 1
      for (int e = tid; e < all; e += 16 * 256) {
        float x[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) x[j] = p.sum_partial[(size_t)(e + 256 * j < all ? e + 256 * j : all - 1) * 3];
#pragma unroll
        for (int j = 0; j < 16; ++j) l += e + 256 * j < all ? (double)x[j] : 0.0;
      }
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) l += __shfl_xor(l, d, 64);
      if (lane == 0) loss[wave] = l;
    }
  }

  // P's pieces: this wave's block of 32 input channels, four chunks of 16 output channels
  uintx4 w[4][3];
  {
    const int nblk = p.w_blocks;
    const int blk = c0 / 32 + cb < nblk ? c0 / 32 + cb : nblk - 1;        // (a block past the last is never stored)
    const uintx4 *const src = reinterpret_cast<const uintx4 *>(p.wpk) + (size_t)blk * nk * 192 + lane;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int ks = (KH ? 4 * hi : 0) + i;
#pragma unroll
      for (int pc = 0; pc < 3; ++pc) w[i][pc] = src[(size_t)(ks < nk ? ks : nk - 1) * 192 + pc * 64];
    }
  }

  floatx16 acc[MBW];
#pragma unroll
  for (int a = 0; a < MBW; ++a)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[a][r] = 0.f;
  floatx16 t;                                              // the tile of du

  // operand addresses
  const int i16 = lane & 15;
  const int tr_px = (KH ? 0 : 32 * hi) + 16 * ((lane >> 4) & 1) + 4 * (i16 & 3);
  float *const tile = tiles + (KH ? hi * TILE : 0) + (32 * cb + l31) * bwd_tile_row(BM) + (KH ? 0 : 32 * hi) + 4 * lh;
  __syncthreads();                                         // the channel sums are there (for the loaders)
  if (SRC > 1 && p.loss_out && lin == 0 && tid == 0) p.loss_out[0] = (float)(((loss[0] + loss[1]) + (loss[2] + loss[3])) * (double)p.loss_scale);
#pragma unroll
  for (int i = 0; i < 4; ++i)                              // (no such chunk of channels: multiplied all the same, a branch would cost more)
    if ((KH ? 4 * hi : 0) + i >= nk) w[i][0] = w[i][1] = w[i][2] = uintx4{0u, 0u, 0u, 0u};
  __syncthreads();                                         // chunk 0 is staged
  for (int c = 0; c < nch; ++c) {
    const char *const copy = lds + (c & 1) * COPY;
    // Steps of du (16 channels) and of dP (16 pixels, a block of 32 rows) in turn, the next one's operands on their way while one
    // multiplies.  Fenced: left alone the compiler moves every read down to its product and the wave waits for LDS a dozen times a chunk.
    uintx4 x[3], a[3], b[3];
    auto read_x = [&](int i) {
      const int ks = (KH ? 4 * hi : 0) + i;
      const int o0 = 16 * ks < p.Co - 16 ? 16 * ks : p.Co - 16;      // the ragged last chunk reaches back; its weights there are zero
      const char *const src = copy + (o0 + 8 * lh + (i16 >> 2)) * PITCH + 2 * tr_px;
#pragma unroll
      for (int pc = 2; pc >= 0; --pc) {
        const uintx2 lo = read_transposed(src + pc * PLANE), up = read_transposed(src + pc * PLANE + 4 * PITCH);
        x[pc] = uintx4{lo[0], lo[1], up[0], up[1]};
      }
    };
    const char *const S = copy + l31 * PITCH + 16 * lh;
    auto read_ab = [&](int i) {
      const int s = i / MBW, mb = i % MBW;
#pragma unroll
      for (int pc = 2; pc >= 0; --pc) {
        a[pc] = *reinterpret_cast<const uintx4 *>(S + pc * PLANE + (wm * MBW + mb) * 32 * PITCH + 32 * s);
        if (mb == 0) b[pc] = *reinterpret_cast<const uintx4 *>(S + pc * PLANE + (BM + wn * 32) * PITCH + 32 * s);
      }
    };
    read_x(0);
    floatx16 part;                                         // du over DU_SUM chunks of channels
    static_assert(PX / 16 * MBW == 4, "four steps each");
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      read_ab(i);
      if (i % DU_SUM == 0) {
#pragma unroll
        for (int r = 0; r < 16; ++r) part[r] = 0.f;
      }
      __builtin_amdgcn_sched_barrier(0);
      constexpr int PW[6] = {0, 0, 1, 2, 1, 0}, PXC[6] = {2, 1, 1, 0, 0, 0};       // weights by dz, small products first
#pragma unroll
      for (int q = 0; q < 6; ++q)
        part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x[PXC[q]]), __builtin_bit_cast(bf16x8, w[i][PW[q]]), part, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (i < 3) read_x(i + 1);
      __builtin_amdgcn_sched_barrier(0);
      constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};        // dz by u
#pragma unroll
      for (int q = 0; q < 6; ++q)
        acc[i % MBW] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[PA[q]]), __builtin_bit_cast(bf16x8, b[PB[q]]),
                                                               acc[i % MBW], 0, 0, 0);
      if (i % DU_SUM == DU_SUM - 1) t = i < DU_SUM ? part : t + part;
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)                            // register 4 r + e: pixel 8 r + 4 (lane / 32) + e of channel lane % 32
      *reinterpret_cast<f4 *>(tile + (c & 1) * (TILES * TILE) + 8 * r) = f4{t[4 * r], t[4 * r + 1], t[4 * r + 2], t[4 * r + 3]};
    __syncthreads();                                       // chunk c consumed; chunk c + 1 is staged
  }

  // ---- dP: accumulator register r of lane l holds row 8*(r/4) + 4*(l/32) + r%4, column l%32
  float *const dst = p.partial + (size_t)split * p.Co * p.Ci;
  const int col = c0 + wn * 32 + l31;
  float odd = 0.f;
#pragma unroll
  for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int o = (wm * MBW + mb) * 32 + 8 * (r / 4) + 4 * lh + r % 4;
      if (o < p.Co && col < p.Ci) dst[(size_t)o * p.Ci + col] = acc[mb][r];
      odd = fmaf(acc[mb][r], 0.f, odd);
    }
  if (__any(odd != odd)) {
#pragma unroll 1
    for (int i = 0; i < 16 * MBW; ++i) {
      const int r = i & 15, o = (wm * MBW + (i >> 4)) * 32 + 8 * (r / 4) + 4 * lh + r % 4;
      if (o >= p.Co || col >= p.Ci) continue;
      float *const q = dst + (size_t)o * p.Ci + col;
      if (*q == *q) continue;
      float s = 0.f;
      Cursor<POOL> g(p, first, 1);
#pragma unroll 1
      for (int j = 0; j < nch * PER && g.n < p.N && s == s; ++j, g.next()) {
        const int px = g.pixel(p);
#pragma unroll 1
        for (int e = POOL ? 0 : 4 * g.b - px; e < 4 * VA; ++e) {
          const int at_px = px + (e >> 2) * p.W + (e & 3);
          s = fmaf(dz_value<SRC, HS>(p, sums, g.n, o, at_px), p.u[((size_t)g.n * p.Ci + col) * HW + at_px], s);
        }
      }
      *q = s;
    }
  }
}

bool pw_bwd_geom(int N, int Co, int Ci, int H, int W, bool pooled, const PwGeom &pdg, PwBwdGeom &g) {
  const unsigned long long HW = (unsigned long long)H * W;
  if (!pdg.split || pdg.K != Co || Co < 16 || Co > 128 || HW < 4) return false;
  if (pooled && (W % 4 || H % 2)) return false;
  if ((unsigned long long)N * (Co > Ci ? Co : Ci) * HW * sizeof(float) > (1ull << 31)) return false;
  g = PwBwdGeom{};
  g.bm = Co <= 64 ? 64 : 128;
  g.pooled = pooled;
  g.tiles_n = cdiv(Ci, 64);
  const int per = bwd_px(g.bm) / (pooled ? 8 : 4);
  const long long units = (long long)N * (pooled ? HW / 8 : (HW + 3) / 4);
  const int nchunks = (int)((units + per - 1) / per);
  int want = 256 / g.tiles_n;                              // one workgroup per compute unit (its LDS allows no more)
  if (want < 1) want = 1;
  if (want > nchunks) want = nchunks;
  g.chunks_per_split = cdiv(nchunks, want);
  g.splits = cdiv(nchunks, g.chunks_per_split);
  g.lds_bytes = bwd_lds(g.bm);
  return true;
}

namespace {
template <class F>
hipError_t bwd_each(F f) {
  hipError_t e;
#define PBKD_BWD(BM)                                                \
  if ((e = f(&pw_bwd_kernel<BM, 0, false>, BM, 0, false)) != hipSuccess) return e; \
  if ((e = f(&pw_bwd_kernel<BM, 1, false>, BM, 1, false)) != hipSuccess) return e; \
  if ((e = f(&pw_bwd_kernel<BM, 2, false>, BM, 2, false)) != hipSuccess) return e; \
  if ((e = f(&pw_bwd_kernel<BM, 2, true>, BM, 2, true)) != hipSuccess) return e;   \
  if ((e = f(&pw_bwd_kernel<BM, 3, false>, BM, 3, false)) != hipSuccess) return e; \
  if ((e = f(&pw_bwd_kernel<BM, 3, true>, BM, 3, true)) != hipSuccess) return e;
  PBKD_BWD(64)
  PBKD_BWD(128)
#undef PBKD_BWD
  return hipSuccess;
}
}  // namespace

hipError_t init_pw_bwd_attributes() {
  return bwd_each([](void (*k)(PwBwdArgs), int bm, int, bool) {
    return hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bwd_lds(bm));
  });
}

hipError_t launch_pw_bwd(const PwBwdArgs &a, hipStream_t s) {
  const PwBwdGeom &g = a.geo;
  const unsigned long long HW = (unsigned long long)a.H * a.W;
  const bool head = a.src >= 2;
  if (a.N < 1 || a.Co < 16 || a.Co > g.bm || (g.bm != 64 && g.bm != 128) || a.Ci < 1 || g.tiles_n != cdiv(a.Ci, 64) || HW < 4 ||
      a.src < 0 || a.src > 3 || (a.src == 3) != g.pooled || (a.src == 3 && (a.W % 4 || a.H % 2)) || a.w_blocks < cdiv(a.Ci, 32) ||
      (unsigned long long)a.N * (a.Co > a.Ci ? a.Co : a.Ci) * HW * sizeof(float) > (1ull << 31) || g.splits < 1 ||
      (long long)g.splits * g.tiles_n > 65535)
    return hipErrorInvalidValue;
  const long long units = (long long)a.N * (g.pooled ? HW / 8 : (HW + 3) / 4), per = bwd_px(g.bm) / (g.pooled ? 8 : 4);
  if ((long long)g.splits * g.chunks_per_split * per < units) return hipErrorInvalidValue;
  if (!a.u || !a.du || !a.partial || !a.wpk || !a.w || (a.src < 2 && !a.g) || (head && (!a.t || !a.shift)) || (a.zs && !head) ||
      (a.src > 0 && (!a.z || !a.scale || !a.mean || !a.rstd || !a.dgamma || !a.dbeta)) || (a.zs && !a.identity_skip && (!a.scale_s || !a.shift_s)))
    return hipErrorInvalidValue;
  bool found = false;
  const hipError_t e = bwd_each([&](void (*k)(PwBwdArgs), int bm, int src, bool hs) {
    if (bm != g.bm || src != a.src || hs != (a.zs != nullptr)) return hipSuccess;
    found = true;
    hipLaunchKernelGGL(k, dim3(g.splits * g.tiles_n), dim3(kThreads), g.lds_bytes, s, a);
    return hipGetLastError();
  });
  return e != hipSuccess ? e : found ? hipSuccess : hipErrorInvalidValue;
}

}  // namespace pbkd
