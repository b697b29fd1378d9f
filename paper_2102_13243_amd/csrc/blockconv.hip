// fp32 3x3 / stride 1 / padding 1 convolutions of 16, 32 or 64 channels in and out: the layers of a CIFAR ResNet, alone or
// with the BatchNorms on either side of them inside the same launch.
//
// Such a layer moves 8 to 17 MB and multiplies for 4 us; as separate kernels its convolution, the statistics, the
// normalisation and, backward, the two passes of the BatchNorm's pullback each cost a launch, a ramp and a drain (4 to 6 us
// around 1.5 us of traffic).  Here a workgroup owns a band of whole rows of one image, and
//   forward: x = act(BN(z) (+ residual)) is made while the band's input patch is brought into LDS, from z, the output of the
//     convolution before, and that convolution's table of partial sums; the band's own rows of x are stored; the convolution
//     runs out of LDS and leaves the partial sums of the BatchNorm behind it;
//   backward: the same with dz, the cotangent that BN's pullback gives its convolution, made from the cotangent of BN's output
//     (and the residual's cotangent stored); the convolution is the input pullback (the filter turned by 180 degrees, its
//     channel axes swapped), and the sums that the pullback of the BatchNorm before it needs are taken from its result.
// The patch's border of one pixel is made twice, by neighbours, from the same numbers.
//
// Measured in the steps of a ResNet-56 (us per launch, beside the second stream's filter gradients), 128 x 32 x 32 x 16 and its
// halvings: forward convolution 12.8 + statistics 4.3 + application 4.3, three launches, before; 14.7 to 15.9 now.  Backward 5.7 +
// 5.8 + 12.5 before; 15.6 to 18.7 now (59 MB at 16 channels, of which a step has to move that much).  The rest of a launch:
// 3 us of start and drain, 4.3 of MFMAs, the loads in front of them.  Batch 128: 3.09 -> 2.47 ms, batch 50 with 40 x 40 images, whose widths the
// kernel before did not take, 3.14 -> 2.16.
// One big workgroup per CU, for each repeats the sum over the table in front; 64-channel layers need more than 64 KB of LDS.
//
// Matrix part: v_mfma_f32_16x16x4_f32, a wavefront multiplies G blocks of 16 pixels by 16 outputs; a lane's four MFMA steps
// take four adjacent channels, so that both operands are read 16 bytes at a time.  Patch pixels are C + 4 floats apart, and the
// 16-byte chunks of filter row n are permuted by (n / 4) % 4: the lanes of either read fall into different banks.
#include "s4tf_internal.h"
#include "igemm_args.h"

namespace s4tf {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

struct BlockArgs {
  BlockConv b;
  int RB, bands, PW, OBW, WPX;  // rows per band, bands per image, patch width, blocks of 16 outputs and of G*16 pixels per workgroup
  uint32_t magicPW, magicW, magicPeriod;
  int shiftPW, shiftW, shiftPeriod;
  double inv_M, inv_rows, inv_last;
  float inv_band[2], inv_rest[2];  // of a whole band and of an image's last: 1 / its pixels, 1 / those of its last, partial wavefront
};

__device__ inline f32x4 load4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ inline __amdgpu_buffer_rsrc_t make_buffer(const float* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, (int)bytes, 0x00020000);
}
__device__ inline f32x4 buffer_load4(__amdgpu_buffer_rsrc_t r, int element) {  // zeros for element -1
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, element * 4, 0, 0));
}

// A barrier for what lies in LDS: unlike __syncthreads it does not wait for stores to global memory (nor for loads that nobody
// has used yet)
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory"); }

// v + the same of another lane: within a row of 16 lanes by DPP, which costs a few cycles where a shuffle through LDS takes
// a hundred; every step of a sum over 2^k lanes leaves the partial sum in all of them
template <int CTRL> __device__ inline double dpp_add(double v) {
  const uint64_t bits = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)bits, CTRL, 0xf, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(bits >> 32), CTRL, 0xf, 0xf, true);
  return v + __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ inline double lanes_sum(double v, int lanes) {
  if (lanes > 1) v = dpp_add<0xB1>(v);   // quad_perm [1,0,3,2]
  if (lanes > 2) v = dpp_add<0x4E>(v);   // quad_perm [2,3,0,1]
  if (lanes > 4) v = dpp_add<0x141>(v);  // row_half_mirror: the other four of eight
  if (lanes > 8) v = dpp_add<0x140>(v);  // row_mirror: the other eight of sixteen
  if (lanes > 16) v += __shfl_xor(v, 16, 64);
  if (lanes > 32) v += __shfl_xor(v, 32, 64);
  return v;
}

// BatchNorm in front of the patch: per-channel coefficients into coef[5][C].  Every workgroup adds up the whole table (16 to
// 130 KB, from L2), and nothing else can run before it is done: its loads are issued first of all (issue), as many at once as
// the registers hold, and waited for while those of the patch are on their way (finish).
template <int C, bool FLIP> struct Table {
  static constexpr int NF = 2, ND = 4;
  f32x4 sv[NF], qv[NF];  // forward: runs of this thread's channel
  f64x2 dv[ND];          // backward: rows of two adjacent columns
  int lpc, c, l, count;

  __device__ inline void load_f(const BlockConv& b, int i0) {
    const float* __restrict__ srow = b.part + (long long)c * count;
    const float* __restrict__ qrow = b.part + ((long long)C + c) * count;
#pragma unroll
    for (int u = 0; u < NF; ++u) {
      const int i = 4 * (i0 + u * lpc);
      sv[u] = qv[u] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (i + 3 < count) {
        sv[u] = *reinterpret_cast<const f32x4u*>(srow + i);
        qv[u] = *reinterpret_cast<const f32x4u*>(qrow + i);
      } else {
#pragma unroll
        for (int e = 0; e < 3; ++e)
          if (i + e < count) { sv[u][e] = srow[i + e]; qv[u][e] = qrow[i + e]; }
      }
    }
  }
  __device__ inline void load_d(const BlockConv& b, int z0) {
    const f64x2* __restrict__ rows = reinterpret_cast<const f64x2*>(b.dpart) + c;
#pragma unroll
    for (int u = 0; u < ND; ++u) dv[u] = z0 + u * lpc < count ? rows[(long long)(z0 + u * lpc) * C] : f64x2{0.0, 0.0};
  }
  __device__ inline void issue(const BlockConv& b) {
    const int T = blockDim.x, tid = threadIdx.x;
    count = b.runs.count;
    if constexpr (!FLIP) {
      lpc = 64;
      while (lpc * C > T) lpc >>= 1;
      c = tid / lpc;
      l = tid - c * lpc;
      if (c >= C) c = 0, l = count;  // (threads beyond the last channel)
      load_f(b, l);
    } else {
      lpc = T / C;
      l = tid / C;
      c = tid & (C - 1);
      load_d(b, l);
    }
  }
  // sh: scratch of 2*C doubles per wavefront
  __device__ inline void finish(const BlockArgs& a, float (*coef)[C], double* sh) {
    const BlockConv& b = a.b;
    const int T = blockDim.x, tid = threadIdx.x;
    const bool first = blockIdx.x == 0 && blockIdx.y == 0;
    if constexpr (!FLIP) {  // mean and 1/std out of sums and squared deviations (see bn_stats_from_runs_kernel)
      double S = 0.0, Q = 0.0;  // Q: squared deviations plus sum of s*s/n
      const bool even = b.runs.last == b.runs.rows;
      for (int i0 = l; 4 * i0 < count; i0 += NF * lpc) {
        if (i0 != l) load_f(b, i0);
#pragma unroll
        for (int u = 0; u < NF; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e) {  // (runs beyond the last are zeros)
            const double v = (double)sv[u][e];
            double inv = a.inv_rows;
            if (!even) {
              const int i = 4 * (i0 + u * lpc) + e;
              if (i - div_magic(i, a.magicPeriod, a.shiftPeriod) * b.runs.period == b.runs.period - 1) inv = a.inv_last;
            }
            S += v;
            Q += fma(v * inv, v, (double)qv[u][e]);
          }
      }
      S = lanes_sum(S, lpc);
      Q = lanes_sum(Q, lpc);
      if (l == 0) {
        const double m = S * a.inv_M;
        double var = (Q - S * m) * a.inv_M;
        if (var < 0.0) var = 0.0;
        const float mu = (float)m, is = (float)(1.0 / sqrt(var + (double)b.eps));
        coef[0][c] = mu;
        coef[1][c] = b.gamma[c] * is;
        coef[2][c] = b.beta[c];
        if (first) {
          b.mean[c] = mu;
          b.invstd[c] = is;
        }
      }
    } else {  // the pullback's coefficients out of the sums of dz and dz*xhat (see bn_vjp_apply_wide_kernel)
      f64x2 s = {0.0, 0.0};
      for (int z0 = l; z0 < count; z0 += ND * lpc) {
        if (z0 != l) load_d(b, z0);
#pragma unroll
        for (int u = 0; u < ND; ++u) s += dv[u];
      }
      if constexpr (C < 32) { s[0] += __shfl_xor(s[0], 16, 64); s[1] += __shfl_xor(s[1], 16, 64); }
      if constexpr (C < 64) { s[0] += __shfl_xor(s[0], 32, 64); s[1] += __shfl_xor(s[1], 32, 64); }
      if ((tid & 63) < C) *reinterpret_cast<f64x2*>(sh + (tid >> 6) * 2 * C + 2 * c) = s;
      lds_barrier();
      for (int k = tid; k < 2 * C; k += T) {
        double t = 0.0;
#pragma unroll 4
        for (int w = 0; w < (T >> 6); ++w) t += sh[w * 2 * C + k];
        const int ch = k & (C - 1);
        const float mean_s = (float)t * (float)a.inv_M, is = b.invstd[ch], gs = b.gamma[ch] * is;
        if (k < C) {
          coef[0][ch] = b.mean[ch];
          coef[1][ch] = gs;
          coef[2][ch] = b.mask_y ? 0.f : b.beta[ch];
          coef[3][ch] = gs * mean_s;
        } else {
          coef[4][ch] = gs * (is * mean_s);
        }
        if (first) (k < C ? b.dbeta : b.dgamma)[ch] = (float)t;
      }
    }
    lds_barrier();
  }
};

// FLIP: input pullback.  BN: the BatchNorm in front.
template <int C, int G, bool FLIP, bool BN>
__global__ __launch_bounds__(1024) void block_conv_kernel(const BlockArgs a) {
  extern __shared__ float smem[];
  constexpr int C4 = C / 4, C16 = C / 16, CS = C + 4, U = BN ? 3 : 4, FB = 4;
  __shared__ float coef[BN ? 5 : 1][C];
  const BlockConv& b = a.b;
  const int H = b.g.H, W = b.g.W, PW = a.PW, KT = C, OBW = a.OBW;
  float* wl = smem;                       // [OBW][9][C16][16 outputs][16 channels]
  float* patch = wl + OBW * 9 * C * 16;   // [RB + 2][PW][CS]
  const int T = blockDim.x, tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = blockIdx.x / a.bands, p0 = (blockIdx.x - n * a.bands) * a.RB, rows = min(a.RB, H - p0), n0 = blockIdx.y * OBW * 16;
  const long long img = (long long)n * H * W;

  // ---- loads of the first patch pieces and of the filter, before anything waits ----
  const int chunks = (a.RB + 2) * PW * C4, c4 = tid & (C4 - 1);
  const bool has2 = b.src2 != nullptr, has3 = FLIP && b.mask_y != nullptr;
  const uint32_t img_bytes = (uint32_t)H * W * C * 4u;  // loads beyond them (offset -1) give zeros
  const auto src = make_buffer(b.src + img * C, img_bytes), src2 = make_buffer(has2 ? b.src2 + img * C : b.src, img_bytes),
             src3 = make_buffer(has3 ? b.mask_y + img * C : b.src, img_bytes);
  f32x4 v1[U], v2[U], v3[U];
  int off[U], at[U];  // element offset in the image, -1: outside; LDS float, -1: none
  bool own[U];
  auto load = [&](int i0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * T, t = i / C4, pr = div_magic(t, a.magicPW, a.shiftPW), pw = t - pr * PW, h = p0 + pr - 1, w = pw - 1;
      const bool in = (i < chunks) & ((unsigned)h < (unsigned)H) & ((unsigned)w < (unsigned)W);
      at[u] = i < chunks ? t * CS + c4 * 4 : -1;
      off[u] = in ? (h * W + w) * C + c4 * 4 : -1;
      own[u] = in & (pr >= 1) & (pr <= rows) & (blockIdx.y == 0);
      v1[u] = buffer_load4(src, off[u]);
      if (BN && has2) v2[u] = buffer_load4(src2, off[u]);
      if (FLIP && BN && has3) v3[u] = buffer_load4(src3, off[u]);
    }
  };
  Table<C, FLIP> table;
  if constexpr (BN) table.issue(b);
  const int filter = 9 * C * OBW * 4;
  auto filter_source = [&](int i) {  // 16 bytes: forward four outputs of one channel, FLIP four channels of one output
    const int blk = i >> 6, ob = blk / (9 * C16), tc = blk - ob * (9 * C16), tap = tc / C16, cg = tc - tap * C16;
    if constexpr (FLIP) return ((8 - tap) * KT + n0 + ob * 16 + ((i >> 2) & 15)) * C + cg * 16 + (i & 3) * 4;
    else return (tap * C + cg * 16 + (i & 15)) * KT + n0 + ob * 16 + ((i >> 4) & 3) * 4;
  };
  auto filter_store = [&](int i, f32x4 v) {
    float* blk = wl + (i >> 6) * 256;
    if constexpr (FLIP) {
      const int o = (i >> 2) & 15;
      *reinterpret_cast<f32x4*>(blk + o * 16 + (((i & 3) ^ (o >> 2)) << 2)) = v;
    } else {
      const int ci = i & 15, o4 = (i >> 4) & 3;
#pragma unroll
      for (int j = 0; j < 4; ++j) blk[(o4 * 4 + j) * 16 + (((ci >> 2) ^ o4) << 2) + (ci & 3)] = v[j];
    }
  };
  f32x4 fv[FB];
#pragma unroll
  for (int f = 0; f < FB; ++f)
    if (tid + f * T < filter) fv[f] = load4(b.w + filter_source(tid + f * T));
  load(tid);

  if constexpr (BN) table.finish(a, coef, reinterpret_cast<double*>(patch));
#pragma unroll
  for (int f = 0; f < FB; ++f)
    if (tid + f * T < filter) filter_store(tid + f * T, fv[f]);
  for (int i0 = tid + FB * T; i0 < filter; i0 += FB * T) {
#pragma unroll
    for (int f = 0; f < FB; ++f)
      if (i0 + f * T < filter) fv[f] = load4(b.w + filter_source(i0 + f * T));
#pragma unroll
    for (int f = 0; f < FB; ++f)
      if (i0 + f * T < filter) filter_store(i0 + f * T, fv[f]);
  }

  // ---- the patch ----
  {
    f32x4 mu, sc, be, a0, a2;
    if constexpr (BN) {
      mu = load4(&coef[0][c4 * 4]); sc = load4(&coef[1][c4 * 4]); be = load4(&coef[2][c4 * 4]);
      if constexpr (FLIP) { a0 = load4(&coef[3][c4 * 4]); a2 = load4(&coef[4][c4 * 4]); }
    }
    const float lo = b.act != S4TF_ACT_NONE ? 0.f : -__builtin_inff(), hi = b.act == S4TF_ACT_RELU6 ? 6.f : __builtin_inff();
    float* __restrict__ made = b.made ? b.made + img * C : nullptr;
    const bool no_act = b.act == S4TF_ACT_NONE;
    float* dres = FLIP && b.dres ? b.dres + img * C : nullptr;
    for (int i0 = tid; i0 < chunks; i0 += U * T) {
      if (i0 != tid) load(i0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        f32x4 o = v1[u];
        if constexpr (BN) {
          if (off[u] >= 0) {
            f32x4 r;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              if constexpr (!FLIP) {
                float z = fmaf(v1[u][e] - mu[e], sc[e], be[e]);
                if (has2) z += v2[u][e];
                o[e] = fminf(fmaxf(z, lo), hi);
              } else {  // v1: cotangent of BN's output, v2: BN's input, v3: BN's output where a residual went into it
                const float xc = v2[u][e] - mu[e], y = has3 ? v3[u][e] : fmaf(xc, sc[e], be[e]);
                const float dz = (no_act | ((y > 0.f) & (y < hi))) ? v1[u][e] : 0.f;  // (bitwise: no branches)
                r[e] = dz;
                o[e] = fmaf(sc[e], dz, -fmaf(xc, a2[e], a0[e]));
              }
            }
            if (own[u]) {
              *reinterpret_cast<f32x4*>(made + off[u]) = o;
              if (FLIP && dres) {
                if (b.acc_dres) r += load4(dres + off[u]);
                *reinterpret_cast<f32x4*>(dres + off[u]) = r;
              }
            }
          }
        }
        if (at[u] >= 0) *reinterpret_cast<f32x4*>(patch + at[u]) = o;
      }
    }
  }
  lds_barrier();

  // ---- the product ----
  const int PX = rows * W, ob = wave / a.WPX, wp = wave - ob * a.WPX, m0 = wp * G * 16;
  const int live = min(max(PX - m0, 0), G * 16);  // this wavefront's pixels
  int abase[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const int m = min(m0 + g * 16 + l16, PX - 1), row = div_magic(m, a.magicW, a.shiftW), col = m - row * W;
    abase[g] = (row * PW + col) * CS + 4 * g4;
  }
  const int col = n0 + ob * 16 + l16;
  const long long out0 = (img + (long long)p0 * W + m0) * KT + col;
  // backward: what the sums of the BatchNorm in front need, on its way during the product
  float nz[G][4], ny[G][4], old[G][4];
  if constexpr (FLIP) {
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = g * 16 + 4 * g4 + v;
        const bool ok = m < live;
        nz[g][v] = (ok && b.npart) ? b.nz[out0 + (long long)m * KT] : 0.f;
        ny[g][v] = (ok && b.npart && b.ny) ? b.ny[out0 + (long long)m * KT] : 0.f;
        old[g][v] = (ok && b.accumulate) ? b.out[out0 + (long long)m * KT] : 0.f;
      }
  }
  f32x4 acc[G];
#pragma unroll
  for (int g = 0; g < G; ++g) acc[g] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float* wb = wl + ob * (9 * C16 * 256) + l16 * 16 + ((g4 ^ (l16 >> 2)) << 2);
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
      for (int cg = 0; cg < C16; ++cg) {
        f32x4 av[G];
        const f32x4 bv = load4(wb + ((r * 3 + s) * C16 + cg) * 256);
#pragma unroll
        for (int g = 0; g < G; ++g) av[g] = load4(patch + abase[g] + r * PW * CS + s * CS + cg * 16);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[g][e], bv[e], acc[g], 0, 0, 0);
      }

  if constexpr (!FLIP) {
    // (stored before the sums: the barriers do not wait for it)
    const float bias = b.bias ? b.bias[col] : 0.f;
    const float lo = b.conv_act != S4TF_ACT_NONE ? 0.f : -__builtin_inff(), hi = b.conv_act == S4TF_ACT_RELU6 ? 6.f : __builtin_inff();
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = g * 16 + 4 * g4 + v;
        if (m < live) b.out[out0 + (long long)m * KT] = fminf(fmaxf(acc[g][v] + bias, lo), hi);
      }
    if (b.stats) {
      // per output over the band: the sum, and the sum of squared deviations from the band's own mean.  A wavefront sums
      // deviations from its first pixel's value, so that a mean of many standard deviations costs no digits; joined over
      // the wavefronts, theirs are from their own means, plus n_w (mean_w - mean)^2.
      float* red = patch;  // [wavefront][16][2]
      lds_barrier();
      const float pivot = __shfl(acc[0][0], l16, 64);
      float s = 0.f, q = 0.f;
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float dev = g * 16 + 4 * g4 + v < live ? acc[g][v] - pivot : 0.f;
          s += dev;
          q = fmaf(dev, dev, q);
        }
      s += __shfl_xor(s, 16, 64); q += __shfl_xor(q, 16, 64);
      s += __shfl_xor(s, 32, 64); q += __shfl_xor(q, 32, 64);
      if (lane < 16) {
        const float inv = live == G * 16 ? 1.f / (float)(G * 16) : live > 0 ? a.inv_rest[rows == a.RB ? 0 : 1] : 0.f;
        red[(wave * 16 + lane) * 2] = fmaf((float)live, pivot, s);
        red[(wave * 16 + lane) * 2 + 1] = fmaxf(q - s * s * inv, 0.f);
      }
      lds_barrier();
      if (tid < OBW * 16) {
        const f32x2* r = reinterpret_cast<const f32x2*>(red) + (tid >> 4) * a.WPX * 16 + (tid & 15);
        float sum = 0.f, m2 = 0.f, sw[16], qw[16];
#pragma unroll
        for (int w = 0; w < 16; ++w) {
          const f32x2 t = w < a.WPX ? r[w * 16] : f32x2{0.f, 0.f};
          sw[w] = t[0];
          qw[w] = t[1];
          sum += sw[w];
        }
        const float mean = sum * a.inv_band[rows == a.RB ? 0 : 1], full = 1.f / (float)(G * 16);
        const int whole = PX / (G * 16), rest = PX - whole * (G * 16);
        const float inv_rest = a.inv_rest[rows == a.RB ? 0 : 1];
#pragma unroll
        for (int w = 0; w < 16; ++w) {
          const float nw = w < whole ? (float)(G * 16) : w == whole ? (float)rest : 0.f, d = sw[w] * (w < whole ? full : inv_rest) - mean;
          m2 += fmaf(d * d, nw, qw[w]);
        }
        b.stats[(long long)(n0 + tid) * gridDim.x + blockIdx.x] = sum;
        b.stats[(long long)(KT + n0 + tid) * gridDim.x + blockIdx.x] = m2;
      }
    }
  } else {
    float mu = 0.f, is = 0.f, sc = 0.f, be = 0.f, s = 0.f, q = 0.f;
    if (b.npart) {
      mu = b.nmean[col]; is = b.ninvstd[col];
      if (!b.ny) { sc = b.ngamma[col] * is; be = b.nbeta[col]; }
    }
    const float hi = b.nact == S4TF_ACT_RELU6 ? 6.f : __builtin_inff();
    const bool no_nact = b.nact == S4TF_ACT_NONE;
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = g * 16 + 4 * g4 + v;
        const float val = acc[g][v] + old[g][v];
        if (m < live) {
          b.out[out0 + (long long)m * KT] = val;
          const float xc = nz[g][v] - mu, y = b.ny ? ny[g][v] : fmaf(xc, sc, be);
          const float dz = (no_nact | ((y > 0.f) & (y < hi))) ? val : 0.f;
          s += dz;
          q += dz * (xc * is);
        }
      }
    if (b.npart) {
      double* red = reinterpret_cast<double*>(patch);  // [wavefront][2][16]
      lds_barrier();
      s += __shfl_xor(s, 16, 64); q += __shfl_xor(q, 16, 64);
      s += __shfl_xor(s, 32, 64); q += __shfl_xor(q, 32, 64);
      if (lane < 16) {
        red[wave * 32 + lane] = (double)s;
        red[wave * 32 + 16 + lane] = (double)q;
      }
      lds_barrier();
      if (tid < OBW * 32) {
        const int o = tid >> 5, k = tid & 31;
        double t = 0.0;
#pragma unroll 4
        for (int w = 0; w < a.WPX; ++w) t += red[(o * a.WPX + w) * 32 + k];
        b.npart[((long long)blockIdx.x * 2 + (k >> 4)) * KT + n0 + o * 16 + (k & 15)] = t;
      }
    }
  }
}

struct BlockPlan { int G, RB, OBW, WPX; };

constexpr size_t MAX_LDS = 156 << 10;
// what the sums over wavefronts need, in the patch's place
size_t scratch_bytes(int C, int waves) { return (size_t)waves * (2 * C > 64 ? 2 * C : 64) * sizeof(double); }

// Picks rows per band and outputs per workgroup with the least estimated time (cycles): the CUs take whole workgroups, so the
// fullest one decides; it runs them in rounds of what its LDS and 16 wavefronts hold; a round costs its start, the patch at
// about 10 bytes per cycle and CU, and the busiest SIMD's MFMAs of 32 cycles.
bool plan_block(const ConvGeom& g, BlockPlan& best) {
  const int C = g.C;
  double best_cost = -1.0;
  for (int RB = 1; RB <= g.H; ++RB) {
    const int blocks = (RB * g.W + 15) / 16, bands = (g.H + RB - 1) / RB;
    if (blocks > 32) break;
    for (int OBW = 1; OBW <= C / 16 && OBW <= 2; OBW *= 2)
      for (int G = 1; G <= 2; ++G) {
        const int WPX = (blocks + G - 1) / G, waves = WPX * OBW;
        if (waves > 16) continue;
        const size_t patch = (size_t)(RB + 2) * (g.W + 2) * (C + 4) * 4, scratch = scratch_bytes(C, waves);
        const size_t lds = (size_t)9 * C * 16 * OBW * 4 + (patch > scratch ? patch : scratch) + 5 * 64 * 4;
        if (lds > MAX_LDS) continue;
        const long long wgs = (long long)g.N * bands * (C / 16 / OBW), per_cu = (wgs + 255) / 256;
        long long resident = (long long)((160 << 10) / lds);
        if (resident > 16 / waves) resident = 16 / waves;
        if (resident < 1) resident = 1;
        const long long rounds = (per_cu + resident - 1) / resident;
        const double conc = (double)((per_cu + rounds - 1) / rounds);
        const double mfma = (double)((long long)(conc * waves + 3) / 4) * G * 9 * (C / 4) * 32.0;
        const double load = conc * ((double)patch * 2.0 + 9.0 * C * 64.0 * OBW) / 10.0;
        const double cost = rounds * (6000.0 + mfma + load);
        if (best_cost < 0.0 || cost < best_cost) {
          best_cost = cost;
          best = {G, RB, OBW, WPX};
        }
      }
  }
  return best_cost >= 0.0;
}

template <int C, bool FLIP, bool BN> void launch_block(const BlockPlan& p, const BlockArgs& a, dim3 grid, size_t lds, hipStream_t st) {
  const dim3 block((unsigned)(64 * p.WPX * p.OBW));
  if (p.G == 1) hipLaunchKernelGGL((block_conv_kernel<C, 1, FLIP, BN>), grid, block, lds, st, a);
  else hipLaunchKernelGGL((block_conv_kernel<C, 2, FLIP, BN>), grid, block, lds, st, a);
}
template <bool FLIP, bool BN> void launch_block(const BlockPlan& p, const BlockArgs& a, dim3 grid, size_t lds, hipStream_t st) {
  if (a.b.g.C == 16) launch_block<16, FLIP, BN>(p, a, grid, lds, st);
  else if (a.b.g.C == 32) launch_block<32, FLIP, BN>(p, a, grid, lds, st);
  else launch_block<64, FLIP, BN>(p, a, grid, lds, st);
}

}  // namespace

bool block_conv_ok(const ConvGeom& g, int dtype) {
  if (dtype != S4TF_F32 || g.R != 3 || g.S != 3 || g.stride != 1 || g.pad != 1 || g.C != g.K) return false;
  if (g.C != 16 && g.C != 32 && g.C != 64) return false;
  if ((long long)g.H * g.W * g.C >= (1LL << 31) / 4 || (long long)g.N * g.H > (1 << 30)) return false;
  BlockPlan p;
  return plan_block(g, p);
}
StatRuns block_conv_runs(const ConvGeom& g) {
  BlockPlan p;
  plan_block(g, p);
  StatRuns r;
  r.period = (g.H + p.RB - 1) / p.RB;
  r.count = g.N * r.period;
  r.rows = p.RB * g.W;
  r.last = (g.H - (r.period - 1) * p.RB) * g.W;
  return r;
}

size_t block_conv_table_bytes(const ConvGeom& g) { return (size_t)block_conv_runs(g).count * 2 * g.C * sizeof(double); }

int block_conv(const BlockConv& b, bool flip, hipStream_t st) {
  BlockPlan p;
  if (!plan_block(b.g, p)) return fail(S4TF_ERR_UNSUPPORTED, "block_conv: shape");
  BlockArgs a = {};
  a.b = b;
  a.RB = p.RB; a.OBW = p.OBW; a.WPX = p.WPX;
  a.bands = (b.g.H + p.RB - 1) / p.RB;
  a.PW = b.g.W + 2;
  magic_div(a.PW, a.magicPW, a.shiftPW);
  magic_div(b.g.W, a.magicW, a.shiftW);
  magic_div(b.runs.period, a.magicPeriod, a.shiftPeriod);
  for (int k = 0; k < 2; ++k) {
    const int px = (k == 0 ? p.RB : b.g.H - (a.bands - 1) * p.RB) * b.g.W, rest = px % (p.G * 16);
    a.inv_band[k] = 1.f / (float)px;
    a.inv_rest[k] = rest ? 1.f / (float)rest : 0.f;
  }
  a.inv_M = 1.0 / ((double)b.g.N * b.g.H * b.g.W);
  if (b.part) { a.inv_rows = 1.0 / (double)b.runs.rows; a.inv_last = 1.0 / (double)b.runs.last; }
  const int waves = p.WPX * p.OBW;
  const size_t patch = (size_t)(p.RB + 2) * a.PW * (b.g.C + 4) * 4, scratch = scratch_bytes(b.g.C, waves);
  const size_t lds = (size_t)9 * b.g.C * 16 * p.OBW * 4 + (patch > scratch ? patch : scratch);
  const dim3 grid((unsigned)(b.g.N * a.bands), (unsigned)(b.g.C / 16 / p.OBW));
  ProfScope ps(flip ? PC_CONV_DGRAD : PC_CONV_FWD, st);
  const bool bn = b.part || b.dpart;
  if (flip) bn ? launch_block<true, true>(p, a, grid, lds, st) : launch_block<true, false>(p, a, grid, lds, st);
  else bn ? launch_block<false, true>(p, a, grid, lds, st) : launch_block<false, false>(p, a, grid, lds, st);
  return launch_status("block_conv");
}

}  // namespace s4tf
