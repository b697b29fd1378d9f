// fp32 convolutions whose reduction axis is short and not made of 16-byte channel chunks: the first layers of a network
// (1 or 3 channels) and LeNet-sized ones (6 channels), forward, input pullback (stride 1) and filter + bias gradient.
//
// The whole reduction axis k = (tap, channel), at most a few hundred long, is flattened: a workgroup brings the input
// patch of a band of output rows of one image into LDS (a border of zeros around the image), the filter as [k][outputs],
// and multiplies out of LDS with v_mfma_f32_16x16x4_f32.  Element (pixel, k) of the im2col matrix is
// patch[base(pixel) + off(k)], with off() in a table, so neither channel count nor filter shape matters, and nothing is
// padded to vector widths in global memory.
//
// Bound by latency at these sizes: one round of loads, tens to hundreds of MFMAs per wavefront, the stores.  The
// element-wise loaders of igemm.hip, which these layers took, recompute a gather address per element and k-tile.  Measured,
// from -> to, us: 128 x 28 x 28, 1 -> 6, 5x5: forward 17.2 -> 6.6, filter + bias gradient 37 -> 10.7; 128 x 14 x 14, 6 -> 16,
// 5x5: 13.3 -> 8.1, 27 -> 10.1, input pullback 19.3 -> 11.7; 32 x 224 x 224, 3 -> 32, 3x3 / 2 (memory floor 14):
// 48.5 -> 26.9, 41 -> 26.7.
#include "s4tf_internal.h"
#include "igemm_args.h"

namespace s4tf {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

struct SmallArgs {
  const float* x;     // what the patch is taken from: (N, H, W, C)
  const float* w;     // forward: [(r,s,c)][K]; FLIP: (R, S, K, C), read turned by 180 degrees with its channels swapped
  float* y;           // (N, P, Q, K)
  const float* bias;  // forward, optional
  float* stats;       // forward, optional: BatchNorm partial sums per band, see igemm_fwd
  const float* mask;  // input pullback, optional: the layer's input; the result is multiplied by act'(mask)
  int H, W, C, K, P, Q, R, S, stride, pad_h, pad_w;
  int Kred, KP;       // k = (r, s, c), and padded to a multiple of 4
  int RB, bands, PR, PW;  // output rows per band, bands per image, patch rows and columns
  int PS;             // floats per patch pixel: odd, so that 16 pixels' values lie in different LDS banks
  int act, accumulate;
  long long runs;
  uint32_t magicQ, magicRow, magicC, magicS, magicO;  // / Q, / (PW*C), / C, / S, / K
  int shiftQ, shiftRow, shiftC, shiftS, shiftO;
};

// rows p0*stride - pad_h ..., columns -pad_w ... of one image, PS floats per pixel; zeros outside
__device__ inline void load_patch(const float* __restrict__ x, int h0, const SmallArgs& a, float* patch) {
  const int rowf = a.PW * a.C, total = a.PR * rowf, wc = a.W * a.C, lead = a.pad_w * a.C;
  for (int i0 = threadIdx.x; i0 < total; i0 += 4 * 256) {
    float v[4];
    int at[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + u * 256, pr = div_magic(i, a.magicRow, a.shiftRow), j = i - pr * rowf, jx = j - lead, h = h0 + pr;
      const int px = div_magic(j, a.magicC, a.shiftC);
      at[u] = (pr * a.PW + px) * a.PS + j - px * a.C;
      v[u] = ((i < total) & (h >= 0) & (h < a.H) & (jx >= 0) & (jx < wc)) ? x[(long long)h * wc + jx] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i0 + u * 256 < total) patch[at[u]] = v[u];
  }
}
// Four MFMA steps take 16 values of the k axis, step e of them 4*e + g for the lanes of group g: in the tables a lane's four are adjacent
__device__ inline int four_of(int k) { return (k & ~15) + 4 * (k & 3) + ((k >> 2) & 3); }
// offset of k = (r, s, c) from a pixel's base
__device__ inline int k_offset(int k, const SmallArgs& a) {
  const int t = div_magic(k, a.magicC, a.shiftC), c = k - t * a.C, r = div_magic(t, a.magicS, a.shiftS), s = t - r * a.S;
  return (r * a.PW + s) * a.PS + c;
}

// G blocks of 16 pixels at a time share the filter fragments
template <int NB, int G, bool FLIP>
__global__ __launch_bounds__(256, 2) void small_conv_kernel(const SmallArgs a) {
  extern __shared__ float smem[];
  constexpr int CO = NB * 16;
  float* wl = smem;                                        // [KP][CO]
  int* koff = reinterpret_cast<int*>(wl + a.KP * CO);      // [KP]
  float* patch = reinterpret_cast<float*>(koff + a.KP);    // [PR][PW][PS]
  __shared__ float red[4][CO][2];
  __shared__ int cnt[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, g4 = lane >> 4;
  const int n = blockIdx.x / a.bands, band = blockIdx.x - n * a.bands, p0 = band * a.RB;
  for (int i = threadIdx.x; i < a.KP * CO / 4; i += 256) *reinterpret_cast<f32x4*>(wl + 4 * i) = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int k = threadIdx.x; k < a.KP; k += 256) koff[four_of(k)] = k < a.Kred ? k_offset(k, a) : 0;
  load_patch(a.x + (long long)n * a.H * a.W * a.C, p0 * a.stride - a.pad_h, a, patch);
  __syncthreads();
  const int weights = a.Kred * a.K;
  for (int i0 = threadIdx.x; i0 < weights; i0 += 4 * 256) {  // in the order of memory
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = i0 + u * 256 < weights ? a.w[i0 + u * 256] : 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + u * 256;
      int k, o;
      if constexpr (FLIP) {  // tap t of the filter is tap R*S-1-t of the turned one
        const int to = div_magic(i, a.magicC, a.shiftC), c = i - to * a.C, t = div_magic(to, a.magicO, a.shiftO);
        o = to - t * a.K;
        k = (a.R * a.S - 1 - t) * a.C + c;
      } else {
        k = div_magic(i, a.magicO, a.shiftO);
        o = i - k * a.K;
      }
      if (i < weights) wl[k * CO + o] = v[u];
    }
  }
  __syncthreads();

  const int PX = min(a.RB, a.P - p0) * a.Q;
  const long long out0 = ((long long)n * a.P + p0) * a.Q;  // the band's pixels are adjacent in y
  float bias[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) bias[nb] = (!FLIP && a.bias && nb * 16 + l16 < a.K) ? a.bias[nb * 16 + l16] : 0.f;
  const float lo = a.act != S4TF_ACT_NONE ? 0.f : -__builtin_inff(), hi = a.act == S4TF_ACT_RELU6 ? 6.f : __builtin_inff();
  float pivot[NB], s1[NB], q1[NB];
  int seen = 0;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) pivot[nb] = s1[nb] = q1[nb] = 0.f;
  for (int b0 = wave * G; b0 * 16 < PX; b0 += 4 * G) {
    int base[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int m = min((b0 + g) * 16 + l16, PX - 1), p = div_magic(m, a.magicQ, a.shiftQ), q = m - p * a.Q;
      base[g] = (p * a.PW + q) * a.stride * a.PS;
    }
    f32x4 acc[G][NB];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[g][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < a.KP; k0 += 16) {
      const i32x4 ko = *reinterpret_cast<const i32x4*>(koff + k0 + 4 * g4);
      float av[4][G], bv[4][NB];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
#pragma unroll
        for (int g = 0; g < G; ++g) av[e][g] = patch[base[g] + ko[e]];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) bv[e][nb] = wl[(k0 + 4 * e + g4) * CO + nb * 16 + l16];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) acc[g][nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[e][g], bv[e][nb], acc[g][nb], 0, 0, 0);
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int mb = (b0 + g) * 16;
      if (mb < PX) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        if (!FLIP && a.stats && seen == 0 && g == 0) pivot[nb] = __shfl(acc[0][nb][0], l16, 64);
        const int col = nb * 16 + l16;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int m = mb + 4 * g4 + v;
          if (m >= PX || col >= a.K) continue;
          float val = acc[g][nb][v];
          if constexpr (!FLIP) {
            const float d = val - pivot[nb];
            s1[nb] += d;
            q1[nb] = fmaf(d, d, q1[nb]);
          }
          float* dst = a.y + (out0 + m) * a.K + col;
          val += bias[nb];
          if (FLIP && a.accumulate) val += *dst;
          if (FLIP && a.mask) val *= act_mask(a.mask[(out0 + m) * a.K + col], a.act);
          *dst = FLIP ? val : fminf(fmaxf(val, lo), hi);
        }
      }
      seen += min(16, PX - mb);
      }
    }
  }
  if constexpr (!FLIP) {
    if (a.stats) {  // sum and squared deviations from the band's own mean, joined over the wavefronts pairwise
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        float s = s1[nb], q = q1[nb];
        s += __shfl_xor(s, 16, 64); q += __shfl_xor(q, 16, 64);
        s += __shfl_xor(s, 32, 64); q += __shfl_xor(q, 32, 64);
        if (lane < 16) {
          red[wave][nb * 16 + lane][0] = fmaf((float)seen, pivot[nb], s);
          red[wave][nb * 16 + lane][1] = seen ? fmaxf(q - s * s / (float)seen, 0.f) : 0.f;
        }
      }
      if (lane == 0) cnt[wave] = seen;
      __syncthreads();
      const int col = threadIdx.x;
      if (col < CO && col < a.K) {
        float sum = red[0][col][0], m2 = red[0][col][1], nn = (float)cnt[0];
        for (int w = 1; w < 4 && cnt[w] > 0; ++w) {
          const float nb_ = (float)cnt[w], sb = red[w][col][0], d = sb / nb_ - sum / nn;
          m2 += red[w][col][1] + d * d * (nn * nb_ / (nn + nb_));
          sum += sb;
          nn += nb_;
        }
        a.stats[(long long)col * a.runs + blockIdx.x] = sum;
        a.stats[(long long)(a.K + col) * a.runs + blockIdx.x] = m2;
      }
    }
  }
}

// ---- filter and bias gradient -----------------------------------------------------------------------------------
// dw[k][n] = sum over pixels of patch[base(pixel) + off(k)] * dy[pixel][n]: rows k in blocks of 16, the MFMA's k axis over
// 4 pixels.  The wavefronts split the pixels, a workgroup walks some bands and leaves one slab; a second kernel adds the
// slabs in order.  The bias gradient is summed, in double, from the same tile of dy.
struct SmallWgradArgs {
  SmallArgs s;        // x, geometry
  const float* dy;    // (N, P, Q, K)
  double* bias;       // gridDim.x rows of K, or NULL
  float* slabs;       // gridDim.x slabs of Kred * K
  int units;          // images * bands
};

template <int RBLK, int NB>
__global__ __launch_bounds__(256, 2) void small_wgrad_kernel(const SmallWgradArgs b) {
  extern __shared__ float smem[];
  const SmallArgs& a = b.s;
  constexpr int CO = NB * 16;
  const int PXP = (a.RB * a.Q + 15) / 16 * 16;
  float* dyt = smem;                                       // [PXP][CO]
  int* pix = reinterpret_cast<int*>(dyt + PXP * CO);       // [PXP]: a pixel's base
  float* patch = reinterpret_cast<float*>(pix + PXP);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, g4 = lane >> 4;
  int koff[RBLK];
#pragma unroll
  for (int rb = 0; rb < RBLK; ++rb) {
    const int k = rb * 16 + l16;
    koff[rb] = k < a.Kred ? k_offset(k, a) : 0;
  }
  double bsum = 0.0;
  for (int m = threadIdx.x; m < PXP; m += 256) {
    const int p = div_magic(m, a.magicQ, a.shiftQ), q = m - p * a.Q;
    pix[four_of(m)] = m < a.RB * a.Q ? (p * a.PW + q) * a.stride * a.PS : 0;
  }
  if (a.K != CO)
    for (int i = threadIdx.x; i < PXP * CO; i += 256) dyt[i] = 0.f;
  f32x4 acc[RBLK][NB];
#pragma unroll
  for (int rb = 0; rb < RBLK; ++rb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[rb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int u = blockIdx.x; u < b.units; u += gridDim.x) {
    const int n = u / a.bands, p0 = (u - n * a.bands) * a.RB, PX = min(a.RB, a.P - p0) * a.Q;
    __syncthreads();
    load_patch(a.x + (long long)n * a.H * a.W * a.C, p0 * a.stride - a.pad_h, a, patch);
    const float* __restrict__ dy = b.dy + (((long long)n * a.P + p0) * a.Q) * a.K;
    if (a.K == CO) {
      for (int i0 = threadIdx.x; i0 < PXP * CO / 4; i0 += 4 * 256) {
        f32x4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = i0 + u * 256 < PX * CO / 4 ? *reinterpret_cast<const f32x4u*>(dy + (i0 + u * 256) * 4) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (i0 + u * 256 < PXP * CO / 4) *reinterpret_cast<f32x4*>(dyt + (i0 + u * 256) * 4) = v[u];
      }
    } else {
      const int live = PX * a.K;  // the columns from K on stay zero, see above
      for (int i0 = threadIdx.x; i0 < live; i0 += 8 * 256) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = i0 + u * 256 < live ? dy[i0 + u * 256] : 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int i = i0 + u * 256, m = div_magic(i, a.magicO, a.shiftO);
          if (i < live) dyt[m * CO + i - m * a.K] = v[u];
        }
      }
      for (int i = PX * CO + threadIdx.x; i < PXP * CO; i += 256) dyt[i] = 0.f;
    }
    __syncthreads();
    if (b.bias)
      for (int m = threadIdx.x / CO; m < PX; m += 256 / CO) bsum += (double)dyt[m * CO + threadIdx.x % CO];
    for (int m0 = wave * 16; m0 < PX; m0 += 64) {
      const i32x4 pb = *reinterpret_cast<const i32x4*>(pix + m0 + 4 * g4);
      float bv[4][NB], av[4][RBLK];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) bv[e][nb] = dyt[(m0 + 4 * e + g4) * CO + nb * 16 + l16];
#pragma unroll
        for (int rb = 0; rb < RBLK; ++rb) av[e][rb] = patch[pb[e] + koff[rb]];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int rb = 0; rb < RBLK; ++rb)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) acc[rb][nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[e][rb], bv[e][nb], acc[rb][nb], 0, 0, 0);
    }
  }
  // the four wavefronts' sums, added in wavefront order
  float* red = smem;
  constexpr int TILE = RBLK * 16 * CO;
  __syncthreads();
#pragma unroll
  for (int rb = 0; rb < RBLK; ++rb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[wave * TILE + (rb * 16 + 4 * g4 + v) * CO + nb * 16 + l16] = acc[rb][nb][v];
  __syncthreads();
  float* slab = b.slabs + (long long)blockIdx.x * a.Kred * a.K;
  for (int i = threadIdx.x; i < a.Kred * a.K; i += 256) {
    const int k = div_magic(i, a.magicO, a.shiftO), at = k * CO + i - k * a.K;
    slab[i] = ((red[at] + red[TILE + at]) + red[2 * TILE + at]) + red[3 * TILE + at];
  }
  if (b.bias) {
    __syncthreads();
    double* sh = reinterpret_cast<double*>(smem);
    sh[threadIdx.x] = bsum;
    __syncthreads();
    if ((int)threadIdx.x < a.K) {
      double s = 0.0;
      for (int l = 0; l < 256 / CO; ++l) s += sh[l * CO + threadIdx.x];
      b.bias[(long long)blockIdx.x * a.K + threadIdx.x] = s;
    }
  }
}

// 16 outputs x 16 lanes of slabs per workgroup; the workgroups behind those of dw's n values take the bias gradient
__global__ __launch_bounds__(256) void small_reduce_kernel(const float* __restrict__ slabs, const double* __restrict__ bias,
                                                           float* __restrict__ dw, float* __restrict__ db, int n, int K, int count) {
  __shared__ float sh[16][17];
  __shared__ double shd[16][17];
  const int ol = threadIdx.x & 15, zl = threadIdx.x >> 4, wblocks = (n + 15) / 16, i = blockIdx.x * 16 + ol;
  if ((int)blockIdx.x >= wblocks) {
    const int c = ((int)blockIdx.x - wblocks) * 16 + ol;
    double s = 0.0;
    if (c < K) {
#pragma unroll 8
      for (int z = zl; z < count; z += 16) s += bias[(long long)z * K + c];
    }
    shd[zl][ol] = s;
    __syncthreads();
    if (zl == 0 && c < K) {
      for (int l = 1; l < 16; ++l) s += shd[l][ol];
      db[c] = (float)s;
    }
    return;
  }
  float s = 0.f;
  if (i < n) {
#pragma unroll 8
    for (int z = zl; z < count; z += 16) s += slabs[(long long)z * n + i];
  }
  sh[zl][ol] = s;
  __syncthreads();
  if (zl == 0 && i < n) {
    float t = 0.f;
#pragma unroll
    for (int l = 0; l < 16; ++l) t += sh[l][ol];
    dw[i] = t;
  }
}

constexpr int MAX_LDS = 60 << 10;

// Cuts the output into bands of whole rows, at most about `want` pixels each, as the LDS allows; `divide`: rows that
// divide the image's, so that the bands are equal runs of pixels, of at least 32 where there is a choice.  false when not
// even one row fits.
bool cut_bands(SmallArgs& a, int want, int fixed_floats, int floats_per_pixel, bool divide) {
  int best = 0;
  for (int rb = 1; rb <= a.P; ++rb) {
    if (divide && a.P % rb) continue;
    const long long patch = (long long)((rb - 1) * a.stride + a.R) * a.PW * a.PS;
    if ((fixed_floats + patch + (long long)floats_per_pixel * (rb * a.Q + 16)) * 4 > MAX_LDS) break;
    if (best && rb * a.Q > want && best * a.Q >= 32) break;
    best = rb;
  }
  if (!best) return false;
  a.RB = best;
  a.bands = (a.P + best - 1) / best;
  a.PR = (best - 1) * a.stride + a.R;
  magic_div(a.Q, a.magicQ, a.shiftQ);
  magic_div(a.PW * a.C, a.magicRow, a.shiftRow);
  magic_div(a.C, a.magicC, a.shiftC);
  magic_div(a.S, a.magicS, a.shiftS);
  magic_div(a.K, a.magicO, a.shiftO);
  return true;
}

SmallArgs fwd_args(const ConvGeom& g) {
  SmallArgs a = {};
  a.H = g.H; a.W = g.W; a.C = g.C; a.K = g.K; a.P = g.P; a.Q = g.Q; a.R = g.R; a.S = g.S; a.stride = g.stride;
  a.pad_h = a.pad_w = g.pad;
  a.Kred = g.R * g.S * g.C;
  a.PS = g.C | 1;
  a.KP = (a.Kred + 15) / 16 * 16;
  a.PW = (g.Q - 1) * g.stride + g.S;
  return a;
}
SmallArgs dgrad_args(const ConvGeom& g) {  // a stride-1 convolution of dy
  SmallArgs a = {};
  a.H = g.P; a.W = g.Q; a.C = g.K; a.K = g.C; a.P = g.H; a.Q = g.W; a.R = g.R; a.S = g.S; a.stride = 1;
  a.pad_h = g.R - 1 - g.pad; a.pad_w = g.S - 1 - g.pad;
  a.Kred = g.R * g.S * g.K;
  a.PS = g.K | 1;
  a.KP = (a.Kred + 15) / 16 * 16;
  a.PW = g.W + g.S - 1;
  return a;
}
int blocks16(int k) { return (k + 15) / 16; }
// pixels per band: enough workgroups for every CU to have some, 64 to 256 pixels
int band_pixels(long long px) {
  const long long per = px / 1024;
  return per < 64 ? 64 : per > 256 ? 256 : (int)per;
}
bool cut_conv(const ConvGeom& g, SmallArgs& a, bool divide) {
  return cut_bands(a, band_pixels((long long)g.N * a.P * a.Q), a.KP * (blocks16(a.K) * 16 + 1), 0, divide);
}
bool cut_wgrad(SmallArgs& a) { return cut_bands(a, 256, 0, blocks16(a.K) * 16 + 1, false); }

}  // namespace

// Layers of few channels with a filter wider than one tap: where whole 16-channel k-steps would be mostly padding
bool small_conv_ok(int pass, const ConvGeom& g, int dtype) {
  if (dtype != S4TF_F32 || g.R * g.S == 1 || (long long)g.N * g.H * g.W * g.C >= (1LL << 31) || (long long)g.N * g.P * g.Q * g.K >= (1LL << 31))
    return false;
  if (pass == PASS_DGRAD) {
    if (g.stride != 1 || g.R - 1 < g.pad || g.S - 1 < g.pad || g.C > 12 || g.R * g.S * g.K > 416) return false;
    SmallArgs a = dgrad_args(g);
    return cut_conv(g, a, false);
  }
  if (g.C > 8 || g.K > 32 || g.R * g.S * g.C > 159) return false;
  SmallArgs a = fwd_args(g);
  return pass == PASS_FWD ? cut_conv(g, a, false) : (g.K <= 16 || a.Kred <= 32) && cut_wgrad(a);
}

int small_conv_fwd(const ConvGeom& g, const float* x, const float* w, const float* bias, int act, float* y, float* stats,
                   int* stats_rows, hipStream_t st) {
  SmallArgs a = fwd_args(g);
  if (stats && (!cut_conv(g, a, true) || a.RB * a.Q < 32)) stats = nullptr;
  if (!stats && !cut_conv(g, a, false)) return fail(S4TF_ERR_UNSUPPORTED, "small_conv: shape");
  a.x = x; a.w = w; a.y = y; a.bias = bias; a.act = act; a.stats = stats;
  a.runs = (long long)g.N * a.bands;
  if (stats) *stats_rows = a.RB * a.Q;
  const int nb = blocks16(a.K);
  const size_t lds = ((size_t)a.KP * (nb * 16 + 1) + (size_t)a.PR * a.PW * a.PS) * sizeof(float);
  const dim3 grid((unsigned)a.runs);
  // up to 64 pixels per band: a block for each wavefront
  if (nb == 1 && a.RB * a.Q <= 64) hipLaunchKernelGGL((small_conv_kernel<1, 1, false>), grid, dim3(256), lds, st, a);
  else if (nb == 1) hipLaunchKernelGGL((small_conv_kernel<1, 2, false>), grid, dim3(256), lds, st, a);
  else hipLaunchKernelGGL((small_conv_kernel<2, 2, false>), grid, dim3(256), lds, st, a);
  return launch_status("small_conv");
}

// mask (optional): the layer's own input x; dx is then multiplied by act'(x), the pullback of the activation that made it
int small_conv_dgrad(const ConvGeom& g, const float* dy, const float* w, float* dx, int accumulate, const float* mask, int mask_act,
                     hipStream_t st) {
  SmallArgs a = dgrad_args(g);
  if (!cut_conv(g, a, false)) return fail(S4TF_ERR_UNSUPPORTED, "small_conv: shape");
  a.x = dy; a.w = w; a.y = dx; a.accumulate = accumulate; a.mask = mask; a.act = mask_act;
  const size_t lds = ((size_t)a.KP * (16 + 1) + (size_t)a.PR * a.PW * a.PS) * sizeof(float);
  const dim3 grid((unsigned)(g.N * a.bands));
  if (a.RB * a.Q <= 64) hipLaunchKernelGGL((small_conv_kernel<1, 1, true>), grid, dim3(256), lds, st, a);
  else hipLaunchKernelGGL((small_conv_kernel<1, 2, true>), grid, dim3(256), lds, st, a);
  return launch_status("small_conv");
}

namespace {
int wgrad_blocks(const ConvGeom& g, const SmallArgs& a) {
  const long long units = (long long)g.N * a.bands;
  return (int)(units < 768 ? units : 768);
}
}  // namespace

size_t small_wgrad_workspace(const ConvGeom& g) {
  SmallArgs a = fwd_args(g);
  if (!cut_wgrad(a)) return 0;
  return (size_t)wgrad_blocks(g, a) * a.K * (a.Kred * sizeof(float) + sizeof(double));
}

// db (optional): the bias gradient, a row of the same product
int small_wgrad(const ConvGeom& g, const float* x, const float* dy, float* dw, float* db, void* ws, hipStream_t st) {
  SmallWgradArgs b = {};
  b.s = fwd_args(g);
  if (!cut_wgrad(b.s)) return fail(S4TF_ERR_UNSUPPORTED, "small_conv: shape");
  const SmallArgs& a = b.s;
  b.s.x = x;
  const int blocks = wgrad_blocks(g, a), nb = blocks16(a.K), rblk = a.Kred <= 32 ? 2 : 10, co = nb * 16;
  b.dy = dy; b.units = g.N * a.bands;
  double* bias = static_cast<double*>(ws);  // the workspace: bias rows, then slabs
  b.bias = db ? bias : nullptr;
  b.slabs = reinterpret_cast<float*>(bias + (size_t)blocks * a.K);
  const int pxp = (a.RB * a.Q + 15) / 16 * 16;
  size_t lds = ((size_t)pxp * (co + 1) + (size_t)a.PR * a.PW * a.PS) * sizeof(float);
  const size_t red = (size_t)4 * rblk * 16 * co * sizeof(float);
  if (lds < red) lds = red;
  if (lds < 256 * sizeof(double)) lds = 256 * sizeof(double);
  {
    ProfScope ps(PC_CONV_WGRAD, st);
    if (rblk == 2 && nb == 1) hipLaunchKernelGGL((small_wgrad_kernel<2, 1>), dim3(blocks), dim3(256), lds, st, b);
    else if (rblk == 2) hipLaunchKernelGGL((small_wgrad_kernel<2, 2>), dim3(blocks), dim3(256), lds, st, b);
    else hipLaunchKernelGGL((small_wgrad_kernel<10, 1>), dim3(blocks), dim3(256), lds, st, b);
    const int rc = launch_status("small_wgrad");
    if (rc != S4TF_OK) return rc;
  }
  ProfScope ps(PC_WGRAD_REDUCE, st);
  const int n = a.Kred * a.K;
  hipLaunchKernelGGL(small_reduce_kernel, dim3((n + 15) / 16 + (db ? (a.K + 15) / 16 : 0)), dim3(256), 0, st, b.slabs, bias, dw, db, n, a.K, blocks);
  return launch_status("small_reduce");
}

}  // namespace s4tf
