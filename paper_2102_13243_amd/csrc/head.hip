// Head of the network: global average pool + dense + mean softmax cross-entropy, value and pullback in one call
// (`softmaxCrossEntropy(logits:labels:)` of the paper's training loop).
//   pbar = mean_{h,w} x;  z = pbar W + b;  loss = mean_n (logsumexp(z_n) - z_n[label_n])
//   dz = (softmax(z) - onehot)/n;  dW = pbar^T dz;  db = sum_n dz;  dx = (dz W^T)/(h*w)
// Latency bound throughout: the work is tiny, each kernel a few microseconds.  Two ways through it:
//   * small heads (W of at most 32 KB): everything that concerns one sample, pooled features to dx, by one workgroup that
//     keeps W in LDS; then one kernel for what sums over the batch (dW, db, loss).  2 launches instead of 9: the tiny
//     block's head 85 -> 12 us, of which a single workgroup's pooling was 39;
//   * others (1000 classes): pooling, two products on the wavefront-tile GEMM (logits with the bias in its epilogue,
//     cotangent of the pooled features), softmax, dW on the same GEMM, one kernel for db and the loss.
// What the parameters' gradients need is kept apart (head_params), so that a training step can run it on its second
// stream.
#include "s4tf_internal.h"
#include "igemm_args.h"
#include "pack.h"

namespace s4tf {
namespace {

constexpr int SMALL_W = 8192;      // floats of W a workgroup keeps in LDS
constexpr int SMALL_X = 1 << 16;   // elements of a sample one workgroup pools
constexpr int SMALL_C = 1024, SMALL_K = 256;

// Sum over pixels of V channels per thread: threads (pixel lane, channel vector), the lanes added in order.
// part: LDS, lanes * cvs * V floats; the result for channel c (of this block's cvs * V) ends up in part[c].
template <typename T, int V>
__device__ inline void pool_pixels(const T* __restrict__ x, int HW, int C, int cvs, int lanes, float* part) {
  const int cv = threadIdx.x % cvs, pl = threadIdx.x / cvs;
  float s[V];
#pragma unroll
  for (int e = 0; e < V; ++e) s[e] = 0.f;
  if (pl < lanes) {
    const T* p = x + cv * V;
    int j = pl;
    for (; j + 3 * lanes < HW; j += 4 * lanes) {
      Pack<T, V> v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = ldp<T, V>(p + (long long)(j + u * lanes) * C);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int e = 0; e < V; ++e) s[e] += v[u].get(e);
    }
    for (; j < HW; j += lanes) {
      const Pack<T, V> v = ldp<T, V>(p + (long long)j * C);
#pragma unroll
      for (int e = 0; e < V; ++e) s[e] += v.get(e);
    }
#pragma unroll
    for (int e = 0; e < V; ++e) part[(pl * cvs + cv) * V + e] = s[e];
  }
  __syncthreads();
  for (int c = threadIdx.x; c < cvs * V; c += blockDim.x) {
    float t = 0.f;
    for (int l = 0; l < lanes; ++l) t += part[l * cvs * V + c];
    part[c] = t;  // read by this thread alone until the next barrier
  }
  __syncthreads();
}

// dx[hw][c] = dp[c] (LDS) for this block's cvs * V channels, added to what dx holds when it accumulates (one rounding)
template <typename T, int V>
__device__ inline void spread_pixels(const float* dp, T* dx, int HW, int C, int cvs, int lanes, int accumulate) {
  const int cv = threadIdx.x % cvs, pl = threadIdx.x / cvs;
  if (pl >= lanes) return;
  float v[V];
#pragma unroll
  for (int e = 0; e < V; ++e) v[e] = dp[cv * V + e];
  const Pack<T, V> o = pack_of<T, V>(v);
  T* p = dx + cv * V;
  for (int j = pl; j < HW; j += lanes) {
    if (accumulate) {
      const Pack<T, V> old = ldp<T, V>(p + (long long)j * C);
      float w[V];
#pragma unroll
      for (int e = 0; e < V; ++e) w[e] = old.get(e) + v[e];
      stp<T, V>(p + (long long)j * C, pack_of<T, V>(w));
    } else {
      stp<T, V>(p + (long long)j * C, o);
    }
  }
}

// over the 256 threads of a block; sh: 4 floats of LDS
__device__ inline float block_max(float v, float* sh) {
  for (int off = 1; off < 64; off <<= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  v = fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
  __syncthreads();
  return v;
}
__device__ inline float block_sum(float v, float* sh) {
  for (int off = 1; off < 64; off <<= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  v = (sh[0] + sh[1]) + (sh[2] + sh[3]);
  __syncthreads();
  return v;
}

// one workgroup per sample: pooled features, logits, softmax, dz, and the sample's dx
template <typename T, int V>
__global__ __launch_bounds__(256) void head_sample_kernel(const T* __restrict__ x, const float* __restrict__ W,
                                                          const float* __restrict__ b, const int32_t* __restrict__ labels,
                                                          float* __restrict__ pbar, float* __restrict__ z, float* __restrict__ dz,
                                                          float* __restrict__ rowloss, T* dx, int N, int HW, int C, int K,
                                                          int accumulate, int mask_act) {
  __shared__ float Wl[SMALL_W], part[SMALL_C > 256 * V ? SMALL_C : 256 * V], dzl[SMALL_K], red[256], sh[4];
  const int n = blockIdx.x, t = threadIdx.x;
  for (int i = t; i < C * K; i += 256) Wl[i] = W[i];
  const int CV = C / V, lanes = 256 / CV;
  if (lanes > 0) {
    pool_pixels<T, V>(x + (long long)n * HW * C, HW, C, CV, lanes, part);
  } else {  // more channel vectors than threads
    for (int c = t; c < C; c += 256) {
      float s = 0.f;
      for (int j = 0; j < HW; ++j) s += to_f32<T>(x[((long long)n * HW + j) * C + c]);
      part[c] = s;
    }
    __syncthreads();
  }
  const float hw = (float)HW;
  for (int c = t; c < C; c += 256) {
    part[c] /= hw;
    pbar[n * C + c] = part[c];
  }
  __syncthreads();
  // logits: 256 / K threads per class, added in order
  const int parts = 256 / K, j = t % K, pt = t / K;
  float s = 0.f;
  if (pt < parts)
    for (int c = pt; c < C; c += parts) s = fmaf(part[c], Wl[c * K + j], s);
  red[t] = s;
  __syncthreads();
  float zj = -INFINITY;
  if (t < K) {
    zj = 0.f;
    for (int l = 0; l < parts; ++l) zj += red[l * K + t];
    zj += b[t];
    z[n * K + t] = zj;
  }
  const float m = block_max(zj, sh);
  const float lse = m + logf(block_sum(t < K ? expf(zj - m) : 0.f, sh));
  const int lab = labels[n];
  if (t < K) {
    const float d = (expf(zj - lse) - (t == lab ? 1.f : 0.f)) * (1.0f / (float)N);
    dzl[t] = d;
    dz[n * K + t] = d;
    if (t == lab) rowloss[n] = lse - zj;
  }
  if (t == 0 && (lab < 0 || lab >= K)) rowloss[n] = 0.f;
  if (!dx) return;
  __syncthreads();
  for (int c = t; c < C; c += 256) {
    float d = 0.f;
    for (int l = 0; l < K; ++l) d = fmaf(dzl[l], Wl[c * K + l], d);
    part[c] = d / hw;
    if (mask_act) part[c] *= act_mask(to_f32<T>(x[(long long)n * C + c]), mask_act);  // HW is 1, see head_can_mask
  }
  __syncthreads();
  T* out = dx + (long long)n * HW * C;
  if (lanes > 0) {
    spread_pixels<T, V>(part, out, HW, C, CV, lanes, accumulate);
  } else {
    for (int i = t; i < HW * C; i += 256) out[i] = from_f32<T>(accumulate ? to_f32<T>(out[i]) + part[i % C] : part[i % C]);
  }
}

// The mean of the losses, in double, by one workgroup: thread sums of a stride, then a tree
__device__ inline void mean_loss(const float* __restrict__ rowloss, float* __restrict__ loss, int N, double* sh) {
  double s = 0.0;
  for (int n = threadIdx.x; n < N; n += 256) s += (double)rowloss[n];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) sh[threadIdx.x] += sh[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = (float)(sh[0] / (double)N);
}

// Sums over the batch of a small head: output o = (c, j) of [pbar | 1]^T dz (row C is db), 16 lanes of samples each; the
// last workgroup takes the loss.
__global__ __launch_bounds__(256) void head_batch_kernel(const float* __restrict__ pbar, const float* __restrict__ dz,
                                                         const float* __restrict__ rowloss, float* __restrict__ dW,
                                                         float* __restrict__ db, float* __restrict__ loss, int N, int C, int K) {
  __shared__ double shd[256];
  if (blockIdx.x == gridDim.x - 1) {
    mean_loss(rowloss, loss, N, shd);
    return;
  }
  float* red = reinterpret_cast<float*>(shd);
  const int ol = threadIdx.x & 15, nl = threadIdx.x >> 4, o = blockIdx.x * 16 + ol;
  const int c = o / K, j = o - c * K;
  float s = 0.f;
  if (c <= C) {
#pragma unroll 8
    for (int n = nl; n < N; n += 16) s = fmaf(c < C ? pbar[n * C + c] : 1.f, dz[n * K + j], s);
  }
  red[nl * 16 + ol] = s;
  __syncthreads();
  if (nl == 0 && c <= C) {
    float t = 0.f;
#pragma unroll
    for (int l = 0; l < 16; ++l) t += red[l * 16 + ol];
    if (c < C) dW[o] = t;
    else db[j] = t;
  }
}

// ---- other heads ---------------------------------------------------------------------------------------------------
template <typename T, int V>
__global__ __launch_bounds__(256) void gap_kernel(const T* __restrict__ x, float* __restrict__ pbar, int HW, int C, int cvs) {
  __shared__ float part[256 * V];
  const int c0 = blockIdx.x * cvs * V, n = blockIdx.y;
  const int live = min(cvs, C / V - (int)blockIdx.x * cvs);  // the last block of channels may be narrower
  pool_pixels<T, V>(x + (long long)n * HW * C + c0, HW, C, live, 256 / live, part);
  for (int c = threadIdx.x; c < live * V; c += 256) pbar[(long long)n * C + c0 + c] = part[c] / (float)HW;
}
template <typename T, int V>
__global__ __launch_bounds__(256) void gap_vjp_kernel(const float* __restrict__ part, int splits, T* dx, int N, int HW, int C,
                                                      int cvs, int accumulate) {
  __shared__ float dp[256 * V];
  const int c0 = blockIdx.x * cvs * V, n = blockIdx.y;
  const int live = min(cvs, C / V - (int)blockIdx.x * cvs);
  for (int c = threadIdx.x; c < live * V; c += 256) {
    float v = 0.f;
    for (int s = 0; s < splits; ++s) v += part[((long long)s * N + n) * C + c0 + c];
    dp[c] = v / (float)HW;
  }
  __syncthreads();
  spread_pixels<T, V>(dp, dx + (long long)n * HW * C + c0, HW, C, live, 256 / live, accumulate);
}

// part[s][m][j] = sum over the k of split s of A[m][k] * Bm(k, j), with Bm(k, j) = B[k][j] (B is [K][J]) or,
// BT, B[j][k] (B is [J][K]).  64x64 outputs per workgroup, 4x4 per thread, 32 k per LDS step.
constexpr int SK_T = 64, SK_KC = 32;
template <bool BT>
__global__ __launch_bounds__(256) void skinny_gemm_kernel(const float* __restrict__ A, const float* __restrict__ B,
                                                          float* __restrict__ part, int M, int J, int K, int kper) {
  __shared__ float As[SK_KC][SK_T + 4], Bs[SK_KC][SK_T + 4];
  const int t = threadIdx.x, tx = t & 15, ty = t >> 4;
  const int j0 = blockIdx.x * SK_T, m0 = blockIdx.z * SK_T;
  const int k0 = blockIdx.y * kper, k1 = min(K, k0 + kper);
  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;
  for (int kb = k0; kb < k1; kb += SK_KC) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {  // A[m][k]: k fastest
      const int k = t & 31, m = (t >> 5) + 8 * i;
      As[k][m] = (m0 + m < M && kb + k < k1) ? A[(long long)(m0 + m) * K + kb + k] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (BT) {
        const int k = t & 31, j = (t >> 5) + 8 * i;
        Bs[k][j] = (j0 + j < J && kb + k < k1) ? B[(long long)(j0 + j) * K + kb + k] : 0.f;
      } else {
        const int j = t & 63, k = (t >> 6) + 4 * i;
        Bs[k][j] = (j0 + j < J && kb + k < k1) ? B[(long long)(kb + k) * J + j0 + j] : 0.f;
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < SK_KC; ++k) {
      const float4 a = *reinterpret_cast<const float4*>(&As[k][ty * 4]);
      const float4 b = *reinterpret_cast<const float4*>(&Bs[k][tx * 4]);
      const float av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] += av[i] * bv[j];
    }
    __syncthreads();
  }
  float* dst = part + (long long)blockIdx.y * M * J;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + ty * 4 + i;
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int col = j0 + tx * 4 + j;
      if (col < J) dst[(long long)m * J + col] = acc[i][j];
    }
  }
}

struct SkinnyPlan { int splits, kper; dim3 grid; };
SkinnyPlan skinny_plan(int M, int J, int K) {
  SkinnyPlan p;
  const int jt = (J + SK_T - 1) / SK_T, mt = (M + SK_T - 1) / SK_T;
  int want = 256 / (jt * mt);
  const int maxs = (K + SK_KC - 1) / SK_KC;
  if (want > maxs) want = maxs;
  if (want < 1) want = 1;
  p.kper = ((K + want - 1) / want + SK_KC - 1) / SK_KC * SK_KC;
  p.splits = (K + p.kper - 1) / p.kper;
  p.grid = dim3(jt, p.splits, mt);
  return p;
}

// one block per sample: logits (split-k partial sums added in order, plus the bias; or, part == nullptr, complete in z),
// max, sum of exponentials, loss term, dz.  A thread meets the same classes in every phase, so it reads back only
// logits it wrote itself.
__global__ __launch_bounds__(256) void softmax_xent_kernel(const float* __restrict__ part, int splits,
                                                           const float* __restrict__ bias, float* __restrict__ z,
                                                           const int32_t* __restrict__ labels, float* __restrict__ dz,
                                                           float* __restrict__ rowloss, int N, int K) {
  __shared__ float sh[4];
  const int n = blockIdx.x, t = threadIdx.x;
  float* zr = z + (long long)n * K;
  float m = -INFINITY;
  for (int j = t; j < K; j += 256) {
    float v;
    if (part) {
      v = 0.f;
      for (int s = 0; s < splits; ++s) v += part[((long long)s * N + n) * K + j];
      v += bias[j];
      zr[j] = v;
    } else {
      v = zr[j];
    }
    m = fmaxf(m, v);
  }
  m = block_max(m, sh);
  float se = 0.f;
  for (int j = t; j < K; j += 256) se += expf(zr[j] - m);
  const float lse = m + logf(block_sum(se, sh));
  const int lab = labels[n];
  const float invN = 1.0f / (float)N;
  for (int j = t; j < K; j += 256) {
    const float p = expf(zr[j] - lse);
    dz[(long long)n * K + j] = (p - (j == lab ? 1.f : 0.f)) * invN;
    if (j == lab) rowloss[n] = lse - zr[j];
  }
  if (t == 0 && (lab < 0 || lab >= K)) rowloss[n] = 0.f;
}

// db (16 classes per workgroup, 16 lanes of samples each) and, in the last workgroup, the loss
__global__ __launch_bounds__(256) void head_bias_kernel(const float* __restrict__ dz, const float* __restrict__ rowloss,
                                                        float* __restrict__ db, float* __restrict__ loss, int N, int K) {
  __shared__ double shd[256];
  if (blockIdx.x == gridDim.x - 1) {
    mean_loss(rowloss, loss, N, shd);
    return;
  }
  float* red = reinterpret_cast<float*>(shd);
  const int ol = threadIdx.x & 15, nl = threadIdx.x >> 4, j = blockIdx.x * 16 + ol;
  float s = 0.f;
  if (j < K) {
#pragma unroll 4
    for (int n = nl; n < N; n += 16) s += dz[(long long)n * K + j];
  }
  red[nl * 16 + ol] = s;
  __syncthreads();
  if (nl == 0 && j < K) {
    float t = 0.f;
#pragma unroll
    for (int l = 0; l < 16; ++l) t += red[l * 16 + ol];
    db[j] = t;
  }
}

ConvGeom dense_geom(int N, int C, int K) {
  ConvGeom g;
  g.N = N; g.H = 1; g.W = 1; g.C = C; g.K = K; g.R = 1; g.S = 1; g.stride = 1; g.pad = 0; g.P = 1; g.Q = 1;
  return g;
}

bool small_head(const s4tf_head_desc& d) {
  return (long long)d.c * d.classes <= SMALL_W && d.c <= SMALL_C && d.classes <= SMALL_K && (long long)d.h * d.w * d.c <= SMALL_X;
}
// products on the wavefront-tile GEMM (it loads 4 adjacent channels or classes at a time)
bool wave_head(const s4tf_head_desc& d, const void* W, const void* logits) {
  const ConvGeom g = dense_geom(d.n, d.c, d.classes);
  return wave_gemm_ok(PASS_FWD, g, S4TF_F32) && wave_gemm_ok(PASS_DGRAD, g, S4TF_F32) && aligned16(W) && aligned16(logits);
}

struct Layout {
  size_t pbar, logits, dz, rowloss, part, wg, total;  // part: partial sums of either product
};
Layout layout(const s4tf_head_desc& d) {
  Layout l;
  size_t o = 0;
  l.pbar = o; o += align_up((size_t)d.n * d.c * 4, 256);
  l.logits = o; o += align_up((size_t)d.n * d.classes * 4, 256);
  l.dz = o; o += align_up((size_t)d.n * d.classes * 4, 256);
  l.rowloss = o; o += align_up((size_t)d.n * 4, 256);
  const size_t pf = (size_t)skinny_plan(d.n, d.classes, d.c).splits * d.n * d.classes;
  const size_t pb = (size_t)skinny_plan(d.n, d.c, d.classes).splits * d.n * d.c;
  l.part = o; o += align_up((pf > pb ? pf : pb) * 4, 256);
  l.wg = o; o += align_up(igemm_wgrad_workspace(dense_geom(d.n, d.c, d.classes), S4TF_F32), 256);
  l.total = o;
  return l;
}

// KERNEL<T, V> with 16-byte accesses where the channel count allows them
#define HEAD_LAUNCH(KERNEL, grid, ...)                                                                     \
  do {                                                                                                     \
    if (d.dtype == S4TF_BF16) {                                                                            \
      typedef bf16_t T;                                                                                    \
      if (V > 1) hipLaunchKernelGGL((KERNEL<T, 8>), grid, dim3(256), 0, st, __VA_ARGS__);                  \
      else hipLaunchKernelGGL((KERNEL<T, 1>), grid, dim3(256), 0, st, __VA_ARGS__);                        \
    } else {                                                                                               \
      typedef float T;                                                                                     \
      if (V > 1) hipLaunchKernelGGL((KERNEL<T, 4>), grid, dim3(256), 0, st, __VA_ARGS__);                  \
      else hipLaunchKernelGGL((KERNEL<T, 1>), grid, dim3(256), 0, st, __VA_ARGS__);                        \
    }                                                                                                      \
  } while (0)

}  // namespace

size_t head_workspace(const s4tf_head_desc& d) { return layout(d).total; }

bool head_can_mask(const s4tf_head_desc& d) { return small_head(d) && d.h * d.w == 1 && !d.accumulate_dx; }
int head_value(const s4tf_head_desc& d, const void* x, const float* W, const float* b, const int32_t* labels, void* dx,
               float* logits_out, void* ws, hipStream_t st, int mask_act) {
  const Layout l = layout(d);
  char* base = static_cast<char*>(ws);
  float* pbar = reinterpret_cast<float*>(base + l.pbar);
  float* logits = logits_out ? logits_out : reinterpret_cast<float*>(base + l.logits);
  float* dz = reinterpret_cast<float*>(base + l.dz);
  float* rowloss = reinterpret_cast<float*>(base + l.rowloss);
  float* part = reinterpret_cast<float*>(base + l.part);
  const int HW = d.h * d.w, vec = d.dtype == S4TF_BF16 ? 8 : 4;
  const int V = d.c % vec == 0 ? vec : 1;
  int rc;
  if (small_head(d)) {
    ProfScope ps(PC_HEAD, st);
    HEAD_LAUNCH(head_sample_kernel, dim3(d.n), (const T*)x, W, b, labels, pbar, logits, dz, rowloss, (T*)dx, d.n, HW, d.c, d.classes,
                d.accumulate_dx, mask_act);
    return launch_status("head_sample");
  }
  // channel vectors per workgroup of the pooling kernels: 64, and narrower where that leaves the chip empty
  int cvs = d.c / V < 64 ? d.c / V : 64;
  while (cvs > 8 && (long long)d.n * ((d.c / V + cvs - 1) / cvs) < 256) cvs = (cvs + 1) / 2;
  const dim3 pool_grid((unsigned)((d.c / V + cvs - 1) / cvs), (unsigned)d.n);
  {
    ProfScope ps(PC_HEAD, st);
    HEAD_LAUNCH(gap_kernel, pool_grid, (const T*)x, pbar, HW, d.c, cvs);
    if ((rc = launch_status("gap")) != S4TF_OK) return rc;
  }
  const bool waves = wave_head(d, W, logits);
  const ConvGeom g = dense_geom(d.n, d.c, d.classes);
  const SkinnyPlan sp = skinny_plan(d.n, d.classes, d.c), sb = skinny_plan(d.n, d.c, d.classes);
  {
    ProfScope ps(PC_HEAD, st);
    if (waves) {
      if ((rc = wave_gemm_fwd(g, pbar, W, b, S4TF_ACT_NONE, logits, nullptr, nullptr, st)) != S4TF_OK) return rc;
    } else {
      hipLaunchKernelGGL(skinny_gemm_kernel<false>, sp.grid, dim3(256), 0, st, pbar, W, part, d.n, d.classes, d.c, sp.kper);
      if ((rc = launch_status("head logits")) != S4TF_OK) return rc;
    }
    hipLaunchKernelGGL(softmax_xent_kernel, dim3(d.n), dim3(256), 0, st, waves ? nullptr : part, sp.splits, b, logits, labels, dz,
                       rowloss, d.n, d.classes);
    if ((rc = launch_status("softmax_xent")) != S4TF_OK) return rc;
  }
  if (!dx) return S4TF_OK;
  ProfScope ps(PC_HEAD, st);  // dpbar[n][c] = sum_j dz[n][j] W[c][j]
  if (waves) {
    if ((rc = wave_gemm_dgrad(g, dz, W, part, 0, nullptr, S4TF_ACT_NONE, st)) != S4TF_OK) return rc;
  } else {
    hipLaunchKernelGGL(skinny_gemm_kernel<true>, sb.grid, dim3(256), 0, st, dz, W, part, d.n, d.c, d.classes, sb.kper);
    if ((rc = launch_status("head dpbar")) != S4TF_OK) return rc;
  }
  HEAD_LAUNCH(gap_vjp_kernel, pool_grid, part, waves ? 1 : sb.splits, (T*)dx, d.n, HW, d.c, cvs, d.accumulate_dx);
  return launch_status("gap_vjp");
}

int head_params(const s4tf_head_desc& d, float* loss, float* dW, float* db, void* ws, hipStream_t st) {
  const Layout l = layout(d);
  char* base = static_cast<char*>(ws);
  const float* pbar = reinterpret_cast<const float*>(base + l.pbar);
  const float* dz = reinterpret_cast<const float*>(base + l.dz);
  const float* rowloss = reinterpret_cast<const float*>(base + l.rowloss);
  if (small_head(d)) {
    ProfScope ps(PC_HEAD, st);
    hipLaunchKernelGGL(head_batch_kernel, dim3(((d.c + 1) * d.classes + 15) / 16 + 1), dim3(256), 0, st, pbar, dz, rowloss, dW, db,
                       loss, d.n, d.c, d.classes);
    return launch_status("head_batch");
  }
  int rc = igemm_wgrad(dense_geom(d.n, d.c, d.classes), S4TF_F32, pbar, dz, dW, base + l.wg, l.total - l.wg, st);
  if (rc != S4TF_OK) return rc;
  ProfScope ps(PC_HEAD, st);
  hipLaunchKernelGGL(head_bias_kernel, dim3((d.classes + 15) / 16 + 1), dim3(256), 0, st, dz, rowloss, db, loss, d.n, d.classes);
  return launch_status("head_bias");
}

int head_fwd_vjp(const s4tf_head_desc& d, const void* x, const float* W, const float* b, const int32_t* labels, float* loss,
                 void* dx, float* dW, float* db, float* logits_out, void* ws, hipStream_t st) {
  const int rc = head_value(d, x, W, b, labels, dx, logits_out, ws, st);
  return rc != S4TF_OK ? rc : head_params(d, loss, dW, db, ws, st);
}

}  // namespace s4tf
