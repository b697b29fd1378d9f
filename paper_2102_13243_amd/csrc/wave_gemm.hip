// fp32 implicit GEMM in which every wavefront works for itself: forward, input pullback and filter gradient of dense
// convolutions whose channel counts are multiples of 4 (the GEMM view is that of igemm.hip), and the head's products.
//
//   D[m][n] = sum_k A[m][k] B[k][n]
//
// The matrix rate of gfx950 in fp32 is a sixteenth of the bf16 one (v_mfma_f32_16x16x4_f32: 32 cycles for 2 KFLOP), so
// a 32 x 64 tile of one wavefront spends 1024 cycles on a k-step of 16 and needs 6 KB of operands for it: bandwidth is
// no concern at that tile size.  What bounds these layers (a few thousand such wavefront tiles, 9 to 80 k-steps each) is
// latency: with operand tiles shared by a workgroup, every k-tile paid a memory latency and two barriers.  Here a
// wavefront owns a ring of STAGES LDS slots, fills it with 16-byte direct loads (buffer_load ... lds) and waits only on
// its own vmcnt: no barrier in the loop, and wavefronts of a SIMD drift apart and cover each other.  Forward, batch 32,
// staged per workgroup / here: 14x14 576 -> 96 22.3 / 13.1 us, 7x7 960 -> 160 18.2 / 9.8; batch 5, 5x5 960 -> 160
// 17.7 / 6.7.  (Fragments loaded from global memory straight into registers were measured too: adjacent lanes then lie
// in different rows, four cache accesses per 64 bytes, and the address unit becomes the bound: 15.4, 12.7 and 11.3.)
//
// k-step: 16 values of k; MFMA e takes k = 4*(l/16) + e from lane l, so a lane's four values are adjacent.
//   * operands contiguous along k (A of forward and dgrad: rows of pixels; B of dgrad: filter rows) lie in LDS as
//     [row][16 k], 64 bytes a row, the 16-byte chunk XOR-ed with (row >> 2) & 3: 16 rows x one chunk, the ds_read_b128
//     of a fragment, touches every bank once (block j of dgrad's B is every F-th filter row, which gives its outputs the layout below);
//   * operands contiguous along the GEMM row (B of forward: filters; both operands of wgrad: pixels x channels) lie as
//     [k][16*F rows], and lane l reads the F adjacent rows F*(l%16) .. of one k in one instruction: block j of the MFMA
//     output then holds rows (columns) F*(l%16) + j, and a lane's F outputs are adjacent in memory.
// GEMMs with few tiles split the k-steps over the WK wavefronts of a workgroup (added through LDS in wavefront order);
// filter gradients also over workgroups (slabs, added by splitk_reduce_kernel in order).
// Padding, strides, ragged edges and channel counts that are no multiple of 16 are out-of-range buffer offsets: zeros.
#include "s4tf_internal.h"
#include "igemm_args.h"

namespace s4tf {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

struct WaveArgs {
  const float* a;
  const float* b;
  float* out;
  const float* bias;  // forward, optional
  const float* mask;  // dgrad, optional: the layer's input, the result is multiplied by the derivative of the activation that made it
  float* db;          // wgrad, optional: column sums of b
  float* stats;       // forward, optional: BatchNorm partial sums per run of one workgroup's rows, see igemm_fwd
  int M, N, K;        // K: channels per tap (forward, dgrad), pixels (wgrad)
  int C;              // wgrad: channels of x
  int H, W, S, stride, pad;  // forward, wgrad: the image A gathers from; dgrad: P x Q of dy
  int P, Q;           // forward, dgrad: rows are (image, p, q); wgrad: k is (image, p, q)
  int taps, spt, steps;      // k-steps per tap and in all
  int act, accumulate;
  int tiles_m, tiles_n, splits;
  uint32_t a_bytes, b_bytes;
  uint32_t magicQ, magicP, magicC, magicS;
  int shiftQ, shiftP, shiftC, shiftS;
};

constexpr uint32_t OOB = 0x80000000u;  // past every tensor on this path: such a load writes zeros
constexpr int KS = 16;
constexpr int FM = 2;  // 32 rows per wavefront

__device__ inline i32x4 make_rsrc(const void* base, uint32_t bytes) {
  const uint64_t p = (uint64_t)base;
  i32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)p);
  r[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32));
  r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
  r[3] = 0x00020000;
  return r;
}
// 16 bytes per lane from buffer[voff] to LDS[lds + lane*16]; inline assembly so that the compiler does not count these
// loads and put full waits into the loop
__device__ inline void dma16(uint32_t voff, i32x4 rsrc, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds" : : "v"(voff), "s"(rsrc), "s"(lds) : "memory");
}
template <int N> __device__ inline void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory"); }
__device__ inline void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory"); }

template <int F> struct Vec;
template <> struct Vec<1> { typedef float type; };
template <> struct Vec<2> { typedef f32x2 type; };
template <> struct Vec<4> { typedef f32x4 type; };
template <int F> __device__ inline float elem(const typename Vec<F>::type& v, int j) { if constexpr (F == 1) return v; else return v[j]; }
template <typename T> __device__ inline T lds_read(uint32_t at) {
  return *(const __attribute__((address_space(3))) T*)(uintptr_t)at;
}

__device__ inline int div_stride(int x, int stride) { return stride == 1 ? x : stride == 2 ? x >> 1 : x / stride; }  // x >= 0

// POINT: a plain matrix product (1x1 / stride 1 / no padding layers, dense layers)
template <int PASS, bool POINT, int FN, int WM, int WK, int STAGES>
__global__ __launch_bounds__(64 * WM * WK, 2) void wave_gemm_kernel(const WaveArgs g) {
  constexpr bool AROW = PASS == PASS_WGRAD, BROW = PASS != PASS_DGRAD;  // contiguous along the GEMM row, not along k
  constexpr int BM = WM * FM * 16, BN = FN * 16, LOADS = FM + FN, SLOT = LOADS * 1024, RING = STAGES * SLOT;
  constexpr int NW = WM * WK, REDB = (WK - 1) * WM * FM * FN * 4 * 64 * 4, STATB = WM * BN * 2 * 4;
  constexpr int SMEM = NW * RING > REDB ? NW * RING : REDB;
  static_assert(STATB <= SMEM, "");
  __shared__ __attribute__((aligned(1024))) char smem[SMEM];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave % WM, wk = wave / WM, l16 = lane & 15, g4 = lane >> 4;
  // Workgroup ids are dealt round-robin to the XCDs: each gets a contiguous run of (split, row tile, column tile),
  // columns fastest, so that what neighbours share stays in one L2.
  const int tiles = g.tiles_m * g.tiles_n, units = tiles * g.splits, per = (units + NUM_XCD - 1) / NUM_XCD;
  const int u = (int)(blockIdx.x % NUM_XCD) * per + (int)(blockIdx.x / NUM_XCD);
  if constexpr (PASS == PASS_WGRAD) {
    if ((int)(blockIdx.x / NUM_XCD) >= per) {  // behind the last tile: workgroups that sum 16 columns of dy each, the bias gradient
      constexpr int LANES = 4 * WM * WK;
      double* sh = reinterpret_cast<double*>(smem);
      const int c = threadIdx.x & 15, l = threadIdx.x >> 4, col = ((int)blockIdx.x - NUM_XCD * per) * 16 + c;
      double s = 0.0;  // bias cotangents cancel heavily: in double
      if (col < g.N) {
#pragma unroll 4
        for (int px = l; px < g.K; px += LANES) s += (double)g.b[(long long)px * g.N + col];
      }
      sh[threadIdx.x] = s;
      __syncthreads();
      if (l == 0 && col < g.N) {
        for (int i = 1; i < LANES; ++i) s += sh[i * 16 + c];
        g.db[col] = (float)s;
      }
      return;
    }
  }
  if ((int)(blockIdx.x / NUM_XCD) >= per || u >= units) return;
  const int split = u / tiles, t = u - split * tiles, tm = t / g.tiles_n, tn = t - tm * g.tiles_n;
  const int m0 = tm * BM + wm * FM * 16, n0 = tn * BN;
  const uint32_t ring = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)smem) + wave * RING;
  const i32x4 ra = make_rsrc(g.a, g.a_bytes), rb = make_rsrc(g.b, g.b_bytes);

  // ---- what this lane fetches ----
  // k-contiguous: instruction i fetches rows i*16 + lane/4, the lane's chunk lane%4 of the row holds k-chunk kc
  // row-contiguous, F blocks: the 16 x 16*F values of a step are F KB, instruction i the i-th of them
  const int kc4 = ((lane & 3) ^ (g4 & 3)) * 4;
  int abase[FM], ak[FM];  // element offset that does not depend on the step; k inside a step (row-contiguous)
  uint32_t amask[FM];     // taps inside the image (k-contiguous), or whether the rows exist (row-contiguous)
  int ah[FM], aw[FM];     // wgrad: tap offset (r - pad, s - pad) of this lane's rows
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    if constexpr (AROW) {
      ak[i] = i * (16 / FM) + lane / (4 * FM);
      const int m = m0 + (lane % (4 * FM)) * 4;
      amask[i] = m < g.M;
      if constexpr (POINT) {
        abase[i] = m;
        ah[i] = aw[i] = 0;
      } else {
        const int t2 = div_magic(m, g.magicC, g.shiftC), c = m - t2 * g.C, r = div_magic(t2, g.magicS, g.shiftS), s = t2 - r * g.S;
        abase[i] = c;
        ah[i] = r - g.pad;
        aw[i] = s - g.pad;
      }
    } else {
      ak[i] = kc4;
      const int m = m0 + i * 16 + (lane >> 2);
      if constexpr (POINT) {
        amask[i] = m < g.M;
        abase[i] = m * g.K + kc4;
      } else {
        const int tq = div_magic(m, g.magicQ, g.shiftQ), q = m - tq * g.Q, n = div_magic(tq, g.magicP, g.shiftP), p = tq - n * g.P;
        uint32_t mask = 0;
        if constexpr (PASS == PASS_FWD) {
          const int h = p * g.stride - g.pad, w = q * g.stride - g.pad;
          abase[i] = ((n * g.H + h) * g.W + w) * g.K + kc4;
          if (m < g.M)
            for (int tap = 0, r = 0, s = 0; tap < g.taps; ++tap) {
              if (h + r >= 0 && h + r < g.H && w + s >= 0 && w + s < g.W) mask |= 1u << tap;
              if (++s == g.S) { s = 0; ++r; }
            }
        } else {  // pixel (p, q) of dx meets dy at ((p + pad - r)/stride, (q + pad - s)/stride) where that is whole
          const int hp = p + g.pad, wp = q + g.pad, h = div_stride(hp, g.stride), w = div_stride(wp, g.stride), hr = hp - h * g.stride, wr = wp - w * g.stride;
          abase[i] = ((n * g.H + h) * g.W + w) * g.K + kc4;
          if (m < g.M)
            for (int tap = 0, r = 0, s = 0; tap < g.taps; ++tap) {
              const int rd = div_stride(r, g.stride), sd = div_stride(s, g.stride);
              if (r - rd * g.stride == hr && s - sd * g.stride == wr && h - rd >= 0 && h - rd < g.H && w - sd >= 0 && w - sd < g.W)
                mask |= 1u << tap;
              if (++s == g.S) { s = 0; ++r; }
            }
        }
        amask[i] = mask;
      }
    }
  }
  int bbase[FN], bk[FN];
  bool bin[FN];
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    if constexpr (BROW) {
      bk[j] = j * (16 / FN) + lane / (4 * FN);
      const int n = n0 + (lane % (4 * FN)) * 4;
      bin[j] = n < g.N;
      bbase[j] = bk[j] * g.N + n;
    } else {
      bk[j] = kc4;
      const int n = n0 + FN * (lane >> 2) + j;  // block j takes every FN-th column, as in the other layout
      bin[j] = n < g.N;
      bbase[j] = n * g.K + kc4;
    }
  }

  // ---- k-steps of this wavefront ----
  const int part = split * WK + wk, parts = g.splits * WK;
  const int s0 = (int)((long long)g.steps * part / parts), s1 = (int)((long long)g.steps * (part + 1) / parts);
  int ls = s0, tap = 0, c0, rr = 0, ss = 0;  // the next step to load: its tap and first k (wavefront-uniform)
  if constexpr (POINT || AROW) {
    c0 = s0 * KS;
  } else {
    tap = s0 / g.spt;
    c0 = (s0 - tap * g.spt) * KS;
    rr = tap / g.S;
    ss = tap - rr * g.S;
  }
  auto load = [&](uint32_t slot) {
    const bool live = ls < s1;
    int ua = c0, ub;  // element offsets of this step
    if constexpr (PASS == PASS_FWD) {
      if (!POINT) ua = (rr * g.W + ss) * g.K + c0;
      ub = (tap * g.K + c0) * g.N;
    } else if constexpr (PASS == PASS_DGRAD) {
      if (!POINT) ua = c0 - (div_stride(rr, g.stride) * g.W + div_stride(ss, g.stride)) * g.K;
      ub = tap * g.N * g.K + c0;
    } else {
      ub = c0 * g.N;
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      uint32_t off;
      if constexpr (!AROW) {
        const bool ok = live & (c0 + ak[i] < g.K) & (((amask[i] >> (POINT ? 0 : tap)) & 1) != 0);
        off = ok ? (uint32_t)(abase[i] + ua) * 4u : OOB;
      } else if constexpr (POINT) {
        const int px = c0 + ak[i];
        off = (live & (amask[i] != 0) & (px < g.K)) ? (uint32_t)(px * g.C + abase[i]) * 4u : OOB;
      } else {
        const int px = c0 + ak[i];
        const int tq = div_magic(px, g.magicQ, g.shiftQ), q = px - tq * g.Q, n = div_magic(tq, g.magicP, g.shiftP), p = tq - n * g.P;
        const int h = p * g.stride + ah[i], w = q * g.stride + aw[i];
        const bool ok = live & (amask[i] != 0) & (px < g.K) & ((unsigned)h < (unsigned)g.H) & ((unsigned)w < (unsigned)g.W);
        off = ok ? (uint32_t)(((n * g.H + h) * g.W + w) * g.C + abase[i]) * 4u : OOB;
      }
      dma16(off, ra, slot + i * 1024);
    }
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const bool ok = live & bin[j] & (c0 + bk[j] < g.K);
      dma16(ok ? (uint32_t)(bbase[j] + ub) * 4u : OOB, rb, slot + (FM + j) * 1024);
    }
    ++ls;
    c0 += KS;
    if (!POINT && !AROW && c0 >= g.K) {
      c0 = 0;
      ++tap;
      if (++ss == g.S) { ss = 0; ++rr; }
    }
  };

  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // fragment addresses inside a slot
  const uint32_t fk = ring + l16 * 64 + ((g4 ^ ((l16 >> 2) & 3)) * 16);               // k-contiguous
  const uint32_t fra = ring + g4 * 4 * FM * 64 + l16 * FM * 4;                          // row-contiguous: A
  const uint32_t frb = ring + FM * 1024 + g4 * 4 * FN * 64 + l16 * FN * 4;              // row-contiguous: B
#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s) load(ring + s * SLOT);
  for (int s = s0; s < s1; s += STAGES) {
    // written out once per slot; steps beyond the last multiply zeros
#pragma unroll
    for (int d = 0; d < STAGES; ++d) {
      if (d > 0 && s + d >= s1) break;
      wait_vmcnt<(STAGES - 2) * LOADS>();  // the step's operands have landed
      f32x4 ac[FM];                        // k-contiguous: [block] -> its four k
      typename Vec<FM>::type ar[4];        // row-contiguous: [k] -> its blocks
      f32x4 bc[FN];
      typename Vec<FN>::type br[4];
      if constexpr (AROW) {
#pragma unroll
        for (int e = 0; e < 4; ++e) ar[e] = lds_read<typename Vec<FM>::type>(fra + d * SLOT + e * FM * 64);
      } else {
#pragma unroll
        for (int i = 0; i < FM; ++i) ac[i] = lds_read<f32x4>(fk + d * SLOT + i * 1024);
      }
      if constexpr (BROW) {
#pragma unroll
        for (int e = 0; e < 4; ++e) br[e] = lds_read<typename Vec<FN>::type>(frb + d * SLOT + e * FN * 64);
      } else {
#pragma unroll
        for (int j = 0; j < FN; ++j) bc[j] = lds_read<f32x4>(fk + d * SLOT + (FM + j) * 1024);
      }
      // the slot of the step before this one was read completely before its MFMAs: refill it
      load(ring + ((d + STAGES - 1) % STAGES) * SLOT);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            const float av = AROW ? elem<FM>(ar[e], i) : ac[i][e];
            const float bv = BROW ? elem<FN>(br[e], j) : bc[j][e];
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv, acc[i][j], 0, 0, 0);
          }
      wait_lds();  // (all of this step's reads are long done: the MFMAs consumed them)
    }
  }
  wait_vmcnt<0>();  // direct loads of steps beyond the last still write this wavefront's ring

  float* red = reinterpret_cast<float*>(smem);
  if constexpr (WK > 1) {  // the accumulators of wavefronts wk = 1 .. WK-1 are added to those of wk = 0, in that order
    __syncthreads();
    if (wk > 0) {
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          *reinterpret_cast<f32x4*>(red + ((((wk - 1) * WM + wm) * FM + i) * FN + j) * 256 + lane * 4) = acc[i][j];
    }
    __syncthreads();
    if (wk == 0) {
#pragma unroll
      for (int k = 0; k < WK - 1; ++k)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j)
            acc[i][j] += *reinterpret_cast<const f32x4*>(red + (((k * WM + wm) * FM + i) * FN + j) * 256 + lane * 4);
    }
  }

  // block (i, j), register v of a lane: row and column inside the wavefront's tile
  auto row_of = [&](int i, int v) { return AROW ? FM * (4 * g4 + v) + i : i * 16 + 4 * g4 + v; };
  auto col_of = [&](int j) { return FN * l16 + j; };

  if constexpr (PASS == PASS_FWD) {
    if (g.stats) {
      // per output channel over the workgroup's rows: the sum, and the sum of squared deviations from the rows' own
      // mean.  A wavefront sums deviations from a pivot, its first row's value, so that a channel mean of many
      // standard deviations costs no digits; the WM row blocks are joined with the pairwise formula.
      __syncthreads();
      const long long runs = g.tiles_m;
      if (wk == 0) {
        const int rows = min(max(g.M - m0, 0), FM * 16);
        const float inv = rows > 0 ? 1.f / (float)rows : 0.f;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const float pivot = __shfl(acc[0][j][0], l16, 64);
          float s = 0.f, q = 0.f;
#pragma unroll
          for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const float dev = row_of(i, v) < rows ? acc[i][j][v] - pivot : 0.f;
              s += dev;
              q = fmaf(dev, dev, q);
            }
          s += __shfl_xor(s, 16, 64); q += __shfl_xor(q, 16, 64);
          s += __shfl_xor(s, 32, 64); q += __shfl_xor(q, 32, 64);
          if (lane < 16) {
            red[(wm * BN + col_of(j)) * 2] = fmaf((float)rows, pivot, s);
            red[(wm * BN + col_of(j)) * 2 + 1] = fmaxf(q - s * s * inv, 0.f);
          }
        }
      }
      __syncthreads();
      const int col = n0 + (int)threadIdx.x;
      if ((int)threadIdx.x < BN && col < g.N) {
        float sum = red[threadIdx.x * 2], m2 = red[threadIdx.x * 2 + 1], n = (float)min(g.M - tm * BM, FM * 16);
#pragma unroll
        for (int w = 1; w < WM; ++w) {
          const int left = min(g.M - tm * BM - w * FM * 16, FM * 16);
          if (left <= 0) break;
          const float nb = (float)left, sb = red[(w * BN + threadIdx.x) * 2], mb = red[(w * BN + threadIdx.x) * 2 + 1];
          const float d = sb / nb - sum / n;
          m2 += mb + d * d * (n * nb / (n + nb));
          sum += sb;
          n += nb;
        }
        g.stats[(long long)col * runs + tm] = sum;
        g.stats[(long long)(g.N + col) * runs + tm] = m2;
      }
    }
  }
  if (WK > 1 && wk > 0) return;
  float* out = g.out + (PASS == PASS_WGRAD ? (long long)split * g.M * g.N : 0);
  const float lo = (PASS == PASS_FWD && g.act != S4TF_ACT_NONE) ? 0.f : -__builtin_inff();
  const float hi = (PASS == PASS_FWD && g.act == S4TF_ACT_RELU6) ? 6.f : __builtin_inff();
  typedef typename Vec<FN>::type V;
  const int col = n0 + FN * l16;  // FN adjacent columns per lane
  if (col >= g.N) return;
  if (FN == 1 || g.N % FN == 0) {
    float bias[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) bias[j] = (PASS == PASS_FWD && g.bias) ? g.bias[col + j] : 0.f;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = m0 + row_of(i, v);
        if (row >= g.M) continue;
        V* dst = reinterpret_cast<V*>(out + (long long)row * g.N + col);
        V o, old, y;
        if (PASS == PASS_DGRAD && g.accumulate) old = *dst;
        if (PASS == PASS_DGRAD && g.mask) y = *reinterpret_cast<const V*>(g.mask + (long long)row * g.N + col);
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          float val = acc[i][j][v];
          if constexpr (PASS == PASS_FWD) val = fminf(fmaxf(val + bias[j], lo), hi);
          if (PASS == PASS_DGRAD && g.accumulate) val += elem<FN>(old, j);
          if (PASS == PASS_DGRAD && g.mask) val *= act_mask(elem<FN>(y, j), g.act);
          if constexpr (FN == 1) o = val; else o[j] = val;
        }
        *dst = o;
      }
  } else {  // input pullbacks of layers with an odd number of input channels
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      if (col + j >= g.N) break;
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = m0 + row_of(i, v);
          if (row >= g.M) continue;
          const long long at = (long long)row * g.N + col + j;
          float val = g.accumulate ? acc[i][j][v] + out[at] : acc[i][j][v];
          if (PASS == PASS_DGRAD && g.mask) val *= act_mask(g.mask[at], g.act);
          out[at] = val;
        }
    }
  }
}

// Ring slots: a step is 256 (FN = 1) to 1024 cycles long, so two slots hide an L2 latency once a SIMD holds two or three
// wavefronts; the filter gradient's operands come from farther away and its grids are exact, it takes three.
constexpr int stages_of(int pass) { return pass == PASS_WGRAD ? 3 : 2; }

// How a GEMM is cut: FN blocks of 16 columns per wavefront, WM x WK wavefronts per workgroup, splits over workgroups.
struct WavePlan { int FN, WM, WK, splits; };

// Picks the cut with the least estimated time.  The estimate (in cycles) counts what was seen to matter, with constants
// fitted to 3800 timings of 40 shapes in all cuts (on average the pick takes 3 % longer than the best cut): the CUs
// take whole workgroups, so the fullest CU decides; it runs them in rounds of what its LDS and wavefront slots hold; a
// round costs its start and its steps, a step 256 cycles of matrix work per column block and wavefront of the SIMD plus
// the loads, but no less than the latency the ring leaves exposed; adding accumulators over WK wavefronts, and slabs
// over workgroups, cost extra.
WavePlan plan_for(int pass, int M, int N, long long steps) {
  const int stages = stages_of(pass);
  WavePlan best = {1, 4, 1, 1};
  double best_cost = -1.0;
  static const int kSplits[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256};
  const double slab_bytes = 4.0 * M * N;
  for (int FN = 1; FN <= 4; FN *= 2) {
    if (FN > 1 && 8 * FN >= N) break;  // half of the columns would be padding
    for (int WK = 1; WK <= 8; WK *= 2) {
      if (WK > 1 && WK > steps) break;
      const int WM = WK >= 4 ? 1 : 4 / WK, nw = WM * WK;
      const long long tiles = (long long)((M + 32 * WM - 1) / (32 * WM)) * ((N + 16 * FN - 1) / (16 * FN));
      const int cap = min(160 / (nw * stages * (2 + FN)), 32 / nw);  // workgroups a CU holds
      for (int sp : kSplits) {
        if (sp > 1 && (pass != PASS_WGRAD || steps < 2LL * sp * WK || tiles * sp * nw > 8192)) break;
        const long long per_cu = (tiles * sp + 255) / 256, rounds = (per_cu + cap - 1) / cap;
        double waves = (double)per_cu / (double)rounds * nw / 4.0;  // per SIMD
        if (waves < 1.0) waves = 1.0;
        double step = waves * (256.0 * FN + 21.0 * (2 + FN));
        if (step < 850.0) step = 850.0;
        double cost = (double)rounds * (5500.0 + (double)((steps + (long long)WK * sp - 1) / ((long long)WK * sp)) * step) + 58.0 * (WK - 1) * FN * waves;
        if (sp > 1) cost += 5200.0 + 3500e-6 * sp * slab_bytes;
        if (best_cost < 0.0 || cost < best_cost) {
          best_cost = cost;
          best = {FN, WM, WK, sp};
        }
      }
    }
  }
  return best;
}

template <int PASS, bool POINT, int FN, int WM, int WK> int launch_wave(WaveArgs& a, int splits, hipStream_t st) {
  a.tiles_m = (a.M + WM * FM * 16 - 1) / (WM * FM * 16);
  a.tiles_n = (a.N + FN * 16 - 1) / (FN * 16);
  a.splits = splits;
  const int units = a.tiles_m * a.tiles_n * splits, bias = PASS == PASS_WGRAD && a.db ? (a.N + 15) / 16 : 0;
  hipLaunchKernelGGL((wave_gemm_kernel<PASS, POINT, FN, WM, WK, stages_of(PASS)>), dim3(NUM_XCD * ((units + NUM_XCD - 1) / NUM_XCD) + bias),
                     dim3(64 * WM * WK), 0, st, a);
  return launch_status("wave_gemm");
}
template <int PASS, bool POINT, int FN> int launch_wave(const WavePlan& p, WaveArgs& a, hipStream_t st) {
  switch (p.WK) {
    case 1: return launch_wave<PASS, POINT, FN, 4, 1>(a, p.splits, st);
    case 2: return launch_wave<PASS, POINT, FN, 2, 2>(a, p.splits, st);
    case 4: return launch_wave<PASS, POINT, FN, 1, 4>(a, p.splits, st);
    default: return launch_wave<PASS, POINT, FN, 1, 8>(a, p.splits, st);
  }
}
template <int PASS> int launch_wave(const WavePlan& p, bool point, WaveArgs& a, hipStream_t st) {
  a.spt = (a.K + KS - 1) / KS;
  a.steps = PASS == PASS_WGRAD ? a.spt : a.taps * a.spt;
  if (!point) {
    magic_div(a.Q, a.magicQ, a.shiftQ);
    magic_div(a.P, a.magicP, a.shiftP);
    magic_div(a.C, a.magicC, a.shiftC);
    magic_div(a.S, a.magicS, a.shiftS);
  }
  if (p.FN == 4) return point ? launch_wave<PASS, true, 4>(p, a, st) : launch_wave<PASS, false, 4>(p, a, st);
  if (p.FN == 2) return point ? launch_wave<PASS, true, 2>(p, a, st) : launch_wave<PASS, false, 2>(p, a, st);
  return point ? launch_wave<PASS, true, 1>(p, a, st) : launch_wave<PASS, false, 1>(p, a, st);
}

bool is_point(const ConvGeom& g) { return g.R == 1 && g.S == 1 && g.stride == 1 && g.pad == 0; }
long long steps_of(int pass, const ConvGeom& g) {
  if (pass == PASS_WGRAD) return ((long long)g.N * g.P * g.Q + KS - 1) / KS;
  return (long long)g.R * g.S * (((pass == PASS_FWD ? g.C : g.K) + KS - 1) / KS);
}
WavePlan plan_of(int pass, const ConvGeom& g) {
  if (pass == PASS_FWD) return plan_for(pass, g.N * g.P * g.Q, g.K, steps_of(pass, g));
  if (pass == PASS_DGRAD) return plan_for(pass, g.N * g.H * g.W, g.C, steps_of(pass, g));
  return plan_for(pass, g.R * g.S * g.C, g.K, steps_of(pass, g));
}

}  // namespace

// 16-byte chunks along the channels; byte offsets are 32-bit and stay below OOB; a lane's taps are bits of one word
bool wave_gemm_ok(int pass, const ConvGeom& g, int dtype) {
  const unsigned long long x = 4ull * g.N * g.H * g.W * g.C, y = 4ull * g.N * g.P * g.Q * g.K, w = 4ull * g.R * g.S * g.C * g.K;
  if (dtype != S4TF_F32 || x >= OOB || y >= OOB || w >= OOB || g.R * g.S > 32) return false;
  if (g.K % 4 || (pass != PASS_DGRAD && g.C % 4)) return false;
  // a k-step of 16 lies inside one tap: few channels (the first layers of a net) waste most of it
  const int ch = pass == PASS_DGRAD ? g.K : g.C;
  return pass == PASS_WGRAD || g.R * g.S == 1 || 3 * ch >= 2 * ((ch + KS - 1) / KS * KS);
}

int wave_gemm_fwd(const ConvGeom& g, const float* x, const float* w, const float* bias, int act, float* y, float* stats,
                  int* stats_rows, hipStream_t st) {
  const WavePlan p = plan_of(PASS_FWD, g);
  WaveArgs a = {};
  a.a = x; a.b = w; a.out = y; a.bias = bias; a.act = act; a.stats = stats;
  a.M = g.N * g.P * g.Q; a.N = g.K; a.K = a.C = g.C;
  a.H = g.H; a.W = g.W; a.S = g.S; a.stride = g.stride; a.pad = g.pad; a.P = g.P; a.Q = g.Q; a.taps = g.R * g.S;
  a.a_bytes = 4u * (unsigned)(g.N * g.H * g.W * g.C);
  a.b_bytes = 4u * (unsigned)(a.taps * g.C * g.K);
  if (stats) *stats_rows = p.WM * FM * 16;
  return launch_wave<PASS_FWD>(p, is_point(g), a, st);
}

// mask (optional): the layer's own input; dx is then multiplied by act'(mask), the pullback of the activation that made it
int wave_gemm_dgrad(const ConvGeom& g, const float* dy, const float* w, float* dx, int accumulate, const float* mask, int mask_act,
                    hipStream_t st) {
  WaveArgs a = {};
  a.a = dy; a.b = w; a.out = dx; a.accumulate = accumulate; a.mask = mask; a.act = mask_act;
  a.M = g.N * g.H * g.W; a.N = g.C; a.K = a.C = g.K;
  a.H = g.P; a.W = g.Q; a.S = g.S; a.stride = g.stride; a.pad = g.pad; a.P = g.H; a.Q = g.W; a.taps = g.R * g.S;
  a.a_bytes = 4u * (unsigned)(g.N * g.P * g.Q * g.K);
  a.b_bytes = 4u * (unsigned)(a.taps * g.C * g.K);
  return launch_wave<PASS_DGRAD>(plan_of(PASS_DGRAD, g), is_point(g), a, st);
}

// Up to 4096 pixels a workgroup's walk down 16 columns is shorter than the tiles beside it (dense layers at batch 128: the
// separate column sum took 8 us, this nothing that shows); longer ones need the two-stage sum.
bool wave_gemm_bias_ok(const ConvGeom& g) { return (long long)g.N * g.P * g.Q < 4096; }
int wave_gemm_wgrad_splits(const ConvGeom& g) { return plan_of(PASS_WGRAD, g).splits; }

// `out`: wave_gemm_wgrad_splits(g) slabs of (R, S, C, K); db (optional, see wave_gemm_bias_ok): the bias gradient
int wave_gemm_wgrad(const ConvGeom& g, const float* x, const float* dy, float* out, float* db, hipStream_t st) {
  WaveArgs a = {};
  a.a = x; a.b = dy; a.out = out; a.db = db;
  a.M = g.R * g.S * g.C; a.N = g.K; a.K = g.N * g.P * g.Q; a.C = g.C;
  a.H = g.H; a.W = g.W; a.S = g.S; a.stride = g.stride; a.pad = g.pad; a.P = g.P; a.Q = g.Q; a.taps = g.R * g.S;
  a.a_bytes = 4u * (unsigned)(g.N * g.H * g.W * g.C);
  a.b_bytes = 4u * (unsigned)(g.N * g.P * g.Q * g.K);
  return launch_wave<PASS_WGRAD>(plan_of(PASS_WGRAD, g), is_point(g), a, st);
}

}  // namespace s4tf
