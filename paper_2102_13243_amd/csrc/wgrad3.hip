// bf16 filter gradients of 3x3 / stride 1 / padding 1 layers whose channel counts are multiples of 32.
//
// The general kernel (igemm_dma.hip) gathers x once per tap: a 64x128 tile of dw takes 24 KB through the CU's 64-byte-per-cycle
// load path for every 256 cycles of MFMAs, and spends most of its time there (22 to 24 % of the matrix rate).  Here a workgroup
// owns 32 input channels x 32 output channels of all nine taps.  It brings the pixels of a band of rows (or of some whole small
// images) into LDS once, x with a border of zeros and dy, 64 bytes a pixel each, and multiplies all taps out of it: tap (r, s)
// reads x at a fixed distance from dy's pixel.  To make that true for 16 consecutive positions wherever they lie, both are laid
// out with W + 1 positions a row, the extra one zero, and run on over row ends: (W + 1) / W of the work, and no index
// arithmetic in the loop.
//   * v_mfma_f32_32x32x16_bf16: 32 input channels x 32 output channels, 16 positions; both operands are read with ds_read_b64_tr_b16
//     (four positions of 64 bytes are one sweep over the banks);
//   * the eight wavefronts, two per SIMD so that one's waits are the other's MFMAs, take every eighth group of 16 positions and
//     keep nine accumulators each, added through LDS at the end in wavefront order;
//   * the next band's direct loads are issued between the groups of this one (all of them ahead of the first group cost a fifth:
//     the load path takes them no faster); one workgroup per CU.
// Of 40 k cycles at 64x56x56, 64 channels, 18 k are the MFMAs of a SIMD's two wavefronts, 8 k waits for a band and for each
// other, 7 k the adding at the end, 2.5 k the first band; the rest of a call is the slabs that the splits of the pixels leave.
// Measured, with the reduction, us, general kernel -> this one: 64x56x56, 64 channels 51.2 -> 25.9; 64x28x28, 128 33.3 -> 25.0;
// 64x14x14, 256 35.5 -> 27.0; 64x7x7, 512 30.8 -> 21.5; 32x28x28, 128 24.1 -> 19.3; 13x11x11, 256 14.9 -> 13.1.
#include "s4tf_internal.h"
#include "igemm_args.h"

namespace s4tf {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr uint32_t OOB = 0x80000000u;  // a byte offset past every tensor on this path: such a load writes zeros
constexpr int POS = 64;                // bytes per position: 32 channels
constexpr int TILE = 9 * 32 * 32;
constexpr int LDS_LIMIT = 156 << 10;
constexpr int WAVES = 8;               // two per SIMD: one's waits are the other's MFMAs
constexpr int MAX_LOADS = 6;           // per wavefront and tensor of a unit

struct Wgrad3Args {
  const void* x;   // (N, H, W, C)
  const void* dy;  // (N, H, W, K)
  float* out;      // splits slabs of (3, 3, C, K)
  int N, H, W, C, K;
  int RB, imgs, bands;    // rows per unit of one image, or (imgs > 1) whole images per unit, a row of zeros between two
  int PW;                 // W + 1
  int units, splits;
  int groups;             // of 16 positions of dy in a unit
  int xpos, dpos;         // positions in LDS, multiples of 16
  uint32_t magicPW, magicH1, magicBands;  // / PW, / (H + 1), / bands
  int shiftPW, shiftH1, shiftBands;
};

__device__ inline i32x4 make_rsrc(const void* base, uint32_t bytes) {
  const uint64_t p = (uint64_t)base;
  i32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)p);
  r[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32));
  r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
  r[3] = 0x00020000;
  return r;
}
// 16 bytes per lane from buffer[voff] to LDS[lds + lane*16]
__device__ inline void dma16(uint32_t voff, i32x4 rsrc, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds" : : "v"(voff), "s"(rsrc), "s"(lds) : "memory");
}
__device__ inline bf16x8 read_fragment(uint32_t at) {  // 8 positions of this lane's channel
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(uintptr_t)at);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(uintptr_t)(at + 4 * POS));
  const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8, v);
}

__global__ __launch_bounds__(64 * WAVES, 2) void wgrad3_kernel(const Wgrad3Args a) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)smem);
  // Workgroup ids are dealt round-robin to the XCDs: each gets a contiguous run of (split, tile), tiles fastest, so that the
  // tiles of one split, which read the same pixels, share an L2.
  const int ct = a.C / 32, tiles = ct * (a.K / 32), all = tiles * a.splits, per = (all + NUM_XCD - 1) / NUM_XCD;
  const int u = (int)(blockIdx.x % NUM_XCD) * per + (int)(blockIdx.x / NUM_XCD);
  if ((int)(blockIdx.x / NUM_XCD) >= per || u >= all) return;
  const int split = u / tiles, tile = u - split * tiles, c0 = (tile % ct) * 32, k0 = (tile / ct) * 32;
  const int u0 = (int)((long long)a.units * split / a.splits), u1 = (int)((long long)a.units * (split + 1) / a.splits);
  const int buffer = (a.xpos + a.dpos) * POS;

  // The direct loads of a unit: 16 positions per instruction, lane l the 16-byte chunk l % 4 of position l / 4; wavefront w
  // issues every fourth.  A position's offset from the unit's first image is the same for every band but for the band's first
  // row: computed once.  The buffer is the unit's images: rows above and below them are out of its range and load as zeros.
  uint32_t xrel[MAX_LOADS], drel[MAX_LOADS];
  const int xloads = (a.xpos / 16 - wave + WAVES - 1) / WAVES, dloads = (a.dpos / 16 - wave + WAVES - 1) / WAVES;
#pragma unroll
  for (int k = 0; k < MAX_LOADS; ++k) {
    if (k >= xloads) break;
    const int at = (wave + WAVES * k) * 16 + (lane >> 2), ch = (lane & 3) * 8;
    const int row = div_magic(at, a.magicPW, a.shiftPW), col = at - row * a.PW, t = row - 1;
    int xn = 0, xh = t, dn = 0, dh = row;
    bool xok = col > 0, dok = (col < a.W) & (row < a.RB);
    if (a.imgs > 1) {  // (a row H of one image is the row -1 of the next: zeros)
      xn = t < 0 ? 0 : div_magic(t, a.magicH1, a.shiftH1);
      xh = t - xn * (a.H + 1);
      dn = div_magic(row, a.magicH1, a.shiftH1);
      dh = row - dn * (a.H + 1);
      xok = xok & (xh < a.H);
      dok = (col < a.W) & (dh < a.H);
    }
    xrel[k] = xok ? (uint32_t)((((xn * a.H + xh) * a.W + col - 1) * a.C + c0 + ch) * 2) : OOB;
    drel[k] = dok ? (uint32_t)((((dn * a.H + dh) * a.W + col) * a.K + k0 + ch) * 2) : OOB;
  }
  i32x4 rx, rd;
  uint32_t xbase = 0, dbase = 0, to = 0;  // of the unit being loaded
  auto aim = [&](int un, uint32_t lds) {
    int n0 = un * a.imgs, p0 = 0;
    if (a.imgs == 1) {
      n0 = div_magic(un, a.magicBands, a.shiftBands);
      p0 = (un - n0 * a.bands) * a.RB;
    }
    const int px = min(a.N - n0, a.imgs) * a.H * a.W;
    const long long first = (long long)n0 * a.H * a.W;
    rx = make_rsrc(static_cast<const char*>(a.x) + first * a.C * 2, (uint32_t)(px * a.C * 2));
    rd = make_rsrc(static_cast<const char*>(a.dy) + first * a.K * 2, (uint32_t)(px * a.K * 2));
    xbase = (uint32_t)(p0 * a.W * a.C * 2);
    dbase = (uint32_t)(p0 * a.W * a.K * 2);
    to = __builtin_amdgcn_readfirstlane(lds + wave * 1024);
  };
  auto load_x = [&](int k) {
    int n = xloads;
    asm volatile("" : "+s"(n));  // (compared where it is used: two dozen conditions kept in registers would not fit)
    if (k < n) dma16(xrel[k] + xbase, rx, to + k * (WAVES * 1024));
  };
  auto load_d = [&](int k) {
    int n = dloads;
    asm volatile("" : "+s"(n));
    if (k < n) dma16(drel[k] + dbase, rd, to + a.xpos * POS + k * (WAVES * 1024));
  };

  f32x16 acc[9];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
  // where this lane's part of a fragment lies: positions 8*(lane/32) .. +7, four channels each
  const uint32_t frag = (uint32_t)((8 * (lane >> 5) + ((lane & 15) >> 2)) * POS + ((lane >> 4) & 1) * 32 + (lane & 3) * 8);

  if (u0 < u1) {
    aim(u0, lds0);
#pragma unroll
    for (int k = 0; k < MAX_LOADS; ++k) { load_x(k); load_d(k); }
  }
  for (int un = u0; un < u1; ++un) {
    const uint32_t cur = lds0 + ((un - u0) & 1) * buffer;
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
    __syncthreads();  // this unit has landed, and everyone is done with the one before
    const bool more = un + 1 < u1;
    if (more) aim(un + 1, lds0 + ((un + 1 - u0) & 1) * buffer);
    const uint32_t x0 = cur + frag, d0 = x0 + a.xpos * POS;
#pragma unroll
    for (int k = 0; k < MAX_LOADS; ++k) {  // (groups <= WAVES * MAX_LOADS)
      if (more) {
        load_x(k);
        load_d(k);
      }
      const int g = wave + WAVES * k;
      if (g >= a.groups) continue;
      const uint32_t xg = x0 + g * (16 * POS);
      const bf16x8 bf = read_fragment(d0 + g * (16 * POS));
      bf16x8 af[9];
#pragma unroll
      for (int t = 0; t < 9; ++t) af[t] = read_fragment(xg + (t / 3) * a.PW * POS + (t % 3) * POS);
#pragma unroll
      for (int t = 0; t < 9; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[t], bf, acc[t], 0, 0, 0);
    }
  }
  // the wavefronts' accumulators, added in wavefront order
  __syncthreads();
  f32x4* red = reinterpret_cast<f32x4*>(smem);
#pragma unroll
  for (int half = 1; half >= 0; --half) {  // the upper four wavefronts hand theirs to the lower ones, those to everyone
    if (wave / 4 == half) {
#pragma unroll
      for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          f32x4& r = red[(wave & 3) * (TILE / 4) + (t * 4 + v) * 64 + lane];
          const f32x4 mine = {acc[t][4 * v], acc[t][4 * v + 1], acc[t][4 * v + 2], acc[t][4 * v + 3]};
          if (half == 1) r = mine;
          else r += mine;
        }
    }
    __syncthreads();
  }
  float* out = a.out + (long long)split * 9 * a.C * a.K + (long long)(c0 + 4 * (lane >> 5)) * a.K + k0 + (lane & 31);
#pragma unroll
  for (int k = 0; k < 5; ++k) {  // register group v of tap t: rows 8*v + 4*(lane/32) .. +3, column lane % 32
    const int tv = wave + WAVES * k, t = tv >> 2, v = tv & 3;
    if (tv >= 36) break;
    const f32x4* r = red + tv * 64 + lane;
    const f32x4 sum = ((r[0] + r[TILE / 4]) + r[2 * (TILE / 4)]) + r[3 * (TILE / 4)];
#pragma unroll
    for (int e = 0; e < 4; ++e) out[((long long)t * a.C + 8 * v + e) * a.K] = sum[e];
  }
}

struct Wgrad3Plan { int RB, imgs, groups, xpos, dpos, units, splits; };

// Rows or images per unit, and over how many workgroups the units of a tile are split: the least of rounds of 256 workgroups x
// (9000 cycles of prologue and end + units per workgroup x (600 per group of the busiest wavefront, of which two share a SIMD,
// + 700 for the unit's barrier and first reads)) + what the slabs cost the reduction.  Only the largest bands that
// fit and a few smaller ones are looked at: a call plans on the host each time.
bool plan_wgrad3(const ConvGeom& g, Wgrad3Plan& best) {
  const int PW = g.W + 1, tiles = (g.C / 32) * (g.K / 32);
  double best_cost = -1.0;
  auto look = [&](int RB, int imgs) {
    const int rows = imgs == 1 ? RB : imgs * (g.H + 1);
    Wgrad3Plan p;
    p.RB = RB;
    p.imgs = imgs;
    p.groups = (rows * PW + 15) / 16;
    p.dpos = p.groups * 16;
    p.xpos = (p.dpos + 2 * PW + 2 + 15) / 16 * 16;
    if (2 * (p.xpos + p.dpos) * POS > LDS_LIMIT || p.xpos > MAX_LOADS * WAVES * 16) return false;
    p.units = imgs == 1 ? g.N * ((g.H + RB - 1) / RB) : (g.N + imgs - 1) / imgs;
    for (int target = 32; target <= 512; target *= 2) {  // workgroups
      int s = target / tiles;
      if (s > p.units) s = p.units;
      if (s < 1) s = 1;
      const int per = (p.units + s - 1) / s;
      s = (p.units + per - 1) / per;
      const double rounds = (double)((tiles * s + 255) / 256);
      const double slabs = s > 1 ? 6000.0 + 72.0 * g.C * g.K * s / 2500.0 : 0.0;  // written and read, 2500 bytes a cycle
      const double cost = rounds * (9000.0 + per * (600.0 * ((p.groups + WAVES - 1) / WAVES) + 700.0)) + slabs;
      p.splits = s;
      if (best_cost < 0.0 || cost < best_cost) {
        best_cost = cost;
        best = p;
      }
    }
    return true;
  };
  int fitting = 0;
  for (int bands = 1; bands <= g.H && fitting < 4; ++bands) fitting += look((g.H + bands - 1) / bands, 1);
  for (int imgs = 2; imgs <= 16 && imgs <= g.N; imgs *= 2)
    if (!look(g.H, imgs)) break;
  return best_cost >= 0.0;
}

}  // namespace

bool wgrad3_ok(const ConvGeom& g, int dtype) {
  if (dtype != S4TF_BF16 || g.R != 3 || g.S != 3 || g.stride != 1 || g.pad != 1 || g.C % 32 || g.K % 32) return false;
  if ((long long)g.N * g.H * g.W < 512) return false;  // the general kernel has less to start up: 7x7, 512 channels 6.0 us, here 7.2; 13x6x6 10.0, 10.0
  const unsigned long long x = 2ull * g.N * g.H * g.W * g.C, y = 2ull * g.N * g.H * g.W * g.K;
  Wgrad3Plan p;
  return x < OOB && y < OOB && plan_wgrad3(g, p);
}
int wgrad3_splits(const ConvGeom& g) {
  Wgrad3Plan p;
  plan_wgrad3(g, p);
  return p.splits;
}

// `out`: wgrad3_splits(g) slabs of (3, 3, C, K)
int wgrad3(const ConvGeom& g, const void* x, const void* dy, float* out, hipStream_t st) {
  Wgrad3Plan p;
  if (!plan_wgrad3(g, p)) return fail(S4TF_ERR_UNSUPPORTED, "wgrad3: shape");
  Wgrad3Args a = {};
  a.x = x; a.dy = dy; a.out = out;
  a.N = g.N; a.H = g.H; a.W = g.W; a.C = g.C; a.K = g.K;
  a.RB = p.RB; a.imgs = p.imgs; a.bands = (g.H + p.RB - 1) / p.RB;
  a.PW = g.W + 1;
  a.units = p.units; a.splits = p.splits; a.groups = p.groups; a.xpos = p.xpos; a.dpos = p.dpos;
  magic_div(a.PW, a.magicPW, a.shiftPW);
  magic_div(g.H + 1, a.magicH1, a.shiftH1);
  magic_div(a.bands, a.magicBands, a.shiftBands);
  size_t lds = (size_t)2 * (p.xpos + p.dpos) * POS;
  if (lds < 4 * TILE * sizeof(float)) lds = 4 * TILE * sizeof(float);
  const int all = (g.C / 32) * (g.K / 32) * p.splits;
  hipLaunchKernelGGL(wgrad3_kernel, dim3(NUM_XCD * ((all + NUM_XCD - 1) / NUM_XCD)), dim3(64 * WAVES), lds, st, a);
  return launch_status("wgrad3");
}

}  // namespace s4tf
