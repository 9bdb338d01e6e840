// Learned peak filter: a 3D CNN that scores each threshold peak from the
// 5 x 5 x 5 votes around it (the paper's call for efficiency and purity
// improvements of the peak finding, section "Summary").
//
// Precision contract (identical in the oracle): bfloat16 inputs, weights and
// activations, float32 accumulation; bias after the sum; ReLU; activations
// rounded to bfloat16 (round to nearest even) before the next layer.
//
// Inference runs on the matrix cores with gfx950's v_mfma_f32_16x16x32_bf16
// (A: 16 x 32 bf16 with row m = lane % 16 and k = 8 (lane / 16) + i in
// element i; B likewise with column n = lane % 16; D: row 4 (lane / 16) + i,
// column lane % 16; checked on the device against a host product).  One
// wave scores 16 windows, the columns of every product:
//   conv1  one k-step per output position (27 taps padded to 32): M = 16
//          channels, the B operand built from the window's rows;
//   conv2  14 k-steps of two positions x 16 input channels each, right after
//          the conv1 of its two positions and from their registers;
//   fc1    4 m-tiles of 16 features with the K = 16 instruction; fc2 a dot
//          product on the VALU.
// ht_cnn_score builds each wave's 16 windows in LDS straight from the
// accumulator (no window buffer in HBM).  Training (offline) runs the same
// forward, keeps the activations, and computes the gradients with the matrix
// cores as well (see backward_kernel).
#include "ht_internal.h"

namespace ht {
namespace {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) {
  bf16x8 r;
  __builtin_memcpy(&r, &v, 16);
  return r;
}

constexpr int kWin = HT_CNN_WINDOW;  // bf16 per window (125 used)

__device__ __forceinline__ uint16_t to_bf16(float f) {
  const uint32_t u = __float_as_uint(f);
  const uint32_t lsb = (u >> 16) & 1u;
  return (uint16_t)((u + 0x7FFFu + lsb) >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// parameter offsets in the flat float32 vector
constexpr int oW1 = 0, ob1 = oW1 + 16 * 27, oW2 = ob1 + 16, ob2 = oW2 + 16 * 16 * 27,
              oW3 = ob2 + 16, ob3 = oW3 + 64 * 16, oW4 = ob3 + 64, ob4 = oW4 + 64;
static_assert(ob4 + 1 == HT_CNN_PARAMS, "parameter layout");

constexpr int kC2Steps = 14;  // conv2 k-steps: two positions x 16 channels (position 27 zero)

struct alignas(16) Packed {
  uint16_t w1[64 * 8];             // conv1 operand per lane (K = 32: taps, padded)
  uint16_t w2[kC2Steps * 64 * 8];  // conv2 operand per k-step and lane (K = 32)
  uint16_t w3[4 * 64 * 4];         // fc1 operand per feature tile and lane (K = 16)
  float b1[16], b2[16], b3[64], w4[64], b4[4];
};
static_assert(sizeof(Packed) % 16 == 0, "packed weights are copied in 16-byte chunks");

// conv1's order within a lane's eight taps (lane group g holds taps 8 g .. 8 g +
// 7; -1: zero weight): two rows of three cells and two single cells, so that
// the window's rows are read whole (see forward_kernel)
__device__ constexpr int8_t kTap[4][8] = {{0, 1, 3, 4, 2, 5, 6, 7},
                                          {9, 10, 12, 13, 11, 14, 8, 15},
                                          {18, 19, 21, 22, 20, 23, 16, 17},
                                          {24, 25, -1, -1, 26, -1, -1, -1}};
// conv1's result row 4 g + i is channel chan_of(g) + i
__device__ __forceinline__ int chan_of(int g) { return 8 * (g & 1) + 4 * (g >> 1); }

// The weights in operand order; with zero, a training step's gradient (and its
// loss) cleared beside them.  One element per thread (one workgroup took 8 us).
constexpr int kPackW1 = 64 * 8, kPackW2 = kC2Steps * 64 * 8, kPackW3 = 4 * 64 * 4;
constexpr int kPackAll = kPackW1 + kPackW2 + kPackW3 + 64;
__global__ __launch_bounds__(256) void pack_kernel(const float* __restrict__ P, Packed* __restrict__ W,
                                                   float* __restrict__ zero,
                                                   float* __restrict__ loss) {
  int e = blockIdx.x * 256 + threadIdx.x;
  if (zero && e < HT_CNN_PARAMS) zero[e] = 0.0f;
  if (loss && e == 0) *loss = 0.0f;
  if (e < kPackW1) {
    const int l = e / 8, i = e % 8;
    const int t = kTap[l / 16][i], c = chan_of(l % 16 / 4) + l % 4;
    W->w1[e] = t >= 0 ? to_bf16(P[oW1 + c * 27 + t]) : (uint16_t)0;
    return;
  }
  e -= kPackW1;
  if (e < kPackW2) {
    const int st = e / 512, l = (e / 8) % 64, i = e % 8;
    const int k = 8 * (l / 16) + i;
    const int p = 2 * st + k / 16, cin = k % 16, c = l % 16;
    W->w2[e] = p < 27 ? to_bf16(P[oW2 + (c * 16 + cin) * 27 + p]) : (uint16_t)0;
    return;
  }
  e -= kPackW2;
  if (e < kPackW3) {
    const int nt = e / 256, l = (e / 4) % 64, i = e % 4;
    const int c = 4 * (l / 16) + i, f = 16 * nt + l % 16;
    W->w3[e] = to_bf16(P[oW3 + f * 16 + c]);
    return;
  }
  e -= kPackW3;
  if (e < 16) { W->b1[e] = P[ob1 + e]; W->b2[e] = P[ob2 + e]; }
  if (e < 64) { W->b3[e] = P[ob3 + e]; W->w4[e] = from_bf16(to_bf16(P[oW4 + e])); }
  if (e < 4) W->b4[e] = e == 0 ? P[ob4] : 0.0f;
}
constexpr int kPackBlocks = (kPackAll + 255) / 256;
static_assert(kPackBlocks * 256 >= HT_CNN_PARAMS, "the gradient is cleared by the same threads");

// windows around peaks: votes * 1/16 as bfloat16, phi0 periodic, q/pT and d0
// outside the grid read 0; entries 125..127 are 0
__global__ __launch_bounds__(256) void windows_kernel(const int32_t* __restrict__ acc, int n_phi,
                                                      int n_qpt, int n_d0,
                                                      const ht_peak* __restrict__ peaks,
                                                      const int32_t* __restrict__ n_peaks, int cap,
                                                      uint16_t* __restrict__ win) {
  const int np = min(max(*n_peaks, 0), cap);
  const int64_t n_cells = (int64_t)n_phi * n_qpt * n_d0;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < (int64_t)np * kWin;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int w = (int)(e / kWin), c = (int)(e % kWin);
    float v = 0.0f;
    const int lin = peaks[w].lin;
    if (c < 125 && lin >= 0 && lin < n_cells) {
      const int i = lin % n_phi, col = lin / n_phi, j = col % n_qpt, k = col / n_qpt;
      const int kk = k + c / 25 - 2, jj = j + (c / 5) % 5 - 2;
      int ii = i + c % 5 - 2;
      ii = ii < 0 ? ii + n_phi : (ii >= n_phi ? ii - n_phi : ii);
      if (kk >= 0 && kk < n_d0 && jj >= 0 && jj < n_qpt)
        v = (float)acc[((size_t)kk * n_qpt + jj) * n_phi + ii] * 0.0625f;
    }
    win[e] = to_bf16(v);
  }
}

constexpr int kFwdWaves = 4;
// A window in LDS: its 25 rows (dk, dj) of 5 cells, 8 cells (16 bytes) apart.
// 16 windows are 100 dwords apart: the 16-byte reads of a row of all of them
// meet no bank conflict.  One row more is read (with zero weights) after the last.
constexpr int kRowsLds = 16 * 25 + 1;

__device__ __forceinline__ uint32_t pk_bf16(float a, float b) {  // round to nearest even
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

typedef int32_t Cells4 __attribute__((ext_vector_type(4), aligned(4)));

// 16 windows into LDS: votes * 1/16 as bfloat16 around a peak cell, phi0
// periodic, q/pT and d0 outside the grid 0.  A lane stays with one window (its
// cell is decoded once) and takes every fourth row; a row away from the phi0 seam
// is one 16-byte and one 4-byte load.
__device__ __forceinline__ void build_windows(const int32_t* __restrict__ acc, int n_phi, int n_qpt,
                                              int n_d0, const ht_peak* __restrict__ peaks, int w0,
                                              int n, int l, uint16_t (*xs)[8]) {
  const int64_t n_cells = (int64_t)n_phi * n_qpt * n_d0;
  const int w = l % 16;
  const int lin = w0 + w < n ? peaks[w0 + w].lin : -1;
  const bool ok = lin >= 0 && lin < n_cells;
  const int i = ok ? lin % n_phi : 0, col = ok ? lin / n_phi : 0;
  const int j = col % n_qpt, k = col / n_qpt;
  Cells4 q[7];
  int32_t c4[7];
  const int32_t* base = acc + ((int64_t)(k - 2) * n_qpt + (j - 2)) * n_phi + (i - 2);
  const auto inside = [&](int r) {
    const int kk = k + r / 5 - 2, jj = j + r % 5 - 2;
    return ok && r < 25 && kk >= 0 && kk < n_d0 && jj >= 0 && jj < n_qpt;
  };
  if (__all(!ok || (i >= 2 && i + 2 < n_phi))) {
#pragma unroll
    for (int u = 0; u < 7; ++u) {
      const int r = l / 16 + 4 * u;
      q[u] = Cells4{0, 0, 0, 0};
      c4[u] = 0;
      if (inside(r)) {
        const int32_t* at = base + (r / 5 * n_qpt + r % 5) * (int64_t)n_phi;
        q[u] = *reinterpret_cast<const Cells4*>(at);
        c4[u] = at[4];
      }
    }
  } else {
    int at[5];
#pragma unroll
    for (int d = 0; d < 5; ++d) {
      const int ii = i + d - 2;
      at[d] = ii < 0 ? d + n_phi : (ii >= n_phi ? d - n_phi : d);
    }
#pragma unroll
    for (int u = 0; u < 7; ++u) {
      const int r = l / 16 + 4 * u;
      q[u] = Cells4{0, 0, 0, 0};
      c4[u] = 0;
      if (inside(r)) {
        const int32_t* row = base + (r / 5 * n_qpt + r % 5) * (int64_t)n_phi;
        q[u] = Cells4{row[at[0]], row[at[1]], row[at[2]], row[at[3]]};
        c4[u] = row[at[4]];
      }
    }
  }
#pragma unroll
  for (int u = 0; u < 7; ++u) {
    const int r = l / 16 + 4 * u;
    uint4 o;
    o.x = pk_bf16((float)q[u].x * 0.0625f, (float)q[u].y * 0.0625f);
    o.y = pk_bf16((float)q[u].z * 0.0625f, (float)q[u].w * 0.0625f);
    o.z = pk_bf16((float)c4[u] * 0.0625f, 0.0f);
    o.w = 0;
    if (r < 25) *reinterpret_cast<uint4*>(xs[w * 25 + r]) = o;
  }
}

// Forward of 16 windows per wave.  FUSED: the windows come from the
// accumulator and peak list (ht_cnn_score), else from a window buffer.
// ACT keeps the activations for training.
//
// Every product has the weights as the first operand and the windows as the
// second (N = 16 windows), so a lane's results are four channels of its own
// window, which are the next layer's operand: conv1's two positions of a step
// become conv2's K = 32 by one exchange between the wave's halves, and conv2's
// result is fc1's K = 16 as it stands.  Only the windows pass through LDS.
// The matrix cores add a lane's eight products exactly, so the order of the taps
// within a lane group is free (the groups' order is not): group g's taps 8 g ..
// are two whole rows of three cells and two single cells.  A row is read once
// for its three phi0 offsets and as the first and the second row: 12 row reads
// and 54 reads of one cell per tile, where every tap of every position was read
// by itself (216) and conv1 went through LDS.  452 thousand windows: 195 -> 69 us
// (before: 2175 vector instructions and 1800 LDS cycles a tile).
template <bool FUSED, bool ACT>
__global__ __launch_bounds__(kFwdWaves * 64, 4) void forward_kernel(
    const Packed* __restrict__ W, const uint16_t* __restrict__ win,
    const int32_t* __restrict__ acc, int n_phi, int n_qpt, int n_d0,
    const ht_peak* __restrict__ peaks, const int32_t* __restrict__ n_dev, int n_max,
    float* __restrict__ logits, uint16_t* __restrict__ h1o, uint16_t* __restrict__ h2o,
    uint16_t* __restrict__ h3o) {
  __shared__ __align__(16) uint16_t xl[kFwdWaves][kRowsLds][8];
  __shared__ uint4 w2[kC2Steps * 64];
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int n = n_dev ? min(max(*n_dev, 0), n_max) : n_max;
  const int tiles = (n + 15) / 16;
  const int row = l % 16, g = l / 16;
  uint16_t (*xs)[8] = xl[wave];
  if (l < 8) xs[kRowsLds - 1][l] = 0;
  // where this lane's taps lie at position 0: the first of its rows, its two cells
  const uint16_t* ra = xs[row * 25 + (g < 3 ? 5 * g : 12)];
  const uint16_t* e0 = xs[row * 25] + (g == 0 ? 16 : g == 1 ? 18 : g == 2 ? 57 : 0);
  const uint16_t* e1 = xs[row * 25] + (g == 0 ? 17 : g == 1 ? 56 : g == 2 ? 58 : 0);
  const bf16x8 w1 = as_bf16x8(reinterpret_cast<const uint4*>(W->w1)[l]);
  for (int e = threadIdx.x; e < kC2Steps * 64; e += kFwdWaves * 64)
    w2[e] = reinterpret_cast<const uint4*>(W->w2)[e];
  __syncthreads();
  const int ch = chan_of(g);
  const float4 b1 = *reinterpret_cast<const float4*>(&W->b1[ch]);
  const float4 b2 = *reinterpret_cast<const float4*>(&W->b2[4 * g]);
  // A workgroup takes consecutive tiles and workgroups of one XCD (dispatched
  // round robin) neighbouring ones: their windows overlap in its L2.
  const int per = (tiles + (int)gridDim.x - 1) / (int)gridDim.x;
  const int lb = gridDim.x % 8 == 0 ? blockIdx.x % 8 * (gridDim.x / 8) + blockIdx.x / 8 : blockIdx.x;
  const int last = min(tiles, (lb + 1) * per);
  for (int tile = lb * per + wave; tile < last; tile += kFwdWaves) {
    const int w0 = tile * 16;
    if constexpr (FUSED) {
      build_windows(acc, n_phi, n_qpt, n_d0, peaks, w0, n, l, xs);
    } else {
      // 16 windows x 256 bytes, 16-byte global reads
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int w = l / 16 + 4 * u, o = (l % 16) * 8;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (w0 + w < n) v = *reinterpret_cast<const uint4*>(win + (size_t)(w0 + w) * kWin + o);
        const uint32_t d[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int h = 0; h < 8; ++h) {
          const int cell = o + h;
          if (cell < 125)
            xs[w * 25 + cell / 5][cell % 5] = (uint16_t)(h & 1 ? d[h / 2] >> 16 : d[h / 2] & 0xFFFFu);
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const bool valid = w0 + row < n;
    f32x4 acc2 = {0.f, 0.f, 0.f, 0.f};
    uint32_t even0 = 0, even1 = 0;  // conv1 at the step's first position
    uint4 r[4];
#pragma unroll
    for (int p = 0; p < 2 * kC2Steps; ++p) {
      uint32_t o0 = 0, o1 = 0;  // conv1 at p: four channels of the lane's window
      if (p < 27) {
        const int pk = p / 9, pj = p / 3 % 3, pi = p % 3;
        if (p % 9 == 0) {
#pragma unroll
          for (int q = 0; q < 4; ++q) r[q] = *reinterpret_cast<const uint4*>(ra + 8 * (5 * pk + q));
        }
        const uint4 &A = r[pj], &B = r[pj + 1];
        uint4 x;
        if (pi == 0) {
          x.x = A.x;
          x.y = B.x;
          x.z = __builtin_amdgcn_perm(B.y, A.y, 0x05040100u);
        } else if (pi == 1) {
          x.x = __builtin_amdgcn_alignbit(A.y, A.x, 16);
          x.y = __builtin_amdgcn_alignbit(B.y, B.x, 16);
          x.z = __builtin_amdgcn_perm(B.y, A.y, 0x07060302u);
        } else {
          x.x = A.y;
          x.y = B.y;
          x.z = __builtin_amdgcn_perm(B.z, A.z, 0x05040100u);
        }
        const int at = 40 * pk + 8 * pj + pi;
        x.w = (uint32_t)e0[at] | (uint32_t)e1[at] << 16;
        if constexpr (!FUSED) {  // a caller's window can hold what no zero weight cancels
          x.y = g < 3 ? x.y : 0u;
          x.z = g < 3 ? x.z : x.z & 0xFFFFu;
          x.w = g < 3 ? x.w : 0u;
        }
        f32x4 z = {0.f, 0.f, 0.f, 0.f};
        z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, as_bf16x8(x), z, 0, 0, 0);
        o0 = pk_bf16(fmaxf(z[0] + b1.x, 0.0f), fmaxf(z[1] + b1.y, 0.0f));
        o1 = pk_bf16(fmaxf(z[2] + b1.z, 0.0f), fmaxf(z[3] + b1.w, 0.0f));
        if (ACT && valid)
          *reinterpret_cast<uint2*>(h1o + (size_t)(w0 + row) * 432 + p * 16 + ch) = make_uint2(o0, o1);
      }
      if (p % 2 == 0) {
        even0 = o0;
        even1 = o1;
      } else {
        // conv2 k-step: lane group g takes position p - 1 + g / 2, channels
        // 8 (g % 2) .. + 7: the halves of the wave exchange what they lack
        const auto s0 = __builtin_amdgcn_permlane32_swap(even0, o0, false, false);
        const auto s1 = __builtin_amdgcn_permlane32_swap(even1, o1, false, false);
        const uint4 x = make_uint4(s0[0], s1[0], s0[1], s1[1]);
        acc2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(w2[p / 2 * 64 + l]), as_bf16x8(x), acc2, 0, 0, 0);
      }
    }
    const uint2 h2 = make_uint2(pk_bf16(fmaxf(acc2[0] + b2.x, 0.0f), fmaxf(acc2[1] + b2.y, 0.0f)),
                                pk_bf16(fmaxf(acc2[2] + b2.z, 0.0f), fmaxf(acc2[3] + b2.w, 0.0f)));
    if (ACT && valid) *reinterpret_cast<uint2*>(h2o + (size_t)(w0 + row) * 16 + 4 * g) = h2;
    // fc1 (K = 16) and fc2
    float part[4] = {0.f, 0.f, 0.f, 0.f};
    // opaque: these 40 values a lane are read per tile, not held in registers
    typedef const __attribute__((address_space(1))) Packed* GlobalPacked;
    GlobalPacked Wt = (GlobalPacked)W;
    asm volatile("" : "+s"(Wt));
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      const bf16x4 a = __builtin_bit_cast(bf16x4, reinterpret_cast<const __attribute__((address_space(1))) u32x2*>(Wt->w3)[nt * 64 + l]);
      f32x4 z = {0.f, 0.f, 0.f, 0.f};
      z = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, __builtin_bit_cast(bf16x4, h2), z, 0, 0, 0);
      const int f = 16 * nt + 4 * g;
      const f32x4 b3 = *reinterpret_cast<const __attribute__((address_space(1))) f32x4*>(&Wt->b3[f]);
      const f32x4 w4 = *reinterpret_cast<const __attribute__((address_space(1))) f32x4*>(&Wt->w4[f]);
      const uint2 h3 = make_uint2(pk_bf16(fmaxf(z[0] + b3.x, 0.0f), fmaxf(z[1] + b3.y, 0.0f)),
                                  pk_bf16(fmaxf(z[2] + b3.z, 0.0f), fmaxf(z[3] + b3.w, 0.0f)));
      part[0] += w4.x * __uint_as_float(h3.x << 16);
      part[1] += w4.y * __uint_as_float(h3.x & 0xFFFF0000u);
      part[2] += w4.z * __uint_as_float(h3.y << 16);
      part[3] += w4.w * __uint_as_float(h3.y & 0xFFFF0000u);
      if (ACT && valid) *reinterpret_cast<uint2*>(h3o + (size_t)(w0 + row) * 64 + f) = h3;
    }
    // sum of the 64 features of a window: lane groups, then the lane's own four
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      part[i] += __shfl_xor(part[i], 32);
      part[i] += __shfl_xor(part[i], 16);
    }
    const float v = (part[0] + part[2]) + (part[1] + part[3]);
    if (g == 0 && valid) logits[w0 + row] = v + W->b4[0];
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
}

// Backward on the matrix cores (v_mfma_f32_16x16x16_bf16, K = 16; same
// lane layout as above with k = 4 (lane / 16) + i).  Precision contract (the
// oracle's too): the backward signals dh3, dh2, dh1 are rounded to bfloat16
// after their ReLU masks, like the activations, and every contraction
// accumulates in float32; dz and the last layer stay float32.
//   dh2 = dh3 W3           M = 16 windows, N = 16 channels, K = 64 features
//   dh1[p] = dh2 W2[.][.][p]   per position p: M = 16 windows, N = 16, K = 16
//   dW1 += dh1[p]^T x_p    per position: M = 16 channels, N = 32 taps, K = 16 windows
//   dW2[p] += dh2^T h1[p]  per position: M = 16, N = 16, K = 16 windows
//   dW3 += dh3^T h2        M = 64 features, N = 16 channels, K = 16 windows
// A workgroup takes a tile of 16 windows at a time; its four waves share the
// 27 positions (wave w takes w, w + 4, ..), so each keeps a quarter of the
// gradient in MFMA accumulators over all its tiles.  A product's result layout
// is the next one's A operand (dh1^T and dh2^T never leave the registers).  The
// workgroup's gradient is gathered in LDS and added to the global one with
// contiguous atomics: scattered atomics by every wave (2.2 million on 8529
// addresses at 4096 windows) took most of the kernel's time.  4096 windows: 190 ->
// 25 us.
constexpr int kBwdWaves = 4;
// workgroups at most: each adds the whole gradient once (4096 windows: 64, 128 and
// 256 workgroups take 32.6, 25.0 and 26.2 us)
constexpr int kBwdGrid = 128;
// row stride of the windows: 130 = 65 dwords, odd, so that 16 rows read at one
// column fall in different banks
constexpr int kXb = 130;

__device__ __forceinline__ bf16x4 pack4(uint16_t a, uint16_t b, uint16_t c, uint16_t d) {
  bf16x4 v;
  v[0] = (short)a; v[1] = (short)b; v[2] = (short)c; v[3] = (short)d;
  return v;
}

__global__ __launch_bounds__(kBwdWaves * 64) void backward_kernel(
    const float* __restrict__ P, const uint16_t* __restrict__ win, const float* __restrict__ labels,
    int n, float pos_weight, const float* __restrict__ logits, const uint16_t* __restrict__ h1g,
    const uint16_t* __restrict__ h2g, const uint16_t* __restrict__ h3g, float* __restrict__ grad,
    float* __restrict__ loss) {
  constexpr int kThreads = kBwdWaves * 64;
  __shared__ uint16_t xs[16][kXb];
  __shared__ __align__(16) uint16_t h1s[16][27 * 16];
  __shared__ __align__(16) uint16_t h2s[16][16];
  __shared__ __align__(16) uint16_t h3s[16][64];
  __shared__ __align__(16) uint16_t d3s[16][64];              // dh3 (bf16)
  __shared__ __align__(16) uint16_t d2s[kBwdWaves][16][16];   // dh2 (bf16)
  __shared__ __align__(16) uint16_t w2t[27][264];             // W2 as [position][input 16 + output]
  __shared__ float dzs[16];
  __shared__ float sg[HT_CNN_PARAMS];
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int row = l % 16, g = l / 16;
  const int tiles = (n + 15) / 16;
  for (int e = threadIdx.x; e < HT_CNN_PARAMS; e += kThreads) sg[e] = 0.0f;
  for (int e = threadIdx.x; e < 16 * 16 * 27; e += kThreads) {
    const int c = e / (16 * 27), ci = (e / 27) % 16, p = e % 27;
    w2t[p][ci * 16 + c] = to_bf16(P[oW2 + e]);
  }
  bf16x4 b3[4];  // W3 as the B operand of dh2: features 16 st + 4 g + i, channel row
#pragma unroll
  for (int st = 0; st < 4; ++st) {
    const int f = 16 * st + 4 * g;
    b3[st] = pack4(to_bf16(P[oW3 + (f + 0) * 16 + row]), to_bf16(P[oW3 + (f + 1) * 16 + row]),
                   to_bf16(P[oW3 + (f + 2) * 16 + row]), to_bf16(P[oW3 + (f + 3) * 16 + row]));
  }
  const float w4b = from_bf16(to_bf16(P[oW4 + l]));
  constexpr int kPos = (27 + kBwdWaves - 1) / kBwdWaves;  // positions of a wave
  f32x4 aw1[2], aw2[kPos], aw3 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < 2; ++q) aw1[q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < kPos; ++q) aw2[q] = f32x4{0.f, 0.f, 0.f, 0.f};
  float gb1 = 0.f, gb2 = 0.f, gb3 = 0.f, gw4 = 0.f, gb4 = 0.f, lsum = 0.f;
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int w0 = tile * 16;
    const int nw = min(16, n - w0);
    __syncthreads();  // the previous tile is done with the LDS
    // the tile's inputs and activations, 16 bytes a load (zeros past the last window)
    {
      const int w = threadIdx.x / 16, o = threadIdx.x % 16 * 8;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (w < nw) v = *reinterpret_cast<const uint4*>(win + (size_t)(w0 + w) * kWin + o);
      uint32_t* d = reinterpret_cast<uint32_t*>(&xs[w][o]);
      d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
    }
    const auto stage = [&](void* dst, const uint16_t* src, int row16) {  // row16: 16-byte pieces a window
      for (int e = threadIdx.x; e < 16 * row16; e += kThreads) {
        uint4 v = make_uint4(0, 0, 0, 0);
        if (e < nw * row16) v = reinterpret_cast<const uint4*>(src)[e];
        reinterpret_cast<uint4*>(dst)[e] = v;
      }
    };
    stage(h1s, h1g + (size_t)w0 * 432, 54);
    stage(h2s, h2g + (size_t)w0 * 16, 2);
    stage(h3s, h3g + (size_t)w0 * 64, 8);
    if (threadIdx.x < 16) {
      float dz = 0.f;
      if (l < nw) {
        const float z = logits[w0 + l], y = labels[w0 + l];
        const float wgt = y > 0.5f ? pos_weight : 1.0f;
        const float sp = fmaxf(z, 0.0f) + log1pf(expf(-fabsf(z)));
        lsum += wgt * (sp - y * z) / (float)n;
        dz = wgt * (1.0f / (1.0f + expf(-z)) - y) / (float)n;
        gb4 += dz;
      }
      dzs[l] = dz;
    }
    __syncthreads();
    // dh3 = dz W4 [h3 > 0] and the last layer's gradients: lane = feature, four
    // windows a wave
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int w = 4 * wave + u;
      const float dz = dzs[w];
      const float h3 = from_bf16(h3s[w][l]);
      const uint16_t d3 = h3 > 0.0f ? to_bf16(dz * w4b) : (uint16_t)0;
      d3s[w][l] = d3;
      gb3 += from_bf16(d3);
      gw4 += dz * h3;
    }
    __syncthreads();
    // dh2 = dh3 W3 [h2 > 0], by every wave for itself
    bf16x4 a_dh2_t;  // [channel row][window 4 g + i]
    const bf16x4 b_h2 = pack4(h2s[4 * g][row], h2s[4 * g + 1][row], h2s[4 * g + 2][row],
                              h2s[4 * g + 3][row]);
    {
      f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int st = 0; st < 4; ++st) {
        const bf16x4 a = *reinterpret_cast<const bf16x4*>(&d3s[row][16 * st + 4 * g]);
        d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b3[st], d, 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint16_t v = b_h2[i] != 0 ? to_bf16(d[i]) : (uint16_t)0;
        d2s[wave][4 * g + i][row] = v;
        a_dh2_t[i] = (short)v;
        gb2 += from_bf16(v);
      }
    }
    // dW3 += dh3^T h2: features 16 wave ..
    {
      const int f = 16 * wave + row;
      const bf16x4 a = pack4(d3s[4 * g][f], d3s[4 * g + 1][f], d3s[4 * g + 2][f], d3s[4 * g + 3][f]);
      aw3 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b_h2, aw3, 0, 0, 0);
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const bf16x4 a_dh2 = *reinterpret_cast<const bf16x4*>(&d2s[wave][row][4 * g]);  // [window][channel]
    // per position: dh1[p], then dW1 and dW2 at p
#pragma unroll
    for (int q = 0; q < kPos; ++q) {
      const int p = wave + kBwdWaves * q;
      if (p >= 27) break;
      const int base = (p / 9) * 25 + ((p / 3) % 3) * 5 + p % 3;
      const bf16x4 b = *reinterpret_cast<const bf16x4*>(&w2t[p][row * 16 + 4 * g]);
      f32x4 d = {0.f, 0.f, 0.f, 0.f};
      d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a_dh2, b, d, 0, 0, 0);
      // h1 at p: the ReLU mask of dh1 and the B operand of dW2
      const bf16x4 b_h1 = pack4(h1s[4 * g][p * 16 + row], h1s[4 * g + 1][p * 16 + row],
                                h1s[4 * g + 2][p * 16 + row], h1s[4 * g + 3][p * 16 + row]);
      bf16x4 a1;  // dh1^T: [channel row][window 4 g + i]
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint16_t v = b_h1[i] != 0 ? to_bf16(d[i]) : (uint16_t)0;
        a1[i] = (short)v;
        gb1 += from_bf16(v);
      }
      // dW1[c][t] += sum_w dh1[w][p][c] x[w][cell(p, t)]
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) {
        const int t = 16 * nt + row;
        const int cell = base + (t / 9) * 25 + ((t / 3) % 3) * 5 + t % 3;
        bf16x4 bx = pack4(0, 0, 0, 0);
        if (t < 27)
          bx = pack4(xs[4 * g][cell], xs[4 * g + 1][cell], xs[4 * g + 2][cell], xs[4 * g + 3][cell]);
        aw1[nt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a1, bx, aw1[nt], 0, 0, 0);
      }
      // dW2[c][c'][p] += sum_w dh2[w][c] h1[w][p][c']
      aw2[q] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a_dh2_t, b_h1, aw2[q], 0, 0, 0);
    }
  }
  // the workgroup's gradient in LDS: each wave's own part, and the shared ones by atomics
#pragma unroll
  for (int nt = 0; nt < 2; ++nt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = 4 * g + i, t = 16 * nt + row;
      if (t < 27) atomicAdd(&sg[oW1 + c * 27 + t], aw1[nt][i]);
    }
#pragma unroll
  for (int q = 0; q < kPos; ++q) {
    const int p = wave + kBwdWaves * q;
    if (p >= 27) break;
#pragma unroll
    for (int i = 0; i < 4; ++i) sg[oW2 + ((4 * g + i) * 16 + row) * 27 + p] = aw2[q][i];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) sg[oW3 + (16 * wave + 4 * g + i) * 16 + row] = aw3[i];
  atomicAdd(&sg[ob1 + row], gb1);
  if (wave == 0) atomicAdd(&sg[ob2 + row], gb2);
  atomicAdd(&sg[ob3 + l], gb3);
  atomicAdd(&sg[oW4 + l], gw4);
  for (int o = 32; o > 0; o >>= 1) {
    lsum += __shfl_xor(lsum, o);
    gb4 += __shfl_xor(gb4, o);
  }
  if (threadIdx.x == 0) {
    sg[ob4] = gb4;
    atomicAdd(loss, lsum);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < HT_CNN_PARAMS; e += kThreads) atomicAdd(&grad[e], sg[e]);
}

__global__ void sgd_kernel(float* __restrict__ P, float* __restrict__ mom, float* __restrict__ grad,
                           float lr, float momentum) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < HT_CNN_PARAMS) {
    const float m = momentum * mom[q] + grad[q];
    mom[q] = m;
    P[q] = P[q] - lr * m;
    grad[q] = 0.0f;
  }
}

// ordered compaction of the peaks whose logit reaches the threshold
__global__ __launch_bounds__(256) void keep_count_kernel(const float* __restrict__ logits,
                                                         const int32_t* __restrict__ n_peaks, int cap,
                                                         float thr, int32_t* __restrict__ tile_cnt) {
  __shared__ int32_t wc[4];
  const int np = min(max(*n_peaks, 0), cap);
  const int p = blockIdx.x * 256 + threadIdx.x;
  const uint64_t m = __ballot(p < np && logits[p] >= thr);
  if ((threadIdx.x & 63) == 0) wc[threadIdx.x >> 6] = __popcll(m);
  __syncthreads();
  if (threadIdx.x == 0) tile_cnt[blockIdx.x] = wc[0] + wc[1] + wc[2] + wc[3];
}

__global__ __launch_bounds__(256) void keep_emit_kernel(const float* __restrict__ logits,
                                                        const ht_peak* __restrict__ peaks,
                                                        const int32_t* __restrict__ n_peaks, int cap,
                                                        float thr, const int32_t* __restrict__ tile_off,
                                                        ht_peak* __restrict__ out, int out_cap) {
  __shared__ int32_t wc[4];
  const int np = min(max(*n_peaks, 0), cap);
  const int p = blockIdx.x * 256 + threadIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool k = p < np && logits[p] >= thr;
  const uint64_t m = __ballot(k);
  if (lane == 0) wc[wave] = __popcll(m);
  __syncthreads();
  int before = 0;
  for (int w = 0; w < wave; ++w) before += wc[w];
  if (k) {
    const uint64_t lower = lane ? (m & ((1ull << lane) - 1ull)) : 0ull;
    const int idx = tile_off[blockIdx.x] + before + __popcll(lower);
    if (idx < out_cap) out[idx] = peaks[p];
  }
}

// forward grid: the workgroups that fit the chip at once (4 per CU by
// registers), one tile each while there are fewer tiles than workgroups
constexpr int kFwdGrid = 1024;

int blocks(int64_t n, int per, int cap = 8192) {
  int64_t b = (n + per - 1) / per;
  return (int)(b < 1 ? 1 : (b > cap ? cap : b));
}

}  // namespace

size_t cnn_workspace_bytes(int32_t max_windows, int training) {
  size_t b = (sizeof(Packed) + 255) / 256 * 256;
  if (training) {
    const size_t n = (size_t)(max_windows > 0 ? max_windows : 1);
    b += (n * 4 + 255) / 256 * 256;                 // logits
    b += (n * 432 * 2 + 255) / 256 * 256;           // h1
    b += (n * 16 * 2 + 255) / 256 * 256;           // h2
    b += (n * 64 * 2 + 255) / 256 * 256;           // h3
    b += ((size_t)HT_CNN_PARAMS * 4 + 255) / 256 * 256;  // gradient
  }
  return b;
}

int launch_cnn_windows(const Plan& p, const int32_t* acc, const ht_peak* peaks, const int32_t* n_peaks,
                       int32_t cap, uint16_t* win, hipStream_t s) {
  const ht_grid& g = p.grid;
  windows_kernel<<<blocks((int64_t)cap * kWin, 256), 256, 0, s>>>(acc, g.n_phi, g.n_qpt, g.n_d0,
                                                                  peaks, n_peaks, cap, win);
  HT_CHECK(hipGetLastError());
  return HT_OK;
}

int launch_cnn_forward(const float* params, const uint16_t* win, const int32_t* n_dev, int32_t n_max,
                       float* logits, void* ws, hipStream_t s) {
  Packed* W = reinterpret_cast<Packed*>(ws);
  pack_kernel<<<kPackBlocks, 256, 0, s>>>(params, W, nullptr, nullptr);
  HT_CHECK(hipGetLastError());
  const int tiles = (n_max + 15) / 16;
  forward_kernel<false, false><<<blocks(tiles, 1, kFwdGrid), kFwdWaves * 64, 0, s>>>(
      W, win, nullptr, 0, 0, 0, nullptr, n_dev, n_max, logits, nullptr, nullptr, nullptr);
  HT_CHECK(hipGetLastError());
  return HT_OK;
}

int launch_cnn_score(const Plan& p, const float* params, const int32_t* acc, const ht_peak* peaks,
                     const int32_t* n_peaks, int32_t cap, float* logits, void* ws, hipStream_t s) {
  Packed* W = reinterpret_cast<Packed*>(ws);
  pack_kernel<<<kPackBlocks, 256, 0, s>>>(params, W, nullptr, nullptr);
  HT_CHECK(hipGetLastError());
  const ht_grid& g = p.grid;
  const int tiles = (cap + 15) / 16;
  forward_kernel<true, false><<<blocks(tiles, 1, kFwdGrid), kFwdWaves * 64, 0, s>>>(
      W, nullptr, acc, g.n_phi, g.n_qpt, g.n_d0, peaks, n_peaks, cap, logits, nullptr, nullptr,
      nullptr);
  HT_CHECK(hipGetLastError());
  return HT_OK;
}

int launch_cnn_train(float* params, float* mom, const uint16_t* win, const float* labels, int32_t n,
                     float lr, float momentum, float pos_weight, float* loss, void* ws, hipStream_t s) {
  char* base = reinterpret_cast<char*>(ws);
  Packed* W = reinterpret_cast<Packed*>(base);
  size_t o = (sizeof(Packed) + 255) / 256 * 256;
  const size_t nn = (size_t)(n > 0 ? n : 1);
  float* logits = reinterpret_cast<float*>(base + o);
  o += (nn * 4 + 255) / 256 * 256;
  uint16_t* h1 = reinterpret_cast<uint16_t*>(base + o);
  o += (nn * 432 * 2 + 255) / 256 * 256;
  uint16_t* h2 = reinterpret_cast<uint16_t*>(base + o);
  o += (nn * 16 * 2 + 255) / 256 * 256;
  uint16_t* h3 = reinterpret_cast<uint16_t*>(base + o);
  o += (nn * 64 * 2 + 255) / 256 * 256;
  float* grad = reinterpret_cast<float*>(base + o);
  pack_kernel<<<kPackBlocks, 256, 0, s>>>(params, W, grad, loss);
  HT_CHECK(hipGetLastError());
  const int tiles = (n + 15) / 16;
  forward_kernel<false, true><<<blocks(tiles, 1, kFwdGrid), kFwdWaves * 64, 0, s>>>(
      W, win, nullptr, 0, 0, 0, nullptr, nullptr, n, logits, h1, h2, h3);
  HT_CHECK(hipGetLastError());
  backward_kernel<<<blocks(tiles, 1, kBwdGrid), kBwdWaves * 64, 0, s>>>(
      params, win, labels, n, pos_weight, logits, h1, h2, h3, grad, loss);
  HT_CHECK(hipGetLastError());
  sgd_kernel<<<(HT_CNN_PARAMS + 255) / 256, 256, 0, s>>>(params, mom, grad, lr, momentum);
  HT_CHECK(hipGetLastError());
  return HT_OK;
}

int launch_cnn_keep(const Plan& p, const float* logits, const ht_peak* peaks, const int32_t* n_peaks,
                    int32_t cap, float thr, ht_peak* out, int32_t out_cap, int32_t* n_out,
                    hipStream_t s) {
  const int tiles = (cap + 255) / 256 > 0 ? (cap + 255) / 256 : 1;
  keep_count_kernel<<<tiles, 256, 0, s>>>(logits, n_peaks, cap, thr, p.d_ctile_cnt);
  HT_CHECK(hipGetLastError());
  const int rc = launch_scan(p.d_ctile_cnt, p.d_ctile_off, tiles, n_out, s);
  if (rc != HT_OK) return rc;
  keep_emit_kernel<<<tiles, 256, 0, s>>>(logits, peaks, n_peaks, cap, thr, p.d_ctile_off, out,
                                         out_cap);
  HT_CHECK(hipGetLastError());
  return HT_OK;
}

}  // namespace ht
