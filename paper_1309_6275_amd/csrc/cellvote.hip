// Band (cell) vote, a variant of the first transform: each valid hit votes
// for every phi0 bin its curve reaches while (kappa, d0) range over a
// column's cell, instead of the point at the column centre (the paper's
// instances are cells of the parameter space, section "Hough Transform
// Algorithm").  u = sin(phi - phi0) is increasing in kappa and d0 over the
// cell, so the band runs between the phi0 of two corners: (smallest kappa,
// lower d0 edge) and (largest kappa, upper d0 edge), each from the float32
// vote formula with that corner's tables; u is clipped to [-1, 1], and no
// vote is cast when the whole cell lies beyond |u| = 1.
//
// Same gfx950 mapping as the point vote: a workgroup owns 64 q/pT columns of
// one d0 plane in LDS (lane = column), waves split the hits and broadcast
// them through SGPRs, and the two corners' arcsines of the hits' distinct radii
// (the layers of a barrel tracker) are computed once per column into a table.
// With 32-bit counters a band is two LDS atomics, +1 at its first bin and -1
// after its last, and the tile is summed along phi0 at the end.  3600 hits on the
// displaced-jet grid: 208 -> 58 us (two arcsines per hit and column and an atomic
// per bin, about four a column, before; 41 us of it were the vote total, added
// by one global atomic per wave to the same word).  What is left is the issue
// of 26 vector instructions per hit and column wave.  16-bit counters (n_phi >
// 604) cannot hold differences of 65535 votes and take an atomic per bin.
// Grids with few tiles also split the hits into slices that add their tiles
// into a cleared accumulator, as the point vote does.
#include "ht_internal.h"

namespace ht {
namespace {

constexpr int kCellWaves = 16;
constexpr int kCellThreads = kCellWaves * kWave;
constexpr int kLdsBytes = 160 * 1024;
constexpr int kCast = 8;  // hits of known radius in flight per wave (64 % kCast == 0)

__device__ __forceinline__ float bcast(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

struct CellTable {
  float lo[kMaxRadii][kWave], hi[kMaxRadii][kWave];  // corner arcsines per (radius, column)
};
static_assert(kMaxRadii * 2 >= kCellWaves, "the tile's sums reuse the table");
// LDS of a CU less the kernel's static arrays
constexpr int kCellLds = kLdsBytes - (int)sizeof(RadiusSet) - (int)sizeof(CellTable) - 8 * kCellWaves;
// odd dword strides; 32-bit rows have a word to spare
int wide_stride(int n_phi) { return (n_phi + 1) | 1; }
bool cell_wide(int n_phi) { return (size_t)kWave * wide_stride(n_phi) * 4 <= (size_t)kCellLds; }
int cell_stride(int n_phi) { return cell_wide(n_phi) ? wide_stride(n_phi) : ((n_phi + 1) / 2) | 1; }

__device__ __forceinline__ int floor_i32(float x) {  // x finite and in range where it counts
  int i;
  asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(i) : "v"(x));
  return i;
}

// The arcsines of a column's two corners for radius r (r2 = r r, ir = 1 / r),
// the smaller in lo; lo is NaN where the cell casts no vote.  The bin of an
// arcsine does not increase with it (every rounded step is monotone), so a band runs
// from hi's bin to lo's.
__device__ __forceinline__ void corners(bool col_ok, float r2, float ir, float ckl, float cql,
                                        float ctl, float ckh, float cqh, float cth, float& lo,
                                        float& hi) {
  const float ulo = ((ckl * r2 + cql) * ir) * ctl;
  const float uhi = ((ckh * r2 + cqh) * ir) * cth;
  const bool ok = col_ok && !(ulo > 1.0f) && !(uhi < -1.0f);
  const float a = asin_f(fmaxf(ulo, -1.0f)), b = asin_f(fminf(uhi, 1.0f));
  lo = ok ? fminf(a, b) : __builtin_nanf("");
  hi = fmaxf(a, b);
}

template <bool WIDE, bool POW2>
__global__ __launch_bounds__(kCellThreads) void cell_vote_kernel(
    const float* __restrict__ r, const float* __restrict__ phi, int n_all,
    const float* __restrict__ kl, const float* __restrict__ kh, const float* __restrict__ ql,
    const float* __restrict__ tl, const float* __restrict__ qh, const float* __restrict__ th,
    int n_phi, int n_qpt, float phi_lo, float invw, int stride, int32_t* __restrict__ acc,
    unsigned long long* __restrict__ n_votes) {
  extern __shared__ uint32_t lds[];
  __shared__ RadiusSet R;
  __shared__ unsigned long long s_votes[kCellWaves];
  __shared__ CellTable T;
  const int n_slices = gridDim.z;
  const int chunk = ((n_all + n_slices - 1) / n_slices + kWave - 1) / kWave * kWave;
  const int h0 = (int)blockIdx.z * chunk;
  const int n_hits = min(n_all, h0 + chunk);
  if (n_slices > 1 && h0 >= n_hits) return;  // an empty slice adds nothing
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x >> 6;
  const int j0 = blockIdx.x * kWave;
  const int k = blockIdx.y;
  const int j = j0 + lane;
  const bool col_ok = j < n_qpt;

  for (int w = threadIdx.x; w < kWave * stride; w += kCellThreads) lds[w] = 0u;
  float ckl = 0.0f, ckh = 0.0f, cql = 0.0f, ctl = 0.0f, cqh = 0.0f, cth = 0.0f;
  if (col_ok) {
    const size_t c = (size_t)k * n_qpt + j;
    ckl = kl[j];
    ckh = kh[j];
    cql = ql[c];
    ctl = tl[c];
    cqh = qh[c];
    cth = th[c];
  }
  radius_set_build(R, r, phi, h0, n_hits);
  for (int t = threadIdx.x; t < R.n * kWave; t += kCellThreads) {  // the thread's own column
    const float rv = R.r[t >> 6];
    corners(col_ok, rv * rv, 1.0f / rv, ckl, cql, ctl, ckh, cqh, cth, T.lo[t >> 6][lane],
            T.hi[t >> 6][lane]);
  }
  __syncthreads();
  // the lane's column of the table in registers, indexed by the wave-uniform
  // radius index; the last entry is the invalid hit's
  float rlo[kMaxRadii + 1], rhi[kMaxRadii + 1];
#pragma unroll
  for (int a = 0; a <= kMaxRadii; ++a) {
    rlo[a] = a < kMaxRadii && a < R.n ? T.lo[a % kMaxRadii][lane] : __builtin_nanf("");
    rhi[a] = a < kMaxRadii && a < R.n ? T.hi[a % kMaxRadii][lane] : 0.0f;
  }

  uint32_t* col = lds + lane * stride;
  uint32_t wraps = 0;  // WIDE: bands that reach bin 0 from the end of the row
  for (int base = h0 + wave * kWave; base < n_hits; base += kCellThreads) {
    const int h = base + lane;
    float hr = 1.0f, hp = 0.0f;
    bool hv = false;
    if (h < n_hits) {
      hr = r[h];
      hp = phi[h];
      hv = hit_ok(hr, hp);
    }
    const int hri = hv ? radius_index(R, hr) : kMaxRadii;
    uint64_t todo = __ballot(hv);
    if (!todo) continue;
    // One band.  Its ends lie in [-n_phi - 1, 2 n_phi + 1): one period of
    // correction, a mask where n_phi is a power of two.  Two arcsines are at
    // most pi apart, so a band has at most n_phi / 2 + 2 <= n_phi bins.
    const auto cast = [&](float ph, float slo, float shi) {
      const bool ok = slo == slo;
      const int a0 = floor_i32(((ph - shi) - phi_lo) * invw);
      const int b0 = floor_i32(((ph - slo) - phi_lo) * invw);
      const auto wrap = [n_phi](int i) {
        if (POW2) return i & (n_phi - 1);
        i = i < 0 ? i + n_phi : i;
        return i >= n_phi ? i - n_phi : i;
      };
      if (WIDE) {
        // from its first bin to the one after its last (a band over every bin
        // ends where it begins); the word after the row takes what casts none
        const int ia = ok ? wrap(a0) : n_phi;
        const int e = ok ? wrap(b0 + 1) : n_phi;
        atomicAdd(&col[ia], 1u);
        atomicAdd(&col[e], ~0u);
        wraps += ok && e <= ia ? 1u : 0u;
      } else if (ok) {
        int i = wrap(a0);
        for (int q = a0; q <= b0; ++q) {
          atomicAdd(&col[i >> 1], (i & 1) ? 65536u : 1u);
          i = i + 1 == n_phi ? 0 : i + 1;
        }
      }
    };
    // kCast hits at a time from fixed lanes (a read of a lane that a register
    // names takes twice as long)
    const int m = kWave - __builtin_clzll(todo);
    if (__ballot(hri < 0) == 0) {
      // every radius is in the table: no test per hit, several hits' chains side by side
#pragma unroll 1
      for (int h8 = 0; h8 < m; h8 += kCast) {
        const float p8 = __shfl(hp, h8 + lane);
        const int r8 = __shfl(hri, h8 + lane);
#pragma unroll
        for (int u = 0; u < kCast; ++u) {
          const int ri = __builtin_amdgcn_readlane(r8, u);
          const float slo = rlo[ri], shi = rhi[ri];
          cast(bcast(p8, u), slo, shi);
        }
      }
      continue;
    }
    const float hr2 = hr * hr;
    const float hir = 1.0f / hr;
    while (todo) {
      const int src = __builtin_ctzll(todo);
      todo &= todo - 1;
      const int ri = __builtin_amdgcn_readlane(hri, src);
      float slo, shi;
      if (ri >= 0) {
        slo = rlo[ri];
        shi = rhi[ri];
      } else {
        corners(col_ok, bcast(hr2, src), bcast(hir, src), ckl, cql, ctl, ckh, cqh, cth, slo, shi);
      }
      cast(bcast(hp, src), slo, shi);
    }
  }
  if (WIDE && wraps) atomicAdd(&col[0], wraps);
  __syncthreads();

  if (WIDE) {
    // running sums along phi0: a wave takes a segment of every column, first
    // its total, then, after the totals of the segments before it, the sums
    uint32_t (*tot)[kWave] = reinterpret_cast<uint32_t (*)[kWave]>(&T.lo[0][0]);
    const int seg = (n_phi + kCellWaves - 1) / kCellWaves;
    const int b0 = min(n_phi, wave * seg), b1 = min(n_phi, b0 + seg);
    uint32_t sum = 0;
#pragma unroll 8
    for (int b = b0; b < b1; ++b) sum += col[b];
    tot[wave][lane] = sum;
    __syncthreads();
    sum = 0;
    for (int w = 0; w < wave; ++w) sum += tot[w][lane];
#pragma unroll 8
    for (int b = b0; b < b1; ++b) {
      sum += col[b];
      col[b] = sum;
    }
    __syncthreads();
  }

  const int ncol = min(kWave, n_qpt - j0);
  int32_t* out = acc + ((size_t)k * n_qpt + j0) * n_phi;
  // the vote count, when asked for, is the sum of the tile's counters
  unsigned long long votes = 0;
  for (int cj = wave; cj < ncol; cj += kCellWaves) {  // a column per wave: no division per cell
    const uint32_t* row = lds + cj * stride;
    for (int i = lane; i < n_phi; i += kWave) {
      const int32_t v = (int32_t)(WIDE ? row[i] : (i & 1 ? row[i >> 1] >> 16 : row[i >> 1] & 0xFFFFu));
      if (n_slices == 1)
        out[cj * n_phi + i] = v;
      else if (v)
        atomicAdd(&out[cj * n_phi + i], v);
      votes += (unsigned long long)v;
    }
  }

  if (n_votes) {
    unsigned long long v = votes;
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    // one global atomic per workgroup: one per wave to the same word took 10 ns each
    if (lane == 0) s_votes[wave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < kCellWaves; ++w) v += s_votes[w];
      if (v) atomicAdd(n_votes, v);
    }
  }
}

__global__ void zero_u64(unsigned long long* p) { *p = 0ull; }

__global__ void zero_i32(int32_t* __restrict__ p, int64_t n) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x)
    p[e] = 0;
}

}  // namespace

int cell_vote_init(int n_phi) {
  const int bytes = kWave * cell_stride(n_phi) * 4;
  const hipFuncAttribute at = hipFuncAttributeMaxDynamicSharedMemorySize;
  HT_CHECK(hipFuncSetAttribute((const void*)cell_vote_kernel<true, true>, at, bytes));
  HT_CHECK(hipFuncSetAttribute((const void*)cell_vote_kernel<true, false>, at, bytes));
  HT_CHECK(hipFuncSetAttribute((const void*)cell_vote_kernel<false, true>, at, bytes));
  HT_CHECK(hipFuncSetAttribute((const void*)cell_vote_kernel<false, false>, at, bytes));
  return HT_OK;
}

int launch_cell_vote(const Plan& p, const float* r, const float* phi, int32_t n_hits,
                     int32_t* acc, unsigned long long* n_votes, hipStream_t s) {
  const ht_grid& g = p.grid;
  const int stride = cell_stride(g.n_phi);
  const size_t lds_bytes = (size_t)kWave * stride * 4;
  if (n_votes) {
    zero_u64<<<1, 1, 0, s>>>(n_votes);
    HT_CHECK(hipGetLastError());
  }
  const int tiles = (g.n_qpt + kWave - 1) / kWave * g.n_d0;
  const int slices = hit_slices(tiles, n_hits);
  dim3 grid((g.n_qpt + kWave - 1) / kWave, g.n_d0, slices);
  if (slices > 1) {
    const int64_t cells = p.n_cells;
    const int64_t blocks = (cells + 1023) / 1024 < 1024 ? (cells + 1023) / 1024 : 1024;
    zero_i32<<<(unsigned)blocks, 256, 0, s>>>(acc, cells);
    HT_CHECK(hipGetLastError());
  }
  const bool wide = cell_wide(g.n_phi), pow2 = (g.n_phi & (g.n_phi - 1)) == 0;
  auto kern = pow2 ? (wide ? cell_vote_kernel<true, true> : cell_vote_kernel<false, true>)
                   : (wide ? cell_vote_kernel<true, false> : cell_vote_kernel<false, false>);
  p.prof_mark(HT_STAGE_VOTE, 0, s);
  kern<<<grid, kCellThreads, lds_bytes, s>>>(r, phi, n_hits, p.d_ckl, p.d_ckh, p.d_cql, p.d_ctl,
                                             p.d_cqh, p.d_cth, g.n_phi, g.n_qpt, p.phi_lo,
                                             p.invw, stride, acc, n_votes);
  HT_CHECK(hipGetLastError());
  p.prof_mark(HT_STAGE_VOTE, 1, s);
  return HT_OK;
}

}  // namespace ht
