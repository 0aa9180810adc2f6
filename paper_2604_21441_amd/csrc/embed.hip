// Mechanical embedding (Theory, eq. 3): the ML-MM coupling left at the MM
// level, Coulomb plus 12-6 Lennard-Jones between every ML atom and every MM
// atom with fixed force-field charges and LJ parameters:
//   E = sum_{i in ML} sum_{j in MM, r < rc} ke q_i q_j / r + 4 eps_ij ((s_ij/r)^12 - (s_ij/r)^6)
// with Lorentz-Berthelot mixing s_ij = (s_i + s_j)/2, eps_ij = sqrt(eps_i eps_j).
//
// A workgroup takes 128 MM atoms, two per lane of each of its 16 wavefronts (4
// beyond 262,144 MM atoms), and the wavefronts share the ML atoms (staged in
// LDS) between them.  Each pair is evaluated in FP32.  An MM atom's force and
// the energy accumulate in FP64 registers and are summed over the wavefronts
// through LDS, in order; an ML atom's force is summed over the lanes in FP32,
// the 64 MM atoms of each tile by themselves, and added with FP64 atomics
// (skipped when no lane is inside the cutoff).
//
// Bound by the chain of one wavefront through its ML atoms (a sphere around
// the ML region holds few of the MM atoms' wavefronts, and these few meet
// nearly every ML atom inside the cutoff) and by the atomics on the few lines
// of ML forces, hence every workgroup begins at another ML atom.  60 x 30,000
// atoms: one wavefront walking all ML atoms for 64 MM atoms 52 us; eight
// sharing them 19; two MM atoms per lane, which halves the sums over lanes and
// the atomics, 15; the turned order 11.5; 16 wavefronts 9.7 (one MM atom per
// lane 13.6, four 14.6).  That was with the two tiles added lane by lane before
// the sum, an FP32 addition more: apart they take 11.2 us against 10.4 (the
// call 15.9 both, bound by the caller).
#include "nnp_internal.h"

namespace nnp {
namespace {

constexpr int kMeWaves = 16;       // wavefronts of a workgroup; with many workgroups
constexpr int kMeWavesMany = 4;    // (launch_me_pairs: more than kMeGroupsMost)
constexpr int kMeGroupsMost = 2048;   // eight per CU
constexpr int kMeBlock = 256;
constexpr int kMeTiles = 2;     // 64 MM atoms each
constexpr int kMeChunk = 256;   // ML atoms per LDS chunk

// v + (v of the lane that the DPP control names; 0 where there is none)
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, false));
}

// Sum over the wavefront, in lane 63 (row shifts by 1, 2, 4 and 8, then the
// rows' totals passed on).
__device__ __forceinline__ float wsum63(float v) {
  v = dpp_add<0x111, 0xf>(v);
  v = dpp_add<0x112, 0xf>(v);
  v = dpp_add<0x114, 0xf>(v);
  v = dpp_add<0x118, 0xf>(v);
  v = dpp_add<0x142, 0xa>(v);
  return dpp_add<0x143, 0xc>(v);
}

__device__ __forceinline__ double wsum_d(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_me_pairs(const float* __restrict__ ml_pos,
                                                         const float* __restrict__ ml_par, int n_ml,
                                                         const float* __restrict__ mm_pos,
                                                         const float* __restrict__ mm_par, int n_mm, Geometry g,
                                                         float rc2, float ke, double* __restrict__ energy,
                                                         double* __restrict__ ml_f, double* __restrict__ mm_f,
                                                         int accumulate) {
  __shared__ float4 sx[kMeChunk];   // ML x, y, z, q
  __shared__ float2 sp[kMeChunk];   // ML sigma, eps
  __shared__ double sf[WAVES][4][64];   // per wavefront and MM atom of a tile: force, energy
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int j0 = blockIdx.x * (64 * kMeTiles) + lane;
  float4 y[kMeTiles];    // MM x, y, z, q
  float2 yp[kMeTiles];   // MM sigma, eps
#pragma unroll
  for (int u = 0; u < kMeTiles; ++u) {
    const int64_t j = 3 * (int64_t)(j0 + 64 * u);
    y[u] = make_float4(0.f, 0.f, 0.f, 0.f);
    yp[u] = make_float2(0.f, 0.f);
    if (j0 + 64 * u < n_mm) {
      y[u] = make_float4(mm_pos[j], mm_pos[j + 1], mm_pos[j + 2], mm_par[j]);
      yp[u] = make_float2(mm_par[j + 1], mm_par[j + 2]);
    }
  }
  double f[kMeTiles][3] = {}, eacc = 0.0;
  for (int c0 = 0; c0 < n_ml; c0 += kMeChunk) {
    const int nc = min(kMeChunk, n_ml - c0);
    __syncthreads();
    for (int t = threadIdx.x; t < nc; t += 64 * WAVES) {
      const int i = c0 + t;
      sx[t] = make_float4(ml_pos[3 * (int64_t)i], ml_pos[3 * (int64_t)i + 1], ml_pos[3 * (int64_t)i + 2],
                          ml_par[3 * (int64_t)i]);
      sp[t] = make_float2(ml_par[3 * (int64_t)i + 1], ml_par[3 * (int64_t)i + 2]);
    }
    __syncthreads();
    const int turn = (int)((blockIdx.x * 29u) % (unsigned)nc);
    for (int k = wave; k < nc; k += WAVES) {
      const int t = k + turn < nc ? k + turn : k + turn - nc;
      const float4 xi = sx[t];
      const float2 pi = sp[t];
      float a[kMeTiles][3] = {};   // on this ML atom, each tile summed by itself
      bool in[kMeTiles] = {};
#pragma unroll
      for (int u = 0; u < kMeTiles; ++u) {
        float dx = y[u].x - xi.x, dy = y[u].y - xi.y, dz = y[u].z - xi.z;
        if (g.periodic) {
          dx -= g.box[0] * rintf(dx * g.inv_box[0]);
          dy -= g.box[1] * rintf(dy * g.inv_box[1]);
          dz -= g.box[2] * rintf(dz * g.inv_box[2]);
        }
        const float r2 = dx * dx + dy * dy + dz * dz;
        if (j0 + 64 * u < n_mm && r2 < rc2) {
          in[u] = true;
          const float ir2 = 1.f / r2;
          const float ir = sqrtf(ir2);
          const float qq = ke * xi.w * y[u].w;
          const float s = 0.5f * (pi.x + yp[u].x);
          const float eps = sqrtf(pi.y * yp[u].y);
          const float s2 = s * s * ir2;
          const float s6 = s2 * s2 * s2;
          const float s12 = s6 * s6;
          const float ec = qq * ir;
          eacc += (double)ec + (double)(4.f * eps * (s12 - s6));
          const float w = (ec + eps * (48.f * s12 - 24.f * s6)) * ir2;   // -dE/dr / r
          a[u][0] = w * dx;
          a[u][1] = w * dy;
          a[u][2] = w * dz;
#pragma unroll
          for (int c = 0; c < 3; ++c) f[u][c] += a[u][c];
        }
      }
      uint64_t any = 0;
#pragma unroll
      for (int u = 0; u < kMeTiles; ++u) any |= __builtin_amdgcn_ballot_w64(in[u]);
      if (any == 0) continue;
      double r[3] = {0.0, 0.0, 0.0};
#pragma unroll
      for (int u = 0; u < kMeTiles; ++u)
#pragma unroll
        for (int c = 0; c < 3; ++c) r[c] += (double)wsum63(a[u][c]);
      if (lane == 63) {
        double* o = ml_f + 3 * (int64_t)(c0 + t);
#pragma unroll
        for (int c = 0; c < 3; ++c) unsafeAtomicAdd(o + c, -r[c]);
      }
    }
  }
  sf[wave][3][lane] = eacc;
#pragma unroll
  for (int u = 0; u < kMeTiles; ++u) {
#pragma unroll
    for (int k = 0; k < 3; ++k) sf[wave][k][lane] = f[u][k];
    __syncthreads();
    // wavefronts 0 to 2 write a component of the MM forces each, 3 adds the energy
    if (wave < 3 || (u == 0 && wave == 3)) {
      double v = 0.0;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) v += sf[w][wave][lane];
      if (wave < 3) {
        if (j0 + 64 * u < n_mm) {
          double* o = mm_f + 3 * (int64_t)(j0 + 64 * u) + wave;
          *o = accumulate ? v + *o : v;
        }
      } else {
        v = wsum_d(v);
        if (lane == 0 && v != 0.0) unsafeAtomicAdd(energy, v);
      }
    }
    if (u + 1 < kMeTiles) __syncthreads();
  }
}

// The outputs that k_me_pairs adds to, cleared in one launch.
__global__ __launch_bounds__(kMeBlock) void k_me_clear(double* __restrict__ energy, double* __restrict__ ml_f,
                                                       int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kMeBlock + threadIdx.x;
  if (i < n) ml_f[i] = 0.0;
  if (i == 0) *energy = 0.0;
}

}  // namespace

hipError_t launch_me_pairs(int n_ml, const float* ml_pos, const float* ml_par, int n_mm, const float* mm_pos,
                           const float* mm_par, const Geometry& g, float cutoff, float ke, double* energy,
                           double* ml_f, double* mm_f, int accumulate, hipStream_t st) {
  if (!accumulate) {
    const int64_t n = 3 * (int64_t)n_ml;
    hipLaunchKernelGGL(k_me_clear, dim3((unsigned)(n / kMeBlock + 1)), dim3(kMeBlock), 0, st, energy, ml_f, n);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (n_mm == 0) return hipSuccess;
  const float rc2 = cutoff > 0.f ? cutoff * cutoff : INFINITY;
  // Most workgroups of a large surrounding have no pair inside the cutoff, and
  // 16 wavefronts then only load, wait for each other and store zeros.  20 ML
  // atoms, cutoff 12 A, 16 wavefronts -> 4: 1,000,000 MM atoms 48 -> 22 us,
  // 400,000 22 -> 13, 200,000 14.3 -> 11.5; 200 ML atoms 97 -> 76, 47 -> 50, 32
  // -> 43.
  const int groups = (n_mm - 1) / (64 * kMeTiles) + 1;
  auto run = [&](auto kernel, int waves) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)groups), dim3((unsigned)(64 * waves)), 0, st, ml_pos, ml_par, n_ml,
                       mm_pos, mm_par, n_mm, g, rc2, ke, energy, ml_f, mm_f, accumulate);
  };
  if (groups <= kMeGroupsMost) run(k_me_pairs<kMeWaves>, kMeWaves);
  else run(k_me_pairs<kMeWavesMany>, kMeWavesMany);
  return hipGetLastError();
}

}  // namespace nnp
