// MM point charges as an extra per-atom network input (electrostatic
// embedding through the model, with forces on MM atoms; Methods: the 2026
// interface passes MM positions and charges, and the model may put forces on
// MM atoms):
//   phi_i = ke * sum_j q_j fc(r_ij; Rm) / r_ij     over MM atoms j, r_ij < Rm
// The passes are all-pairs over (NNP atom, MM atom), each wavefront taking 16
// (forward) or 8 (adjoint) NNP atoms and one MM atom per lane.  A lane keeps
// one running sum per NNP atom; these are reduced across lanes (a DPP
// transposing butterfly within each 16-lane row: 15 exchanges for all 16 sums,
// where a shuffle tree per sum took 96 LDS round trips) and stored as the
// workgroup's partial.  The partials of an NNP atom are added in a fixed order
// (FP64), the forward's by a second launch, the adjoint's by the force gather.
// No atomics on the NNP side: with a small ML region every NNP atom collects
// a term from each of hundreds of workgroups, and FP64 atomics on one address
// serialise (60 NNP atoms, 30,000 charges: 10.9 us forward and 15.7 us
// adjoint with per-wavefront atomics).  Intended for ML regions of up to a
// few thousand atoms.
#include <algorithm>

#include "nnp_internal.h"

namespace nnp {
namespace {

constexpr int kBlock = 256;
constexpr int kNnpChunk = 16;       // NNP atoms per workgroup row (= lanes of a DPP row)
constexpr int kMaxMmBlocks = 512;   // workgroups along the MM atoms
constexpr int kBwdChunk = 8;        // NNP atoms per adjoint wavefront
constexpr int kBwdWaves = 16;       // most wavefronts of an adjoint workgroup
constexpr int kBwdTiles = kBlock / 64;   // MM atoms per lane of the adjoint, or one

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// v[0 .. 16) summed over the 16 lanes of each DPP row: lane l of a row ends
// with the row's total of value l & 15 in v[0].
__device__ __forceinline__ void row_sum16(float* v, int lane) {
  halve<8, kDppMirror>(v, lane & 8);
  halve<4, kDppHalfMirror>(v, lane & 4);
  halve<2, kDppXor2>(v, lane & 2);
  halve<1, kDppXor1>(v, lane & 1);
}

// v[0 .. 8) summed over the wavefront: lane l ends with the total of value l & 7.
__device__ __forceinline__ float wave_sum8(float* v, int lane) {
  halve<4, kDppHalfMirror>(v, lane & 4);
  halve<2, kDppXor2>(v, lane & 2);
  halve<1, kDppXor1>(v, lane & 1);
  float s = v[0];
#pragma unroll
  for (int off = 8; off <= 32; off *= 2) s += __shfl_xor(s, off, 64);
  return s;
}

__device__ __forceinline__ void mm_disp(const float4& pi, float yx, float yy, float yz, const Geometry& g,
                                        float& dx, float& dy, float& dz, float& r2) {
  dx = yx - pi.x; dy = yy - pi.y; dz = yz - pi.z;
  if (g.periodic) {
    dx -= g.box[0] * rintf(dx * g.inv_box[0]);
    dy -= g.box[1] * rintf(dy * g.inv_box[1]);
    dz -= g.box[2] * rintf(dz * g.inv_box[2]);
  }
  r2 = dx * dx + dy * dy + dz * dz;
}

__global__ __launch_bounds__(kBlock) void k_fill_f64(double* p, int n) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) p[t] = 0.0;
}

// part[i * gridDim.x + blockIdx.x] = this workgroup's share of phi_i / ke.
__global__ __launch_bounds__(kBlock) void k_mm_fwd(const float4* __restrict__ spos, int n,
                                                   const float* __restrict__ mm_pos,
                                                   const float* __restrict__ mm_q, int n_mm,
                                                   DescParams p, Geometry g, float* __restrict__ part) {
  __shared__ float red[kBlock / kNnpChunk][kNnpChunk];   // [wavefront row][NNP atom]
  const int lane = threadIdx.x & 63;
  const int i0 = blockIdx.y * kNnpChunk, cnt = min(n - i0, kNnpChunk);
  const float rm2 = p.mm_cutoff * p.mm_cutoff;
  const float inv2rm = 0.5f / p.mm_cutoff;
  float acc[kNnpChunk];
#pragma unroll
  for (int c = 0; c < kNnpChunk; ++c) acc[c] = 0.f;
  for (int j = blockIdx.x * kBlock + threadIdx.x; j < n_mm; j += gridDim.x * kBlock) {
    const float yx = mm_pos[3 * (int64_t)j], yy = mm_pos[3 * (int64_t)j + 1], yz = mm_pos[3 * (int64_t)j + 2];
    const float q = mm_q[j];
#pragma unroll
    for (int c = 0; c < kNnpChunk; ++c) {
      if (c < cnt) {
        const float4 pi = spos[i0 + c];
        float dx, dy, dz, r2;
        mm_disp(pi, yx, yy, yz, g, dx, dy, dz, r2);
        if (r2 < rm2) {
          float ir = __builtin_amdgcn_rsqf(r2);
          float r = r2 * ir;
          float fc = 0.5f * __builtin_amdgcn_cosf(r * inv2rm) + 0.5f;
          acc[c] += q * fc * ir;
        }
      }
    }
  }
  row_sum16(acc, lane);
  red[threadIdx.x >> 4][lane & 15] = acc[0];
  __syncthreads();
  if ((int)threadIdx.x < cnt) {
    float s = red[0][threadIdx.x];
#pragma unroll
    for (int r = 1; r < kBlock / kNnpChunk; ++r) s += red[r][threadIdx.x];
    part[(int64_t)(i0 + threadIdx.x) * gridDim.x + blockIdx.x] = s;
  }
}

// phi_i = ke * (sum of the nbx partials of atom i, in order, FP64); one
// wavefront per NNP atom.  nbx = 0 (no MM atoms) gives phi = 0.
__global__ __launch_bounds__(kBlock) void k_mm_finish(const float* __restrict__ part, int nbx, int n,
                                                      DescParams p, float* __restrict__ x) {
  const int i = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  const int lane = threadIdx.x & 63;
  if (i >= n) return;   // wavefront-uniform
  double s = 0.0;
  for (int b = lane; b < nbx; b += 64) s += (double)part[(int64_t)i * nbx + b];
  s = wave_sum(s);
  if (lane == 0) x[(int64_t)i * p.stride + p.D] = (float)(p.ke * s);
}

// Adjoint: dE/dphi_i = g[i][D] (+ the predicted charge q_i of a network with
// a charge output, whose energy holds q_i phi_i);  dphi_i/dy_j = ke q_j f'(r) u,  f(r) = fc(r)/r,
// u = (y_j - x_i)/r.  MM atom j gets -sum_i dE/dphi_i dphi_i/dy_j, NNP atom i
// the opposite of its column sum, as per-workgroup partials
// part[(3 i + k) * gridDim.x + blockIdx.x].
//
// A lane holds T MM atoms. The wavefronts of a workgroup take 8 NNP atoms each,
// of the same 64 T MM atoms, row after row of the grid; the MM forces of all
// rows are added up in registers, then through LDS: with one grid row the
// workgroup owns them and writes or adds them plainly; grid rows add with FP64
// atomics.  Few NNP atoms: bound by the chain of pairs of the few wavefronts
// inside the cutoff, hence 8 atoms each and T = 1: 60 NNP atoms, 30,000 charges
// 7.4 us (16 atoms and two MM atoms per lane: 11.8), and the partials 1.5 in
// the gather.  Workgroups of 16 NNP atoms that added to cleared MM forces with
// atomics, and a launch for the partials, took 10.5 + 4.1 us and the clearing
// 2.1.  Many: bound by the pairs and the sums over lanes after each 8 T of a
// lane, hence T = 4 (mm_tiles), 30,000 charges, event-timed: 1,000 NNP atoms 43
// us and 4,000 101 (T = 1, the forces exchanged after every row, 81 and 322; a
// workgroup per 256 MM atoms and 16 NNP atoms, with atomics, 55 and 178).
template <int T>
__global__ __launch_bounds__(64 * kBwdWaves) void k_mm_bwd(const float4* __restrict__ spos, int n,
                                                           const float* __restrict__ mm_pos,
                                                           const float* __restrict__ mm_q, int n_mm,
                                                           const float* __restrict__ gx,
                                                           const float* __restrict__ qpred, DescParams p, Geometry g,
                                                           float* __restrict__ part,
                                                           double* __restrict__ mm_forces, int assign) {
  __shared__ double sf[kBwdWaves][3][64];   // MM forces of each wavefront
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), waves = blockDim.x >> 6;
  const int rows = kBwdChunk * waves;
  const float rm2 = p.mm_cutoff * p.mm_cutoff;
  const float inv2rm = 0.5f / p.mm_cutoff;
  const float dfc_s = -0.5f * 3.14159265358979323846f / p.mm_cutoff;
  for (int64_t j0 = (int64_t)blockIdx.x * (64 * T); j0 < n_mm; j0 += (int64_t)gridDim.x * (64 * T)) {
    float4 y[T];   // MM x, y, z, q
    double f[T][3];
#pragma unroll
    for (int u = 0; u < T; ++u) {
      const int64_t j = min(j0 + 64 * u + lane, (int64_t)n_mm - 1);
      y[u] = make_float4(mm_pos[3 * j], mm_pos[3 * j + 1], mm_pos[3 * j + 2], mm_q[j]);
      f[u][0] = f[u][1] = f[u][2] = 0.0;
    }
    for (int r0 = blockIdx.y * rows; r0 < n; r0 += gridDim.y * rows) {
      const int i0 = r0 + kBwdChunk * wave, cnt = min(n - i0, kBwdChunk);
      if (cnt <= 0) break;
      float ax[kBwdChunk], ay[kBwdChunk], az[kBwdChunk];
#pragma unroll
      for (int c = 0; c < kBwdChunk; ++c) {
        ax[c] = ay[c] = az[c] = 0.f;
        if (c >= cnt) continue;
        const int i = i0 + c;
        float gi = gx[(int64_t)i * p.stride + p.D];
        if (qpred != nullptr) gi += qpred[i];
        const float ke_g = (float)p.ke * gi;
        const float4 pi = spos[i];
#pragma unroll
        for (int u = 0; u < T; ++u) {
          float dx, dy, dz, r2;
          mm_disp(pi, y[u].x, y[u].y, y[u].z, g, dx, dy, dz, r2);
          if (j0 + 64 * u + lane < n_mm && r2 < rm2) {
            float ir = __builtin_amdgcn_rsqf(r2);
            float r = r2 * ir;
            float arg = r * inv2rm;
            float fc = 0.5f * __builtin_amdgcn_cosf(arg) + 0.5f;
            float dfc = dfc_s * __builtin_amdgcn_sinf(arg);
            float fp = (dfc - fc * ir) * ir;            // d/dr (fc / r)
            float w = ke_g * y[u].w * fp * ir;   // times u = d / r
            const float vx = w * dx, vy = w * dy, vz = w * dz;
            ax[c] += vx; ay[c] += vy; az[c] += vz;
            f[u][0] -= vx; f[u][1] -= vy; f[u][2] -= vz;
          }
        }
      }
      const float s[3] = {wave_sum8(ax, lane), wave_sum8(ay, lane), wave_sum8(az, lane)};
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (lane < cnt) {
          float* o = part + ((int64_t)(i0 + lane) * 3 + k) * gridDim.x + blockIdx.x;
          *o = j0 < (int64_t)gridDim.x * (64 * T) ? s[k] : *o + s[k];
        }
    }
    if (mm_forces == nullptr) continue;
    const int used = min(waves, (n - (int)blockIdx.y * rows + kBwdChunk - 1) / kBwdChunk);
#pragma unroll
    for (int u = 0; u < T; ++u) {
#pragma unroll
      for (int k = 0; k < 3; ++k) sf[wave][k][lane] = f[u][k];
      __syncthreads();
      for (int t = threadIdx.x; t < 3 * 64; t += blockDim.x) {
        const int c = t / 3, k = t - 3 * c;
        if (j0 + 64 * u + c >= n_mm) continue;
        double v = 0.0;
        for (int w = 0; w < used; ++w) v += sf[w][k][c];
        double* o = mm_forces + 3 * (j0 + 64 * u) + t;
        if (gridDim.y > 1) {
          if (v != 0.0) unsafeAtomicAdd(o, v);
        } else if (assign) {
          *o = v;
        } else if (v != 0.0) {
          *o += v;
        }
      }
      __syncthreads();
    }
  }
}

inline int mm_blocks(int n_mm) {
  const int b = (n_mm + kBlock - 1) / kBlock;
  return b < kMaxMmBlocks ? b : kMaxMmBlocks;
}

// MM atoms per lane of the adjoint: one, for as many wavefronts as there can
// be, while pieces of 8 NNP and 64 MM atoms come to fewer than 16 per CU; four
// from there on, a sum over lanes and an exchange through LDS then being shared
// by 32 pairs instead of 8 (calls, us, one -> four: 60 NNP atoms and 30,000
// charges 70.3 -> 71.1, 100 and 30,000 76.8 -> 74.7, 1,000 and 30,000 156 ->
// 132, 500 and 3,000 84.4 -> 90.7).
inline int mm_tiles(const nnp_model& m, int n, int n_mm) {
  const int64_t rows = (n + kBwdChunk - 1) / kBwdChunk, groups = (n_mm + 63) / 64;
  return groups <= kMaxMmBlocks && rows * groups <= 16 * (int64_t)m.n_cu ? 1 : kBwdTiles;
}

inline int wave_blocks(int n) { return (int)(((int64_t)n * 64 + kBlock - 1) / kBlock); }

}  // namespace

int mm_partial_blocks(const nnp_model& m, int n, int n_mm) {
  return mm_tiles(m, n, n_mm) == 1 ? (n_mm + 63) / 64 : mm_blocks(n_mm);
}

// Three floats per partial: a partial per 256 MM atoms for every atom, or what
// calls with one per 64 can use (mm_tiles).
size_t mm_partial_floats(const nnp_model& m, int max_atoms, int max_mm) {
  const size_t fine = std::min((size_t)max_atoms * std::min((max_mm + 63) / 64, kMaxMmBlocks),
                               (size_t)kBwdChunk * 16 * m.n_cu);
  return 3 * std::max(fine, (size_t)max_atoms * mm_blocks(max_mm));
}

hipError_t launch_mm_fwd(nnp_model& m, int n, int n_mm, const float* mm_pos, const float* mm_q,
                         hipStream_t st) {
  if (n == 0) return hipSuccess;
  const int nbx = n_mm > 0 ? mm_blocks(n_mm) : 0;
  if (nbx > 0) {
    if (m.d_mm_part == nullptr || (size_t)n * nbx > mm_partial_floats(m, m.max_atoms, m.max_mm))
      return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_mm_fwd, dim3(nbx, (n + kNnpChunk - 1) / kNnpChunk), dim3(kBlock), 0, st, m.d_spos, n,
                       mm_pos, mm_q, n_mm, m.dp, m.geo, m.d_mm_part);
  }
  hipLaunchKernelGGL(k_mm_finish, dim3(wave_blocks(n)), dim3(kBlock), 0, st, m.d_mm_part, nbx, n, m.dp, m.d_x);
  return hipGetLastError();
}

hipError_t launch_mm_bwd(nnp_model& m, int n, int n_mm, const float* mm_pos, const float* mm_q, double* mm_forces,
                         int accumulate, hipStream_t st) {
  if (n == 0 || n_mm == 0)
    return mm_forces != nullptr && !accumulate ? launch_fill_f64(mm_forces, 3 * (int64_t)n_mm, st) : hipSuccess;
  const int nbx = mm_partial_blocks(m, n, n_mm);
  if (m.d_mm_part == nullptr || 3 * (size_t)n * nbx > mm_partial_floats(m, m.max_atoms, m.max_mm))
    return hipErrorInvalidValue;
  // as many wavefronts as there are rows of 8 NNP atoms; with more rows than
  // one workgroup takes, grid rows until there are two workgroups per CU
  const int rows = (n + kBwdChunk - 1) / kBwdChunk, waves = std::min(rows, kBwdWaves);
  const int gy = std::min((rows + waves - 1) / waves, std::max(1, 2 * m.n_cu / nbx));
  if (gy > 1 && mm_forces != nullptr && !accumulate) {
    const hipError_t e = launch_fill_f64(mm_forces, 3 * (int64_t)n_mm, st);
    if (e != hipSuccess) return e;
  }
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(nbx, gy), dim3(64 * waves), 0, st, m.d_spos, n, mm_pos, mm_q, n_mm, m.d_g,
                       m.charges ? m.d_q : nullptr, m.dp, m.geo, m.d_mm_part, mm_forces, !accumulate);
  };
  if (mm_tiles(m, n, n_mm) == 1) run(k_mm_bwd<1>);
  else run(k_mm_bwd<kBwdTiles>);
  return hipGetLastError();
}

hipError_t launch_fill_f64(double* p, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_f64, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, p, (int)n);
  return hipGetLastError();
}

}  // namespace nnp
