// Symmetry-function descriptors (forward) and their adjoint (backward with
// the FP64 force scatter), the force gather with the energy reduction, and
// the link-atom chain rule.  The descriptors are those of the ANI family of
// models the paper runs and benchmarks (Methods; performance section); the
// adjoint gives F = -grad E (Theory, eq. 2).
//
// The forward runs one 16-lane row per atom (k_desc_fwd_rows), one wavefront
// per atom (k_desc_fwd), or one to four atoms per wavefront with the lanes
// balanced over chunks of all their work (k_desc_fwd_pool), chosen by elements
// and size (descriptor_variant); the adjoint one wavefront per atom.  An output block is either the radial block of one neighbour
// species (16 outputs) or the angular block of one unordered species pair
// (8 x 4 outputs).
//
// Radial   G[s][k]   = sum_j exp(-eta_r (r - Rs_k)^2) fc(r; Rc)
// Angular  G[p][m][n] = 2^(1-zeta) sum_{j<k} (1 + cos(theta' - theta_n))^zeta
//                         exp(-eta_a (rbar - Ra_m)^2) fc(r_j; Rca) fc(r_k; Rca)
// with theta' = arccos(0.95 cos theta).  cos(theta' - theta_n) is expanded as
// cos theta' cos theta_n + sin theta' sin theta_n, where cos theta' = 0.95 c
// and sin theta' = sqrt(1 - (0.95 c)^2) >= 0.312, so no arccos is evaluated.
//
// Transcendentals use the hardware exp2 / log2 / sin / cos / sqrt / rsq
// instructions (arguments pre-scaled: exp(x) = exp2(x log2 e), cos(pi r/R) =
// cos of r/(2R) revolutions).
#include <climits>

#include "nnp_internal.h"

namespace nnp {
namespace {

constexpr int kBlock = 256;
constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float lg2(float x) { return __builtin_amdgcn_logf(x); }
__device__ __forceinline__ float cos_rev(float x) { return __builtin_amdgcn_cosf(x); }
__device__ __forceinline__ float sin_rev(float x) { return __builtin_amdgcn_sinf(x); }
__device__ __forceinline__ float rsq(float x) { return __builtin_amdgcn_rsqf(x); }

struct Geo {
  float dx, dy, dz, r, ir;
};

__device__ __forceinline__ Geo displacement(const float4& pi, const float4& pj, const MinImage& b) {
  Geo o;
  float dx = pj.x - pi.x, dy = pj.y - pi.y, dz = pj.z - pi.z;
  if (b.on) {
    dx -= b.L[0] * rintf(dx * b.iL[0]);
    dy -= b.L[1] * rintf(dy * b.iL[1]);
    dz -= b.L[2] * rintf(dz * b.iL[2]);
  }
  float r2 = dx * dx + dy * dy + dz * dz;
  float ir = rsq(r2);
  o.dx = dx; o.dy = dy; o.dz = dz;
  o.r = r2 * ir;
  o.ir = ir;
  return o;
}

struct Consts {
  // pre-scaled constants
  float eta_r_l2, eta_a_l2;      // eta * log2(e)
  float inv2rc, inv2rca;         // 1 / (2 Rc): cos(pi r / Rc) = cos_rev(r / (2 Rc))
  float dfc_r, dfc_a;            // -0.5 pi / Rc
};

__device__ __forceinline__ Consts make_consts(const DescParams& p) {
  Consts c;
  c.eta_r_l2 = p.eta_rad * kLog2e;
  c.eta_a_l2 = p.eta_ang * kLog2e;
  c.inv2rc = p.inv2rc;
  c.inv2rca = p.inv2rca;
  c.dfc_r = p.dfc_r;
  c.dfc_a = p.dfc_a;
  return c;
}

// Split the 64 lanes of a wavefront over nb output blocks in proportion to
// their work counts (every block with work gets at least one lane), and
// return this lane's block, its rank in the block and the block's lane count.
__device__ __forceinline__ void split_lanes(const int* cnt, int nb, int lane, int* my_b, int* my_rank, int* my_len,
                                            int* start, int* len) {
  int total = 0;
  for (int b = 0; b < nb; ++b) total += cnt[b];
  const float scale = total > 0 ? 64.f / (float)total : 0.f;
  int used = 0;
  for (int b = 0; b < nb; ++b) {
    len[b] = cnt[b] > 0 ? max(1, (int)((float)cnt[b] * scale)) : 0;
    used += len[b];
  }
  while (used > 64) {  // only when many tiny blocks were rounded up to one lane
    int k = 0;
    for (int b = 1; b < nb; ++b) if (len[b] > len[k]) k = b;
    --len[k];
    --used;
  }
  while (used < 64 && total > 0) {  // spare lanes go to the block with most work per lane
    int k = -1;
    for (int b = 0; b < nb; ++b)
      if (cnt[b] > 0 && (k < 0 || cnt[b] * len[k] > cnt[k] * len[b])) k = b;
    ++len[k];
    ++used;
  }
  int run = 0;
  *my_b = -1;
  *my_rank = 0;
  *my_len = 0;
  for (int b = 0; b < nb; ++b) {
    start[b] = run;
    if (lane >= run && lane < run + len[b]) {
      *my_b = b;
      *my_rank = lane - run;
      *my_len = len[b];
    }
    run += len[b];
  }
}

// Forward descriptors, one wavefront per atom.  Radial phase: the lanes are
// split over the S neighbour-species segments of the radial list, each lane
// accumulating the 16 radial terms of its neighbours in registers.  Angular
// phase: the angular neighbours' geometry is cached in LDS (one array per
// component) and the lanes are split over the P species-pair classes; each
// lane takes a contiguous range of its class's (j, k) pairs, walked without
// divisions, and accumulates the 32 terms in registers.  Each phase ends
// with a fixed-order reduction of the per-lane partial sums through LDS.
struct FwdArgs {
  const int* order;        // bin-major visiting order of the slots
  const float4* spos;
  const int* rad;
  const int* ang;
  const int* rad_off;
  const int* ang_off;
  int max_rad, max_ang, n;
  float* x;
};

constexpr int kPartStride = 33;  // padded row of the per-lane partial sums

__global__ __launch_bounds__(64) void k_desc_fwd(FwdArgs a, DescParams p, Geometry geo) {
  extern __shared__ float smem_f[];
  float* part = smem_f;                      // [64][kPartStride]
  float* gux = part + 64 * kPartStride;      // angular neighbours, one array per component
  float* guy = gux + a.max_ang;
  float* guz = guy + a.max_ang;
  float* gr = guz + a.max_ang;
  float* gfc = gr + a.max_ang;
  const int i = a.order[xcd_block(blockIdx.x, gridDim.x)];
  const int lane = threadIdx.x;
  const Consts c = make_consts(p);
  const float4 pi = a.spos[i];
  const MinImage mi = min_image_at(geo, i);
  const int S1 = p.S + 1;
  const int* roff = a.rad_off + (int64_t)i * S1;
  const int* aoff = a.ang_off + (int64_t)i * S1;
  const int* rrow = a.rad + (int64_t)i * a.max_rad;
  const int* arow = a.ang + (int64_t)i * a.max_ang;
  float* xo = a.x + (int64_t)i * p.stride;
  int cnt[kMaxPairs], st[kMaxPairs], len[kMaxPairs];
  int my_b, my_rank, my_len;

  // ---- radial phase
  for (int s = 0; s < p.S; ++s) cnt[s] = roff[s + 1] - roff[s];
  split_lanes(cnt, p.S, lane, &my_b, &my_rank, &my_len, st, len);
  {
    float acc[kRadShifts];
#pragma unroll
    for (int k = 0; k < kRadShifts; ++k) acc[k] = 0.f;
    if (my_b >= 0) {
      const int t1 = roff[my_b + 1];
      for (int t = roff[my_b] + my_rank; t < t1; t += my_len) {
        Geo d = displacement(pi, a.spos[rrow[t]], mi);
        float fc = 0.5f * cos_rev(d.r * c.inv2rc) + 0.5f;
#pragma unroll
        for (int k = 0; k < kRadShifts; ++k) {
          float tt = d.r - p.rad_shift[k];
          acc[k] += ex2(-c.eta_r_l2 * tt * tt) * fc;
        }
      }
    }
#pragma unroll
    for (int k = 0; k < kRadShifts; ++k) part[lane * kPartStride + k] = acc[k];
  }
  // angular neighbour geometry
  const int na = aoff[p.S];
  for (int u = lane; u < na; u += 64) {
    Geo d = displacement(pi, a.spos[arow[u]], mi);
    gux[u] = d.dx * d.ir;
    guy[u] = d.dy * d.ir;
    guz[u] = d.dz * d.ir;
    gr[u] = d.r;
    gfc[u] = 0.5f * cos_rev(d.r * c.inv2rca) + 0.5f;
  }
  __syncthreads();
  for (int o = lane; o < p.S * kRadShifts; o += 64) {
    const int b = o / kRadShifts, k = o % kRadShifts;
    float v = 0.f;
    for (int l = st[b]; l < st[b] + len[b]; ++l) v += part[l * kPartStride + k];
    xo[o] = v;
  }
  __syncthreads();

  // ---- angular phase
  for (int q = 0; q < p.P; ++q) {
    const int na_ = aoff[p.pair_a[q] + 1] - aoff[p.pair_a[q]];
    const int nb_ = aoff[p.pair_b[q] + 1] - aoff[p.pair_b[q]];
    cnt[q] = p.pair_a[q] == p.pair_b[q] ? na_ * (na_ - 1) / 2 : na_ * nb_;
  }
  split_lanes(cnt, p.P, lane, &my_b, &my_rank, &my_len, st, len);
  {
    float acc[kAngShifts][kAngSects];
#pragma unroll
    for (int m = 0; m < kAngShifts; ++m)
#pragma unroll
      for (int n = 0; n < kAngSects; ++n) acc[m][n] = 0.f;
    if (my_b >= 0) {
      const int sa = p.pair_a[my_b], sb = p.pair_b[my_b];
      const int oa = aoff[sa], ob = aoff[sb];
      const int nB = aoff[sb + 1] - ob;
      const int T = cnt[my_b];
      // contiguous range [r0, r1) of this lane
      const int r0 = (int)(((int64_t)T * my_rank) / my_len);
      const int r1 = (int)(((int64_t)T * (my_rank + 1)) / my_len);
      int uj, uk;      // same pair (j, k): walk k = 1..n-1, j = 0..k-1 (k-major)
      if (sa == sb) {
        int kk = (int)((1.f + __builtin_amdgcn_sqrtf(1.f + 8.f * (float)r0)) * 0.5f);
        while (kk * (kk - 1) / 2 > r0) --kk;
        while ((kk + 1) * kk / 2 <= r0) ++kk;
        uj = r0 - kk * (kk - 1) / 2;
        uk = kk;
      } else {         // different species: j-major over (j, k)
        uj = r0 / max(nB, 1);
        uk = r0 - uj * nB;
      }
      for (int r = r0; r < r1; ++r) {
        const int gj = oa + uj;
        const int gk = (sa == sb ? oa : ob) + uk;
        float cs = gux[gj] * gux[gk] + guy[gj] * guy[gk] + guz[gj] * guz[gk];
        float ct = 0.95f * cs;
        float sn = __builtin_amdgcn_sqrtf(1.f - ct * ct);
        float F = p.ang_pref * gfc[gj] * gfc[gk];
        float rbar = 0.5f * (gr[gj] + gr[gk]);
        float A[kAngSects];
#pragma unroll
        for (int n = 0; n < kAngSects; ++n) {
          float base = 1.f + ct * p.cos_sect[n] + sn * p.sin_sect[n];
          A[n] = F * ex2(p.zeta * lg2(base));
        }
#pragma unroll
        for (int m = 0; m < kAngShifts; ++m) {
          float tt = rbar - p.ang_shift[m];
          float B = ex2(-c.eta_a_l2 * tt * tt);
#pragma unroll
          for (int n = 0; n < kAngSects; ++n) acc[m][n] += B * A[n];
        }
        if (sa == sb) {
          if (++uj == uk) { uj = 0; ++uk; }
        } else {
          if (++uk == nB) { uk = 0; ++uj; }
        }
      }
    }
#pragma unroll
    for (int m = 0; m < kAngShifts; ++m)
#pragma unroll
      for (int n = 0; n < kAngSects; ++n) part[lane * kPartStride + m * kAngSects + n] = acc[m][n];
  }
  __syncthreads();
  const int nang = p.P * kAngShifts * kAngSects;
  for (int o = lane; o < nang; o += 64) {
    const int q = o / (kAngShifts * kAngSects), e = o % (kAngShifts * kAngSects);
    float v = 0.f;
    for (int l = st[q]; l < st[q] + len[q]; ++l) v += part[l * kPartStride + e];
    xo[p.S * kRadShifts + o] = v;
  }
}

// ---------------------------------------------------------------------------
// Row kernels: one 16-lane DPP row per atom, four atoms per wavefront.
//
// The lanes of a row split an output block's pairs (radial: strided over the
// species segment; angular: a contiguous range of the class's (j, k) pairs),
// each lane accumulating the whole block in registers; the row then sums the
// block across its 16 lanes with a transposing butterfly (every step halves
// the values a lane holds, so 16 values cost 15 exchanges and 32 cost 30),
// leaving lane l with outputs [l B/16, (l+1) B/16).  The exchanges are DPP
// row permutations: mirror (l <-> 15-l), half-mirror (l <-> 7-l within each
// half) and the quad swaps xor 2 and xor 1; the pairings are disjoint, so
// after four steps every lane's values cover all 16 lanes exactly once.

// Sum N values over the L = 16 or 8 lanes of a row; lane `sub` ends with
// totals [sub N/L, (sub+1) N/L) in v[0 .. N/L).  An 8-lane row is half of a
// DPP row, whose half-mirror pairs lanes across bit 2 within each half.
template <int N, int L>
__device__ __forceinline__ void row_reduce(float* v, int sub) {
  if constexpr (L == 16) {
    halve<N / 2, kDppMirror>(v, sub & 8);
    halve<N / 4, kDppHalfMirror>(v, sub & 4);
    halve<N / 8, kDppXor2>(v, sub & 2);
    halve<N / 16, kDppXor1>(v, sub & 1);
  } else {
    static_assert(L == 8, "row width");
    halve<N / 2, kDppHalfMirror>(v, sub & 4);
    halve<N / 4, kDppXor2>(v, sub & 2);
    halve<N / 8, kDppXor1>(v, sub & 1);
  }
}

// Start of a lane's contiguous range [r0, r1) of T unordered pairs within a
// class, decoded to (j, k): same species: k-major over j < k; different
// species: j-major over (j, k).
__device__ __forceinline__ void pair_start(int r0, bool same, int nB, int* j, int* k) {
  if (same) {
    int kk = (int)((1.f + __builtin_amdgcn_sqrtf(1.f + 8.f * (float)r0)) * 0.5f);
    if (kk * (kk - 1) / 2 > r0) --kk;      // the sqrt is within an ulp: one step each way
    if ((kk + 1) * kk / 2 <= r0) ++kk;
    *k = kk;
    *j = r0 - kk * (kk - 1) / 2;
  } else {
    const int jj = (int)(((float)r0 + 0.5f) * __builtin_amdgcn_rcpf((float)max(nB, 1)));
    *j = jj;
    *k = r0 - jj * nB;
  }
}

// L lanes per atom (16 or 8), 256 / L atoms per 256-thread workgroup.
template <int L>
__global__ __launch_bounds__(256) void k_desc_fwd_rows(FwdArgs a, DescParams p, Geometry geo) {
  constexpr int kAtoms = 256 / L;
  extern __shared__ float4 smem_r[];
  const int row = threadIdx.x / L, sub = threadIdx.x % L;
  float4* G = smem_r + row * a.max_ang;                                      // (u, r hq)
  float* W = reinterpret_cast<float*>(smem_r + kAtoms * a.max_ang) + row * a.max_ang;  // fc sq_pref
  const int li = xcd_block(blockIdx.x, gridDim.x) * kAtoms + row;   // place in the visiting order
  const bool valid = li < a.n;
  const Consts c = make_consts(p);
  const int S1 = p.S + 1;
  const int ii = valid ? a.order[li] : 0;
  const float4 pi = a.spos[ii];
  const MinImage mi = min_image_at(geo, ii);
  const int* roff = a.rad_off + (int64_t)ii * S1;
  const int* aoff = a.ang_off + (int64_t)ii * S1;
  const int* rrow = a.rad + (int64_t)ii * a.max_rad;
  const int* arow = a.ang + (int64_t)ii * a.max_ang;
  float* xo = a.x + (int64_t)ii * p.stride;

  // angular neighbour geometry of this row's atom
  const int na = valid ? aoff[p.S] : 0;
  for (int u = sub; u < na; u += L) {
    Geo d = displacement(pi, a.spos[arow[u]], mi);
    G[u] = make_float4(d.dx * d.ir, d.dy * d.ir, d.dz * d.ir, d.r * p.hq_eta_a);
    W[u] = (0.5f * cos_rev(d.r * c.inv2rca) + 0.5f) * p.sq_pref;
  }

  // radial blocks
  for (int s = 0; s < p.S; ++s) {
    float acc[kRadShifts];
#pragma unroll
    for (int k = 0; k < kRadShifts; ++k) acc[k] = 0.f;
    const int t1 = valid ? roff[s + 1] : 0;
    for (int t = (valid ? roff[s] : 0) + sub; t < t1; t += L) {
#pragma clang fp contract(off)   // keep r sq in a register: one SGPR operand per shift
      Geo d = displacement(pi, a.spos[rrow[t]], mi);
      const float fc = fmaf(0.5f, cos_rev(d.r * c.inv2rc), 0.5f);
      const float rs = d.r * p.sq_eta_r;
#pragma unroll
      for (int k = 0; k < kRadShifts; ++k) {
        const float tt = rs - p.rad_shift_s[k];
        acc[k] = fmaf(ex2(-(tt * tt)), fc, acc[k]);
      }
    }
    row_reduce<kRadShifts, L>(acc, sub);
    if (valid) {
      if constexpr (L == 16) xo[s * kRadShifts + sub] = acc[0];
      else *reinterpret_cast<float2*>(xo + s * kRadShifts + 2 * sub) = make_float2(acc[0], acc[1]);
    }
  }
  __syncthreads();

  // angular blocks
  for (int q = 0; q < p.P; ++q) {
    const int sa = p.pair_a[q], sb = p.pair_b[q];
    const bool same = sa == sb;
    int oa = 0, ob = 0, nA = 0, nB = 0;
    if (valid) {
      oa = aoff[sa];
      nA = aoff[sa + 1] - oa;
      ob = aoff[sb];
      nB = aoff[sb + 1] - ob;
    }
    const int T = same ? nA * (nA - 1) / 2 : nA * nB;
    const int r0 = (T * sub) / L, r1 = (T * (sub + 1)) / L;
    float acc[kAngShifts * kAngSects];
#pragma unroll
    for (int e = 0; e < kAngShifts * kAngSects; ++e) acc[e] = 0.f;
    if (r0 < r1) {
      int j, k;
      pair_start(r0, same, nB, &j, &k);
      const int kbase = same ? oa : ob;
      for (int r = r0; r < r1; ++r) {
        const float4 gj = G[oa + j], gk = G[kbase + k];
        const float F = W[oa + j] * W[kbase + k];
        const float cs = gj.x * gk.x + gj.y * gk.y + gj.z * gk.z;
        const float ct = 0.95f * cs;
        const float sn = __builtin_amdgcn_sqrtf(1.f - ct * ct);
        const float rb = gj.w + gk.w;
        float A[kAngSects];
#pragma unroll
        for (int n = 0; n < kAngSects; ++n) {
          const float base = 1.f + ct * p.cos_sect[n] + sn * p.sin_sect[n];
          A[n] = F * ex2(p.zeta * lg2(base));
        }
#pragma unroll
        for (int m = 0; m < kAngShifts; ++m) {
          const float tt = rb - p.ang_shift_s[m];
          const float B = ex2(-(tt * tt));
#pragma unroll
          for (int n = 0; n < kAngSects; ++n) acc[m * kAngSects + n] = fmaf(B, A[n], acc[m * kAngSects + n]);
        }
        if (same) {
          if (++j == k) { j = 0; ++k; }
        } else {
          if (++k == nB) { k = 0; ++j; }
        }
      }
    }
    row_reduce<kAngShifts * kAngSects, L>(acc, sub);
    if (valid) {
      float* dst = xo + p.S * kRadShifts + q * kAngShifts * kAngSects;
      if constexpr (L == 16)
        *reinterpret_cast<float2*>(dst + 2 * sub) = make_float2(acc[0], acc[1]);
      else
        *reinterpret_cast<float4*>(dst + 4 * sub) = make_float4(acc[0], acc[1], acc[2], acc[3]);
    }
  }
}

// ---------------------------------------------------------------------------
// Pool kernel: AW atoms per wavefront, the lanes balanced over the work of
// all of them.
//
// The radial neighbours of one (atom, neighbour species) and the angular
// pairs of one (atom, species-pair class) form a unit.  The wavefront cuts
// its units into chunks of at most C items, C being (within a few steps) the
// smallest size for which the chunks fit its 64 lanes, and each lane sums one
// chunk's block in registers.  The chunks of a unit then add up pairwise in
// a tree (chunk c + d into chunk c for c a multiple of 2d, d = 1, 2, 4, ...,
// 16 values at a time through LDS), and the unit's first chunk stores the
// block in the descriptor row.
//
// With several elements a class holds few pairs (about 14 per class for
// H/C/N/O molecules against 17 angular neighbours): the row kernels then
// leave most lanes of a row idle and pay a 32-value cross-lane reduction per
// class, which this kernel avoids.  Adding the partials with LDS float
// atomics instead was several times slower.  The radial phase runs first,
// with the first pass of the angular geometry already loaded into registers,
// so that the partial rows can share LDS with the angular geometry (each is
// dead while the other is live).
constexpr int kPoolPitch = 20;   // LDS row of one lane's 16 partial sums (16-byte aligned)

__device__ __forceinline__ int wave_total(int v) {
  return __builtin_amdgcn_readlane(wave_scan_dpp<false>(v), 63);
}

// ceil(x / C) for 0 <= x < 2^20 and C >= 1, with rC = 1 / C: the FP32
// quotient is within one of the true one, and one correction each way fixes it.
__device__ __forceinline__ int ceil_div(int x, int C, float rC) {
  if (x <= 0) return 0;
  const int y = x - 1;
  int q = (int)((float)y * rC);
  q -= q * C > y ? 1 : 0;
  q += (q + 1) * C <= y ? 1 : 0;
  return q + 1;
}

// Chunk size for unit sizes cnt (one unit per lane, 0 elsewhere): with U
// non-empty units and N items, C = ceil(N / (64 - U)) always fits, since the
// chunk count is below N / C + U; smaller sizes are tried while they still fit.
__device__ __forceinline__ int pool_chunk(int cnt) {
  const int N = wave_total(cnt);
  if (N == 0) return 0;
  const int U = (int)__popcll(__ballot(cnt > 0));
  int C = (N + 63 - U) / (64 - U);   // uniform: scalar arithmetic
  for (int step = 0; step < 3 && C > 1; ++step) {
    const int k = ceil_div(cnt, C - 1, __builtin_amdgcn_rcpf((float)(C - 1)));
    if (wave_total(k) > 64) break;
    --C;
  }
  return C;
}

// The wavefronts of a pool workgroup work independently, each in its own LDS
// slice, and synchronise only among their own lanes: LDS accesses of one
// wavefront complete in order, so keeping the compiler from moving them
// across this point is enough.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Hands the chunks out to the lanes in unit order: lane l < K gets unit *unit
// (the lane that holds it), chunk *chunk of that unit and the unit's chunk
// count *nunit; other lanes get unit -1.  Returns the largest chunk count.
__device__ __forceinline__ int pool_assign(int cnt, int C, int lane, int* owner, int* unit, int* chunk,
                                           int* nunit) {
  const int nch = C > 0 ? ceil_div(cnt, C, __builtin_amdgcn_rcpf((float)C)) : 0;
  const int incl = wave_scan_dpp<false>(nch);
  const int K = __builtin_amdgcn_readlane(incl, 63);
  const int excl = incl - nch;
  owner[lane] = 0;
  wave_sync();
  if (nch > 0) owner[excl] = ((lane + 1) << 8) | excl;
  wave_sync();
  const int o = wave_scan_dpp<true>(owner[lane]);
  *unit = lane < K ? (o >> 8) - 1 : -1;
  *chunk = lane < K ? lane - (o & 255) : 0;
  *nunit = __shfl(nch, max(*unit, 0), 64);
  return __builtin_amdgcn_readlane(wave_scan_dpp<true>(nch), 63);
}

// Pairwise tree over the chunks of each unit (chunks of a unit sit on
// consecutive lanes): chunk c + d adds into chunk c for c a multiple of 2d,
// through this lane's LDS row, until chunk 0 holds the unit's sums.
__device__ __forceinline__ void pool_tree16(float* v, float* part, int lane, int unit, int chunk, int nunit,
                                            int maxn) {
  for (int d = 1; d < maxn; d *= 2) {
    wave_sync();
    if (unit >= 0 && (chunk & (2 * d - 1)) == d) {
      float4* row = reinterpret_cast<float4*>(part + lane * kPoolPitch);
#pragma unroll
      for (int e = 0; e < 4; ++e) row[e] = make_float4(v[4 * e], v[4 * e + 1], v[4 * e + 2], v[4 * e + 3]);
    }
    wave_sync();
    if (unit >= 0 && (chunk & (2 * d - 1)) == 0 && chunk + d < nunit) {
      const float4* row = reinterpret_cast<const float4*>(part + (lane + d) * kPoolPitch);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float4 w = row[e];
        v[4 * e] += w.x;
        v[4 * e + 1] += w.y;
        v[4 * e + 2] += w.z;
        v[4 * e + 3] += w.w;
      }
    }
  }
}

__device__ __forceinline__ void store16(float* dst, const float* v) {
  float4* d4 = reinterpret_cast<float4*>(dst);
#pragma unroll
  for (int e = 0; e < 4; ++e) d4[e] = make_float4(v[4 * e], v[4 * e + 1], v[4 * e + 2], v[4 * e + 3]);
}

template <int AW>
__global__ __launch_bounds__(256) void k_desc_fwd_pool(FwdArgs a, DescParams p, Geometry geo) {
  static_assert(AW >= 1 && AW * kMaxPairs <= 40, "units must leave lanes for the chunks");
  extern __shared__ float4 smem_pool[];
  const int S = p.S, P = p.P, S1 = S + 1;
  // per wavefront: [angular geometry | partial rows (aliased: never live together)] [owner]
  const int area = (max(AW * a.max_ang * 5, 64 * kPoolPitch) + 3) & ~3;   // floats
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  float4* smem_p = smem_pool + wave * ((area + 64) / 4);
  float4* G = smem_p;                                             // [AW][max_ang] (u, r hq)
  float* W = reinterpret_cast<float*>(G + AW * a.max_ang);        // [AW][max_ang] fc sq_pref
  float* part = reinterpret_cast<float*>(smem_p);                 // [64][kPoolPitch]
  int* owner = reinterpret_cast<int*>(smem_p) + area;             // [64]
  const int li0 = (xcd_block(blockIdx.x, gridDim.x) * 4 + wave) * AW;
  const Consts c = make_consts(p);
  int slot[AW], na[AW];
  int nat = 0;
#pragma unroll
  for (int t = 0; t < AW; ++t) {
    slot[t] = li0 + t < a.n ? a.order[li0 + t] : 0;
    na[t] = li0 + t < a.n ? a.ang_off[(int64_t)slot[t] * S1 + S] : 0;
    nat += na[t];
  }
  auto atom_of = [&](int t) {
    int ii = slot[0];
#pragma unroll
    for (int k = 1; k < AW; ++k) ii = t == k ? slot[k] : ii;
    return ii;
  };

  // ---- angular units (lane t * kMaxPairs + q), set up first so that their
  // loads and the first pass of the geometry loads overlap the radial phase
  uint64_t pairs = 0;   // species pairs of the classes, four bits each (uniform)
#pragma unroll
  for (int k = 0; k < kMaxPairs; ++k) pairs |= (uint64_t)(p.pair_a[k] | (p.pair_b[k] << 2)) << (4 * k);
  int T = 0, oa = 0, kb = 0, nB = 0, same = 0;
  {
    const int t = lane / kMaxPairs, q = lane % kMaxPairs;
    if (t < AW && q < P && li0 + t < a.n) {
      const int code = (int)(pairs >> (4 * q)) & 15;
      const int sa = code & 3, sb = code >> 2;
      const int ii = atom_of(t);
      const int* aoff = a.ang_off + (int64_t)ii * S1;
      oa = aoff[sa];
      const int nA = aoff[sa + 1] - oa;
      const int ob = aoff[sb];
      nB = aoff[sb + 1] - ob;
      same = sa == sb;
      kb = same ? oa : ob;
      T = same ? nA * (nA - 1) / 2 : nA * nB;
      if (T == 0) {   // no pairs in this class
        const float zero[kRadShifts] = {};
        float* dst = a.x + (int64_t)ii * p.stride + S * kRadShifts + q * kAngShifts * kAngSects;
        store16(dst, zero);
        store16(dst + 16, zero);
      }
    }
  }
  // angular neighbour geometry, flattened over the atoms: the first pass is
  // loaded now and stored to LDS after the radial phase (whose partial rows
  // share that LDS)
  auto split = [&](int f, int* tt, int* uu) {
    int t = 0, u = f;
#pragma unroll
    for (int k = 0; k + 1 < AW; ++k)
      if (t == k && u >= na[k]) { u -= na[k]; t = k + 1; }
    *tt = t;
    *uu = u;
  };
  int g_t = 0, g_u = 0, g_ii = 0;
  float4 g_pi = make_float4(0.f, 0.f, 0.f, 0.f), g_pj = g_pi;
  if (lane < nat) {
    split(lane, &g_t, &g_u);
    g_ii = atom_of(g_t);
    g_pi = a.spos[g_ii];
    g_pj = a.spos[a.ang[(int64_t)g_ii * a.max_ang + g_u]];
  }

  // ---- radial units (lane t * kMaxSpecies + s) and chunks
  {
    const int t = lane / kMaxSpecies, s = lane % kMaxSpecies;
    int beg = 0, cnt = 0, ii = 0;
    if (t < AW && s < S && li0 + t < a.n) {
      ii = atom_of(t);
      const int* roff = a.rad_off + (int64_t)ii * S1;
      beg = roff[s];
      cnt = roff[s + 1] - beg;
      if (cnt == 0) {   // no neighbours of this species
        const float zero[kRadShifts] = {};
        store16(a.x + (int64_t)ii * p.stride + s * kRadShifts, zero);
      }
    }
    const int C = pool_chunk(cnt);
    int unit, chunk, nunit;
    const int maxn = pool_assign(cnt, C, lane, owner, &unit, &chunk, &nunit);
    const int src = max(unit, 0);
    const int ub = __shfl(beg, src, 64), ue = __shfl(beg + cnt, src, 64), ui = __shfl(ii, src, 64);
    float acc[kRadShifts];
#pragma unroll
    for (int k = 0; k < kRadShifts; ++k) acc[k] = 0.f;
    if (unit >= 0) {
      const int b0 = ub + chunk * C, b1 = min(b0 + C, ue);
      const float4 pi = a.spos[ui];
      const MinImage mi = min_image_at(geo, ui);
      const int* rrow = a.rad + (int64_t)ui * a.max_rad;
      for (int q = b0; q < b1; ++q) {
#pragma clang fp contract(off)   // keep r sq in a register: one SGPR operand per shift
        const Geo d = displacement(pi, a.spos[rrow[q]], mi);
        const float fc = fmaf(0.5f, cos_rev(d.r * c.inv2rc), 0.5f);
        const float rs = d.r * p.sq_eta_r;
#pragma unroll
        for (int k = 0; k < kRadShifts; ++k) {
          const float tt = rs - p.rad_shift_s[k];
          acc[k] = fmaf(ex2(-(tt * tt)), fc, acc[k]);
        }
      }
    }
    pool_tree16(acc, part, lane, unit, chunk, nunit, maxn);
    if (unit >= 0 && chunk == 0) store16(a.x + (int64_t)ui * p.stride + (src % kMaxSpecies) * kRadShifts, acc);
  }
  wave_sync();

  // ---- angular geometry to LDS
  for (int f = lane; f < nat; f += 64) {
    if (f >= 64) {
      split(f, &g_t, &g_u);
      g_ii = atom_of(g_t);
      g_pi = a.spos[g_ii];
      g_pj = a.spos[a.ang[(int64_t)g_ii * a.max_ang + g_u]];
    }
    const Geo d = displacement(g_pi, g_pj, min_image_at(geo, g_ii));
    G[g_t * a.max_ang + g_u] = make_float4(d.dx * d.ir, d.dy * d.ir, d.dz * d.ir, d.r * p.hq_eta_a);
    W[g_t * a.max_ang + g_u] = (0.5f * cos_rev(d.r * c.inv2rca) + 0.5f) * p.sq_pref;
  }
  wave_sync();

  // ---- angular chunks
  const int C = pool_chunk(T);
  int unit, chunk, nunit;
  const int maxn = pool_assign(T, C, lane, owner, &unit, &chunk, &nunit);
  const int src = max(unit, 0);
  const int uT = __shfl(T, src, 64), uoa = __shfl(oa, src, 64), ukb = __shfl(kb, src, 64);
  const int unB = __shfl(nB, src, 64), usame = __shfl(same, src, 64);
  const int ut = src / kMaxPairs;
  float acc[kAngShifts * kAngSects];
#pragma unroll
  for (int e = 0; e < kAngShifts * kAngSects; ++e) acc[e] = 0.f;
  if (unit >= 0) {
    const float4* Gt = G + ut * a.max_ang;
    const float* Wt = W + ut * a.max_ang;
    const int r0 = chunk * C, r1 = min(r0 + C, uT);
    // (inner, outer) walk: same species k-major over j < k (inner j, limit k),
    // two species j-major (inner k, limit nB)
    int j, k;
    pair_start(r0, usame != 0, unB, &j, &k);
    int in = usame ? j : k, out = usame ? k : j;
    for (int r = r0; r < r1; ++r) {
      const int jj = usame ? in : out, kk = usame ? out : in;
      const float4 gj = Gt[uoa + jj], gk = Gt[ukb + kk];
      const float F = Wt[uoa + jj] * Wt[ukb + kk];
      const float cs = gj.x * gk.x + gj.y * gk.y + gj.z * gk.z;
      const float ct = 0.95f * cs;
      const float sn = __builtin_amdgcn_sqrtf(1.f - ct * ct);
      const float rb = gj.w + gk.w;
      float A[kAngSects];
#pragma unroll
      for (int n = 0; n < kAngSects; ++n) {
        const float base = 1.f + ct * p.cos_sect[n] + sn * p.sin_sect[n];
        A[n] = F * ex2(p.zeta * lg2(base));
      }
#pragma unroll
      for (int m = 0; m < kAngShifts; ++m) {
        const float tt = rb - p.ang_shift_s[m];
        const float B = ex2(-(tt * tt));
#pragma unroll
        for (int n = 0; n < kAngSects; ++n) acc[m * kAngSects + n] = fmaf(B, A[n], acc[m * kAngSects + n]);
      }
      ++in;
      const bool wrap = in == (usame ? out : unB);
      in = wrap ? 0 : in;
      out += wrap ? 1 : 0;
    }
  }
  // the unit sums in two halves of 16 (the geometry is dead from here on)
  constexpr int B = kAngShifts * kAngSects, H = B / 2;
  float* dst = a.x + (int64_t)atom_of(ut) * p.stride + S * kRadShifts + (src % kMaxPairs) * B;
  pool_tree16(acc, part, lane, unit, chunk, nunit, maxn);
  if (unit >= 0 && chunk == 0) store16(dst, acc);
  pool_tree16(acc + H, part, lane, unit, chunk, nunit, maxn);
  if (unit >= 0 && chunk == 0) store16(dst + H, acc + H);
}

// Adjoint, one wavefront per centre atom i (no global atomics).
//
// With d_ij = x_j - x_i, F_i = sum_j dE_i/dd_ij - sum_j dE_j/dd_ji.
//   Radial terms of both centres depend on the same r_ij and differ only in
//   the weights (dE_i/dG of j's species, dE_j/dG of i's species), so atom i
//   adds the two rows of 16 weights and evaluates the pair once for both:
//   nothing has to be handed to j, which does the same from its side.
//   Angular terms of centre i act on its angular neighbours: their totals are
//   summed in FP64 in LDS and handed over, rounded once to FP32, through the
//   centre's slot in each neighbour's own angular list (lists are symmetric
//   and sorted by slot within a species segment; each entry has one writer).
// k_force_gather then sums, per atom and in FP64, its own total and the
// entries of its angular list.
//
// The wavefront
//   1. computes the geometry, one radial neighbour per lane; lanes within the
//      angular cutoff (the lists' own predicate, so ranks equal list places)
//      leave a record in LDS;
//   2. sums the radial terms in quads: a quad of lanes per neighbour, four of
//      the 16 shifts per lane, so that dE_j/dG is read as one 64-byte piece;
//   3. evaluates the angular triplets (adj_triplets);
//   4. finds the places in the neighbours' lists, two lanes per neighbour.
//
// After a list of this call has overflowed its capacity (d_cut says so, for the
// adjoint and the gather alike; the status word outlives the call and can be
// cleared at any time) lists are cut off and no longer symmetric.  The
// wavefront then looks every place up in the radial lists (contrib rows follow
// those), leaves out dE_j/dG for a neighbour whose list does not hold the
// centre, and hands over through the radial entries.
//
// Bound by VALU issue: 932 VALU instructions per wavefront in the water box
// of 98,304 atoms, of which the triplet loop is 515 (210 per pass of 64), take
// 149 of the 160 us to issue, 952 at 261,000 atoms 404 of 428.  Handing over every radial neighbour through a search
// for its slot, as before, took 195 us there and 577 us (now 431) at 261,000
// atoms, and moved 12 bytes per radial instead of per angular neighbour
// through contrib (gather 46 -> 28 us).  Tried: the triplets' contractions on
// the matrix cores (4x4x1 FP32, one product per quad of lanes, weights in
// registers): 12 % fewer VALU instructions, but 461 us at 261,000 atoms, the
// 16 products per pass costing more issue time than they save.
struct BwdArgs {
  const int* order;        // bin-major visiting order of the slots
  const float4* spos;
  const int* rad;
  const int* ang;
  const int* rad_off;
  const int* ang_off;
  int max_rad, max_ang, n;
  float rca2;              // the angular predicate of the neighbour search
  const float* g;
  const float4* shifts;    // the 16 scaled radial shifts
  const int* cut;
  float3* contrib;   // [n][max_ang]; [n][max_rad] after an overflow
  double* self;      // [n][3]
};

typedef double v4d __attribute__((ext_vector_type(4)));

// LDS of the wavefront (bytes, a multiple of 16): two float4 records per
// angular neighbour, their FP64 slots (which share space with the radial
// partial sums, 64 neighbours x 4 lanes x 2), the dE/dx row, and 64 x 8 bytes
// of exchange.
__host__ __device__ __forceinline__ size_t adj_slots_bytes(int max_ang) {
  const size_t slots = sizeof(double) * 3 * (size_t)max_ang, partial = sizeof(float2) * 4 * 64;
  return ((slots > partial ? slots : partial) + 15) & ~(size_t)15;
}
__host__ __device__ __forceinline__ size_t adj_lds(int max_ang, int stride) {
  return sizeof(float4) * 2 * (size_t)max_ang + adj_slots_bytes(max_ang) + sizeof(float) * (size_t)stride +
         sizeof(uint2) * 64;
}

// Sum over the 64 lanes with two FP64 matrix products by ones: the first
// sums over the four 16-lane rows (the product's K), the four accumulators of
// a lane then hold a quarter of the 16 sums, one quarter per row of lanes.
__device__ __forceinline__ double wave_sum_mfma(double v) {
  v4d d = v4d{0.0, 0.0, 0.0, 0.0};
  d = __builtin_amdgcn_mfma_f64_16x16x4f64(v, 1.0, d, 0, 0, 0);
  const double s = (d[0] + d[1]) + (d[2] + d[3]);
  d = v4d{0.0, 0.0, 0.0, 0.0};
  d = __builtin_amdgcn_mfma_f64_16x16x4f64(s, 1.0, d, 0, 0, 0);
  return d[0];
}

__device__ __forceinline__ int lanes_below(uint64_t m) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Place of i in j's radial list (its segment of species si), or -1.
__device__ __forceinline__ int radial_place(const BwdArgs& a, int S1, int i, int si, int j) {
  const int* jrow = a.rad + (int64_t)j * a.max_rad;
  int l = a.rad_off[(int64_t)j * S1 + si], h = a.rad_off[(int64_t)j * S1 + si + 1] - 1;
  while (l < h) {
    const int mid = (l + h) >> 1;
    if (jrow[mid] < i) l = mid + 1; else h = mid;
  }
  return l <= h && jrow[l] == i ? l : -1;
}

// LDS of a wavefront and what its triplet loop needs.
struct AdjWave {
  const float4 *G1, *G2;   // angular neighbours' records
  double *sx, *sy, *sz;    // their FP64 slots
  const float* gl;         // the centre's dE/dx row
  int lane;
};

// The sums over the shifts and sections that a triplet's derivatives need,
// with Ab_n = bs_n^(zeta - 1): SA = sum h_n A_n, SP and SQ = sum h_n Ab_n
// (cos, sin) and sdr = sum h'_n A_n.
struct AdjSums {
  float SA, SP, SQ, sdr;
};

// Derivatives of one triplet (inner neighbour j, outer k) to its two pair
// vectors.
__device__ __forceinline__ void adj_vectors(const DescParams& p, const float4& j1, const float4& j2, const float4& k1,
                                            const float4& k2, float cs, float qq, const AdjSums& t, float3* v,
                                            float3* w) {
#pragma clang fp contract(off)
  const float F = j2.x * k2.x;
  const float dTdc = F * (p.zeta * 0.95f) * fmaf(-qq, t.SQ, t.SP);
  const float hdr = F * (0.5f * p.c_sdr) * t.sdr;
  const float cj = dTdc * j2.z, ck = dTdc * k2.z;
  const float ej = fmaf(-cj, cs, fmaf(j2.y * k2.x, t.SA, hdr));
  const float ek = fmaf(-ck, cs, fmaf(j2.x * k2.y, t.SA, hdr));
  *v = make_float3(fmaf(cj, k1.x, ej * j1.x), fmaf(cj, k1.y, ej * j1.y), fmaf(cj, k1.z, ej * j1.z));
  *w = make_float3(fmaf(ck, j1.x, ek * k1.x), fmaf(ck, j1.y, ek * k1.y), fmaf(ck, j1.z, ek * k1.z));
}

__device__ __forceinline__ void adj_add(const AdjWave& wv, int u, float x, float y, float z) {
  unsafeAtomicAdd(wv.sx + u, (double)x);
  unsafeAtomicAdd(wv.sy + u, (double)y);
  unsafeAtomicAdd(wv.sz + u, (double)z);
}

// Triplets (k-major, j < k, a contiguous range per lane), the weights of each
// triplet's class read from LDS: j's total goes to its FP64 slot with an LDS
// atomic, k's is summed in registers and flushed when k changes.
template <int S>
__device__ __forceinline__ void adj_triplets(const AdjWave& wv, const DescParams& p, int na) {
  const int lane = wv.lane;
  const int T = na * (na - 1) / 2;
  const int r0 = (T * lane) >> 6, r1 = (T * (lane + 1)) >> 6;   // T < 2^15
  if (r0 >= r1) return;
  int j, k;
  pair_start(r0, true, 0, &j, &k);
  const float zm1 = p.zeta - 1.f;
  float kx = 0.f, ky = 0.f, kz = 0.f;   // running total of the current k
  float4 k1 = wv.G1[k], k2 = wv.G2[k];
  for (int r = r0; r < r1; ++r) {
#pragma clang fp contract(off)
    const float4 j1 = wv.G1[j], j2 = wv.G2[j];
    const int sj = __float_as_int(j2.w) & 3, sk = __float_as_int(k2.w) & 3;   // sj <= sk (rows are grouped by species)
    const int q = sj * (2 * S - 1 - sj) / 2 + sk;                             // class of (sj, sk)
    const float4* g4 = reinterpret_cast<const float4*>(wv.gl + S * kRadShifts + q * kAngShifts * kAngSects);
    const float cs = fmaf(j1.x, k1.x, fmaf(j1.y, k1.y, j1.z * k1.z));
    const float rb = j1.w + k1.w;
    float h[kAngSects] = {0.f, 0.f, 0.f, 0.f}, ht[kAngSects] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int m = 0; m < kAngShifts; ++m) {
      const float4 gv = g4[m];
      const float tt = rb - p.ang_shift_s[m];
      const float B = ex2(-(tt * tt)), tB = tt * B;
      h[0] = fmaf(gv.x, B, h[0]);
      h[1] = fmaf(gv.y, B, h[1]);
      h[2] = fmaf(gv.z, B, h[2]);
      h[3] = fmaf(gv.w, B, h[3]);
      ht[0] = fmaf(gv.x, tB, ht[0]);
      ht[1] = fmaf(gv.y, tB, ht[1]);
      ht[2] = fmaf(gv.z, tB, ht[2]);
      ht[3] = fmaf(gv.w, tB, ht[3]);
    }
    const float ct = 0.95f * cs;
    const float s2 = fmaf(-ct, ct, 1.f);
    const float ist = rsq(s2);
    const float st = s2 * ist;
    AdjSums t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int n = 0; n < kAngSects; ++n) {
      const float bs = fmaf(st, p.sin_sect[n], fmaf(ct, p.cos_sect[n], 1.f));
      const float Ab = ex2(zm1 * lg2(bs));   // bs^(zeta - 1)
      const float wn = h[n] * Ab;
      t.SA = fmaf(wn, bs, t.SA);
      t.SP = fmaf(wn, p.cos_sect[n], t.SP);
      t.SQ = fmaf(wn, p.sin_sect[n], t.SQ);
      t.sdr = fmaf(ht[n] * Ab, bs, t.sdr);
    }
    float3 v, w;
    adj_vectors(p, j1, j2, k1, k2, cs, ct * ist, t, &v, &w);
    adj_add(wv, j, v.x, v.y, v.z);
    kx += w.x;
    ky += w.y;
    kz += w.z;
    if (++j == k || r + 1 == r1) {   // k changes, or the range ends
      adj_add(wv, k, kx, ky, kz);
      kx = ky = kz = 0.f;
      j = 0;
      if (r + 1 < r1) {
        ++k;
        k1 = wv.G1[k];
        k2 = wv.G2[k];
      }
    }
  }
}

template <int S>
__global__ __launch_bounds__(64, 7) void k_desc_adj(BwdArgs a, DescParams p, Geometry geo) {
  constexpr int S1 = S + 1, P = S * (S + 1) / 2, D = kRadShifts * S + kAngShifts * kAngSects * P;
  extern __shared__ float4 smem_b[];
  const int lane = threadIdx.x;
  // angular neighbours: (u, r hq) and (fc sq_pref, dfc sq_pref, 1/r, slot * 4 + species)
  float4* G1 = smem_b;
  float4* G2 = G1 + a.max_ang;
  double* sx = reinterpret_cast<double*>(G2 + a.max_ang);   // FP64 slots of the angular neighbours
  double* sy = sx + a.max_ang;
  double* sz = sy + a.max_ang;
  float2* part = reinterpret_cast<float2*>(sx);             // radial partial sums (before the slots are used)
  float* gl = reinterpret_cast<float*>(reinterpret_cast<char*>(sx) + adj_slots_bytes(a.max_ang));   // dE/dx row
  uint2* ex = reinterpret_cast<uint2*>(gl + p.stride);
  const int i = a.order[xcd_block(blockIdx.x, gridDim.x)];
  const bool full = *a.cut != 0;
  const float4 pi = a.spos[i];
  const int si = __float_as_int(pi.w);
  const MinImage mi = min_image_at(geo, i);
  const int nr = a.rad_off[(int64_t)i * S1 + S];
  int ao[S1];   // angular segments of the species (uniform)
#pragma unroll
  for (int s = 0; s < S1; ++s) ao[s] = a.ang_off[(int64_t)i * S1 + s];
  const int* rrow = a.rad + (int64_t)i * a.max_rad;
  const int c4 = lane & 3;
  const float4 sh = a.shifts[c4];
  {
    const float4* g4 = reinterpret_cast<const float4*>(a.g + (int64_t)i * p.stride);
    float4* l4 = reinterpret_cast<float4*>(gl);
#pragma unroll
    for (int q = 0; q < D / 4; q += 64)
      if (D / 4 - q >= 64 || lane < D / 4 - q) l4[q + lane] = g4[q + lane];
  }

  // 1., 2. geometry and radial pairs, 64 neighbours at a time
  double fx = 0.0, fy = 0.0, fz = 0.0;   // this lane's share of the centre's radial total (FP32 terms)
  int na_seen = 0;
  for (int c0 = 0; c0 < nr; c0 += 64) {
    const int cnt = min(64, nr - c0);
    const bool valid = lane < cnt;
    const int j = valid ? rrow[c0 + lane] : i;
    const float4 pj = a.spos[j];
    float dx, dy, dz, r2;
    pair_d_exact(pi, pj, mi, &dx, &dy, &dz, &r2);
    const float ir = rsq(r2), r = r2 * ir;
    const int js = j * 4 + __float_as_int(pj.w);
    ex[lane] = make_uint2(__float_as_uint(r * p.sq_eta_r), (uint32_t)js);
    const bool in_a = valid && r2 < a.rca2;
    const uint64_t ma = __builtin_amdgcn_ballot_w64(in_a);
    const int u = na_seen + lanes_below(ma);
    na_seen += __popcll(ma);
    if (in_a && u < ao[S]) {
      const float arg = r * p.inv2rca;
      G1[u] = make_float4(dx * ir, dy * ir, dz * ir, r * p.hq_eta_a);
      G2[u] = make_float4(fmaf(0.5f, cos_rev(arg), 0.5f) * p.sq_pref, p.dfc_a * sin_rev(arg) * p.sq_pref, ir,
                          __int_as_float(js));
    }
    wave_sync();
    const int np = (cnt + 15) >> 4;
    float4 gj[4];
    uint2 en[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (q < np) {   // neighbours beyond cnt hold the centre itself; their sums are not read
        en[q] = ex[16 * q + (lane >> 2)];
        gj[q] = *reinterpret_cast<const float4*>(a.g + (uint64_t)(en[q].y >> 2) * (uint32_t)p.stride +
                                                 (si * kRadShifts + 4 * c4));
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (q < np) {
#pragma clang fp contract(off)
        const float4 gi = *reinterpret_cast<const float4*>(gl + (en[q].y & 3) * kRadShifts + 4 * c4);
        const float rs = __uint_as_float(en[q].x);
        const float t0 = rs - sh.x, t1 = rs - sh.y, t2 = rs - sh.z, t3 = rs - sh.w;
        const float b0 = (gi.x + gj[q].x) * ex2(-(t0 * t0)), b1 = (gi.y + gj[q].y) * ex2(-(t1 * t1));
        const float b2 = (gi.z + gj[q].z) * ex2(-(t2 * t2)), b3 = (gi.w + gj[q].w) * ex2(-(t3 * t3));
        part[(16 * q + (lane >> 2)) * 4 + c4] =
            make_float2((b0 + b1) + (b2 + b3), fmaf(b3, t3, fmaf(b2, t2, fmaf(b1, t1, b0 * t0))));
      }
    }
    wave_sync();
    if (valid) {
      const float4* q4 = reinterpret_cast<const float4*>(part + 4 * lane);
      const float4 v0 = q4[0], v1 = q4[1];
      float s0 = (v0.x + v0.z) + (v1.x + v1.z), s1 = (v0.y + v0.w) + (v1.y + v1.w);
      if (full && radial_place(a, S1, i, si, j) < 0) {   // j's cut-off list does not hold i: dE_i/dG alone
        s0 = s1 = 0.f;
#pragma unroll 1
        for (int k = 0; k < kRadShifts; ++k) {
          const float t = r * p.sq_eta_r - reinterpret_cast<const float*>(a.shifts)[k];
          const float b = gl[(js & 3) * kRadShifts + k] * ex2(-(t * t));
          s0 += b;
          s1 = fmaf(b, t, s1);
        }
      }
      const float arg = r * p.inv2rc;
      const float fc = fmaf(0.5f, cos_rev(arg), 0.5f);
      const float w = fmaf(p.dfc_r * sin_rev(arg), s0, p.c1_rad * fc * s1) * ir;
      fx += (double)(w * dx);
      fy += (double)(w * dy);
      fz += (double)(w * dz);
    }
    wave_sync();
  }

  // 3. angular triplets
  const int na = min(ao[S], na_seen);   // (equal unless the radial list overflowed)
  for (int u = lane; u < na; u += 64) sx[u] = sy[u] = sz[u] = 0.0;
  wave_sync();
  adj_triplets<S>(AdjWave{G1, G2, sx, sy, sz, gl, lane}, p, na);
  wave_sync();
  // 4. each angular neighbour's total goes to the centre's place in that
  // neighbour's angular list: the entry equal to i in the segment of i's
  // species, 16 entries a round by two lanes with two 16-byte loads each.
  // Entries outside the segment cannot equal i (other species), or are left
  // over from an earlier call beyond the list's end: the first match is the
  // true one.
  if (!full) {
    const bool wide = (a.max_ang & 3) == 0;   // rows start on 16-byte boundaries
    for (int u0 = 0; u0 < na; u0 += 32) {
      const int u = u0 + (lane >> 1);
      if (u < na) {
        const uint32_t j = (uint32_t)__float_as_int(G2[u].w) >> 2;
        const int* jrow = a.ang + (uint64_t)j * (uint32_t)a.max_ang;
        const int* jo = a.ang_off + (uint64_t)j * S1 + si;
        const int lo = jo[0], hi = jo[1];
        int pos = INT_MAX;
        if (wide) {
          for (int e = (lo & ~3) + 8 * (lane & 1); e < hi && pos == INT_MAX; e += 16) {
            const int4 q0 = *reinterpret_cast<const int4*>(jrow + e);
            const int4 q1 = e + 4 < hi ? *reinterpret_cast<const int4*>(jrow + e + 4) : make_int4(-1, -1, -1, -1);
            const int w[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
#pragma unroll
            for (int c = 7; c >= 0; --c) pos = w[c] == i ? e + c : pos;
          }
        } else {
          for (int e = lo + (lane & 1); e < hi; e += 2)
            if (jrow[e] == i) pos = e;
        }
        if (pos < hi)
          a.contrib[(uint64_t)j * (uint32_t)a.max_ang + pos] =
              make_float3((float)-sx[u], (float)-sy[u], (float)-sz[u]);
      }
    }
  } else {
    int seen = 0;
    for (int c0 = 0; c0 < nr; c0 += 64) {
      const bool valid = c0 + lane < nr;
      const int j = valid ? rrow[c0 + lane] : i;
      const bool in_a = valid && pair_r2_exact(pi, a.spos[j], mi) < a.rca2;
      const uint64_t ma = __builtin_amdgcn_ballot_w64(in_a);
      const int u = seen + lanes_below(ma);
      seen += __popcll(ma);
      const int pos = valid ? radial_place(a, S1, i, si, j) : -1;
      const bool any = in_a && u < na;
      if (pos >= 0)
        a.contrib[(int64_t)j * a.max_rad + pos] =
            any ? make_float3((float)-sx[u], (float)-sy[u], (float)-sz[u]) : make_float3(0.f, 0.f, 0.f);
      else if (valid)   // j does not see the centre: nothing comes back from it
        a.contrib[(int64_t)i * a.max_rad + c0 + lane] = make_float3(0.f, 0.f, 0.f);
    }
  }
  // 5. the centre's own total
  double tx = fx, ty = fy, tz = fz;
  for (int u = lane; u < na; u += 64) {
    tx += sx[u];
    ty += sy[u];
    tz += sz[u];
  }
  tx = wave_sum_mfma(tx);
  ty = wave_sum_mfma(ty);
  tz = wave_sum_mfma(tz);
  if (lane < 3) a.self[3 * (int64_t)i + lane] = lane == 0 ? tx : lane == 1 ? ty : tz;
}

// FP64 energy reduction blocks, appended to the gather's grid (one launch for
// both): with per-tile partials from the network kernel (a single system)
// one block sums them; otherwise block `sys` sums that system's atomic
// energies over its species buckets.  Fixed order, hence deterministic.
struct EnergyArgs {
  const double* part;      // per-tile partials, or null
  const float* e;          // atomic energies in sorted order
  const int* bin_start;    // species buckets [s * n_bins, (s + 1) * n_bins)
  int n_bins, S, tile_rows;
  int mixed;               // the network's narrow species used 16-atom tiles
  int sums;                // partials of summed ensemble members (k_mlp_sum), else 0
  int empty;               // no atoms: the energies are zero (the buckets are not read)
  double* out;
  int accumulate;
  int* status;
};

__device__ __forceinline__ void energy_block(const EnergyArgs& ea, int sys) {
  __shared__ double red[kBlock];
  double acc = 0.0;
  if (ea.empty) {
  } else if (ea.part != nullptr) {
    const int narrow = ea.mixed ? narrow_species(ea.bin_start, ea.S, ea.n_bins) : -1;
    int tiles = ea.sums;
    for (int s = 0; s < ea.S && ea.sums == 0; ++s) {
      const int rows = s == narrow ? 16 : ea.tile_rows;
      tiles += (ea.bin_start[(s + 1) * ea.n_bins] - ea.bin_start[s * ea.n_bins] + rows - 1) / rows;
    }
    // eight loads in flight per thread, added in the same order as one at a time
    for (int t0 = threadIdx.x; t0 < tiles; t0 += 8 * kBlock) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = t0 + u * kBlock < tiles ? ea.part[t0 + u * kBlock] : 0.0;
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (t0 + u * kBlock < tiles) acc += v[u];
    }
  } else {
    for (int s = 0; s < ea.S; ++s) {
      const int b0 = ea.bin_start[s * ea.n_bins + sys], b1 = ea.bin_start[s * ea.n_bins + sys + 1];
      for (int t0 = b0 + threadIdx.x; t0 < b1; t0 += 8 * kBlock) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = t0 + u * kBlock < b1 ? ea.e[t0 + u * kBlock] : 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (t0 + u * kBlock < b1) acc += (double)v[u];
      }
    }
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = kBlock / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double v = red[0];
    if (!isfinite(v)) atomicOr(ea.status, kStatusNonFinite);
    ea.out[sys] = ea.accumulate ? ea.out[sys] + v : v;
  }
}

// F_atom += self + sum over the atom's angular list entries (its radial ones
// after a list overflow, see k_desc_adj), and with the MM channel its partials
// of k_mm_bwd (FP64): 16 lanes per atom, each summing a strided part of the
// row, then a shuffle tree.
// With `assign` the sum overwrites F_atom (every row of the output is an NNP
// atom and the call does not accumulate), which saves clearing it first.
// Blocks from gather_blocks on reduce the energies instead.
__global__ __launch_bounds__(kBlock) void k_force_gather(const float3* __restrict__ contrib,
                                                         const double* __restrict__ self,
                                                         const int* __restrict__ rad_off,
                                                         const int* __restrict__ ang_off,
                                                         const int* __restrict__ cut,
                                                         const int* __restrict__ slot_atom, int n, int S,
                                                         int max_rad, int max_ang, double* __restrict__ forces,
                                                         double* __restrict__ link_forces, int assign,
                                                         int gather_blocks, EnergyArgs ea,
                                                         const float* __restrict__ mm_part, int mm_blocks) {
  // the energy blocks come first, so that their serial reduction runs beside
  // the gather instead of after it
  const int energy_blocks = (int)gridDim.x - gather_blocks;
  if ((int)blockIdx.x < energy_blocks) {
    energy_block(ea, (int)blockIdx.x);
    return;
  }
  const int gid = ((int)blockIdx.x - energy_blocks) * blockDim.x + threadIdx.x;
  const int i = gid >> 4;
  const int sub = gid & 15;
  double fx = 0.0, fy = 0.0, fz = 0.0;
  if (i < n) {
    const bool full = *cut != 0;
    const int cnt = (full ? rad_off : ang_off)[(int64_t)i * (S + 1) + S];
    const float3* row = contrib + (int64_t)i * (full ? max_rad : max_ang);   // 16 lanes read 192 contiguous bytes
    for (int t = sub; t < cnt; t += 16) {
      const float3 v = row[t];
      fx += v.x; fy += v.y; fz += v.z;
    }
    const float* mp = mm_part + (int64_t)i * 3 * mm_blocks;   // MM channel: partials of the three components
#pragma unroll 4
    for (int b = sub; b < mm_blocks; b += 16) {
      fx += (double)mp[b];
      fy += (double)mp[b + mm_blocks];
      fz += (double)mp[b + 2 * mm_blocks];
    }
  }
#pragma unroll
  for (int off = 8; off >= 1; off >>= 1) {
    fx += __shfl_xor(fx, off, 64);
    fy += __shfl_xor(fy, off, 64);
    fz += __shfl_xor(fz, off, 64);
  }
  if (i < n && sub == 0) {
    const int a = slot_atom[i];   // a < 0: link atom -1 - a
    double* f = a >= 0 ? forces + 3 * (int64_t)a : link_forces + 3 * (int64_t)(-1 - a);
    fx += self[3 * (int64_t)i];
    fy += self[3 * (int64_t)i + 1];
    fz += self[3 * (int64_t)i + 2];
    if (!assign) {
      fx += f[0];
      fy += f[1];
      fz += f[2];
    }
    f[0] = fx;
    f[1] = fy;
    f[2] = fz;
  }
}

// Chain rule for link atoms (eq. 4): r_L = r_ML + d u/|u|, u = r_MM - r_ML, so
// F_MM += (d/|u|)(F_L - (F_L.u^) u^) and F_ML += F_L - (d/|u|)(F_L - (F_L.u^) u^).
// FP64 atomics: an ML atom may carry several links.
__global__ __launch_bounds__(kBlock) void k_link_redistribute(const double* __restrict__ link_forces,
                                                              const int* __restrict__ ml, const int* __restrict__ mm,
                                                              int n_links, float d, const float* __restrict__ pos,
                                                              Geometry g, double* __restrict__ forces) {
  const int l = blockIdx.x * blockDim.x + threadIdx.x;
  if (l >= n_links) return;
  const int a = ml[l], b = mm[l];
  double ux = (double)pos[3 * (int64_t)b] - pos[3 * (int64_t)a];
  double uy = (double)pos[3 * (int64_t)b + 1] - pos[3 * (int64_t)a + 1];
  double uz = (double)pos[3 * (int64_t)b + 2] - pos[3 * (int64_t)a + 2];
  if (g.periodic) {
    ux -= g.box[0] * rint(ux / g.box[0]);
    uy -= g.box[1] * rint(uy / g.box[1]);
    uz -= g.box[2] * rint(uz / g.box[2]);
  }
  const double inv = 1.0 / sqrt(ux * ux + uy * uy + uz * uz);
  ux *= inv; uy *= inv; uz *= inv;
  const double fx = link_forces[3 * l], fy = link_forces[3 * l + 1], fz = link_forces[3 * l + 2];
  const double s = (double)d * inv;
  const double fu = fx * ux + fy * uy + fz * uz;
  const double px = s * (fx - fu * ux), py = s * (fy - fu * uy), pz = s * (fz - fu * uz);
  unsafeAtomicAdd(forces + 3 * (int64_t)b + 0, px);
  unsafeAtomicAdd(forces + 3 * (int64_t)b + 1, py);
  unsafeAtomicAdd(forces + 3 * (int64_t)b + 2, pz);
  unsafeAtomicAdd(forces + 3 * (int64_t)a + 0, fx - px);
  unsafeAtomicAdd(forces + 3 * (int64_t)a + 1, fy - py);
  unsafeAtomicAdd(forces + 3 * (int64_t)a + 2, fz - pz);
}

}  // namespace

hipError_t launch_link_redistribute(nnp_model& m, const float* pos, double* forces, hipStream_t st) {
  if (m.n_links_dev == 0) return hipSuccess;
  hipLaunchKernelGGL(k_link_redistribute, dim3((m.n_links_dev + kBlock - 1) / kBlock), dim3(kBlock), 0, st,
                     m.d_link_F, m.d_link_ml, m.d_link_mm, m.n_links_dev, m.link_d, pos, m.geo, forces);
  return hipGetLastError();
}

// Forward descriptor variants: 0 = one wavefront per atom, 1 = one 16-lane
// row per atom, 2 = one 8-lane row per atom (fewer idle lanes, half the
// wavefronts), 3 and 4 = the pool kernel with two and four atoms per
// wavefront (3: with one while that still leaves lanes idle, see
// launch_descriptor_fwd).
//
// The default.  With four elements a centre has ten classes of few pairs, which
// rows of lanes walk one after the other: the pool is faster at every size (us,
// variant 1 -> 3): 60 atoms 21.0 -> 11.3, 1,000 atoms 33.8 -> 17, 25,000 atoms
// 104 -> 58.  With two elements the line is drawn by what
// there is to hide latency with: up to 24 atoms per CU the pool's even split
// is faster (192 atoms 14.7 -> 12.8, 5,400 atoms 21.5 -> 18.1), in between
// the rows (12,288 atoms 21.4, pool 22.0 to 23.7), and from 72 atoms per CU
// on four pooled atoms per wavefront waste the fewest lanes (27,000 atoms
// 39.1 -> 36.0, 87,000 atoms 95.1 -> 87.6), while the angular capacity leaves
// five of their workgroups per CU: 98,304 atoms with capacities of 64, 96, 112,
// 128 and 256 rows 106, 108, 113, 113 and 155, pool 95, 102, 112, 130 and 296.
// The BF16 form rounds the descriptors to eight bits; there another order of
// summation turns single roundings over and moves forces by 1e-4, no nearer to
// float64 and no further from it.  Its default stays the row kernel at every
// size, so that a program that asks for nothing keeps its results; nnp_autotune
// is asked for, and chooses among all variants (261,000 atoms 970 -> 935 us per
// call with the pool).
int descriptor_variant(const nnp_model& m, int n) {
  const int v = stage_variant(m, kTuneDescriptor, n);
  if (v >= 0) return v;
  if (m.prec == NNP_BF16) return 1;
  if (m.S > 2) return 3;
  return n <= 24 * m.n_cu ? 3 : n >= 72 * m.n_cu && m.max_ang <= 96 ? 4 : 1;
}

hipError_t launch_descriptor_fwd(nnp_model& m, int n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  FwdArgs a;
  a.order = m.d_order;
  a.spos = m.d_spos;
  a.rad = m.d_nbr_rad;
  a.ang = m.d_nbr_ang;
  a.rad_off = m.d_rad_off;
  a.ang_off = m.d_ang_off;
  a.max_rad = m.max_rad;
  a.max_ang = m.max_ang;
  a.n = n;
  a.x = m.d_x;
  const int v = descriptor_variant(m, n);
  if (v == 3 || v == 4) {
    // Up to two wavefronts of one atom per SIMD run side by side anyway, and
    // one atom's work is the shorter chain: 300 H/C/N/O atoms 20 -> 14 us per
    // descriptor, 900 atoms of water 13.3 -> 12.2; 6,400 H/C/N/O atoms 29.4
    // -> 30.2, 3,000 of water 15.5 -> 16.1.
    const int aw = v == 4 ? 4 : n <= 8 * m.n_cu ? 1 : 2;
    const size_t area = (std::max((size_t)aw * m.max_ang * 5, (size_t)64 * kPoolPitch) + 3) & ~(size_t)3;
    const size_t lds = 4 * sizeof(float) * (area + 64);   // four wavefronts, each with its own slice
    const unsigned blocks = (unsigned)((n + 4 * aw - 1) / (4 * aw));
    if (aw == 1)
      hipLaunchKernelGGL(k_desc_fwd_pool<1>, dim3(blocks), dim3(256), lds, st, a, m.dp, m.geo);
    else if (aw == 2)
      hipLaunchKernelGGL(k_desc_fwd_pool<2>, dim3(blocks), dim3(256), lds, st, a, m.dp, m.geo);
    else
      hipLaunchKernelGGL(k_desc_fwd_pool<4>, dim3(blocks), dim3(256), lds, st, a, m.dp, m.geo);
  } else if (v == 1) {
    const size_t lds = (sizeof(float4) + sizeof(float)) * 16 * (size_t)m.max_ang;
    hipLaunchKernelGGL(k_desc_fwd_rows<16>, dim3((n + 15) / 16), dim3(256), lds, st, a, m.dp, m.geo);
  } else if (v == 2) {
    const size_t lds = (sizeof(float4) + sizeof(float)) * 32 * (size_t)m.max_ang;
    hipLaunchKernelGGL(k_desc_fwd_rows<8>, dim3((n + 31) / 32), dim3(256), lds, st, a, m.dp, m.geo);
  } else {
    const size_t lds = sizeof(float) * (64 * (size_t)kPartStride + 5 * (size_t)m.max_ang);
    hipLaunchKernelGGL(k_desc_fwd, dim3(n), dim3(64), lds, st, a, m.dp, m.geo);
  }
  return hipGetLastError();
}

// The adjoint has one kernel; variants 0 to 2 are accepted and run it.
int adjoint_variant(const nnp_model& m, int n) {
  const int v = stage_variant(m, kTuneAdjoint, n);
  return v >= 0 ? v : 0;
}

hipError_t launch_descriptor_bwd(nnp_model& m, int n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  BwdArgs a;
  a.order = m.d_order;
  a.spos = m.d_spos;
  a.rad = m.d_nbr_rad;
  a.ang = m.d_nbr_ang;
  a.rad_off = m.d_rad_off;
  a.ang_off = m.d_ang_off;
  a.max_rad = m.max_rad;
  a.max_ang = m.max_ang;
  a.n = n;
  a.rca2 = m.dp.rc_ang * m.dp.rc_ang;
  a.g = m.d_g;
  a.shifts = reinterpret_cast<const float4*>(m.d_shifts);
  a.cut = m.d_cut;
  a.contrib = m.d_contrib;
  a.self = m.d_self;
  // one wavefront per workgroup: several, sharing nothing, measured slower
  // (261,000 atoms 456, 458 and 465 us for one, two and four)
  const size_t lds = adj_lds(m.max_ang, m.stride);
  switch (m.S) {
    case 2: hipLaunchKernelGGL(k_desc_adj<2>, dim3(n), dim3(64), lds, st, a, m.dp, m.geo); break;
    case 4: hipLaunchKernelGGL(k_desc_adj<4>, dim3(n), dim3(64), lds, st, a, m.dp, m.geo); break;
    default: return hipErrorInvalidValue;   // nnp_create accepts two- and four-species models
  }
  return hipGetLastError();
}

hipError_t launch_force_gather(nnp_model& m, int n, int n_mm, double* forces, int assign, double* energies,
                               int n_sys, int accumulate, hipStream_t st) {
  EnergyArgs ea;
  const bool single = m.geo.periodic || m.geo.n_bins == 1;
  ea.part = single ? m.d_part : nullptr;
  ea.e = m.d_e;
  ea.bin_start = m.d_bin_start;
  ea.n_bins = m.geo.n_bins;
  ea.S = m.S;
  ea.tile_rows = 16 * m.mlp_cols;
  ea.mixed = m.mlp_mixed;
  ea.sums = m.mlp_sums;
  ea.empty = n == 0;
  ea.out = energies;
  ea.accumulate = accumulate;
  ea.status = m.d_status;
  const int gather_blocks = (int)((16 * (int64_t)n + kBlock - 1) / kBlock);
  const int energy_blocks = single ? 1 : n_sys;
  hipLaunchKernelGGL(k_force_gather, dim3((unsigned)(gather_blocks + energy_blocks)), dim3(kBlock), 0, st,
                     m.d_contrib, m.d_self, m.d_rad_off, m.d_ang_off, m.d_cut, m.d_slot_atom, n, m.S, m.max_rad,
                     m.max_ang, forces, m.d_link_F, assign, gather_blocks, ea, m.d_mm_part,
                     m.extra && n_mm > 0 ? mm_partial_blocks(m, n, n_mm) : 0);
  return hipGetLastError();
}

}  // namespace nnp
