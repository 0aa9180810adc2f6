// Cell-list neighbour search over the atoms of the index group (Methods: the
// interface's ML subsystem): binning, a stable counting sort by
// key = species * n_bins + bin, and per-atom neighbour lists grouped by
// species; also the lists built from a caller's pair list.  A bin is a cell of the periodic box, or a whole system in batched
// mode (open systems small enough for an all-pairs scan per system).
//
// The binning and the distance predicate are integer-exact functions of the
// FP32 inputs: every operation below is a single IEEE FP32 operation in a
// fixed order with floating-point contraction disabled, so an FP32 reference
// that performs the same operations reproduces the bins, the permutation and
// the neighbour sets bit for bit.
#include <algorithm>

#include <cmath>

#include "nnp_internal.h"

namespace nnp {
namespace {

constexpr int kBlock = 256;

// Position of NNP-local atom t: a system atom, or a link atom placed on its
// cut bond (eq. 4; bond vector under the minimum image when periodic).
__device__ __forceinline__ float3 nnp_position(const float* __restrict__ pos, int a, const LinkArgs& L,
                                               const Geometry& g) {
  if (a >= 0) return make_float3(pos[3 * (int64_t)a], pos[3 * (int64_t)a + 1], pos[3 * (int64_t)a + 2]);
  const int l = -1 - a;
  const int ml = L.ml[l], mm = L.mm[l];
  float3 p = make_float3(pos[3 * (int64_t)ml], pos[3 * (int64_t)ml + 1], pos[3 * (int64_t)ml + 2]);
  float ux = pos[3 * (int64_t)mm] - p.x, uy = pos[3 * (int64_t)mm + 1] - p.y, uz = pos[3 * (int64_t)mm + 2] - p.z;
  if (g.periodic) {
    ux -= g.box[0] * rintf(ux * g.inv_box[0]);
    uy -= g.box[1] * rintf(uy * g.inv_box[1]);
    uz -= g.box[2] * rintf(uz * g.inv_box[2]);
  }
  const float s = L.d / sqrtf(ux * ux + uy * uy + uz * uz);
  return make_float3(p.x + s * ux, p.y + s * uy, p.z + s * uz);
}

// Counters of a pair list's radial entries, one per slot, at the start of the
// slot's row of force contributions (unused until the adjoint, and a cache
// line of its own): 52,000 atomics on counters that shared 29 lines took 15
// us, spread out they take 6.  Without a pair list `at` is null.
struct PairCount {
  int* at;
  int stride;
};

inline PairCount pair_count(const nnp_model& m) {
  return PairCount{reinterpret_cast<int*>(m.d_contrib), (int)(sizeof(float3) / sizeof(int)) * m.max_rad};
}

// Bin of one position in the periodic grid.
__device__ __forceinline__ int cell_of(float x, float y, float z, const Geometry& g) {
#pragma clang fp contract(off)
  float c[3] = {x, y, z};
  int ci[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    float t = c[k] * g.inv_box[k];
    float f = floorf(t);
    float fl = f * g.box[k];
    float w = c[k] - fl;
    float sc = w * g.cell_scale[k];
    int q = (int)floorf(sc);
    q = q < 0 ? 0 : q;
    q = q > g.nc[k] - 1 ? g.nc[k] - 1 : q;
    ci[k] = q;
  }
  return (ci[0] * g.nc[1] + ci[1]) * g.nc[2] + ci[2];
}

__global__ __launch_bounds__(kBlock) void k_stage(const float* __restrict__ pos, int n,
                                                  const int* __restrict__ idx,
                                                  const int* __restrict__ sigma,
                                                  const int* __restrict__ sys, Geometry g, LinkArgs L,
                                                  int* __restrict__ key, int* __restrict__ rank,
                                                  float4* __restrict__ stg,
                                                  int* __restrict__ bin_count, int* __restrict__ status,
                                                  int* __restrict__ cut) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  if (t == 0) *cut = 0;
  const float3 p = nnp_position(pos, idx[t], L, g);
  float x = p.x, y = p.y, z = p.z;
  if (g.periodic) stg[t] = make_float4(x, y, z, __int_as_float(sigma[t]));   // for the bin sort
  int bin;
  if (!(isfinite(x) && isfinite(y) && isfinite(z))) {
    atomicOr(status, kStatusNonFinite);
    bin = g.periodic ? 0 : sys[t];
  } else {
    bin = g.periodic ? cell_of(x, y, z, g) : sys[t];
  }
  int k = sigma[t] * g.n_bins + bin;
  key[t] = k;
  if (g.periodic) {
    rank[t] = atomicAdd(&bin_count[k], 1);   // arrival order among the atoms of the key
    return;
  }
  // Open systems (bins are systems): a system's atoms are contiguous, so a
  // wavefront holds few distinct keys and per-atom atomics would queue on the
  // same few counters.  One atomic per distinct key and wavefront instead (the
  // system ranking places the atoms itself; no arrival rank is needed).
  const int lane = threadIdx.x & 63;
  uint64_t todo = __builtin_amdgcn_ballot_w64(true);
  while (todo != 0) {
    const int leader = __builtin_ctzll(todo);
    const int lk = __builtin_amdgcn_readlane(k, leader);
    const uint64_t same = __builtin_amdgcn_ballot_w64(k == lk);
    if (lane == leader) atomicAdd(&bin_count[lk], (int)__popcll(same));
    todo &= ~same;
  }
}

// Exclusive scans of the bin histogram by one workgroup.
//   start: species-major order (key = species * n_bins + bin), the slot
//     order of the sorted arrays;
//   cmstart[bin * S + species]: bin-major order, the order in which the
//     per-atom kernels visit the slots (all species of a cell or system
//     together, so neighbouring atoms are processed close in time).
// Chunks of kScanThreads * PER entries are staged through LDS so that every global
// load and store is coalesced (per-thread runs of consecutive entries read
// straight from memory are several times slower); each thread scans
// PER consecutive entries of the staged chunk, PER being the smallest power
// of two for which one chunk holds the whole histogram (at most 16; larger
// histograms go to the many-workgroup scan, k_scan_part and k_scan_fin).  Sizing the chunk to the histogram
// matters: one workgroup does all of this work, and with 16 entries per
// thread a 1,024-bin scan took 6.8 us.  The histogram itself is left as it
// is (the bin sort clears it).
constexpr int kScanThreads = 1024;
constexpr int kScanPerMax = 16;
constexpr int kScanChunk = kScanThreads * kScanPerMax;   // largest chunk

// LDS index of chunk entry i: one pad word after every PER entries, so the
// per-thread runs start in different banks (stride PER + 1 is odd).
template <int PER>
__device__ __forceinline__ int scan_pad(int i) { return PER == 1 ? i : i + i / PER; }
template <int PER>
constexpr int scan_lds_words() { return PER == 1 ? kScanThreads : kScanThreads * (PER + 1); }

// Exclusive prefix of v over the workgroup (thread order); *total receives the sum.
__device__ __forceinline__ int block_exclusive(int v, int* wsum, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int inc = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int u = __shfl_up(inc, off, 64);
    if (lane >= off) inc += u;
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  if (wave == 0) {
    const int w = lane < kScanThreads / 64 ? wsum[lane] : 0;
    int wi = w;
#pragma unroll
    for (int off = 1; off < kScanThreads / 64; off <<= 1) {
      const int u = __shfl_up(wi, off, 64);
      if (lane >= off) wi += u;
    }
    if (lane < kScanThreads / 64) wsum[kScanThreads / 64 + lane] = wi - w;
    if (lane == kScanThreads / 64 - 1) wsum[2 * (kScanThreads / 64)] = wi;
  }
  __syncthreads();
  const int ex = wsum[kScanThreads / 64 + wave] + inc - v;
  *total = wsum[2 * (kScanThreads / 64)];
  __syncthreads();   // wsum is reused by the next call
  return ex;
}

// Scan of the staged chunk buf[0 .. kScanThreads * PER) in place (exclusive, plus carry).
template <int PER>
__device__ __forceinline__ void scan_chunk(int* buf, int* wsum, int* carry) {
  int v[PER];
  int sum = 0;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    v[u] = buf[scan_pad<PER>(threadIdx.x * PER + u)];
    sum += v[u];
  }
  int total;
  int run = block_exclusive(sum, wsum, &total) + *carry;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    buf[scan_pad<PER>(threadIdx.x * PER + u)] = run;
    run += v[u];
  }
  *carry += total;
  __syncthreads();
}

template <int PER>
__global__ __launch_bounds__(kScanThreads) void k_scan(const int* __restrict__ count, int* __restrict__ start,
                                                       int* __restrict__ cmstart, int S, int n_bins) {
  __shared__ int wsum[2 * (kScanThreads / 64) + 1];
  __shared__ int buf[scan_lds_words<PER>()];
  __shared__ int bufc[scan_lds_words<PER>()];
  const int nb = S * n_bins;
  int carry = 0;
  if (nb <= kScanThreads * PER) {
    // one chunk: the histogram is read once and both scans run from LDS
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int i = u * kScanThreads + threadIdx.x;
      bufc[scan_pad<PER>(i)] = i < nb ? count[i] : 0;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int b = u * kScanThreads + threadIdx.x;
      int t = 0;
#pragma unroll
      for (int s = 0; s < kMaxSpecies; ++s)
        if (s < S && b < n_bins) t += bufc[scan_pad<PER>(s * n_bins + b)];
      buf[scan_pad<PER>(b)] = t;
    }
    __syncthreads();
    scan_chunk<PER>(buf, wsum, &carry);
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int b = u * kScanThreads + threadIdx.x;
      if (b < n_bins) {
        int r = buf[scan_pad<PER>(b)];
#pragma unroll
        for (int s = 0; s < kMaxSpecies; ++s)
          if (s < S) {
            cmstart[b * S + s] = r;
            r += bufc[scan_pad<PER>(s * n_bins + b)];
          }
      }
    }
    __syncthreads();
    carry = 0;
    scan_chunk<PER>(bufc, wsum, &carry);
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int i = u * kScanThreads + threadIdx.x;
      if (i < nb) start[i] = bufc[scan_pad<PER>(i)];
    }
    if (threadIdx.x == 0) start[nb] = carry;
  }
}

// Histograms beyond one chunk: the same two scans over many workgroups, in
// two launches.  Workgroup w < ca takes species-major chunk w (counts), the
// others bin-major chunk w - ca (per-bin totals over the species); each chunk
// holds kScanPartChunk = kScanThreads * 4 entries.  k_scan_part writes the
// chunk totals, k_scan_fin scans each chunk again starting from the sum of
// the earlier chunks of its order.  One workgroup scanning 35,152 bins took
// 38 us.
constexpr int kScanPartPer = kScanPartChunk / kScanThreads;
static_assert(kScanPartPer * kScanThreads == kScanPartChunk, "whole entries per thread");

__device__ __forceinline__ int scan_entry(const int* __restrict__ count, bool bin_major, int e, int S, int n_bins) {
  if (!bin_major) return count[e];
  int t = 0;
#pragma unroll
  for (int s = 0; s < kMaxSpecies; ++s)
    if (s < S) t += count[s * n_bins + e];
  return t;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_part(const int* __restrict__ count, int S, int n_bins,
                                                            int ca, int* __restrict__ part) {
  __shared__ int wsum[2 * (kScanThreads / 64) + 1];
  const bool bin_major = (int)blockIdx.x >= ca;
  const int c = bin_major ? (int)blockIdx.x - ca : (int)blockIdx.x;
  const int len = bin_major ? n_bins : S * n_bins;
  int sum = 0;
#pragma unroll
  for (int u = 0; u < kScanPartPer; ++u) {
    const int e = c * kScanPartChunk + u * kScanThreads + threadIdx.x;
    if (e < len) sum += scan_entry(count, bin_major, e, S, n_bins);
  }
  int total;
  block_exclusive(sum, wsum, &total);
  if (threadIdx.x == 0) part[blockIdx.x] = total;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_fin(const int* __restrict__ count, int* __restrict__ start,
                                                           int* __restrict__ cmstart, int S, int n_bins, int ca,
                                                           const int* __restrict__ part) {
  __shared__ int wsum[2 * (kScanThreads / 64) + 1];
  __shared__ int buf[scan_lds_words<kScanPartPer>()];
  __shared__ int s_carry;
  const bool bin_major = (int)blockIdx.x >= ca;
  const int c = bin_major ? (int)blockIdx.x - ca : (int)blockIdx.x;
  const int first = bin_major ? ca : 0;
  const int nb = S * n_bins, len = bin_major ? n_bins : nb;
  if (threadIdx.x < 64) {   // the earlier chunks of this order
    int v = 0;
    for (int k = first + (int)threadIdx.x; k < (int)blockIdx.x; k += 64) v += part[k];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    if (threadIdx.x == 0) s_carry = v;
  }
  const int c0 = c * kScanPartChunk;
#pragma unroll
  for (int u = 0; u < kScanPartPer; ++u) {
    const int i = u * kScanThreads + threadIdx.x;
    buf[scan_pad<kScanPartPer>(i)] = c0 + i < len ? scan_entry(count, bin_major, c0 + i, S, n_bins) : 0;
  }
  __syncthreads();
  int carry = s_carry;
  scan_chunk<kScanPartPer>(buf, wsum, &carry);
#pragma unroll
  for (int u = 0; u < kScanPartPer; ++u) {
    const int i = u * kScanThreads + threadIdx.x, e = c0 + i;
    if (e < len) {
      int r = buf[scan_pad<kScanPartPer>(i)];
      if (bin_major) {
#pragma unroll
        for (int s = 0; s < kMaxSpecies; ++s)
          if (s < S) {
            cmstart[e * S + s] = r;
            r += count[s * n_bins + e];
          }
      } else {
        start[e] = r;
      }
    }
  }
  if (!bin_major && c0 + kScanPartChunk >= len && threadIdx.x == 0) start[nb] = carry;
}

// Provisional slots: start of the key plus the atom's arrival rank.
__global__ __launch_bounds__(kBlock) void k_scatter(const int* __restrict__ key, const int* __restrict__ rank, int n,
                                                    const int* __restrict__ start, int* __restrict__ tmp) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  tmp[start[key[t]] + rank[t]] = t;
}

// Scan and scatter in one launch, for histograms of at most one chunk: every
// workgroup stages the histogram in LDS and scans it itself (a few KB to a
// few tens of KB from L2, cheaper than a kernel boundary); workgroup 0 also
// writes both scans for the later kernels.  Then each thread places one
// atom at start[key] + rank.
template <int PER>
__global__ __launch_bounds__(kScanThreads) void k_scan_scatter(const int* __restrict__ count, int* __restrict__ start,
                                                               int* __restrict__ cmstart, int S, int n_bins,
                                                               const int* __restrict__ key,
                                                               const int* __restrict__ rank, int n,
                                                               int* __restrict__ tmp) {
  __shared__ int wsum[2 * (kScanThreads / 64) + 1];
  __shared__ int buf[scan_lds_words<PER>()];
  __shared__ int bufc[scan_lds_words<PER>()];
  const int nb = S * n_bins;   // <= kScanThreads * PER (checked by the launcher)
  const int t = blockIdx.x * kScanThreads + threadIdx.x;
  const int k = t < n ? key[t] : 0;
  const int rk = t < n ? rank[t] : 0;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int i = u * kScanThreads + threadIdx.x;
    bufc[scan_pad<PER>(i)] = i < nb ? count[i] : 0;
  }
  __syncthreads();
  int carry = 0;
  if (blockIdx.x == 0) {   // bin-major starts (workgroup-uniform branch)
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int b = u * kScanThreads + threadIdx.x;
      int tot = 0;
#pragma unroll
      for (int s = 0; s < kMaxSpecies; ++s)
        if (s < S && b < n_bins) tot += bufc[scan_pad<PER>(s * n_bins + b)];
      buf[scan_pad<PER>(b)] = tot;
    }
    __syncthreads();
    scan_chunk<PER>(buf, wsum, &carry);
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int b = u * kScanThreads + threadIdx.x;
      if (b < n_bins) {
        int r = buf[scan_pad<PER>(b)];
#pragma unroll
        for (int s = 0; s < kMaxSpecies; ++s)
          if (s < S) {
            cmstart[b * S + s] = r;
            r += bufc[scan_pad<PER>(s * n_bins + b)];
          }
      }
    }
    __syncthreads();
    carry = 0;
  }
  scan_chunk<PER>(bufc, wsum, &carry);   // species-major starts, in place
  if (blockIdx.x == 0) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int i = u * kScanThreads + threadIdx.x;
      if (i < nb) start[i] = bufc[scan_pad<PER>(i)];
    }
    if (threadIdx.x == 0) start[nb] = carry;
  }
  if (t < n) tmp[bufc[scan_pad<PER>(k)] + rk] = t;
}

// Small periodic systems: the whole cell list in one launch, through LDS.
// Every workgroup bins all atoms (U per thread; LDS histogram atomics give
// arrival ranks), scans the histogram and scatters the atoms by key, all in
// its own LDS; then it places kScanThreads atoms of its own: the stable slot
// of an atom is the start of its key plus the number of atoms of that key with
// a smaller index, counted in the key's segment of the scatter.  The same
// outputs, bit for bit, as binning, scan + scatter and bin sort in three
// launches; the device histogram is not touched (it stays zero).
//
// Bound by latency and, with more atoms per thread, by the LDS scatters: 1,500
// atoms 9.0 us (one workgroup alone for all 10.6), 2,100 atoms 9.6 against
// 14.4 for the three launches, 4,100 atoms 10.2 against 14.5, 8,100 atoms 12.7
// against 14.2, but 12,288 atoms 16.9 against 15.2 (event-timed), hence the
// limit.
constexpr int kCellsMost = 8;   // atoms per thread; LDS: 2 padded scan buffers and 16 bits per atom

template <int PER, int U>
__global__ __launch_bounds__(kScanThreads) void k_cells(const float* __restrict__ pos, int n,
                                                        const int* __restrict__ idx,
                                                        const int* __restrict__ sigma, Geometry g, LinkArgs L,
                                                        int S, int* __restrict__ key, int* __restrict__ bin_start,
                                                        int* __restrict__ perm, float4* __restrict__ spos,
                                                        int* __restrict__ slot_atom, int* __restrict__ order,
                                                        int* __restrict__ sbin, int* __restrict__ islot,
                                                        PairCount pc, int* __restrict__ status,
                                                        int* __restrict__ cut) {
  __shared__ int wsum[2 * (kScanThreads / 64) + 1];
  __shared__ int hist[scan_lds_words<PER>()];   // counts per key, then species-major starts
  __shared__ int bmaj[scan_lds_words<PER>()];   // totals per bin, then bin-major starts
  __shared__ uint16_t tmp[U * kScanThreads];     // atoms of each key in arrival order
  const int nb = S * g.n_bins;                   // <= kScanThreads * PER <= 2^14 (checked by the launcher)
  const int tid = threadIdx.x;
  if (blockIdx.x == 0 && tid == 0) *cut = 0;
#pragma unroll
  for (int u = 0; u < PER; ++u) hist[scan_pad<PER>(u * kScanThreads + tid)] = 0;
  const int own = blockIdx.x * kScanThreads + tid;   // the atom this thread places
  const int atom = own < n ? idx[own] : 0;
  const float3 mine = nnp_position(pos, atom, L, g);
  // thread tid bins atoms u * kScanThreads + tid (every load before the first use)
  int aa[U], ss[U], kr[U];   // kr: key | arrival rank << 15
  float3 pp[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int t = min(u * kScanThreads + tid, n - 1);
    aa[u] = idx[t];
    ss[u] = sigma[t];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int64_t at = 3 * (int64_t)max(aa[u], 0);
    pp[u] = make_float3(pos[at], pos[at + 1], pos[at + 2]);
  }
  if (L.n > 0) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (aa[u] < 0) pp[u] = nnp_position(pos, aa[u], L, g);
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int t = u * kScanThreads + tid;
    if (t >= n) continue;
    int bin = 0;
    if (!(isfinite(pp[u].x) && isfinite(pp[u].y) && isfinite(pp[u].z)))
      atomicOr(status, kStatusNonFinite);
    else
      bin = cell_of(pp[u].x, pp[u].y, pp[u].z, g);
    const int k = ss[u] * g.n_bins + bin;
    kr[u] = k | (atomicAdd(&hist[scan_pad<PER>(k)], 1) << 15);
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int b = u * kScanThreads + tid;
    int tot = 0;
#pragma unroll
    for (int s = 0; s < kMaxSpecies; ++s)
      if (s < S && b < g.n_bins) tot += hist[scan_pad<PER>(s * g.n_bins + b)];
    bmaj[scan_pad<PER>(b)] = tot;
  }
  __syncthreads();
  int carry = 0;
  scan_chunk<PER>(bmaj, wsum, &carry);
  carry = 0;
  scan_chunk<PER>(hist, wsum, &carry);
  auto start_of = [&](int k) { return k < nb ? hist[scan_pad<PER>(k)] : n; };
  if (blockIdx.x == 0)
    for (int i = tid; i <= nb; i += kScanThreads) bin_start[i] = start_of(i);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int t = u * kScanThreads + tid;
    if (t < n) tmp[start_of(kr[u] & 0x7fff) + (kr[u] >> 15)] = (uint16_t)t;
  }
  __syncthreads();
  if (own < n) {
    int k = kr[0];
#pragma unroll
    for (int u = 1; u < U; ++u) k = u == (int)blockIdx.x ? kr[u] : k;
    k &= 0x7fff;
    const int b0 = start_of(k), b1 = start_of(k + 1);
    int rank = 0;
    for (int e = b0; e < b1; ++e) rank += tmp[e] < own;
    const int slot = b0 + rank;
    const int sp = k / g.n_bins, bin = k - sp * g.n_bins;
    int o0 = bmaj[scan_pad<PER>(bin)];   // bin-major: earlier bins, then earlier species of this bin
    for (int s = 0; s < sp; ++s) o0 += start_of(s * g.n_bins + bin + 1) - start_of(s * g.n_bins + bin);
    const int cz = bin % g.nc[2], cxy = bin / g.nc[2];
    key[own] = k;
    perm[slot] = own;
    order[o0 + rank] = slot;
    sbin[slot] = ((cxy / g.nc[1]) << 20) | ((cxy % g.nc[1]) << 10) | cz;
    islot[own] = slot;
    if (pc.at != nullptr) pc.at[(int64_t)slot * pc.stride] = 0;
    spos[slot] = make_float4(mine.x, mine.y, mine.z, __int_as_float(sp));
    slot_atom[slot] = atom;
  }
}

// One wavefront per bin: the atomically scattered entries of the bin are
// ranked by atom index (a stable order independent of the atomic order), and
// the sorted positions / species / atom indices are written per slot, and
// each slot's place in the bin-major visiting order.
__global__ __launch_bounds__(kBlock) void k_binsort(const int* __restrict__ start, int n_bins_total,
                                                    const int* __restrict__ tmp,
                                                    const float4* __restrict__ stg,
                                                    const int* __restrict__ idx, Geometry g,
                                                    const int* __restrict__ cmstart, int S,
                                                    int* __restrict__ perm,
                                                    float4* __restrict__ spos,
                                                    int* __restrict__ slot_atom,
                                                    int* __restrict__ order, int* __restrict__ sbin,
                                                    int* __restrict__ islot, PairCount pc,
                                                    int* __restrict__ count) {
  int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  int lane = threadIdx.x & 63;
  if (wave >= n_bins_total) return;
  if (lane == 0) count[wave] = 0;   // the histogram starts from zero in the next call
  int b0 = start[wave], b1 = start[wave + 1];
  const int sp = wave / g.n_bins, bin = wave - sp * g.n_bins;
  const int o0 = cmstart[bin * S + sp];
  // the cell's coordinates, packed for the neighbour search
  const int cz = bin % g.nc[2], cxy = bin / g.nc[2];
  const int packed = ((cxy / g.nc[1]) << 20) | ((cxy % g.nc[1]) << 10) | cz;
  const int cnt = b1 - b0;
  // bins of up to 64 atoms: one entry per lane, ranked against the others
  // with lane reads (no memory round trip per comparison)
  const int mine = lane < cnt ? tmp[b0 + lane] : 0;
  for (int e = b0 + lane; e < b1; e += 64) {
    int t = tmp[e];
    int rank = 0;
    if (cnt <= 64) {
      for (int q = 0; q < cnt; ++q) rank += __builtin_amdgcn_readlane(mine, q) < t;
    } else {
      for (int q = b0; q < b1; ++q) rank += tmp[q] < t;
    }
    int slot = b0 + rank;
    perm[slot] = t;
    order[o0 + rank] = slot;
    sbin[slot] = packed;
    islot[t] = slot;
    if (pc.at != nullptr) pc.at[(int64_t)slot * pc.stride] = 0;
    spos[slot] = stg[t];   // staged by k_stage: no second trip through idx and pos
    slot_atom[slot] = idx[t];
  }
}

// Open systems (one bin per system): the stable slot of every atom is found
// directly, one wavefront per system.  The system's atoms are taken in input
// order, 64 at a time; for each species a ballot gives every atom its rank
// among the earlier atoms of its species, so slot = bin start + rank.  No
// atomics and no in-bin sort are needed, whatever the system size.
__global__ __launch_bounds__(64) void k_rank_systems(const int* __restrict__ sys_off, int n_sys, int S,
                                                      const int* __restrict__ bin_start,
                                                      const int* __restrict__ sigma,
                                                      const int* __restrict__ idx, const float* __restrict__ pos,
                                                      Geometry g, LinkArgs L, const int* __restrict__ cmstart,
                                                      int* __restrict__ perm, float4* __restrict__ spos,
                                                      int* __restrict__ slot_atom, int* __restrict__ order,
                                                      int* __restrict__ count, int* __restrict__ sbin,
                                                      int* __restrict__ islot, PairCount pc) {
  const int m = blockIdx.x;
  const int lane = threadIdx.x;
  if (lane < S) count[lane * n_sys + m] = 0;   // the histogram starts from zero in the next call
  const int t0 = sys_off[m], t1 = sys_off[m + 1];
  const uint64_t lt = __lanemask_lt();
  int base[kMaxSpecies] = {0, 0, 0, 0}, first[kMaxSpecies], cm[kMaxSpecies];
#pragma unroll
  for (int s = 0; s < kMaxSpecies; ++s) {   // per-system constants (wave-uniform)
    first[s] = s < S ? bin_start[s * n_sys + m] : 0;
    cm[s] = s < S ? cmstart[m * S + s] : 0;
  }
  // the next block of 64 atoms is loaded while the current one is placed
  auto fetch = [&](int t, int& sg, int& a) {
    sg = -1;
    a = 0;
    if (t < t1) {
      sg = sigma[t];
      a = idx[t];
    }
  };
  int sg_n, a_n;
  fetch(t0 + lane, sg_n, a_n);
  for (int c0 = t0; c0 < t1; c0 += 64) {
    const int t = c0 + lane;
    const bool ok = t < t1;
    const int sg = sg_n, a = a_n;
    const float3 p = ok ? nnp_position(pos, a, L, g) : make_float3(0.f, 0.f, 0.f);
    if (c0 + 64 < t1) fetch(t + 64, sg_n, a_n);
    int slot = 0, rank = 0, o = 0;
#pragma unroll
    for (int s = 0; s < kMaxSpecies; ++s) {
      if (s < S) {
        const uint64_t mk = __ballot(sg == s);
        if (sg == s) {
          rank = base[s] + __popcll(mk & lt);
          slot = first[s] + rank;
          o = cm[s] + rank;
        }
        base[s] += __popcll(mk);
      }
    }
    if (ok) {
      perm[slot] = t;
      order[o] = slot;
      sbin[slot] = m;
      islot[t] = slot;
      if (pc.at != nullptr) pc.at[(int64_t)slot * pc.stride] = 0;
      spos[slot] = make_float4(p.x, p.y, p.z, __int_as_float(sg));
      slot_atom[slot] = a;
    }
  }
}

struct NeighArgs {
  const int* order;        // bin-major visiting order of the slots
  const int* sbin;         // packed cell coordinates (periodic) or system of each slot
  const float4* spos;
  const int* perm;
  const int* key;
  const int* bin_start;
  int n, S;
  float rc2, rca2;
  float cull2;             // (sqrt(rc2) + kCullMargin)^2: stencil cells beyond it hold no neighbour
  int* rad;
  int* ang;
  int* rad_off;
  int* ang_off;
  int max_rad, max_ang;
  int* status;
  int* cut;                // set if a list of this call was cut off
};

__device__ __forceinline__ void list_overflow(const NeighArgs& a) {
  atomicOr(a.status, kStatusCapacity);
  *a.cut = 1;   // (any number of wavefronts, all the same value)
}

constexpr int kMaxStencil = 27;

// One wavefront per sorted slot i.  For each species, the candidate atoms of
// the (deduplicated) 27-cell stencil are visited in ascending cell order --
// hence ascending slot order -- one candidate per lane, and the accepted ones
// are compacted with a ballot, so every species segment of a list is sorted
// by slot.  Angular neighbours (r < rc_ang) are the same sequence thinned out.
// Lists never hold more than their capacity; an overflow sets the device
// status word.
// Candidates of one species per atom held in LDS (flattened stencil ranges);
// a longer candidate sequence falls back to a binary search over the ranges.
constexpr int kCandCap = 1024;
// Distance (A) added to the cutoff before a stencil cell is skipped.  Cell
// assignment and the distance test round positions to a few FP32 ulps,
// about 1e-3 A for coordinates of 10^4 A, so skipping is exact for inputs
// within many box lengths of the origin.
constexpr float kCullMargin = 0.02f;

// Accepted candidates are appended in lane order: a lane's place is the
// number of accepting lanes below it.
__device__ __forceinline__ unsigned place(uint64_t m, int before) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)before));
}
__device__ __forceinline__ int below(uint64_t m) { return (int)place(m, 0); }

__global__ __launch_bounds__(64) void k_neighbours(NeighArgs a, Geometry g) {
#pragma clang fp contract(off)
  __shared__ int s_start[kMaxStencil];
  __shared__ int s_off[kMaxStencil + 1];
  __shared__ int s_cand[kCandCap];
  const int i = a.order[xcd_block(blockIdx.x, gridDim.x)];
  const int lane = threadIdx.x;
  const float4 pi = a.spos[i];
  const int sb = a.sbin[i];
  const MinImage mi = min_image_at(g, i);
  // Stencil cells in ascending id order: per dimension the (wrapped)
  // coordinates {c-1, c, c+1} are sorted, and ids are lexicographic in
  // (x, y, z).  Lane l < nst takes the l-th of them.
  int nst = 1;
  int my_cell = sb;   // open systems: the system's bin
  bool culled = false;
  if (g.periodic) {
    const int c[3] = {sb >> 20, (sb >> 10) & 1023, sb & 1023};
    int nd[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) nd[k] = g.nc[k] >= 3 ? 3 : g.nc[k];
    nst = nd[0] * nd[1] * nd[2];
    const int l = lane < nst ? lane : 0;
    int o[3];
    if (nst == 27) {
      o[0] = l / 9; o[1] = (l / 3) % 3; o[2] = l % 3;
    } else {
      o[0] = l / (nd[1] * nd[2]); o[1] = (l / nd[2]) % nd[1]; o[2] = l % nd[2];
    }
    // A stencil cell whose nearest point lies beyond the cutoff (plus
    // kCullMargin) holds no neighbour of this centre: its lane offers no
    // candidates.  The gap per dimension is the centre's offset inside its
    // own cell (lower neighbour) or the rest of the cell (upper neighbour).
    const float pc[3] = {pi.x, pi.y, pi.z};
    float gap2 = 0.f;
    int v[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int n = g.nc[k];
      if (n < 3) {   // every cell of the dimension is in the stencil
        v[k] = o[k];
        continue;
      }
      // offset of the o-th sorted coordinate: c = 0 gives {0, 1, n-1},
      // c = n-1 gives {0, n-2, n-1}, otherwise {c-1, c, c+1}
      const int d = c[k] == 0 ? (o[k] == 2 ? -1 : o[k]) : (c[k] == n - 1 ? (o[k] == 0 ? 1 : o[k] - 2) : o[k] - 1);
      const int w = c[k] + d;
      v[k] = w < 0 ? w + n : (w >= n ? w - n : w);
      const float x = pc[k] - floorf(pc[k] * g.inv_box[k]) * g.box[k];
      const float u = x - (float)c[k] * g.cell_len[k];
      const float gap = d == 0 ? 0.f : fmaxf(d > 0 ? g.cell_len[k] - u : u, 0.f);
      gap2 += gap * gap;
    }
    my_cell = (v[0] * g.nc[1] + v[1]) * g.nc[2] + v[2];
    culled = gap2 > a.cull2;
  }

  int* rad = a.rad + (int64_t)i * a.max_rad;
  int* ang = a.ang + (int64_t)i * a.max_ang;
  int nr = 0, na = 0;   // list lengths so far (wavefront-uniform)
  bool overflow = false;
  // candidate ranges of a species, one stencil cell per lane; those of the
  // next species are on their way while this one's candidates are tested
  int st_next = 0, end_next = 0;
  auto fetch = [&](int s) {
    st_next = end_next = 0;
    if (s < a.S && lane < nst && !culled) {
      const int b = s * g.n_bins + my_cell;
      st_next = a.bin_start[b];
      end_next = a.bin_start[b + 1];
    }
  };
  fetch(0);
  for (int s = 0; s < a.S; ++s) {
    if (lane == 0) {
      a.rad_off[(int64_t)i * (a.S + 1) + s] = nr;
      a.ang_off[(int64_t)i * (a.S + 1) + s] = na;
    }
    const int st = st_next, cnt = end_next - st_next;
    fetch(s + 1);
    const int inc = wave_scan_dpp<false>(cnt);
    const int total = __builtin_amdgcn_readlane(inc, 63);
    // one range (an open system): slots follow directly; short per-cell ranges
    // are flattened into LDS by their lanes; otherwise search the ranges
    const int st0 = __builtin_amdgcn_readfirstlane(st);
    const bool flat = nst > 1 && total <= kCandCap;
    __syncthreads();   // the previous species' candidates have been read
    if (lane < nst) {
      s_start[lane] = st;
      s_off[lane] = inc - cnt;
      if (flat)
        for (int q = 0; q < cnt; ++q) s_cand[inc - cnt + q] = st + q;
    }
    __syncthreads();
    // candidate slot at position c of the flattened sequence (-1 beyond it)
    auto candidate = [&](int c) {
      int j = -1;
      if (c < total) {
        if (nst == 1) {
          j = st0 + c;
        } else if (flat) {
          j = s_cand[c];
        } else {
          int lo = 0, hi = nst - 1;
          while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_off[mid] <= c) lo = mid; else hi = mid - 1;
          }
          j = s_start[lo] + (c - s_off[lo]);
        }
      }
      return j;
    };
    // the next step's candidate and position are fetched before this step's
    // test, so the load is in flight while the wavefront works
    int j = candidate(lane);
    float4 pj = a.spos[j >= 0 && j != i ? j : i];
    for (int c0 = 0; c0 < total; c0 += 64) {
      const int jn = candidate(c0 + 64 + lane);
      const float4 pn = a.spos[jn >= 0 && jn != i ? jn : i];
      // straight-line test (invalid lanes read the centre's own position and
      // are masked), so the ballots take the comparison masks directly
      const bool valid = j >= 0 && j != i;
      const float r2 = pair_r2_exact(pi, pj, mi);
      const bool in_r = valid && r2 < a.rc2;
      const uint64_t mr = __builtin_amdgcn_ballot_w64(in_r);
      const int pr = nr + below(mr);
      // angular entries are also in the radial list
      const bool in_a = valid && r2 < a.rca2 && pr < a.max_rad;
      const uint64_t ma = __builtin_amdgcn_ballot_w64(in_a);
      const int pa = na + below(ma);
      if (in_r && pr < a.max_rad) rad[(unsigned)pr] = j;
      if (in_a && pa < a.max_ang) ang[(unsigned)pa] = j;
      nr += __popcll(mr);
      na += __popcll(ma);
      if (nr > a.max_rad || na > a.max_ang) {
        overflow = true;
        nr = min(nr, a.max_rad);
        na = min(na, a.max_ang);
      }
      j = jn;
      pj = pn;
    }
  }
  if (lane == 0) {
    a.rad_off[(int64_t)i * (a.S + 1) + a.S] = nr;
    a.ang_off[(int64_t)i * (a.S + 1) + a.S] = na;
    if (overflow) list_overflow(a);
  }
}

// Same lists as k_neighbours for periodic boxes, a wavefront per cell (or per
// part of its atoms).  The stencil's candidates, all species in list order,
// are flattened once, and their positions are kept in registers, 64 per
// chunk: one shifted copy each, the image nearest to the cell's centre.  The
// centres' positions are shifted the same way, so a pair costs three
// subtractions and r^2 instead of the minimum image.  That r^2 differs from the predicate's
// (pair_r2_exact on the caller's coordinates) by rounding only, so it decides
// unless it falls within eps of a cutoff: two comparisons, one on each side,
// must agree for every lane of a chunk.  A centre with a chunk where they do
// not (about one in twenty), or whose lists would overflow, is done again with
// the predicate itself; where a cell has more candidates than the registers
// hold, the rest of them go through the predicate for every centre.
//
// The shift picks the predicate's image: with at least four cells per
// dimension a stencil pair is at most half a box apart; with three it can be
// further, but the other image is then at least a cell away, which is more
// than the cutoff by kCullMargin (cells_fast).
//
// Bound by instruction issue, scalar and vector: about 18 vector and 14 scalar
// instructions per chunk and centre, 7 chunks per centre in water.
// k_neighbours: 565 vector instructions per atom.  What decides per lane (the
// margin, the capacity) instead of per chunk on scalars took the box of
// 261,000 atoms from 181 to 136 us.
template <int S, int NCH>
__global__ __launch_bounds__(64) void k_neighbours_cell(NeighArgs a, Geometry g, int K) {
  constexpr int kCap = 64 * NCH, kList = kCap + 512;   // candidates in registers, and in LDS
  __shared__ int s_cand[kList];
  __shared__ int s_start[kMaxStencil * S], s_off[kMaxStencil * S + 1];
  const int b = xcd_block(blockIdx.x, gridDim.x);
  const int cell = b / K, part = b - cell * K;
  const int lane = threadIdx.x;
  const MinImage mi = min_image_of_system(g, 0);
  const int cc[3] = {cell / (g.nc[1] * g.nc[2]), (cell / g.nc[2]) % g.nc[1], cell % g.nc[2]};
  // stencil cells in ascending id order (see k_neighbours), one per lane
  int my_cell = 0;
  {
    const int l = lane < kMaxStencil ? lane : 0;
    const int o[3] = {l / 9, (l / 3) % 3, l % 3};
    int v[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int n = g.nc[k], c = cc[k];
      const int d = c == 0 ? (o[k] == 2 ? -1 : o[k]) : (c == n - 1 ? (o[k] == 0 ? 1 : o[k] - 2) : o[k] - 1);
      const int w = c + d;
      v[k] = w < 0 ? w + n : (w >= n ? w - n : w);
    }
    my_cell = (v[0] * g.nc[1] + v[1]) * g.nc[2] + v[2];
  }
  // candidates: ranges of slots, species by species, flattened
  int total = 0, first[S + 1], own_st[S], own_n[S], own_at[S], n_centres = 0;
  const uint64_t own_lane = __ballot(lane < kMaxStencil && my_cell == cell);
  const int own = __ffsll((unsigned long long)own_lane) - 1;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    first[s] = total;
    int st = 0, cnt = 0;
    if (lane < kMaxStencil) {
      const int* r = a.bin_start + s * g.n_bins + my_cell;
      st = r[0];
      cnt = r[1] - st;
    }
    int inc = cnt;
#pragma unroll
    for (int off = 1; off < 32; off <<= 1) {
      const int u = __shfl_up(inc, off, 64);
      if (lane >= off) inc += u;
    }
    const int at = total + inc - cnt;
    if (lane < kMaxStencil) {
      s_start[s * kMaxStencil + lane] = st;
      s_off[s * kMaxStencil + lane] = at;
      for (int q = 0; q < cnt && at + q < kList; ++q) s_cand[at + q] = st + q;
    }
    own_st[s] = __builtin_amdgcn_readlane(st, own);
    own_n[s] = __builtin_amdgcn_readlane(cnt, own);
    own_at[s] = __builtin_amdgcn_readlane(at, own);
    n_centres += own_n[s];
    total += __builtin_amdgcn_readlane(inc, kMaxStencil - 1);
  }
  first[S] = total;
  // this wavefront's centres: the part-th of K equal pieces, all species
  const int chunk = (n_centres + K - 1) / K;
  const int q0 = part * chunk, q1 = min(n_centres, q0 + chunk);
  if (q0 >= q1) return;
  __syncthreads();
  const int nch = (min(total, kCap) + 63) >> 6;
  // candidates in registers, as the image nearest to the cell's centre
  const float mx = ((float)cc[0] + 0.5f) * g.cell_len[0], my = ((float)cc[1] + 0.5f) * g.cell_len[1],
              mz = ((float)cc[2] + 0.5f) * g.cell_len[2];
  auto shift = [](float x, float m, float L, float iL) { return x - L * rintf((x - m) * iL); };
  float cx[NCH], cy[NCH], cz[NCH], reach = 0.f;
  int cj[NCH];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    cj[c] = -1;
    cx[c] = cy[c] = cz[c] = 3e18f;   // beyond every cutoff
    if (c < nch && 64 * c + lane < total) cj[c] = s_cand[64 * c + lane];
  }
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    if (cj[c] >= 0) {
      const float4 q = a.spos[cj[c]];
      cx[c] = shift(q.x, mx, g.box[0], g.inv_box[0]);
      cy[c] = shift(q.y, my, g.box[1], g.inv_box[1]);
      cz[c] = shift(q.z, mz, g.box[2], g.inv_box[2]);
      reach = fmaxf(reach, fmaxf(fabsf(q.x), fmaxf(fabsf(q.y), fabsf(q.z))));
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) reach = fmaxf(reach, __shfl_xor(reach, off, 64));
  // both distances round coordinates of up to reach + 2 L: each component is
  // within 2^-21 (reach + 2 L) of the other, r^2 within 2 sqrt(3) rc times
  // that (and its own rounding)
  const float eps = 8.f * sqrtf(a.rc2) * 0x1p-21f * (reach + 2.f * fmaxf(g.box[0], fmaxf(g.box[1], g.box[2])));
  const unsigned last_r = (unsigned)a.max_rad - 1, last_a = (unsigned)a.max_ang - 1;
  unsigned starts = 0;   // chunks in which a species starts
#pragma unroll
  for (int s = 1; s < S; ++s)
    if (first[s] < kCap) starts |= 1u << (first[s] >> 6);
  auto slot_of = [&](int q) {   // q-th centre of the cell
    int i = 0;
#pragma unroll
    for (int s = 0, at = 0; s < S; ++s) {
      if (q >= at && q < at + own_n[s]) i = own_st[s] + q - at;
      at += own_n[s];
    }
    return i;
  };
  for (int qb = q0; qb < q1; qb += 64) {   // 64 centres at a time, one per lane
    const int my_i = slot_of(min(qb + lane, q1 - 1));
    const float4 pc = a.spos[my_i];
    const float px = shift(pc.x, mx, g.box[0], g.inv_box[0]), py = shift(pc.y, my, g.box[1], g.inv_box[1]),
                pz = shift(pc.z, mz, g.box[2], g.inv_box[2]);
    for (int q = qb; q < min(q1, qb + 64); ++q) {
      const int from = q - qb;
      const int i = __builtin_amdgcn_readlane(my_i, from);
      int* rad = a.rad + (int64_t)i * a.max_rad;
      int* ang = a.ang + (int64_t)i * a.max_ang;
      int nr = 0, na = 0, ro[S], ao[S];
#pragma unroll
      for (int s = 0; s < S; ++s) ro[s] = ao[s] = 0;
      const float x = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(px), from));
      const float y = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(py), from));
      const float z = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pz), from));
      // every comparison counts on scalar instructions too, so the checks are
      // per lane: the least distance of any r^2 to a cutoff, and places held
      // below the capacity (a list that reaches it is done again)
      float margin = 3e18f;
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        if (c < nch) {
          const float dx = cx[c] - x, dy = cy[c] - y, dz = cz[c] - z;
          float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
          r2 = cj[c] == i ? 3e18f : r2;
          const uint64_t mr = __builtin_amdgcn_ballot_w64(r2 < a.rc2), ma = __builtin_amdgcn_ballot_w64(r2 < a.rca2);
          margin = fminf(margin, fminf(fabsf(r2 - a.rc2), fabsf(r2 - a.rca2)));
          const unsigned pr = min(place(mr, nr), last_r), pa = min(place(ma, na), last_a);
          if (starts >> c & 1) {   // a species starts in this chunk
#pragma unroll
            for (int s = 1; s < S; ++s)
              if ((first[s] >> 6) == c) {
                const uint64_t before = (uint64_t(1) << (first[s] & 63)) - 1;
                ro[s] = nr + __popcll(mr & before);
                ao[s] = na + __popcll(ma & before);
              }
          }
          nr += __popcll(mr);
          na += __popcll(ma);
          if (__builtin_amdgcn_inverse_ballot_w64(mr)) rad[pr] = cj[c];
          if (__builtin_amdgcn_inverse_ballot_w64(ma)) ang[pa] = cj[c];
        }
      }
      const bool again = nr > a.max_rad || na > a.max_ang || __ballot(!(margin > eps)) != 0;
#pragma unroll
      for (int s = 1; s < S; ++s)
        if ((first[s] >> 6) >= nch) {   // no candidate of species s or later
          ro[s] = nr;
          ao[s] = na;
        }
      if (again || total > kCap) {   // the predicate itself, with the lists' capacities: all, or the rest
        bool overflow = false;
        const float4 pi = a.spos[i];
        int next = 1;   // species whose start comes next
        int c0 = kCap;
        if (again) {
          nr = na = c0 = 0;
        } else {
#pragma unroll
          for (int s = 1; s < S; ++s) next += first[s] < kCap;
        }
        for (; c0 < total; c0 += 64) {
          const int c = c0 + lane;
          int j = -1;
          if (c < total) {
            if (c < kList) {
              j = s_cand[c];
            } else {
              int lo = 0, hi = S * kMaxStencil - 1;
              while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (s_off[mid] <= c) lo = mid; else hi = mid - 1;
              }
              j = s_start[lo] + (c - s_off[lo]);
            }
          }
          const bool valid = j >= 0 && j != i;
          const float r2 = pair_r2_exact(pi, a.spos[valid ? j : i], mi);
          const uint64_t mr = __ballot(valid && r2 < a.rc2);
          const int pr = nr + below(mr);
          const uint64_t ma = __ballot(valid && r2 < a.rca2 && pr < a.max_rad);
          const int pa = na + below(ma);
#pragma unroll
          for (int s = 1; s < S; ++s)
            if (s == next && first[s] < c0 + 64) {
              const uint64_t before = (uint64_t(1) << (first[s] - c0)) - 1;
              ro[s] = min(nr + __popcll(mr & before), a.max_rad);
              ao[s] = min(na + __popcll(ma & before), a.max_ang);
              ++next;
            }
          if ((mr >> lane & 1) && pr < a.max_rad) rad[pr] = j;
          if ((ma >> lane & 1) && pa < a.max_ang) ang[pa] = j;
          nr += __popcll(mr);
          na += __popcll(ma);
          if (nr > a.max_rad || na > a.max_ang) {
            overflow = true;
            nr = min(nr, a.max_rad);
            na = min(na, a.max_ang);
          }
        }
#pragma unroll
        for (int s = 1; s < S; ++s)
          if (s >= next) {   // species s starts behind the last candidate
            ro[s] = nr;
            ao[s] = na;
          }
        if (overflow && lane == 0) list_overflow(a);
      }
      // species offsets: lanes 0 .. S the radial ones, 16 .. 16 + S the angular ones
      const int t = lane & 15;
      int v = lane < 16 ? nr : na;
#pragma unroll
      for (int s = 0; s < S; ++s)
        if (t == s) v = lane < 16 ? ro[s] : ao[s];
      int* dst = (lane < 16 ? a.rad_off : a.ang_off) + (int64_t)i * (S + 1) + t;
      if (lane < 32 && t <= S) *dst = v;
    }
  }
}

// The cell kernel's conditions: a periodic box of at least three cells per
// dimension, and where there are three, cells longer than the cutoff by the
// margin (see k_neighbours_cell).
bool cells_fast(const Geometry& g, float rc) {
  if (!g.periodic) return false;
  for (int k = 0; k < 3; ++k)
    if (g.nc[k] < 3 || (g.nc[k] == 3 && g.cell_len[k] < rc + kCullMargin)) return false;
  return true;
}

// ---------------------------------------------------------------------------
// Neighbour lists from a pair list supplied by the caller (the MD engine's own
// list, a half list possibly with a buffer beyond the cutoff).  Each pair of
// NNP atoms is re-tested with the same FP32 predicate as the cell-list search
// and appended to both atoms' radial rows in arbitrary order; one wavefront
// per row then sorts it by slot (which groups it by species, slots being
// species-major), derives the species segments and the angular sub-list, so
// the lists are exactly the ones the cell-list search builds.
__device__ __forceinline__ float pair_r2(const float4& pi, const float4& pj, const Geometry& g) {
  return pair_r2_exact(pi, pj, min_image_of_system(g, 0));   // one system: the call's box or none
}

__global__ __launch_bounds__(kBlock) void k_pairs_scatter(const int* __restrict__ pairs, int n_pairs,
                                                          const int* __restrict__ loc, int n_atoms,
                                                          const int* __restrict__ islot,
                                                          const float4* __restrict__ spos, Geometry g, float rc2,
                                                          int* __restrict__ rad, PairCount pc, int max_rad,
                                                          int* __restrict__ status) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n_pairs) return;
  const int a = pairs[2 * (int64_t)p], b = pairs[2 * (int64_t)p + 1];
  if (a < 0 || b < 0 || a >= n_atoms || b >= n_atoms || a == b) {
    atomicOr(status, kStatusInput);
    return;
  }
  const int la = loc[a], lb = loc[b];
  if (la < 0 || lb < 0) return;   // a pair with an atom outside the index group
  const int sa = islot[la], sb = islot[lb];
  if (!(pair_r2(spos[sa], spos[sb], g) < rc2)) return;
  const int pa = atomicAdd(pc.at + (int64_t)sa * pc.stride, 1), pb = atomicAdd(pc.at + (int64_t)sb * pc.stride, 1);
  if (pa < max_rad) rad[(int64_t)sa * max_rad + pa] = sb;
  if (pb < max_rad) rad[(int64_t)sb * max_rad + pb] = sa;
}

// Link atoms (eq. 4) are not atoms of the system, so a caller's pair list
// cannot name them: one wavefront per link atom tests it against every NNP
// atom with the same predicate and appends each pair within the cutoff to
// both rows.  A pair of two link atoms is added by the one with the lower
// index.  The NNP-local indices of the link atoms are [n - n_links, n).
__global__ __launch_bounds__(64) void k_link_pairs(int n, int n_links, const int* __restrict__ islot,
                                                   const float4* __restrict__ spos, Geometry g, float rc2,
                                                   int* __restrict__ rad, PairCount pc, int max_rad) {
  const int tl = n - n_links + (int)blockIdx.x;
  const int sl = islot[tl];
  const float4 pl = spos[sl];
  for (int t = threadIdx.x; t < n; t += 64) {
    if (t >= n - n_links && t <= tl) continue;
    const int st = islot[t];
    if (!(pair_r2(pl, spos[st], g) < rc2)) continue;
    const int pa = atomicAdd(pc.at + (int64_t)sl * pc.stride, 1), pb = atomicAdd(pc.at + (int64_t)st * pc.stride, 1);
    if (pa < max_rad) rad[(int64_t)sl * max_rad + pa] = st;
    if (pb < max_rad) rad[(int64_t)st * max_rad + pb] = sl;
  }
}

// One wavefront per slot: sorts the row by slot, then the species offsets and
// the angular list.  The place of an entry (up to four per lane) is the count
// of smaller ones, read from LDS four at a time; equal entries (a pair given
// twice, an input error) would take the same place and leave the next one
// empty, and are then placed in the order of the row.  While the counting
// runs, the entries' positions arrive, so that each entry carries its angular
// flag (bit 31) to its place.
//
// Bound by the latency of one wavefront's chain: for 900 atoms 5.9 us; with a
// bitonic sort, the positions read after it and the segments counted entry by
// entry, 11.3 us.
constexpr int kPairRank = kPairRowMax / 64;

__global__ __launch_bounds__(64) void k_pairs_lists(NeighArgs a, Geometry g, PairCount pc) {
  __shared__ int4 row4[kPairRowMax / 4];
  __shared__ int sorted[kPairRowMax];
  int* row = reinterpret_cast<int*>(row4);
  const int i = blockIdx.x;
  const int lane = threadIdx.x;
  int* rrow = a.rad + (int64_t)i * a.max_rad;
  const int first = lane < a.max_rad ? rrow[lane] : 0;   // in flight with the count
  const float4 pi = a.spos[i];
  int bound[kMaxSpecies];   // first slot of species s + 1
#pragma unroll
  for (int s = 0; s < kMaxSpecies; ++s) bound[s] = s + 1 < a.S ? a.bin_start[(s + 1) * g.n_bins] : INT_MAX;
  const int cnt = pc.at[(int64_t)i * pc.stride];
  bool overflow = cnt > a.max_rad;
  const int n = min(cnt, a.max_rad);
  const int nk = (n + 63) >> 6;
  int e[kPairRank], place[kPairRank];
#pragma unroll
  for (int k = 0; k < kPairRank; ++k) {
    const int t = 64 * k + lane;
    e[k] = INT_MAX;
    place[k] = 0;
    if (k < nk) {
      if (t < n) e[k] = k == 0 ? first : rrow[t];
      row[t] = e[k];
      sorted[t] = -1;
    }
  }
  __syncthreads();
  float4 pj[kPairRank];
#pragma unroll
  for (int k = 0; k < kPairRank; ++k)
    if (k < nk) pj[k] = a.spos[64 * k + lane < n ? e[k] : i];
  for (int t = 0; t < n; t += 4) {
    const int4 x = row4[t >> 2];
#pragma unroll
    for (int k = 0; k < kPairRank; ++k)
      if (k < nk) place[k] += (x.x < e[k]) + (x.y < e[k]) + (x.z < e[k]) + (x.w < e[k]);
  }
#pragma unroll
  for (int k = 0; k < kPairRank; ++k)
    if (k < nk && 64 * k + lane < n) {
      if (pair_r2(pi, pj[k], g) < a.rca2) e[k] |= INT_MIN;
      sorted[place[k]] = e[k];
    }
  __syncthreads();
  bool dup = false;   // places nothing came to (no slot is INT_MAX, so no entry is -1)
#pragma unroll
  for (int k = 0; k < kPairRank; ++k)
    if (64 * k + lane < n && sorted[64 * k + lane] == -1) dup = true;
  dup = __ballot(dup) != 0;
  if (dup) {
    for (int t = 0; t < n; ++t)
#pragma unroll
      for (int k = 0; k < kPairRank; ++k) place[k] += row[t] == (e[k] & INT_MAX) && t < 64 * k + lane;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPairRank; ++k)
      if (64 * k + lane < n) sorted[place[k]] = e[k];
    __syncthreads();
  }
  int* ang = a.ang + (int64_t)i * a.max_ang;
  int na = 0;
  int seg_r[kMaxSpecies] = {}, seg_a[kMaxSpecies] = {};   // entries below each bound
  for (int c0 = 0; c0 < n; c0 += 64) {
    const int t = c0 + lane;
    const int v = t < n ? sorted[t] : INT_MAX;
    const bool in_a = v < 0;
    const int j = v & INT_MAX;
    if (t < n) rrow[t] = j;
    const uint64_t ma = __ballot(in_a);
    const int pa = na + __popcll(ma & __lanemask_lt());
    if (in_a && pa < a.max_ang) ang[pa] = j;
#pragma unroll
    for (int s = 0; s < kMaxSpecies; ++s)
      if (s + 1 < a.S) {
        seg_r[s] += __popcll(__ballot(j < bound[s]));
        seg_a[s] += __popcll(__ballot(in_a && pa < a.max_ang && j < bound[s]));
      }
    na += __popcll(ma);
  }
  if (na > a.max_ang) {
    overflow = true;
    na = a.max_ang;
  }
  if (lane <= a.S) {   // offset of species `lane`: the entries below its first slot
    int r = 0, q = 0;
#pragma unroll
    for (int s = 0; s < kMaxSpecies; ++s)
      if (s + 1 == lane) {
        r = seg_r[s];
        q = seg_a[s];
      }
    if (lane == a.S) { r = n; q = na; }
    a.rad_off[(int64_t)i * (a.S + 1) + lane] = r;
    a.ang_off[(int64_t)i * (a.S + 1) + lane] = q;
  }
  if (lane == 0 && overflow) list_overflow(a);
  if (lane == 0 && dup) atomicOr(a.status, kStatusInput);
}

inline int blocks_for(int64_t n, int b) { return (int)((n + b - 1) / b); }

// Smallest power of two PER <= kScanPerMax with nb <= kScanThreads * PER
// (kScanPerMax for larger histograms, which are scanned in several chunks).
inline int scan_entries_per_thread(int nb) {
  int per = 1;
  while (per < kScanPerMax && nb > kScanThreads * per) per *= 2;
  return per;
}

template <int PER>
void launch_scan(nnp_model& m, hipStream_t st) {
  const int nb = m.S * m.geo.n_bins;
  if (nb > kScanChunk) {   // many workgroups
    const int ca = (nb + kScanPartChunk - 1) / kScanPartChunk;
    const int cb = (m.geo.n_bins + kScanPartChunk - 1) / kScanPartChunk;
    hipLaunchKernelGGL(k_scan_part, dim3(ca + cb), dim3(kScanThreads), 0, st, m.d_bin_count, m.S, m.geo.n_bins, ca,
                       m.d_scan_part);
    hipLaunchKernelGGL(k_scan_fin, dim3(ca + cb), dim3(kScanThreads), 0, st, m.d_bin_count, m.d_bin_start,
                       m.d_cmstart, m.S, m.geo.n_bins, ca, m.d_scan_part);
    return;
  }
  hipLaunchKernelGGL(k_scan<PER>, dim3(1), dim3(kScanThreads), 0, st, m.d_bin_count, m.d_bin_start, m.d_cmstart,
                     m.S, m.geo.n_bins);
}

template <int PER, int U>
void launch_cells_small(nnp_model& m, const float* pos, int n, const LinkArgs& L, const PairCount& pc,
                        hipStream_t st) {
  hipLaunchKernelGGL((k_cells<PER, U>), dim3(blocks_for(n, kScanThreads)), dim3(kScanThreads), 0, st, pos, n,
                     m.d_idx, m.d_sigma, m.geo, L, m.S, m.d_key, m.d_bin_start, m.d_perm, m.d_spos, m.d_slot_atom,
                     m.d_order, m.d_sbin, m.d_islot, pc, m.d_status, m.d_cut);
}

template <int U>
void launch_cells_small(nnp_model& m, const float* pos, int n, const LinkArgs& L, const PairCount& pc,
                        hipStream_t st) {
  switch (scan_entries_per_thread(m.S * m.geo.n_bins)) {
    case 1: launch_cells_small<1, U>(m, pos, n, L, pc, st); break;
    case 2: launch_cells_small<2, U>(m, pos, n, L, pc, st); break;
    case 4: launch_cells_small<4, U>(m, pos, n, L, pc, st); break;
    case 8: launch_cells_small<8, U>(m, pos, n, L, pc, st); break;
    default: launch_cells_small<16, U>(m, pos, n, L, pc, st); break;
  }
}

template <int PER>
void launch_scan_scatter(nnp_model& m, int n, hipStream_t st) {
  hipLaunchKernelGGL(k_scan_scatter<PER>, dim3(blocks_for(n, kScanThreads)), dim3(kScanThreads), 0, st,
                     m.d_bin_count, m.d_bin_start, m.d_cmstart, m.S, m.geo.n_bins, m.d_key, m.d_rank, n, m.d_tmp);
}

}  // namespace

hipError_t launch_cells(nnp_model& m, const float* pos, int n, bool pair_list, hipStream_t st) {
  const PairCount pc = pair_list ? pair_count(m) : PairCount{nullptr, 0};
  const Geometry& g = m.geo;
  LinkArgs L{m.d_link_ml, m.d_link_mm, m.link_d, m.n_links_dev};
  int nb = m.S * g.n_bins;
  if (n > 0 && g.periodic && n <= kCellsMost * kScanThreads && nb <= kScanChunk) {
    if (n <= 2 * kScanThreads) launch_cells_small<2>(m, pos, n, L, pc, st);
    else if (n <= 4 * kScanThreads) launch_cells_small<4>(m, pos, n, L, pc, st);
    else launch_cells_small<8>(m, pos, n, L, pc, st);
    return hipGetLastError();
  }
  if (n > 0) {
    hipLaunchKernelGGL(k_stage, dim3(blocks_for(n, kBlock)), dim3(kBlock), 0, st, pos, n, m.d_idx,
                       m.d_sigma, m.d_sys, g, L, m.d_key, m.d_rank, m.d_stg, m.d_bin_count, m.d_status,
                       m.d_cut);
  }
  const bool fused = n > 0 && g.periodic && nb <= kScanChunk;
  const int per = scan_entries_per_thread(nb);
  if (fused) {
    switch (per) {
      case 1: launch_scan_scatter<1>(m, n, st); break;
      case 2: launch_scan_scatter<2>(m, n, st); break;
      case 4: launch_scan_scatter<4>(m, n, st); break;
      case 8: launch_scan_scatter<8>(m, n, st); break;
      default: launch_scan_scatter<16>(m, n, st); break;
    }
  } else {
    switch (per) {
      case 1: launch_scan<1>(m, st); break;
      case 2: launch_scan<2>(m, st); break;
      case 4: launch_scan<4>(m, st); break;
      case 8: launch_scan<8>(m, st); break;
      default: launch_scan<16>(m, st); break;
    }
  }
  if (n > 0 && !g.periodic) {
    hipLaunchKernelGGL(k_rank_systems, dim3(g.n_bins), dim3(64), 0, st, m.d_sys_off, g.n_bins, m.S, m.d_bin_start,
                       m.d_sigma, m.d_idx, pos, g, L, m.d_cmstart, m.d_perm, m.d_spos, m.d_slot_atom,
                       m.d_order, m.d_bin_count, m.d_sbin, m.d_islot, pc);
  } else if (n > 0) {
    if (!fused)
      hipLaunchKernelGGL(k_scatter, dim3(blocks_for(n, kBlock)), dim3(kBlock), 0, st, m.d_key, m.d_rank, n,
                         m.d_bin_start, m.d_tmp);
    hipLaunchKernelGGL(k_binsort, dim3(blocks_for((int64_t)nb * 64, kBlock)), dim3(kBlock), 0, st,
                       m.d_bin_start, nb, m.d_tmp, m.d_stg, m.d_idx, g, m.d_cmstart, m.S, m.d_perm,
                       m.d_spos, m.d_slot_atom, m.d_order, m.d_sbin, m.d_islot, pc, m.d_bin_count);
  }
  return hipGetLastError();
}

// Candidates of a cell, on average, and whether that is a filled box of ordinary
// density and cells (water: 380 to 470), for which the registers hold 512 of
// them, a fifth above the average.  (768, used where that is not so, cost a tenth
// more time: 98,304 atoms 71 us against 64.)
float cell_candidates(const nnp_model& m, int n) { return (float)kMaxStencil * (float)n / (float)m.geo.n_bins; }
bool crowded(float avg) { return 1.2f * avg > 512.f; }

// 0: one wavefront per atom; 1 / 2 / 3: the cell kernel with about 16 / 8 / 4
// centres per wavefront (only where its conditions hold).  Without a pinned or
// tuned choice, the cell kernel from 40,000 atoms on, when its wavefronts, each
// a long chain, come to more than a few per SIMD: 27,000 atoms 35 us against 32
// for variant 0, 48,000 atoms 45 against 51, 98,304 atoms 65 against 96, 261,000
// atoms 136 (variant 1) against 225; from 50,000 on where the cells hold more or
// fewer (46,656 atoms, 460 candidates: 51 against 48; 50,653, 405: 47 against 51).
// Not where the average shows that its cells are no good: mostly empty (a ball of
// 46,656 atoms in a box of 300 A, where few wavefronts get all the cells: 1,733
// us against 63; slabs that fill 0.8, 0.7 and 0.5 of a box 60, 67 and 70 against
// 65 to 66) or much larger than the cutoff (thin boxes: 111 against 53), nor in
// boxes so long that rounding of the coordinates sends many centres to the
// exact predicate (16.5 x 16.5 x 2,400 A: 86 against 48).
int neighbour_variant(const nnp_model& m, int n) {
  if (!cells_fast(m.geo, m.dp.rc_rad)) return 0;
  const int v = stage_variant(m, kTuneNeighbours, n);
  if (v >= 0) return v;
  const float avg = cell_candidates(m, n);
  const float longest = std::max(m.geo.box[0], std::max(m.geo.box[1], m.geo.box[2]));
  if (n < (avg < 375.f || crowded(avg) ? 50000 : 40000) || avg < 300.f || 1.2f * avg > 768.f ||
      longest > 100.f * m.dp.rc_rad)
    return 0;
  return m.geo.n_bins < 48 * m.n_cu ? 2 : 1;
}

hipError_t launch_neighbours(nnp_model& m, int n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  NeighArgs a;
  a.order = m.d_order;
  a.sbin = m.d_sbin;
  a.spos = m.d_spos;
  a.perm = m.d_perm;
  a.key = m.d_key;
  a.bin_start = m.d_bin_start;
  a.n = n;
  a.S = m.S;
  a.rc2 = m.dp.rc_rad * m.dp.rc_rad;
  a.rca2 = m.dp.rc_ang * m.dp.rc_ang;
  {
    const float rm = std::sqrt(a.rc2) + kCullMargin;
    a.cull2 = rm * rm;
  }
  a.rad = m.d_nbr_rad;
  a.ang = m.d_nbr_ang;
  a.rad_off = m.d_rad_off;
  a.ang_off = m.d_ang_off;
  a.max_rad = m.max_rad;
  a.max_ang = m.max_ang;
  a.status = m.d_status;
  a.cut = m.d_cut;
  const int v = neighbour_variant(m, n);
  if (v >= 1) {
    // K wavefronts share a cell
    const int target = v == 1 ? 16 : (v == 2 ? 8 : 4);
    const float per_bin = (float)n / (float)m.geo.n_bins;
    const int K = std::max(1, std::min(64, (int)std::lround(per_bin / target)));
    const bool more = crowded(cell_candidates(m, n));
    auto run = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)(m.geo.n_bins * K)), dim3(64), 0, st, a, m.geo, K);
    };
    if (m.S == 2) run(more ? k_neighbours_cell<2, 12> : k_neighbours_cell<2, 8>);
    else run(more ? k_neighbours_cell<4, 12> : k_neighbours_cell<4, 8>);   // nnp_create accepts two or four species
  } else {
    hipLaunchKernelGGL(k_neighbours, dim3(n), dim3(64), 0, st, a, m.geo);
  }
  return hipGetLastError();
}

hipError_t launch_pair_lists(nnp_model& m, int n, int n_atoms, int n_pairs, const int* pairs, hipStream_t st) {
  if (n == 0) return hipSuccess;
  const PairCount pc = pair_count(m);
  if (n_pairs > 0) {
    hipLaunchKernelGGL(k_pairs_scatter, dim3(blocks_for(n_pairs, kBlock)), dim3(kBlock), 0, st, pairs, n_pairs,
                       m.d_loc, n_atoms, m.d_islot, m.d_spos, m.geo, m.dp.rc_rad * m.dp.rc_rad, m.d_nbr_rad,
                       pc, m.max_rad, m.d_status);
  }
  if (m.n_links_dev > 0) {
    hipLaunchKernelGGL(k_link_pairs, dim3(m.n_links_dev), dim3(64), 0, st, n, m.n_links_dev, m.d_islot, m.d_spos,
                       m.geo, m.dp.rc_rad * m.dp.rc_rad, m.d_nbr_rad, pc, m.max_rad);
  }
  NeighArgs a;
  a.order = m.d_order;
  a.sbin = m.d_sbin;
  a.spos = m.d_spos;
  a.perm = m.d_perm;
  a.key = m.d_key;
  a.bin_start = m.d_bin_start;
  a.n = n;
  a.S = m.S;
  a.rc2 = m.dp.rc_rad * m.dp.rc_rad;
  a.rca2 = m.dp.rc_ang * m.dp.rc_ang;
  {
    const float rm = std::sqrt(a.rc2) + kCullMargin;
    a.cull2 = rm * rm;
  }
  a.rad = m.d_nbr_rad;
  a.ang = m.d_nbr_ang;
  a.rad_off = m.d_rad_off;
  a.ang_off = m.d_ang_off;
  a.max_rad = m.max_rad;
  a.max_ang = m.max_ang;
  a.status = m.d_status;
  a.cut = m.d_cut;
  hipLaunchKernelGGL(k_pairs_lists, dim3(n), dim3(64), 0, st, a, m.geo, pc);
  return hipGetLastError();
}

}  // namespace nnp
