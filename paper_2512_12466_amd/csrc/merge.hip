// Source merging on the GPU (Sec. "Source Merging Algorithm", Alg. source_merge).
//
//   1. snap every source to its cell, sort by (cell, input index) and merge
//      same-cell sources by summing rates in input order;
//   2. max_radius: one wavefront per source grows shells r = k dr <= R_max;
//      the shell's samples are the distinct cells floor(centre + r d_q) over
//      the HEALPix directions d_q of `shell_level` (told apart in LDS, by a
//      bitmap of the cube around the source for radii to 14.5 cells in boxes of
//      31 and more, else by a hash set); a shell passes iff N_ion / N_tot >=
//      f_req, or, below N_min samples, iff every sample is ionized;
//   3. pairs with min-image d^2 <= (f_ov (r_a + r_b))^2 + eps and r_a, r_b > 0
//      are united in a lock-free union-find (the larger root is hooked under
//      the smaller, so a group's root is its lowest member); candidates come
//      from a uniform binning whose bins are wider than any overlap distance;
//   4. (root, index) pairs are sorted so each group's members are contiguous
//      and in order; one wavefront per group sums rates, takes the largest
//      radius, forms the flux-weighted centroid with periodic unwrapping
//      relative to the lowest member, rounds it (floor(c + 1/2)), wraps it and
//      snaps it to the nearest member cell (ties: lowest member);
//   5. the merged catalogue is sorted lexicographically by (i, j, k).
// Every decision uses the FP64 operations written here in this order.
#include <algorithm>
#include <cstring>

#include "healpix.h"
#include "internal.h"

namespace nrt {
namespace {

constexpr unsigned long long kPad = ~0ull;

__device__ __forceinline__ int64_t wrap64(int64_t i, int64_t n) {
  const int64_t r = i % n;
  return r < 0 ? r + n : r;
}

// minimum image of a difference of two cell coordinates, |d| < n <= 4096: a
// step of n instead of an integer division (100 instructions a pair and axis)
__device__ __forceinline__ int min_image(int d, int n, int periodic) {
  if (!periodic) return d;
  d = d < 0 ? d + n : d;
  return 2 * d > n ? d - n : d;
}

// ---- bitonic sort of (key, value) pairs, keys compared then values ----
// Stages whose partners lie within kTile run in LDS, a launch for all of them;
// only the wider ones go through memory, a launch each (2^18 pairs: 36
// launches instead of 171, at 4 us each).
constexpr int kTile = 2048;

__device__ __forceinline__ bool pair_greater(unsigned long long ka, uint32_t va,
                                             unsigned long long kb, uint32_t vb) {
  return ka > kb || (ka == kb && va > vb);
}

__global__ void k_bitonic(unsigned long long* key, uint32_t* val, int64_t count, int64_t k,
                          int64_t j) {
  const int64_t q = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (2 * q >= count) return;
  const int64_t i = 2 * q - (q & (j - 1)), l = i + j;  // the pair's lower index has bit j clear
  const unsigned long long ki = key[i], kl = key[l];
  const uint32_t vi = val[i], vl = val[l];
  if (((i & k) == 0) == pair_greater(ki, vi, kl, vl)) {
    key[i] = kl;
    key[l] = ki;
    val[i] = vl;
    val[l] = vi;
  }
}

// stages (k, j) with k_first <= k <= k_last and j < tile, in LDS; `tile` pairs
// a block (a power of two, at most kTile)
__global__ __launch_bounds__(kTile / 2) void k_bitonic_tile(unsigned long long* key, uint32_t* val,
                                                            int tile, int64_t k_first,
                                                            int64_t k_last) {
  __shared__ unsigned long long sk[kTile];
  __shared__ uint32_t sv[kTile];
  const int64_t base = int64_t(blockIdx.x) * tile;
  for (int i = threadIdx.x; i < tile; i += blockDim.x) {
    sk[i] = key[base + i];
    sv[i] = val[base + i];
  }
  for (int64_t k = k_first; k <= k_last; k <<= 1)
    for (int j = int(k >> 1 < tile >> 1 ? k >> 1 : tile >> 1); j > 0; j >>= 1) {
      __syncthreads();
      const int q = threadIdx.x;
      if (2 * q < tile) {
        const int i = 2 * q - (q & (j - 1)), l = i + j;
        const unsigned long long ki = sk[i], kl = sk[l];
        const uint32_t vi = sv[i], vl = sv[l];
        if ((((base + i) & k) == 0) == pair_greater(ki, vi, kl, vl)) {
          sk[i] = kl;
          sk[l] = ki;
          sv[i] = vl;
          sv[l] = vi;
        }
      }
    }
  __syncthreads();
  for (int i = threadIdx.x; i < tile; i += blockDim.x) {
    key[base + i] = sk[i];
    val[base + i] = sv[i];
  }
}

// ---- step 1: keys of the input sources ----
__global__ void k_source_keys(const double* pos, int64_t m, int64_t pow2, int64_t n,
                              unsigned long long* key, uint32_t* val) {
  const int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s >= pow2) return;
  if (s < m) {
    const int64_t i = int64_t(floor(pos[3 * s])), j = int64_t(floor(pos[3 * s + 1])),
                  k = int64_t(floor(pos[3 * s + 2]));
    key[s] = static_cast<unsigned long long>((i * n + j) * n + k);
    val[s] = uint32_t(s);
  } else {
    key[s] = kPad;
    val[s] = 0xffffffffu;
  }
}

// head flag of each run of equal keys (sorted)
__global__ void k_run_heads(const unsigned long long* key, int64_t m, uint32_t* flag) {
  const int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s >= m) return;
  flag[s] = (s == 0 || key[s] != key[s - 1]) ? 1u : 0u;
}

// exclusive scan, block level: 1024 threads x 1 item; block sums out
__global__ void k_scan_block(const uint32_t* in, uint32_t* out, uint32_t* block_sums,
                             int64_t count) {
  __shared__ uint32_t sh[1024];
  const int64_t i = int64_t(blockIdx.x) * 1024 + threadIdx.x;
  const uint32_t v = i < count ? in[i] : 0u;
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const uint32_t t = threadIdx.x >= unsigned(off) ? sh[threadIdx.x - off] : 0u;
    __syncthreads();
    sh[threadIdx.x] += t;
    __syncthreads();
  }
  if (i < count) out[i] = sh[threadIdx.x] - v;
  if (threadIdx.x == 1023) block_sums[blockIdx.x] = sh[1023];
}

__global__ void k_scan_add(uint32_t* out, const uint32_t* block_offsets, int64_t count) {
  const int64_t i = int64_t(blockIdx.x) * 1024 + threadIdx.x;
  if (i < count) out[i] += block_offsets[blockIdx.x];
}

// dedupe: the head of each run sums the run's rates in input order
__global__ void k_dedupe(const unsigned long long* key, const uint32_t* val, const uint32_t* flag,
                         const uint32_t* slot, const double* ndot, int64_t m, int64_t n,
                         int32_t* cells, double* flux) {
  const int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s >= m || !flag[s]) return;
  double f = ndot[val[s]];
  for (int64_t t = s + 1; t < m && !flag[t]; ++t) f += ndot[val[t]];
  const int64_t o = slot[s];
  const int64_t kk = int64_t(key[s]);
  cells[3 * o] = int32_t(kk / (n * n));
  cells[3 * o + 1] = int32_t((kk / n) % n);
  cells[3 * o + 2] = int32_t(kk % n);
  flux[o] = f;
}

__global__ void k_shell_dirs(int level, int64_t count, double* dirs) {
  const int64_t q = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (q >= count) return;
  double x, y, z;
  healpix_dir(level, uint32_t(q), x, y, z);
  dirs[3 * q] = x;
  dirs[3 * q + 1] = y;
  dirs[3 * q + 2] = z;
}

// ---- step 2: max_radius, one wavefront per source ----
constexpr int kHash = 4096;  // >= 2 x samples per shell (768 at level 3)
constexpr int kWavesPerBlock = 2;

__global__ __launch_bounds__(64 * kWavesPerBlock) void k_max_radius(
    const int32_t* cells, int64_t m, const double* x, int64_t n, int periodic,
    const double* dirs, int nsamp, double dr, double x_th, double f_req, int n_min, double r_max,
    double* radius) {
  __shared__ unsigned long long table[kWavesPerBlock][kHash];
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int64_t s = int64_t(blockIdx.x) * kWavesPerBlock + wave;
  if (s >= m) return;  // whole wavefront leaves together
  unsigned long long* tab = table[wave];
  const int64_t ci = cells[3 * s], cj = cells[3 * s + 1], ck = cells[3 * s + 2];
  if (x[ci + n * (cj + n * ck)] < x_th) {
    if (lane == 0) radius[s] = 0.0;
    return;
  }
  double result = r_max;
  for (int64_t kk = 1;; ++kk) {
    const double r = double(kk) * dr;
    if (!(r <= r_max)) break;
    for (int q = lane; q < kHash; q += 64) tab[q] = kPad;
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    int ntot = 0, nion = 0;
    for (int q = lane; q < nsamp; q += 64) {
      const double p0 = (double(ci) + 0.5) + r * dirs[3 * q];
      const double p1 = (double(cj) + 0.5) + r * dirs[3 * q + 1];
      const double p2 = (double(ck) + 0.5) + r * dirs[3 * q + 2];
      int64_t v0 = int64_t(floor(p0)), v1 = int64_t(floor(p1)), v2 = int64_t(floor(p2));
      if (periodic) {
        v0 = wrap64(v0, n);
        v1 = wrap64(v1, n);
        v2 = wrap64(v2, n);
      } else if (v0 < 0 || v0 >= n || v1 < 0 || v1 >= n || v2 < 0 || v2 >= n) {
        continue;
      }
      const unsigned long long cell = static_cast<unsigned long long>(v0 + n * (v1 + n * v2));
      unsigned h = unsigned((cell * 0x9E3779B97F4A7C15ull) >> 52) & (kHash - 1);
      for (;;) {
        const unsigned long long prev = atomicCAS(&tab[h], kPad, cell);
        if (prev == kPad) {  // first time this cell is seen
          ++ntot;
          if (x[cell] >= x_th) ++nion;
          break;
        }
        if (prev == cell) break;
        h = (h + 1) & (kHash - 1);
      }
    }
    for (int off = 32; off > 0; off >>= 1) {
      ntot += __shfl_xor(ntot, off);
      nion += __shfl_xor(nion, off);
    }
    bool pass;
    if (ntot < n_min)
      pass = (nion == ntot);
    else
      pass = !(double(nion) / double(ntot) < f_req);
    __builtin_amdgcn_wave_barrier();
    if (!pass) {
      result = r - dr;
      break;
    }
  }
  if (lane == 0) radius[s] = result;
}

// The same for radii within kNearReach - 1 cells: a shell's samples lie in the
// cube of 2 kNearReach + 1 cells around the source, so a bitmap of the cube
// tells which cells were seen (distinct offsets are distinct cells while the
// cube fits the box, so the caller checks n).  A bitmap of 4 KB a wavefront in
// place of a 32 KB hash table gives 8 times the wavefronts a CU, and the
// wrapped coordinates come from one conditional step each instead of an
// integer division (1024^3, 262144 sources: 12.4 ms by the hash table).
constexpr int kNearReach = 15;
constexpr int kNearWords = 32 * 32;  // bit x + 1 of word (y + 16) + 32 (z + 16)
constexpr int kNearWaves = 4;

__global__ __launch_bounds__(64 * kNearWaves) void k_max_radius_near(
    const int32_t* __restrict__ cells, int64_t m, const double* __restrict__ x, int n,
    int periodic, const double* __restrict__ dirs, int nsamp, double dr, double x_th,
    double f_req, int n_min, double r_max, double* radius) {
  __shared__ uint32_t seen[kNearWaves][kNearWords];
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int64_t s = int64_t(blockIdx.x) * kNearWaves + wave;
  if (s >= m) return;  // whole wavefront leaves together
  uint32_t* bits = seen[wave];
  const int ci = cells[3 * s], cj = cells[3 * s + 1], ck = cells[3 * s + 2];
  if (x[ci + int64_t(n) * (cj + int64_t(n) * ck)] < x_th) {
    if (lane == 0) radius[s] = 0.0;
    return;
  }
  double result = r_max;
  for (int64_t kk = 1;; ++kk) {
    const double r = double(kk) * dr;
    if (!(r <= r_max)) break;
    for (int q = lane; q < kNearWords; q += 64) bits[q] = 0u;
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    int ntot = 0, nion = 0;
    for (int q = lane; q < nsamp; q += 64) {
      int v0 = int(floor((double(ci) + 0.5) + r * dirs[3 * q]));
      int v1 = int(floor((double(cj) + 0.5) + r * dirs[3 * q + 1]));
      int v2 = int(floor((double(ck) + 0.5) + r * dirs[3 * q + 2]));
      const uint32_t bit = 1u << (v0 - ci + kNearReach + 1);
      const int word = (v1 - cj + kNearReach + 1) + 32 * (v2 - ck + kNearReach + 1);
      if (periodic) {
        v0 = v0 < 0 ? v0 + n : (v0 >= n ? v0 - n : v0);
        v1 = v1 < 0 ? v1 + n : (v1 >= n ? v1 - n : v1);
        v2 = v2 < 0 ? v2 + n : (v2 >= n ? v2 - n : v2);
      } else if (v0 < 0 || v0 >= n || v1 < 0 || v1 >= n || v2 < 0 || v2 >= n) {
        continue;
      }
      if (!(atomicOr(&bits[word], bit) & bit)) {  // first time this cell is seen
        ++ntot;
        if (x[v0 + int64_t(n) * (v1 + int64_t(n) * v2)] >= x_th) ++nion;
      }
    }
    for (int off = 32; off > 0; off >>= 1) {
      ntot += __shfl_xor(ntot, off);
      nion += __shfl_xor(nion, off);
    }
    bool pass;
    if (ntot < n_min)
      pass = (nion == ntot);
    else
      pass = !(double(nion) / double(ntot) < f_req);
    __builtin_amdgcn_wave_barrier();
    if (!pass) {
      result = r - dr;
      break;
    }
  }
  if (lane == 0) radius[s] = result;
}

// ---- step 3: binning and union-find ----
__global__ void k_bin_count(const int32_t* cells, const double* radius, int64_t m, int64_t n,
                            int64_t nb, uint32_t* bin_of, uint32_t* counts) {
  const int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s >= m) return;
  if (!(radius[s] > 0.0)) {
    bin_of[s] = 0xffffffffu;
    return;
  }
  const int64_t b = (cells[3 * s] * nb / n) + nb * ((cells[3 * s + 1] * nb / n) +
                                                    nb * (cells[3 * s + 2] * nb / n));
  bin_of[s] = uint32_t(b);
  atomicAdd(&counts[b], 1u);
}

__global__ void k_bin_fill(const uint32_t* bin_of, int64_t m, uint32_t* cursor,
                           uint32_t* members) {
  const int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s >= m || bin_of[s] == 0xffffffffu) return;
  const uint32_t p = atomicAdd(&cursor[bin_of[s]], 1u);
  members[p] = uint32_t(s);
}

__device__ int uf_find(int* parent, int a) {
  for (;;) {
    const int p = __hip_atomic_load(&parent[a], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (p == a) return a;
    a = p;
  }
}

__device__ void uf_unite(int* parent, int a, int b) {
  for (;;) {
    a = uf_find(parent, a);
    b = uf_find(parent, b);
    if (a == b) return;
    if (a < b) {
      const int t = a;
      a = b;
      b = t;
    }  // hook the larger root a under the smaller b
    if (atomicCAS(&parent[a], a, b) == a) return;
  }
}

__device__ bool overlaps(const int32_t* ca, const int32_t* cb, double ra, double rb, int64_t n,
                         int periodic, double f_ov, double eps) {
  if (!(ra > 0.0 && rb > 0.0)) return false;
  double d2 = 0.0;
  for (int ax = 0; ax < 3; ++ax) {
    const double dd = double(min_image(ca[ax] - cb[ax], int(n), periodic));
    d2 += dd * dd;
  }
  const double rsum = f_ov * (ra + rb);
  return d2 <= rsum * rsum + eps;
}

// Half a wavefront per source: 27 lanes look up the bins around it, and the 32
// share the candidates of each bin that is not empty.  The kernel waits for
// dependent loads: a thread per source walks all its candidates one after
// another (512^3, 32768 sources: 418 us), a wavefront per source leaves too few
// sources in flight (1024^3, 262144 sources: 1519 us).
constexpr int kPairBlock = 256;

__global__ __launch_bounds__(kPairBlock) void k_pairs_binned(
    const int32_t* __restrict__ cells, const double* __restrict__ radius,
    const uint32_t* __restrict__ bin_of, const uint32_t* __restrict__ start,
    const uint32_t* __restrict__ counts, const uint32_t* __restrict__ members, int64_t m,
    int64_t n, int nb, int periodic, double f_ov, double eps, int* parent) {
  const int64_t a = int64_t(blockIdx.x) * (kPairBlock / 32) + threadIdx.x / 32;
  const int lane = threadIdx.x % 32;
  if (a >= m || bin_of[a] == 0xffffffffu) return;  // the source's 32 lanes leave together
  const int b0 = int(bin_of[a]);
  int qx = b0 % nb + lane % 3 - 1, qy = b0 / nb % nb + lane / 3 % 3 - 1,
      qz = b0 / (nb * nb) + lane / 9 - 1;
  bool in = lane < 27;
  if (periodic) {
    qx = qx < 0 ? qx + nb : (qx >= nb ? qx - nb : qx);
    qy = qy < 0 ? qy + nb : (qy >= nb ? qy - nb : qy);
    qz = qz < 0 ? qz + nb : (qz >= nb ? qz - nb : qz);
  } else {
    in = in && qx >= 0 && qx < nb && qy >= 0 && qy < nb && qz >= 0 && qz < nb;
  }
  uint32_t first = 0, count = 0;
  if (in) {
    const int q = qx + nb * (qy + nb * qz);
    first = start[q];
    count = counts[q];
  }
  for (uint32_t left = uint32_t(__ballot(count != 0) >> (threadIdx.x & 32)); left;
       left &= left - 1) {
    const int q = __builtin_ctz(left);
    const uint32_t t0 = __shfl(first, q, 32), e = t0 + __shfl(count, q, 32);
    for (uint32_t t = t0 + lane; t < e; t += 32) {
      const int64_t b = members[t];
      if (b > a && overlaps(cells + 3 * a, cells + 3 * b, radius[a], radius[b], n, periodic,
                            f_ov, eps))
        uf_unite(parent, int(a), int(b));
    }
  }
}

__global__ void k_pairs_all(const int32_t* cells, const double* radius, int64_t m, int64_t n,
                            int periodic, double f_ov, double eps, int* parent) {
  const int64_t a = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (a >= m || !(radius[a] > 0.0)) return;
  for (int64_t b = a + 1; b < m; ++b)
    if (overlaps(cells + 3 * a, cells + 3 * b, radius[a], radius[b], n, periodic, f_ov, eps))
      uf_unite(parent, int(a), int(b));
}

__global__ void k_iota(int* parent, int64_t m) {
  const int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s < m) parent[s] = int(s);
}

// ---- step 4: groups ----
__global__ void k_root_keys(int* parent, int64_t m, int64_t pow2, unsigned long long* key,
                            uint32_t* val) {
  const int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s >= pow2) return;
  if (s < m) {
    key[s] = static_cast<unsigned long long>(uf_find(parent, int(s)));
    val[s] = uint32_t(s);
  } else {
    key[s] = kPad;
    val[s] = 0xffffffffu;
  }
}

// One wavefront per group: its lanes load 64 members at a time, and every lane
// sums them in member order from the others' registers (the rates and the
// centroid keep the order of a serial loop, without its chain of loads: 512^3,
// 32768 sources: 259 us with a thread per group).
constexpr int kGroupWaves = 4;

__global__ __launch_bounds__(64 * kGroupWaves) void k_collapse(
    const uint32_t* __restrict__ member, const uint32_t* __restrict__ head, int64_t groups,
    int64_t m, const int32_t* __restrict__ cells, const double* __restrict__ flux,
    const double* __restrict__ radius, int n, int periodic, int32_t* out_cells, double* out_flux,
    double* out_radius) {
  const int64_t o = int64_t(blockIdx.x) * kGroupWaves + threadIdx.x / 64;
  const int lane = threadIdx.x % 64;
  if (o >= groups) return;  // whole wavefront leaves together
  const int64_t s = head[o], e = o + 1 < groups ? int64_t(head[o + 1]) : m;
  const int64_t a = member[s];  // lowest member
  const int a0 = cells[3 * a], a1 = cells[3 * a + 1], a2 = cells[3 * a + 2];
  double ftot = 0.0, rmax = 0.0, c0 = 0.0, c1 = 0.0, c2 = 0.0;
  if (e - s == 1) {
    ftot = flux[a];
    rmax = radius[a];
  }
  for (int64_t t = s; t < e && e - s > 1; t += 64) {
    const int have = int(e - t < 64 ? e - t : 64);
    double f = 0.0, r = 0.0, u0 = 0.0, u1 = 0.0, u2 = 0.0;
    if (lane < have) {
      const int64_t b = member[t + lane];
      f = flux[b];
      r = radius[b];
      u0 = f * double(a0 + min_image(cells[3 * b] - a0, n, periodic));
      u1 = f * double(a1 + min_image(cells[3 * b + 1] - a1, n, periodic));
      u2 = f * double(a2 + min_image(cells[3 * b + 2] - a2, n, periodic));
    }
    for (int q = 0; q < have; ++q) {
      ftot += __shfl(f, q);
      const double rq = __shfl(r, q);
      if (rq > rmax) rmax = rq;
      c0 += __shfl(u0, q);
      c1 += __shfl(u1, q);
      c2 += __shfl(u2, q);
    }
  }
  int64_t best = a;
  if (e - s > 1) {
    int rnd[3];
    const double cen[3] = {c0 / ftot, c1 / ftot, c2 / ftot};
    for (int ax = 0; ax < 3; ++ax) {
      const int64_t v = int64_t(floor(cen[ax] + 0.5));
      rnd[ax] = int(periodic ? wrap64(v, n) : v);
    }
    // nearest member cell, the lowest-sorted of equals
    unsigned long long low = ~0ull;
    for (int64_t t = s + lane; t < e; t += 64) {
      const int64_t b = member[t];
      unsigned long long d2 = 0;
      for (int ax = 0; ax < 3; ++ax) {
        const int64_t dd = min_image(cells[3 * b + ax] - rnd[ax], n, periodic);
        d2 += static_cast<unsigned long long>(dd * dd);
      }
      const unsigned long long w = d2 << 32 | static_cast<unsigned long long>(t - s);
      low = w < low ? w : low;
    }
    for (int off = 32; off > 0; off >>= 1) {
      const unsigned long long w = __shfl_xor(low, off);
      low = w < low ? w : low;
    }
    best = member[s + int64_t(low & 0xffffffffull)];
  }
  if (lane < 3) out_cells[3 * o + lane] = cells[3 * best + lane];
  if (lane == 0) {
    out_flux[o] = ftot;
    out_radius[o] = rmax;
  }
}

// first member of each group
__global__ void k_group_heads(const uint32_t* flag, const uint32_t* slot, int64_t m,
                              uint32_t* head) {
  const int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s < m && flag[s]) head[slot[s]] = uint32_t(s);
}

// ---- step 5: final order ----
__global__ void k_cell_keys(const int32_t* cells, int64_t m, int64_t pow2, int64_t n,
                            unsigned long long* key, uint32_t* val) {
  const int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s >= pow2) return;
  if (s < m) {
    key[s] = static_cast<unsigned long long>((int64_t(cells[3 * s]) * n + cells[3 * s + 1]) * n +
                                             cells[3 * s + 2]);
    val[s] = uint32_t(s);
  } else {
    key[s] = kPad;
    val[s] = 0xffffffffu;
  }
}

__global__ void k_emit(const uint32_t* order, int64_t m, const int32_t* cells, const double* flux,
                       const double* radius, double* out) {
  const int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s >= m) return;
  const int64_t g = order[s];
  out[6 * s] = double(cells[3 * g]) + 0.5;
  out[6 * s + 1] = double(cells[3 * g + 1]) + 0.5;
  out[6 * s + 2] = double(cells[3 * g + 2]) + 0.5;
  out[6 * s + 3] = flux[g];
  out[6 * s + 4] = radius[g];
  out[6 * s + 5] = 0.0;
}

unsigned blocks_for(int64_t items, int block) {
  return unsigned(std::max<int64_t>(1, (items + block - 1) / block));
}


static size_t align256z(size_t x) { return (x + 255) & ~size_t(255); }

// exclusive scan of count uint32 values; tmp holds >= 3 (count / 1024 + 16) words
static hipError_t scan_u32(const uint32_t* in, uint32_t* out, int64_t count, uint32_t* tmp,
                           hipStream_t st) {
  const int64_t nb1 = (count + 1023) / 1024;
  hipLaunchKernelGGL(k_scan_block, dim3(unsigned(std::max<int64_t>(nb1, 1))), dim3(1024), 0, st,
                     in, out, tmp, count);
  if (nb1 > 1) {
    uint32_t* sums = tmp;
    uint32_t* offs = tmp + nb1;
    uint32_t* next = offs + nb1;
    hipError_t e = scan_u32(sums, offs, nb1, next, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_scan_add, dim3(unsigned(nb1)), dim3(1024), 0, st, out, offs, count);
  }
  return hipGetLastError();
}

static void bitonic(unsigned long long* key, uint32_t* val, int64_t pow2, hipStream_t st) {
  const int tile = int(std::min<int64_t>(pow2, kTile));
  if (tile < 2) return;
  const dim3 tiles(unsigned(pow2 / tile)), threads(tile / 2);
  hipLaunchKernelGGL(k_bitonic_tile, tiles, threads, 0, st, key, val, tile, int64_t(2),
                     int64_t(tile));
  for (int64_t k = 2 * int64_t(tile); k <= pow2; k <<= 1) {
    for (int64_t j = k >> 1; j >= tile; j >>= 1)
      hipLaunchKernelGGL(k_bitonic, dim3(blocks_for(pow2 / 2, 256)), dim3(256), 0, st, key, val,
                         pow2, k, j);
    hipLaunchKernelGGL(k_bitonic_tile, tiles, threads, 0, st, key, val, tile, k, k);
  }
}

static hipError_t read_count(const uint32_t* slot, const uint32_t* flag, int64_t m,
                             hipStream_t st, int64_t* out) {
  uint32_t v[2] = {0, 0};
  hipError_t e = hipMemcpyAsync(&v[0], slot + m - 1, 4, hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipMemcpyAsync(&v[1], flag + m - 1, 4, hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  *out = int64_t(v[0]) + v[1];
  return e;
}

}  // namespace

size_t merge_bytes_per_source() { return 256; }

// Runs the merge of the context's m sources (positions already on the
// device in src_pos, rates given on the host); out6 receives, per merged
// source in lexicographic order, (x, y, z, rate, radius, 0).
hipError_t run_merge(nrt_ctx* c, const nrt_merge_params& mp, const double* h_ndot, int64_t m,
                     std::vector<double>& out6, std::string& why) {
  const int64_t n = c->desc.n;
  const int periodic = c->desc.periodic;
  hipStream_t st = c->stream;
  int64_t pow2 = 1;
  while (pow2 < m) pow2 <<= 1;
  char* base = c->ws + c->lay.srcaux;
  char* p = base;
  auto take = [&](size_t bytes) {
    char* q = p;
    p += align256z(bytes);
    return q;
  };
  auto* key = reinterpret_cast<unsigned long long*>(take(size_t(pow2) * 8));
  auto* val = reinterpret_cast<uint32_t*>(take(size_t(pow2) * 4));
  auto* flag = reinterpret_cast<uint32_t*>(take(size_t(m) * 4));
  auto* slot = reinterpret_cast<uint32_t*>(take(size_t(m) * 4));
  auto* cells = reinterpret_cast<int32_t*>(take(size_t(m) * 12));
  auto* flux = reinterpret_cast<double*>(take(size_t(m) * 8));
  auto* radius = reinterpret_cast<double*>(take(size_t(m) * 8));
  auto* parent = reinterpret_cast<int*>(take(size_t(m) * 4));
  auto* bin_of = reinterpret_cast<uint32_t*>(take(size_t(m) * 4));
  auto* members = reinterpret_cast<uint32_t*>(take(size_t(m) * 4));
  auto* ocells = reinterpret_cast<int32_t*>(take(size_t(m) * 12));
  auto* oflux = reinterpret_cast<double*>(take(size_t(m) * 8));
  auto* orad = reinterpret_cast<double*>(take(size_t(m) * 8));
  auto* d_ndot = reinterpret_cast<double*>(take(size_t(m) * 8));
  auto* d_out6 = reinterpret_cast<double*>(take(size_t(m) * 48));
  if (size_t(p - base) > size_t(c->lay.max_sources) * merge_bytes_per_source() + 16 * 256) {
    why = "merge scratch exceeds the source area";
    return hipErrorInvalidValue;
  }
  // general scratch: shell directions, scan temporaries, bins
  const int nsamp = 12 << (2 * mp.shell_level);
  const double reach = 2.0 * mp.f_ov * mp.r_max + std::sqrt(std::max(mp.eps, 0.0)) + 1.0;
  auto scratch_need = [&](int64_t nbins) {
    const int64_t big = std::max(m, nbins);
    return align256z(size_t(nsamp) * 24) + align256z((size_t(big) / 1024 + 16) * 12) +
           3 * align256z(size_t(nbins) * 4);
  };
  const int64_t nb = merge_bins(n, reach, c->scratch_bytes, scratch_need);
  if (scratch_need(nb * nb * nb) > c->scratch_bytes) {
    why = "merge scratch exceeds the workspace scratch";
    return hipErrorInvalidValue;
  }
  const int64_t nbin = nb * nb * nb;
  char* g = c->scratch;
  auto gtake = [&](size_t bytes) {
    char* q = g;
    g += align256z(bytes);
    return q;
  };
  auto* dirs = reinterpret_cast<double*>(gtake(size_t(nsamp) * 24));
  auto* scan_tmp = reinterpret_cast<uint32_t*>(gtake((size_t(std::max(m, nbin)) / 1024 + 16) * 12));
  auto* bcount = reinterpret_cast<uint32_t*>(gtake(size_t(nbin) * 4));
  auto* bstart = reinterpret_cast<uint32_t*>(gtake(size_t(nbin) * 4));
  auto* bcursor = reinterpret_cast<uint32_t*>(gtake(size_t(nbin) * 4));

  hipError_t e = hipMemcpyAsync(d_ndot, h_ndot, size_t(m) * 8, hipMemcpyHostToDevice, st);
  if (e != hipSuccess) return e;

  // 1. snap, sort by (cell, input index), merge same-cell sources
  hipLaunchKernelGGL(k_source_keys, dim3(blocks_for(pow2, 256)), dim3(256), 0, st, c->src_pos, m,
                     pow2, n, key, val);
  bitonic(key, val, pow2, st);
  hipLaunchKernelGGL(k_run_heads, dim3(blocks_for(m, 256)), dim3(256), 0, st, key, m, flag);
  if ((e = scan_u32(flag, slot, m, scan_tmp, st)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_dedupe, dim3(blocks_for(m, 256)), dim3(256), 0, st, key, val, flag, slot,
                     d_ndot, m, n, cells, flux);
  int64_t m1 = 0;
  if ((e = read_count(slot, flag, m, st, &m1)) != hipSuccess) return e;

  // 2. bubble radii
  hipLaunchKernelGGL(k_shell_dirs, dim3(blocks_for(nsamp, 256)), dim3(256), 0, st,
                     mp.shell_level, int64_t(nsamp), dirs);
  // samples lie within floor(1/2 + r) <= kNearReach cells of the source's
  if (mp.r_max <= kNearReach - 0.5 && n >= 2 * kNearReach + 1)
    hipLaunchKernelGGL(k_max_radius_near, dim3(blocks_for(m1, kNearWaves)),
                       dim3(64 * kNearWaves), 0, st, cells, m1, c->x, int(n), periodic, dirs,
                       nsamp, mp.dr, mp.x_th, mp.f_req, mp.n_min, mp.r_max, radius);
  else
    hipLaunchKernelGGL(k_max_radius, dim3(blocks_for(m1, kWavesPerBlock)),
                       dim3(64 * kWavesPerBlock), 0, st, cells, m1, c->x, n, periodic, dirs,
                       nsamp, mp.dr, mp.x_th, mp.f_req, mp.n_min, mp.r_max, radius);

  // 3. overlaps and union-find
  hipLaunchKernelGGL(k_iota, dim3(blocks_for(m1, 256)), dim3(256), 0, st, parent, m1);
  if (nb == 1) {
    hipLaunchKernelGGL(k_pairs_all, dim3(blocks_for(m1, 256)), dim3(256), 0, st, cells, radius,
                       m1, n, periodic, mp.f_ov, mp.eps, parent);
  } else {
    if ((e = hipMemsetAsync(bcount, 0, size_t(nbin) * 4, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_bin_count, dim3(blocks_for(m1, 256)), dim3(256), 0, st, cells, radius,
                       m1, n, nb, bin_of, bcount);
    if ((e = scan_u32(bcount, bstart, nbin, scan_tmp, st)) != hipSuccess) return e;
    e = hipMemcpyAsync(bcursor, bstart, size_t(nbin) * 4, hipMemcpyDeviceToDevice, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bin_fill, dim3(blocks_for(m1, 256)), dim3(256), 0, st, bin_of, m1,
                       bcursor, members);
    hipLaunchKernelGGL(k_pairs_binned, dim3(blocks_for(m1, kPairBlock / 32)), dim3(kPairBlock),
                       0, st, cells, radius, bin_of, bstart, bcount, members, m1, n, int(nb),
                       periodic, mp.f_ov, mp.eps, parent);
  }

  // 4. collapse each group (members contiguous and in order after the sort)
  int64_t pow2b = 1;
  while (pow2b < m1) pow2b <<= 1;
  hipLaunchKernelGGL(k_root_keys, dim3(blocks_for(pow2b, 256)), dim3(256), 0, st, parent, m1,
                     pow2b, key, val);
  bitonic(key, val, pow2b, st);
  hipLaunchKernelGGL(k_run_heads, dim3(blocks_for(m1, 256)), dim3(256), 0, st, key, m1, flag);
  if ((e = scan_u32(flag, slot, m1, scan_tmp, st)) != hipSuccess) return e;
  // the bins are no longer needed: their members' array takes the group heads
  hipLaunchKernelGGL(k_group_heads, dim3(blocks_for(m1, 256)), dim3(256), 0, st, flag, slot, m1,
                     members);
  int64_t m2 = 0;
  if ((e = read_count(slot, flag, m1, st, &m2)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_collapse, dim3(blocks_for(m2, kGroupWaves)), dim3(64 * kGroupWaves), 0, st,
                     val, members, m2, m1, cells, flux, radius, int(n), periodic, ocells, oflux,
                     orad);

  // 5. lexicographic order
  int64_t pow2c = 1;
  while (pow2c < m2) pow2c <<= 1;
  hipLaunchKernelGGL(k_cell_keys, dim3(blocks_for(pow2c, 256)), dim3(256), 0, st, ocells, m2,
                     pow2c, n, key, val);
  bitonic(key, val, pow2c, st);
  hipLaunchKernelGGL(k_emit, dim3(blocks_for(m2, 256)), dim3(256), 0, st, val, m2, ocells, oflux,
                     orad, d_out6);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  out6.resize(size_t(m2) * 6);
  e = hipMemcpyAsync(out6.data(), d_out6, size_t(m2) * 48, hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  return e;
}

}  // namespace nrt
