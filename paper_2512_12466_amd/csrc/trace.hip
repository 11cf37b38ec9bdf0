// Ray-tracing kernels for gfx950: absorber preparation and the march.
//
// The march (Alg. trace_rays, Alg. functors) runs one ray per lane.  Rays
// are held in level queues (structure of arrays); a launch takes a range of
// one level's queue, marches every ray until it stops, accumulates the
// photon budget per lane, and appends the four children of every ray that
// splits to the next level's queue.  Children are allocated per wavefront:
// a ballot of the splitting lanes, one atomicAdd by the first of them, and
// each lane's slot from a masked lane count.
//
// Decisions (next cell, split, stop tests, face of the overlap correction)
// are FP64 in both precisions and use only correctly rounded + - * / (the
// library is compiled with FP contraction off).  The optical depth that the
// tau_max stop reads is one of them: both precisions accumulate it in FP64
// from the FP64 absorber by the same operations, so the two paths march the
// same segments and split the same rays.  MIXED = true computes the
// attenuation, the deposits and the correction factors in FP32 (the
// neighbour's absorber rounded from its FP64 word), sums the deposits of
// HEALPix levels 0..4 in FP32 and of the deeper ones in FP64 (template V),
// and tracks the transmitted fraction in FP64.  POLY = true integrates the flux
// over a source spectrum with the table of Phi(tau) = -ln F(tau) built at
// context set-up (spectrum.hip).  The march is instantiated per precision,
// correction mode, boundary, spectrum, type of the sums and of the cell index.
#include <cfloat>
#include <cmath>
#include <type_traits>

#include "healpix.h"
#include "internal.h"

namespace nrt {

namespace {

// wrapped coordinate; cells lie within a few box lengths of the box, so
// whole-box steps replace the integer division (which the compiler would make
// of the loops again, hence the empty asm)
__device__ __forceinline__ int wrap_cell(int i, int n) {
#pragma unroll 1
  while (i < 0) {
    i += n;
    asm volatile("" : "+v"(i));
  }
#pragma unroll 1
  while (i >= n) {
    i -= n;
    asm volatile("" : "+v"(i));
  }
  return i;
}

// Flat index of the wrapped cell (w0, w1, w2), x fastest.  n <= 4096, so the
// plane index w1 + n w2 fits 24 bits and one 32 x 32 -> 64 multiply-add
// finishes the index.
__device__ __forceinline__ int64_t cell_index(int w0, int w1, int w2, int n) {
  const uint32_t plane = uint32_t(w1) + __umul24(uint32_t(n), uint32_t(w2));
  return int64_t(uint64_t(uint32_t(w0)) + uint64_t(uint32_t(n)) * uint64_t(plane));
}

// start cell of a ray at q = o + s d: floor(q), except that an exact integer
// with a negative direction component belongs to the cell below
__device__ __forceinline__ int start_cell(double o, double s, double d) {
  const double q = o + s * d;
  const double f = floor(q);
  int i = int(f);
  if (q == f && d < 0.0) i -= 1;
  return i;
}

__device__ __forceinline__ unsigned lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi(unsigned(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo(unsigned(mask), 0u));
}

__device__ __forceinline__ unsigned long long read_lane64(unsigned long long v, int lane) {
  const unsigned lo = __builtin_amdgcn_readlane(unsigned(v), lane);
  const unsigned hi = __builtin_amdgcn_readlane(unsigned(v >> 32), lane);
  return (static_cast<unsigned long long>(hi) << 32) | lo;
}

// The march's argument block, read through a pointer that the compiler must
// treat as new at every use: values read this way are re-read from the
// (scalar-cached) argument segment where they are used instead of being held
// in scalar registers across the whole loop.  The ray set-up reads its many
// pointers like this, which leaves the per-step path its registers.
using ArgsK = const MarchArgs __attribute__((address_space(4)));
__device__ __forceinline__ ArgsK& fresh_args() {
  ArgsK* p = (ArgsK*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *p;
}

struct LaneAcc {
  double absorbed = 0.0, escaped = 0.0, truncated = 0.0;
  uint32_t segments = 0;  // of one lane, since they were last added up
};

// Per-wavefront Gamma accumulator in LDS.  A wavefront marches rays claimed
// in runs of consecutive queue entries; nested HEALPix order is a Z-order
// curve and children are queued next to each other, so such a run is a
// bundle of neighbouring pixels of one source and level, and by the split
// rule it crosses each cell several times.  Deposits are summed in a hash
// table whose slots are 64-byte lines of Gamma (kLine consecutive cells along
// x), and folded into Gamma when enough of the slots are taken: the device
// performs FP64 atomics per 64-byte line request, so the flush, in which
// lanes 8j..8j+7 of an instruction cover the cells of one line, costs one
// request per line instead of one per cell.
//
// What bounds it is the LDS pipe.  Measured on MI355X with 16 wavefronts a
// CU, in cycles per wavefront instruction: a 4-byte read 7.8 whatever the
// addresses; a compare-and-swap 10.6, but 35 / 64 when 4 / 8 lanes share an
// address; an FP64 add 13.6, 48 / 96; an FP32 add 198, 244 / 253 (it takes the
// lanes one by one).  So a deposit reads its slot's key and swaps only where
// its line is new, instead of a swap by every lane, and deposits are summed
// in FP64 (see march_kernel for the exception).  A deposit that finds no slot
// within kProbe probes goes straight to Gamma, and on grids whose lines do not
// fit the 32-bit keys (n >= 3251; the 64-bit cell index only) all of them do.
constexpr int kWaves = kBlock / 64;
constexpr int kLine = 8;
constexpr int kProbe = 16;
constexpr uint32_t kEmpty = 0xffffffffu;

// Sizes at which the march's cell index, table and counts change.  A second
// build of the library, for the tests, sets them so that small grids take the
// 64-bit index, both sides of the table's limit and the early sums.
#ifndef NRT_NARROW_CELLS
#define NRT_NARROW_CELLS (int64_t(1) << 32)  // most cells of the 32-bit index
#endif
#ifndef NRT_TABLE_LINES
#define NRT_TABLE_LINES int64_t(kEmpty)  // lines below this many have a key
#endif

#ifndef NRT_SEGMENT_FOLD
#define NRT_SEGMENT_FOLD (uint32_t(1) << 31)  // a lane's segments that are added up early
#endif

template <typename V, typename Idx>
struct LineTable {
  // line slots per wavefront: 37 KiB (FP32 sums) or 34.5 KiB (FP64) per block
  static constexpr int kLog2Lines = sizeof(V) == 4 ? kLog2LinesFp32 : kLog2LinesFp64;
  static constexpr int kLines = 1 << kLog2Lines;
  // slots in use that make a fold, checked every 8 cells (about 35 new lines):
  // at an eighth (FP64) against a quarter 128^3 mixed takes 10.59 / 10.75 ms; at
  // three eighths 11.2, at a half 11.9, for probes in a fuller table
  static constexpr int kFlushAt = sizeof(V) == 4 ? kLines / 4 : kLines / 8;
  static constexpr size_t kWaveBytes =
      kLines * (sizeof(uint32_t) + sizeof(uint8_t) + kLine * sizeof(V));

  uint32_t* key;  // [kLines] line index (cell >> 3) or kEmpty
  V* val;         // [kLines * kLine] partial sums of the line's cells
  uint8_t* list;  // [kLines] slots in use, compacted by a flush
  uint32_t mul;   // multiplier of the slot hash (line_multiplier)
  bool keys_fit;  // of a grid with the 64-bit index

  __device__ __forceinline__ bool staged() const { return sizeof(Idx) == 4 || keys_fit; }

  // First slot of the line of cell c and the key it holds, read ahead of the
  // arithmetic that precedes the deposit.
  struct Look {
    uint32_t k, h, old;
  };
  __device__ __forceinline__ Look look(Idx c) const {
    Look l;
    l.k = uint32_t(c >> 3);
    uint32_t product;  // full rate; the compiler would take the 32-bit multiply
    asm("v_mul_u32_u24 %0, %1, %2" : "=v"(product) : "s"(mul), "v"(l.k));
    l.h = (product >> (24 - kLog2Lines)) & uint32_t(kLines - 1);
    l.old = key[l.h];
    return l;
  }

  // Take the slot of a line that it did not hold when it was read (lanes with
  // claim); counts a new line in `inserted`.  After it, l.old == l.k tells
  // that the slot is the line's.
  __device__ __forceinline__ void claim(Look& l, bool claim, int& inserted) const {
    if (claim && l.old != l.k && staged()) {
      l.old = atomicCAS(&key[l.h], kEmpty, l.k);
      if (l.old == kEmpty) {
        l.old = l.k;
        ++inserted;
      }
    }
  }

  // add v for cell c (lanes with want) to the line's slot, probing further
  // (lanes with claim) if its first slot belongs to another line
  __device__ __forceinline__ void deposit(Look& l, Idx c, V v, bool claim, bool want,
                                          int& inserted) const {
    if (!staged()) {
      if (want) atomicAdd(fresh_args().gamma + c, double(v));
      return;
    }
    const uint32_t sub = uint32_t(c) & uint32_t(kLine - 1);
    if (claim && l.old != l.k) {
#pragma unroll 1
      for (int probe = 1; probe < kProbe; ++probe) {
        l.h = (l.h + 1) & uint32_t(kLines - 1);
        l.old = atomicCAS(&key[l.h], kEmpty, l.k);
        if (l.old == kEmpty || l.old == l.k) break;
      }
      if (l.old == kEmpty) {
        l.old = l.k;
        ++inserted;
      }
      if (want && l.old != l.k) atomicAdd(fresh_args().gamma + c, double(v));
    }
    if (want && l.old == l.k) atomicAdd(&val[l.h * kLine + sub], v);
  }

  // whole wavefront: fold the table into Gamma and clear it (LDS operations
  // of one wavefront complete in program order).  The slots in use are listed
  // first, so that the fold takes 8 lines an iteration however few they are.
  // Cells of a line that got no deposit hold zero and are skipped, so no
  // address past the grid is formed.
  __device__ __forceinline__ void flush(int lane) const {
    double* gamma = fresh_args().gamma;
    __builtin_amdgcn_wave_barrier();
    int used = 0;
#pragma unroll
    for (int q = 0; q < kLines; q += 64) {
      const bool full = key[q + lane] != kEmpty;
      const uint64_t m = __ballot(full);
      if (full) list[used + int(lanes_below(m))] = uint8_t(q + lane);
      used += __popcll(m);
    }
    __builtin_amdgcn_wave_barrier();
    const int sub = lane & (kLine - 1);
    for (int q = lane / kLine; q < used; q += 64 / kLine) {
      const uint32_t slot = list[q];
      const uint32_t k = key[slot];
      const V v = val[slot * kLine + sub];
      if (v != V(0)) {
        atomicAdd(gamma + ((int64_t(k) << 3) + sub), double(v));
        val[slot * kLine + sub] = V(0);
      }
    }
    __builtin_amdgcn_wave_barrier();
    for (int q = lane; q < kLines; q += 64) key[q] = kEmpty;
    __builtin_amdgcn_wave_barrier();
  }
};

// outcome of a step: keep marching, escaped, truncated, or split
constexpr int kGoOn = 0, kEscaped = 1, kTruncated = 2, kSplit = 3;
// cells a busy lane marches per iteration of the wavefront loop (measured on
// the 128^3, 512^3 and 1024^3 workloads: 1 -> 3 gains 4-5 %, 3 -> 4 about
// 1 %, 4 -> 8 another 0.5-3 %; the polychromatic march 1 -> 8 gains 5-11 %);
// a cell takes at most 2 new table slots, so a lane's count per iteration
// fits 5 bits
constexpr int kCellsPerIteration = 8;

// State of the ray a lane is marching.  The axes along which the ray points
// down are mirrored (origin and planes negated, exactly), so that every ray
// runs upwards on every axis: the next plane of an axis is the cell's upper
// one, a step adds 1 to it, and "ahead" and "behind" replace upper and lower.
// Rounding is symmetric, so every value equals the unmirrored one up to its
// sign.  Planes are unwrapped, which keeps crossings exact across periodic
// wraps; the wrapped flat cell index and signed strides address memory.
template <typename Idx>
struct RayState {
  double o0, o1, o2, d0, d1, d2;  // mirrored origin, |direction|
  double r0, r1, r2;              // RN(1 / d); kFarRate for a zero component
  double p0, p1, p2;              // next plane of each axis (an integer)
  double s, L;
  double tau;       // optical depth at the threshold (FP64, both paths)
  double P;         // photons carried (FP64 path)
  double T;         // mixed path: transmitted fraction
  float s_rate;     // mixed path: L / h^3 in FP32
  double a64;       // absorber of the current cell, loaded ahead
  double so;        // sqrt of the pixel solid angle
  // a crossing at s <= s_in leaves a cell off the box's boundary layer for
  // another one: neither it nor a face neighbour's index wraps or leaves
  double s_in;
  Idx c;            // wrapped flat index of the current cell
  int st0, st1, st2;  // signed strides: +-1, +-n, +-n^2
  uint32_t src, pix;
};

// reciprocal of a zero component: crossings of its planes come last
constexpr double kFarRate = 1e290;

// (p - o) / d, correctly rounded, from r = RN(1 / d): q1 is within 2^-104 of
// the quotient before its rounding, so faithful, and Markstein's theorem (a
// faithful quotient corrected once by its exact remainder times RN(1 / d)
// rounds correctly) makes q2 the IEEE quotient.  Six full-rate operations
// where the division takes fourteen, one of them quarter rate; cheap enough
// to form all three axes' crossings every step instead of selecting and
// storing back the one that moved (18 operations against 28).
__device__ __forceinline__ double crossing(double p, double o, double d, double r) {
  const double a = p - o;
  const double q0 = a * r;
  const double q1 = fma(fma(-q0, d, a), r, q0);
  return fma(fma(-q1, d, a), r, q1);
}

// ---- polychromatic sources: Phi(tau) = -ln F(tau) from the table ----
struct SpecPos {
  int q;         // interval
  double x;      // local coordinate in [0, 1)
  double inv_w;  // 1 / interval width in tau (a power of two)
};

// interval and local coordinate of tau >= 0, exactly, from the bits of 1 + tau
__device__ __forceinline__ SpecPos spec_pos(double tau) {
  constexpr int kShift = 52 - kSpecLog2Sub;
  const double v = 1.0 + tau;
  const uint64_t b = uint64_t(__double_as_longlong(v));
  const int e = int(b >> 52) - 1023;
  SpecPos p;
  p.q = (e << kSpecLog2Sub) + int((b >> kShift) & uint64_t(kSpecSub - 1));
  p.inv_w = __longlong_as_double((long long)(1023 + kSpecLog2Sub - e) << 52);
  p.x = (v - __longlong_as_double((long long)(b & ~((uint64_t(1) << kShift) - 1)))) * p.inv_w;
  return p;
}

// (p(x2) - p(x1)) / (x2 - x1) for p = c0 + c1 x + ... + c5 x^5, given
// c[0..4] = c1..c5, as sum_k c_k h_{k-1}(x1, x2) with h_j the complete
// homogeneous polynomial of degree j; free of cancellation, and p'(x1) when
// x2 = x1
template <typename T>
__device__ __forceinline__ T spec_slope(const T* c, T x1, T x2) {
  const T h1 = x1 + x2;
  const T x1s = x1 * x1;
  const T h2 = fma(x2, h1, x1s);
  const T x1c = x1s * x1;
  const T h3 = fma(x2, h2, x1c);
  const T h4 = fma(x2, h3, x1c * x1);
  return fma(c[4], h4, fma(c[3], h3, fma(c[2], h2, fma(c[1], h1, c[0]))));
}

// c1..c5 of interval q in the path's precision
template <bool MIXED, typename Args, typename V>
__device__ __forceinline__ void spec_coef(Args& A, int q, V* c) {
  if constexpr (MIXED) {
    const float4 lo = *reinterpret_cast<const float4*>(A.spec32[q].c);
    c[0] = lo.x;
    c[1] = lo.y;
    c[2] = lo.z;
    c[3] = lo.w;
    c[4] = A.spec32[q].c[4];
  } else {
    const double2* r = reinterpret_cast<const double2*>(A.spec64[q].c);
    const double2 a = r[0], b = r[1];
    c[0] = a.x;
    c[1] = a.y;
    c[2] = b.x;
    c[3] = b.y;
    c[4] = A.spec64[q].c[4];
  }
}

template <bool MIXED, typename Args>
__device__ __forceinline__ double spec_c0(Args& A, int q) {
  return MIXED ? A.spec32[q].c0 : A.spec64[q].c[5];
}

// Phi(tau) in FP64 (ray set-up); +inf past the table
template <typename Args>
__device__ double spec_phi(Args& A, double tau) {
  const SpecPos p = spec_pos(tau);
  if (p.q >= A.spec_nint) return __builtin_inf();
  double c[5];
  spec_coef<false>(A, p.q, c);
  return A.spec64[p.q].c[5] + p.x * spec_slope(c, 0.0, p.x);
}

// Rise of Phi over [tau, tau + dtau]: the optical depth that attenuates the
// whole spectrum across the cell, so that the cell absorbs the share
// 1 - e^{-rise} of the photons the ray carries.  `slope` receives the mean
// dPhi/dtau over the cell when the cell lies within one interval, which is
// dPhi/dtau at tau when dtau = 0 (the thin-cell limit).  Past the table's end
// the rise is infinite: the cell absorbs everything the ray still carries.
template <bool MIXED, typename Args, typename V>
__device__ __forceinline__ V spec_rise(Args& A, double tau, V dtau, V& slope) {
  const SpecPos p1 = spec_pos(tau);
  const SpecPos p2 = spec_pos(tau + double(dtau));
  V c[5];
  spec_coef<MIXED>(A, p1.q, c);
  if (p2.q == p1.q) {
    const V sl = spec_slope(c, V(p1.x), V(p2.x));
    slope = sl * V(p1.inv_w);
    return (dtau * V(p1.inv_w)) * sl;
  }
  slope = V(0);
  if (p2.q >= A.spec_nint) return V(__builtin_inf());
  // rest of the first interval, whole intervals between, start of the last
  const V first = (V(1) - V(p1.x)) * spec_slope(c, V(p1.x), V(1));
  spec_coef<MIXED>(A, p2.q, c);
  const V last = V(p2.x) * spec_slope(c, V(0), V(p2.x));
  const double mid = spec_c0<MIXED>(A, p2.q) - spec_c0<MIXED>(A, p1.q + 1);
  return (first + last) + V(mid);
}

// One ray of a launch as queued: source, HEALPix pixel, path length and
// optical depth at the threshold.  For injected rays `src` holds the ray's
// index.
struct Entry {
  uint32_t src, pix;
  double s, w;
};

// Entry r of the launch: a virtual spawn index, a queue slot or an injected
// ray's index.
template <typename Args>
__device__ __forceinline__ Entry load_entry(Args& A, int64_t r) {
  Entry e;
  if (A.level < 0) {
    e.src = uint32_t(r);
    e.pix = 0;
    e.s = 0.0;
    e.w = 0.0;
  } else if (A.spawn) {
    if (r < (int64_t(1) << 32)) {
      const uint32_t r32 = uint32_t(r);
      e.src = uint32_t(A.src_begin) + r32 / 12u;
      e.pix = r32 % 12u;
    } else {
      e.src = uint32_t(A.src_begin + r / 12);
      e.pix = uint32_t(r % 12);
    }
    e.s = 0.0;
    e.w = 0.0;
  } else {
    e.src = A.in.src[r];
    e.pix = A.in.pix[r];
    e.s = A.in.s[r];
    e.w = A.in.w[r];
  }
  return e;
}

// The box plane ahead of the cell below plane p, on one (mirrored) axis: box
// planes are the multiples of n, and (p - 1/2) / n is at least 1/(2n) from an
// integer, so the rounded reciprocal of n decides its floor rightly.
__device__ __forceinline__ double box_plane(double p, double n, double inv_n) {
  return (floor((p - 0.5) * inv_n) + 1.0) * n;
}

// Path length up to which a ray's crossings stay off the boundary layer, from
// its distances f to the box planes h ahead (in cells, 0 in the last cell):
// -1 in the layer; else 1e-12 short of its entry, so rounding cannot put it
// late.
template <typename Idx>
__device__ __forceinline__ double inner_length(const RayState<Idx>& R, double f0, double f1,
                                               double f2, double h0, double h1, double h2,
                                               double n) {
  const double e0 = ((h0 - 1.0) - R.o0) * R.r0;
  const double e1 = ((h1 - 1.0) - R.o1) * R.r1;
  const double e2 = ((h2 - 1.0) - R.o2) * R.r2;
  const double lo = fmin(fmin(f0, f1), f2), hi = fmax(fmax(f0, f1), f2);
  return lo >= 1.0 && hi <= n - 2.0 ? fmin(fmin(e0, e1), e2) * (1.0 - 1e-12) : -1.0;
}

// Start the ray of entry e: direction, start cell and first absorber.
// Returns kEscaped if it starts outside an open box, else kGoOn.
template <bool MIXED, bool PERIODIC, bool POLY, typename Idx, typename Args>
__device__ __forceinline__ int ray_init(RayState<Idx>& R, Args& A, const Entry& e) {
  double w = e.w;
  int level;
  double o0, o1, o2, d0, d1, d2;
  if (A.level < 0) {  // injected rays: never split
    const int64_t r = e.src;
    o0 = A.inj_origin[3 * r];
    o1 = A.inj_origin[3 * r + 1];
    o2 = A.inj_origin[3 * r + 2];
    d0 = A.inj_dir[3 * r];
    d1 = A.inj_dir[3 * r + 1];
    d2 = A.inj_dir[3 * r + 2];
    R.L = A.inj_L[r];
    level = A.inj_level[r];
    R.s = 0.0;
    R.src = R.pix = 0;
  } else {
    R.src = e.src;
    R.pix = e.pix;
    R.s = e.s;
    level = A.level;
    o0 = A.src_pos[3 * int64_t(R.src)];
    o1 = A.src_pos[3 * int64_t(R.src) + 1];
    o2 = A.src_pos[3 * int64_t(R.src) + 2];
    R.L = ldexp(A.src_l0[R.src], -2 * level);
    if (level <= A.dir_max_level) {  // the table holds this device function's values
      const double* d = A.dirs + 3 * (dir_table_offset(level) + int64_t(R.pix));
      d0 = d[0];
      d1 = d[1];
      d2 = d[2];
    } else {
      healpix_dir(level, R.pix, d0, d1, d2);
    }
  }
  // sqrt of the pixel solid angle: sqrt(Omega(0)) 2^-level, exactly
  R.so = ldexp(A.sqrt_omega_tab[0], -level);
  const int n = A.n;
  const int i0 = start_cell(o0, R.s, d0);
  const int i1 = start_cell(o1, R.s, d1);
  const int i2 = start_cell(o2, R.s, d2);
  // components that no crossing in any box can see count as zero (injected
  // rays only; the smallest nonzero component of a pixel centre is ~1e-5)
  auto axis = [](double o, double d, int i, int stride, double& ro, double& rd, double& rr,
                 double& rp, int& rst) {
    const bool down = d < 0.0;
    const double m = fabs(d);
    ro = down ? -o : o;
    rd = m > 1e-280 ? m : 0.0;
    rr = m > 1e-280 ? 1.0 / m : kFarRate;
    rp = double(down ? -i : i + 1);
    rst = down ? -stride : stride;
  };
  axis(o0, d0, i0, 1, R.o0, R.d0, R.r0, R.p0, R.st0);
  axis(o1, d1, i1, n, R.o1, R.d1, R.r1, R.p1, R.st1);
  axis(o2, d2, i2, n * n, R.o2, R.d2, R.r2, R.p2, R.st2);
  R.tau = w;
  // transmitted share of the ray's photons: e^{-tau}, or e^{-Phi(tau)} for a
  // spectrum (exactly 1 at a source)
  const double T = w == 0.0 ? 1.0 : exp(POLY ? -spec_phi(A, w) : -w);
  if (MIXED) {
    R.T = T;
    R.s_rate = float(R.L * A.inv_h3);
  } else {
    R.P = R.L * T;
  }
  const bool out = i0 < 0 || i0 >= n || i1 < 0 || i1 >= n || i2 < 0 || i2 >= n;
  if (!PERIODIC && out) return kEscaped;
  R.c = Idx(PERIODIC ? cell_index(wrap_cell(i0, n), wrap_cell(i1, n), wrap_cell(i2, n), n)
                     : cell_index(i0, i1, i2, n));
  R.a64 = A.a64[R.c];
  const double nd = double(n);
  const double h0 = box_plane(R.p0, nd, A.inv_n), h1 = box_plane(R.p1, nd, A.inv_n),
               h2 = box_plane(R.p2, nd, A.inv_n);
  R.s_in = inner_length(R, h0 - R.p0, h1 - R.p1, h2 - R.p2, h0, h1, h2, nd);
  return kGoOn;
}


// Arguments every step reads, held in scalar registers for the whole
// launch.  Read from the argument block where they are used, the compiler
// would reload them there (scalar registers are scarce in the march), and the
// wait for such a load also waits for every LDS operation in flight.  An
// empty asm statement makes each value the output of an instruction, which
// cannot be reloaded, so it stays in a register.
struct StepConst {
  double s_stop, tau_stop, sigma0;
  __device__ explicit StepConst(const MarchArgs& A)
      : s_stop(A.s_stop), tau_stop(A.tau_stop), sigma0(A.sigma0) {
    asm volatile("" : "+s"(s_stop));
    asm volatile("" : "+s"(tau_stop));
    asm volatile("" : "+s"(sigma0));
  }
};

// Why a ray whose path length or optical depth reached the launch's bound
// stops, in the method's order: the end of a periodic ray, the optical-depth
// cap (for a spectrum: the threshold optical depth at which the share of
// photons left falls to e^{-tau_max}), then the split.
template <bool PERIODIC, typename Args, typename Idx>
__device__ __forceinline__ int stop_code(const Args& A, const RayState<Idx>& R) {
  if (PERIODIC && R.s >= A.s_max) return kEscaped;
  if (R.tau >= A.tau_stop) return kTruncated;
  return A.level >= A.l_max ? kTruncated : kSplit;
}

// Stop tests at the current cell boundary, then one cell segment: optical
// depth, Eq. lut_eqn deposit with the overlap correction, advance.  The
// caller books the photons of a ray that stops.  `inserted` counts new table
// slots taken by this call's deposits.  Memory latency is hidden by order:
// the cell's absorber was loaded at the end of the previous step; the
// neighbour's is requested by every lane (its own cell's when it needs no
// neighbour), so that the wait for the cell's word leaves that request in
// flight; the table's keys are read before the attenuation, new lines are
// claimed after it and before the advance, whose arithmetic covers the claims
// and the neighbour's load, and the deposits come last.
template <bool MIXED, int CORR, bool PERIODIC, bool POLY, typename V, typename Idx>
__device__ __forceinline__ int ray_step(RayState<Idx>& R, const MarchArgs& A,
                                        const LineTable<V, Idx>& tab, LaneAcc& acc, int& inserted,
                                        const StepConst& K) {
  constexpr bool neighbours = CORR == NRT_CORR_CONSERVATIVE || CORR == NRT_CORR_NAIVE;
  if (R.s >= K.s_stop || R.tau >= K.tau_stop) return stop_code<PERIODIC>(fresh_args(), R);
  const Idx c = R.c;
  auto l1 = tab.look(c);
  // next crossing: lowest axis wins exact ties
  const double t0 = crossing(R.p0, R.o0, R.d0, R.r0);
  const double t1 = crossing(R.p1, R.o1, R.d1, R.r1);
  const double t2 = crossing(R.p2, R.o2, R.d2, R.r2);
  const bool x1 = t1 < t0;
  const double t01 = fmin(t0, t1);
  const bool x2 = t2 < t01;
  const double tn = fmin(t01, t2);
  const double ds = fmax(tn - R.s, 0.0);
  const int st0 = R.st0, st1 = R.st1, st2 = R.st2;
  const int st_x = x2 ? st2 : (x1 ? st1 : st0);
  Idx cn = c + Idx(st_x);

  // ---- overlap geometry (Eqs. correction .. new_secondary): nearest face
  // of the segment midpoint, and the neighbour across it ----
  bool near = false;
  double dedge = 0.0, lpix = 1.0;
  bool neighbour = false;  // the neighbour's absorber is needed
  Idx c2 = c;
  double raw2_64 = 0.0;
  bool behind = false, f1 = false, f2 = false;  // the face: side and axis
  if constexpr (CORR != NRT_CORR_NONE) {
    const double rm = 0.5 * (R.s + tn);
    lpix = rm * R.so;
    // per axis: distance to the nearer face; an exact tie goes the way the
    // ray points (ahead); the first axis wins ties between axes
    const double m0 = R.o0 + rm * R.d0, m1 = R.o1 + rm * R.d1, m2 = R.o2 + rm * R.d2;
    const double b0 = m0 - (R.p0 - 1.0), a0 = R.p0 - m0;
    const double b1 = m1 - (R.p1 - 1.0), a1 = R.p1 - m1;
    const double b2 = m2 - (R.p2 - 1.0), a2 = R.p2 - m2;
    const double e0 = fmin(b0, a0), e1 = fmin(b1, a1), e2 = fmin(b2, a2);
    f1 = e1 < e0;
    const double e01 = fmin(e0, e1);
    f2 = e2 < e01;
    dedge = fmin(e01, e2);
    near = dedge < 0.5 * lpix;
    if constexpr (neighbours) {
      neighbour = near;
      const bool h0 = b0 < a0, h1 = b1 < a1, h2 = b2 < a2;
      behind = f2 ? h2 : (f1 ? h1 : h0);
      const int st_f = f2 ? st2 : (f1 ? st1 : st0);
      c2 = near ? c + Idx(behind ? -st_f : st_f) : c;
    }
  }
  // cells on the box's boundary layer, where a step or a neighbour wraps or
  // leaves: from the planes themselves, without branches.  Rare on large
  // grids (6/n of the cells), so the other cells carry no wrapped coordinates.
  bool escaped = false;
  if (!(tn <= R.s_in)) {
    ArgsK& F = fresh_args();
    const double n = double(F.n), inv_n = F.inv_n;
    double h0 = box_plane(R.p0, n, inv_n), h1 = box_plane(R.p1, n, inv_n),
           h2 = box_plane(R.p2, n, inv_n);
    // cells ahead of this one: 0 in the last before the box plane
    double g0 = h0 - R.p0, g1 = h1 - R.p1, g2 = h2 - R.p2;
    if constexpr (neighbours) {
      const double g = f2 ? g2 : (f1 ? g1 : g0);
      if (near && g == (behind ? n - 1.0 : 0.0)) {
        neighbour = PERIODIC;
        const int st_f = f2 ? st2 : (f1 ? st1 : st0);
        const Idx whole = Idx(st_f) * Idx(F.n);
        c2 = !PERIODIC ? c : (behind ? c2 + whole : c2 - whole);
      }
    }
    const double g = x2 ? g2 : (x1 ? g1 : g0);
    const bool over = g == 0.0;
    escaped = !PERIODIC && over;
    if (over) cn = PERIODIC ? cn - Idx(st_x) * Idx(F.n) : c;  // one that left reads its last cell
    // the new cell's distances and planes
    const double up = over ? n : 0.0, gx = over ? n - 1.0 : g - 1.0;
    g0 = x1 || x2 ? g0 : gx;
    g1 = x1 && !x2 ? gx : g1;
    g2 = x2 ? gx : g2;
    h0 += x1 || x2 ? 0.0 : up;
    h1 += x1 && !x2 ? up : 0.0;
    h2 += x2 ? up : 0.0;
    R.s_in = inner_length(R, g0, g1, g2, h0, h1, h2, n);
  }
  // requested by every lane, whether or not it needs a neighbour, so the
  // load is never skipped by a branch and the wait for this cell's word
  // below can leave it in flight
  auto l2 = l1;
  if constexpr (neighbours) {
    raw2_64 = A.a64[c2];
    l2 = tab.look(c2);
  }

  // ---- segment physics (Eq. lut_eqn, Eq. optical_depth) ----
  // the cell's optical depth in FP64, the same operations in both paths
  const double a64 = fabs(R.a64);
  const double dl = ds * A.h_cm;
  const double dtau64 = K.sigma0 * a64 * dl;
  double G64 = 0.0;
  float G32 = 0.0f, a32 = 0.0f;
  if (MIXED) {
    a32 = float(a64);
    const float dsf = float(ds);
    float dtau = float(dtau64);
    float slope32 = 1.0f;
    if constexpr (POLY) {  // the whole spectrum's attenuation across the cell
      const float dtau0 = dtau;
      dtau = spec_rise<true>(A, R.tau, dtau0, slope32);
    }
    R.tau += dtau64;
    // surviving share e = exp(-dtau) from the hardware base-2 exponential
    // (1 ulp); absorbed share em = 1 - e, which for dtau < 1/8 comes from
    // its series (relative truncation error below dtau^5/720 < 5e-8) since
    // 1 - e would cancel there
    const float e = __builtin_amdgcn_exp2f(dtau * -1.44269504f);
    const float poly =
        dtau * fmaf(dtau, fmaf(dtau, fmaf(dtau, fmaf(dtau, 1.0f / 120.0f, -1.0f / 24.0f),
                                          1.0f / 6.0f), -0.5f), 1.0f);
    const float em = dtau < 0.125f ? poly : 1.0f - e;
    // transmitted fraction in FP64: the absorbed part for weak absorption,
    // the surviving part for strong absorption (where em rounds towards 1)
    const bool weak = em < 0.5f;
    const double part = R.T * double(weak ? em : e);
    const double rest = R.T - part;
    const double dT = weak ? part : rest;
    const float Tf = float(R.T);
    R.T = weak ? rest : part;
    acc.absorbed = fma(R.L, dT, acc.absorbed);
    // an absorber below FP32's normal range takes the thin limit, which is
    // exact there
    G32 = a32 >= FLT_MIN ? (R.s_rate * float(dT)) * __builtin_amdgcn_rcpf(a32)
                         : R.s_rate * Tf * (A.kf * dsf) * slope32;
  } else {
    double rise = dtau64, slope64 = 1.0;
    if constexpr (POLY) rise = spec_rise<false>(A, R.tau, dtau64, slope64);
    const double dN = R.P * (-expm1(-rise));
    G64 = a64 > 0.0 ? dN / (a64 * A.h3) : R.P * A.sigma0 * dl * slope64 / A.h3;
    acc.absorbed += dN;
    R.P -= dN;
    R.tau += dtau64;
  }

  // ---- claims of new lines, in flight during the advance ----
  tab.claim(l1, true, inserted);
  if constexpr (neighbours) tab.claim(l2, neighbour, inserted);

  // ---- advance one cell; the next cell's absorber is consumed by the next
  // step ----
  R.s = tn;
  R.p0 += x1 || x2 ? 0.0 : 1.0;
  R.p1 += x1 && !x2 ? 1.0 : 0.0;
  R.p2 += x2 ? 1.0 : 0.0;
  R.c = cn;
  R.a64 = A.a64[cn];
  acc.segments += 1;

  // ---- overlap correction values (the decision above is FP64; the factor
  // is FP32 in the mixed path) ----
  using R_t = typename std::conditional<MIXED, float, double>::type;
  R_t fc = R_t(1);
  bool secondary = false;
  float raw2_32 = 0.0f;
  if constexpr (CORR != NRT_CORR_NONE) {
    const bool usable = neighbour && !__builtin_signbit(raw2_64);
    // the mixed path's FP32 neighbour absorber, floored at the smallest
    // normal so that its reciprocal stays finite
    if (MIXED) raw2_32 = fmaxf(float(raw2_64), FLT_MIN);
    R_t f;
    if constexpr (MIXED)
      f = 0.5f + float(dedge) * __builtin_amdgcn_rcpf(float(lpix));
    else
      f = near ? 0.5 + dedge / lpix : 1.0;
    if constexpr (CORR == NRT_CORR_LINEAR) {
      fc = near ? f : R_t(1);
    } else if constexpr (CORR == NRT_CORR_SQUARED) {
      fc = near ? f * f : R_t(1);
    } else if constexpr (CORR == NRT_CORR_CONSERVATIVE) {
      fc = usable ? f : R_t(1);
      secondary = usable;
    } else {  // NAIVE
      fc = near ? f : R_t(1);
      secondary = usable;
    }
  }

  // ---- deposit ----
  if constexpr (MIXED) {
    tab.deposit(l1, c, V(fc * G32), true, true, inserted);
    if constexpr (neighbours)
      tab.deposit(l2, c2, V(((1.0f - fc) * (a32 * __builtin_amdgcn_rcpf(raw2_32))) * G32),
                  neighbour, secondary, inserted);
  } else {
    tab.deposit(l1, c, V(fc * G64), true, true, inserted);
    if constexpr (neighbours) {
      double v2 = 0.0;
      if (secondary) v2 = ((1.0 - fc) * (a64 / raw2_64)) * G64;
      tab.deposit(l2, c2, V(v2), neighbour, secondary, inserted);
    }
  }
  return escaped ? kEscaped : kGoOn;
}

// Whole wavefront: append the four children of every lane with a pending
// split to the next level's queue (one atomicAdd for the wavefront).
__device__ __forceinline__ void push_pending(unsigned long long* count, const RayQueue& out,
                                             int64_t out_cap, unsigned long long* overflow,
                                             int lane, bool& pend, uint32_t p_src,
                                             uint32_t p_pix, double p_s, double p_w) {
  const uint64_t pm = __ballot(pend);
  if (!pm) return;
  const int leader = __builtin_ctzll(pm);
  unsigned long long slot0 = 0;
  if (lane == leader) slot0 = atomicAdd(count, 4ull * static_cast<unsigned long long>(__popcll(pm)));
  slot0 = read_lane64(slot0, leader);
  if (pend) {
    const unsigned long long slot = slot0 + 4ull * lanes_below(pm);
    if (slot + 4 <= static_cast<unsigned long long>(out_cap)) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        out.src[slot + k] = p_src;
        out.pix[slot + k] = 4u * p_pix + uint32_t(k);
        out.s[slot + k] = p_s;
        out.w[slot + k] = p_w;
      }
    } else {
      atomicAdd(overflow, 1ull);
    }
    pend = false;
  }
}

// Size of a wavefront's next run of rays.  The claims are same-address atomics,
// about 130 M/s for the device, which bound launches of short rays (39^3, 8
// cells a ray: runs of 64 / 128 / 256 take 8.5 / 7.1 / 6.6 ms); long runs
// leave a long tail where rays are long (1024^3, 100 cells a ray: 221 / 234 /
// 262 ms).  So the run follows the cells that 64 rays of the last one took,
// within the wavefront's even share of what is left.  The share is rounded down
// to whole wavefronts, but up in launches of brief rays (kBriefStop), whose
// second 64 take less time than one more claim by every wavefront (128^3, FP64,
// 1.7 / 3 / 10 cells a ray: 113 / 610 / 2334 us rounded down, 84 / 532 / 1793
// up; where rays are longer, rounding up costs: 1024^3 +2 %).
__device__ __forceinline__ int64_t run_size(int64_t cells_per_64, bool brief, int64_t left,
                                            float share, int64_t lo, int64_t hi) {
  const int64_t by_cells = cells_per_64 <= 16 ? 256 : (cells_per_64 <= 32 ? 128 : 64);
  const int64_t even = int64_t(float(left) * share + (brief ? 63.99f : 0.0f)) & ~int64_t(63);
  const int64_t r = by_cells < even ? by_cells : even;
  return r < lo ? lo : (r > hi ? hi : r);
}

// Bound on the path length of a launch whose rays are brief, 16 cells or fewer: a
// level's rays start at half of it, and take 1.5 cells a unit of length.
constexpr double kBriefStop = 21.0;

// Persistent march: every wavefront takes runs of rays of the launch's range
// (its first by position, the rest from a shared counter; their size from
// run_size), refills idle lanes from its run once A.refill_min of them are idle,
// advances every busy lane by up to 8 cells per iteration, and folds its
// LDS table into Gamma when enough slots are taken.  A lane whose ray splits
// keeps the children's start state in registers; the wavefront appends the children of
// all pending splits to the next level's queue with one atomicAdd once every
// lane holds one (or a pending lane splits again, or the wavefront is done):
// fewer same-address atomics than a push at 32 (1024^3: +1.3 % mixed, +4 %
// FP64).
// The march is held to 128 VGPRs, which keeps 4 waves per SIMD as its LDS
// allows: it waits for memory in a third of its cycles, and a fourth wave gains
// more than the words that spill cost (periodic FP64 23 of them, 128^3: 14.15 ms
// with 3 waves and none spilled, 13.15 with 4; blackbody, 41: 26.8 and 24.7).
// Only the open-box polychromatic FP64 one is faster with 3 (96^3: 1.27 / 1.41).
template <bool MIXED, int CORR, bool PERIODIC, bool POLY, typename V, typename Idx>
__global__ __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu((MIXED || PERIODIC || !POLY) ? 4 : 3, 8))) void k_march(
    MarchArgs A) {
  if (A.skip && *A.skip) return;  // a replayed pass after its iteration stopped
  int64_t total = A.end - A.begin;
  if (A.count_src) {
    const int64_t k = int64_t(*A.count_src);
    total = k < A.in_cap ? k : A.in_cap;
  }
  // Wavefront w starts with rays [w run, (w+1) run) of the launch's range
  // without touching the shared counter, which hands out the runs after the
  // first nwaves * run.  A block with no first run leaves at once: the idle
  // part of a persistent grid (small and empty levels) clears no tables and
  // issues no atomics.
  const int64_t nwaves = int64_t(gridDim.x) * kWaves;
  const float share = 1.0f / float(nwaves);
  // brief rays: the even share, so that often no run is left to claim
  const bool brief = A.s_stop <= kBriefStop;
  int64_t run = run_size(0, brief, total, brief ? share : 0.25f * share, A.claim_min, A.claim);
  const int64_t first_runs = nwaves * run;
  if (int64_t(blockIdx.x) * kWaves * run >= total) return;
  // per-wavefront deposit tables, reused for the budget reduction at the end
  using Tab = LineTable<V, Idx>;
  __shared__ __align__(16) unsigned char lds[kWaves * Tab::kWaveBytes];
  const int wave = threadIdx.x >> 6;
  const int lane = __lane_id();
  uint32_t* key = reinterpret_cast<uint32_t*>(lds) + wave * Tab::kLines;
  V* val = reinterpret_cast<V*>(lds + kWaves * Tab::kLines * sizeof(uint32_t)) +
           wave * Tab::kLines * kLine;
  uint8_t* list = lds + kWaves * Tab::kLines * (sizeof(uint32_t) + kLine * sizeof(V)) +
                  wave * Tab::kLines;
  uint32_t mul = sizeof(V) == 4 ? A.line_mul[0] : A.line_mul[1];
  asm volatile("" : "+s"(mul));
  const Tab tab{key, val, list, mul, (int64_t(A.n) * A.n * A.n) >> 3 < NRT_TABLE_LINES};
  for (int q = lane; q < Tab::kLines; q += 64) key[q] = kEmpty;
  for (int q = lane; q < Tab::kLines * kLine; q += 64) val[q] = V(0);
  __builtin_amdgcn_wave_barrier();

  LaneAcc acc;
  RayState<Idx> R;
  bool busy = false;
  // pending split of this lane: children start state
  bool pend = false;
  uint32_t p_src = 0, p_pix = 0;
  double p_s = 0.0, p_w = 0.0;
  // the run bounds are wavefront-uniform: derive them from a uniform wave
  // index so that they stay in scalar registers
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  int64_t pool = (int64_t(blockIdx.x) * kWaves + wave_u) * run;
  int64_t pool_end = pool + run < total ? pool + run : total;
  bool exhausted = pool >= total;
  if (exhausted) pool = pool_end = 0;
  const StepConst K(A);
  int iterations = 0;              // since the last claim
  int fill = 0;                    // wavefront-uniform occupied line slots
  for (;;) {
    const uint64_t idle = __ballot(!busy);
    const int n_idle = __popcll(idle);
    if (!exhausted && (n_idle >= A.refill_min || n_idle == 64)) {
      ArgsK& F = fresh_args();
      // The first runs were all: no claim is needed to tell.  (FP32 sums: the wait
      // for one is part of the timing that orders the children they are queued
      // with, and so of the sums' rounding, which otherwise moves by 3e-9.)
      if (sizeof(V) == 8 && pool == pool_end && first_runs >= total) {
        exhausted = true;
      } else if (pool == pool_end) {
        // a run is at most 65536 rays of 12300 cells, so that a lane's 32-bit
        // count cannot pass 2^32 before the next claim
        if (acc.segments >= NRT_SEGMENT_FOLD) {
          atomicAdd(&F.acc->segments, static_cast<unsigned long long>(acc.segments));
          acc.segments = 0;
        }
        // what is left by this wavefront's last run (others may have taken more)
        const int64_t left = total - (pool > first_runs ? pool : first_runs);
        run = run_size(int64_t(iterations) * kCellsPerIteration * 64 / run, brief, left, share,
                       F.claim_min, F.claim);
        iterations = 0;
        unsigned long long b = 0;
        if (lane == 0) b = atomicAdd(F.claim_ctr, static_cast<unsigned long long>(run));
        b = read_lane64(b, 0) + static_cast<unsigned long long>(first_runs);
        if (int64_t(b) >= total) {
          exhausted = true;
        } else {
          pool = int64_t(b);
          pool_end = int64_t(b) + run < total ? int64_t(b) + run : total;
        }
      }
      if (!exhausted) {
        const int64_t avail = pool_end - pool;
        const unsigned rank = lanes_below(idle);
        if (!busy && int64_t(rank) < avail) {
          const Entry e = load_entry(F, F.begin + pool + rank);
          const int start = ray_init<MIXED, PERIODIC, POLY>(R, F, e);
          busy = start == kGoOn;
          if (!busy) acc.escaped += MIXED ? R.L * R.T : R.P;
        }
        pool += int64_t(n_idle) < avail ? int64_t(n_idle) : avail;
      }
    }
    if (__ballot(busy) == 0) {
      if (exhausted) break;
      continue;
    }
    // a few cells per busy lane between the wavefront's bookkeeping (refill,
    // split pushes, table occupancy); a lane that stops sits out the rest
    ++iterations;
    int code = kGoOn, inserted = 0;
#pragma unroll 1
    for (int k = 0; k < kCellsPerIteration && busy; ++k) {
      code = ray_step<MIXED, CORR, PERIODIC, POLY>(R, A, tab, acc, inserted, K);
      if (code != kGoOn) {
        busy = false;
        const double carried = MIXED ? R.L * R.T : R.P;
        acc.escaped += code == kEscaped ? carried : 0.0;
        acc.truncated += code == kTruncated ? carried : 0.0;
      }
    }
    fill += __popcll(__ballot(inserted & 1)) + 2 * __popcll(__ballot(inserted & 2)) +
            4 * __popcll(__ballot(inserted & 4)) + 8 * __popcll(__ballot(inserted & 8)) +
            16 * __popcll(__ballot(inserted & 16));
    const bool splits = code == kSplit;
    if (__ballot(splits && pend)) {  // a lane splits again
      ArgsK& F = fresh_args();
      const RayQueue out{F.out.src, F.out.pix, F.out.s, F.out.w};
      push_pending(&F.acc->out_count[F.level + 1], out, F.out_cap, &F.acc->overflow, lane, pend,
                   p_src, p_pix, p_s, p_w);
    }
    if (splits) {
      pend = true;
      p_src = R.src;
      p_pix = R.pix;
      p_s = R.s;
      p_w = R.tau;
    }
    if (__ballot(pend) == ~0ull) {  // every lane holds a pending split
      ArgsK& F = fresh_args();
      const RayQueue out{F.out.src, F.out.pix, F.out.s, F.out.w};
      push_pending(&F.acc->out_count[F.level + 1], out, F.out_cap, &F.acc->overflow, lane, pend,
                   p_src, p_pix, p_s, p_w);
    }
    if (fill >= Tab::kFlushAt) {
      tab.flush(lane);
      fill = 0;
    }
  }
  push_pending(&A.acc->out_count[A.level + 1], A.out, A.out_cap, &A.acc->overflow, lane, pend,
               p_src, p_pix, p_s, p_w);
  tab.flush(lane);

  // block reduction of the lane budgets, then one atomic per block and term
  __syncthreads();
  static_assert(kWaves * Tab::kWaveBytes >= kBlock * 32, "reduction space");
  double(*red_d)[kBlock] = reinterpret_cast<double(*)[kBlock]>(lds);
  unsigned long long* red_u = reinterpret_cast<unsigned long long*>(lds + 3 * kBlock * 8);
  red_d[0][threadIdx.x] = acc.absorbed;
  red_d[1][threadIdx.x] = acc.escaped;
  red_d[2][threadIdx.x] = acc.truncated;
  red_u[threadIdx.x] = acc.segments;
  __syncthreads();
  for (int h = kBlock / 2; h > 0; h >>= 1) {
    if (int(threadIdx.x) < h) {
      red_d[0][threadIdx.x] += red_d[0][threadIdx.x + h];
      red_d[1][threadIdx.x] += red_d[1][threadIdx.x + h];
      red_d[2][threadIdx.x] += red_d[2][threadIdx.x + h];
      red_u[threadIdx.x] += red_u[threadIdx.x + h];
    }
    __syncthreads();
  }
  // a term that is zero adds nothing: these are same-address atomics too, 8 us
  // a term and launch (l_max 4 at 128^3: 648 -> 630 us)
  if (threadIdx.x == 0) {
    if (red_d[0][0] != 0.0) atomicAdd(&A.acc->absorbed, red_d[0][0]);
    if (red_d[1][0] != 0.0) atomicAdd(&A.acc->escaped, red_d[1][0]);
    if (red_d[2][0] != 0.0) atomicAdd(&A.acc->truncated, red_d[2][0]);
    if (red_u[0] != 0) atomicAdd(&A.acc->segments, red_u[0]);
  }
}

// a = (1 - x) n_H with the neighbour flag in the sign bit: a cell is a
// usable neighbour (Eqs. new_correction / new_secondary) iff n_H >= n_th and
// a > 0; otherwise -a is stored (-0.0 for a = 0).  Invalid inputs are counted.
__device__ __forceinline__ bool prep_cell(double nh, double xx, double n_th, double* a64) {
  const double a = (1.0 - xx) * nh;
  const bool usable = nh >= n_th && a > 0.0;
  *a64 = usable ? a : -a;
  return !(nh >= 0.0) || isinf(nh) || !(xx >= 0.0 && xx <= 1.0);
}

__global__ void k_prep(const double* __restrict__ n_H, const double* __restrict__ x, double n_th,
                       int64_t ncell, double* a64, Accum* acc) {
  unsigned long long bad = 0;
  for (int64_t c = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; c < ncell;
       c += int64_t(gridDim.x) * blockDim.x)
    bad += prep_cell(n_H[c], x[c], n_th, a64 + c) ? 1 : 0;
  if (bad) atomicAdd(&acc->invalid, bad);
}

// The threshold optical depth at which a spectrum's Phi reaches tau_max:
// the smallest tau with Phi(tau) >= tau_max on the FP64 table, to the last
// bit, by bisection of [0, hi] (Phi(0) = 0 < tau_max and Phi(hi) >= tau_max
// at the table's end).  The march stops a ray once its threshold optical
// depth reaches it, which is the photon-share cap F <= e^{-tau_max} taken on
// an FP64 quantity that both precisions accumulate alike.  One thread.
struct SpecTable {
  int32_t spec_nint;
  const SpecRec64* spec64;
  const SpecRec32* spec32;
};

__global__ void k_spec_stop(SpecTable t, double tau_max, double hi, double* out) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  double lo = 0.0;
  for (int it = 0; it < 4096; ++it) {
    const double mid = lo + 0.5 * (hi - lo);
    if (!(mid > lo && mid < hi)) break;
    if (spec_phi(t, mid) >= tau_max)
      hi = mid;
    else
      lo = mid;
  }
  *out = hi;
}

// clear the accumulators (one block)
__device__ __forceinline__ void clear_accum(Accum* acc) {
  unsigned long long* p = reinterpret_cast<unsigned long long*>(acc);
  for (int i = threadIdx.x; i < int(sizeof(Accum) / sizeof(unsigned long long)); i += blockDim.x)
    p[i] = 0ull;
}

// Clear Gamma and, unless acc is NULL, the accumulators for a pass: one launch,
// since small passes are launches (about 4 us each) and little else.  With n_H,
// also the absorber of a radiation step's pass from its ionized fraction (as
// k_prep); invalid cells are counted in *invalid, which this kernel does not clear.
__global__ void k_begin_pass(double* gamma, int64_t count, Accum* acc,
                             const double* __restrict__ n_H, const double* __restrict__ x,
                             double n_th, double* a64, unsigned long long* invalid,
                             const unsigned long long* skip) {
  if (skip && *skip) return;
  if (acc && blockIdx.x == 0) clear_accum(acc);
  unsigned long long bad = 0;
  for (int64_t c = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; c < count;
       c += int64_t(gridDim.x) * blockDim.x) {
    gamma[c] = 0.0;
    if (n_H) bad += prep_cell(n_H[c], x[c], n_th, a64 + c) ? 1 : 0;
  }
  if (bad) atomicAdd(invalid, bad);
}

__global__ void k_zero_accum(Accum* acc) { clear_accum(acc); }

__global__ void k_healpix(int level, int64_t first, int64_t count, double* out) {
  const int64_t q = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (q >= count) return;
  double x, y, z;
  healpix_dir(level, uint32_t(first + q), x, y, z);
  out[3 * q] = x;
  out[3 * q + 1] = y;
  out[3 * q + 2] = z;
}

// Entry q of the direction table: levels 0..top in turn, each pixel's vector
// from the geometry (IEEE operations, so the host's values) and the host's
// cosine and sine of its azimuth.  A launch holds the azimuths [lo, hi) in cs
// and writes their pixels; the pixels without an azimuth of their own go with
// the first launch.
__global__ void k_directions(int64_t total, int64_t lo, int64_t hi,
                             const double2* __restrict__ cs, double* out) {
  const int64_t q = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (q >= total) return;
  // a level's entries start at 4 (4^level - 1)
  const int level = (31 - __clz(uint32_t(q / 4 + 1))) / 2;
  const HpAngle a = healpix_angle(level, uint32_t(q - dir_table_offset(level)));
  double2 t{1.0, 0.0};
  if (a.fold >= 2) {
    const int64_t i = hp_azimuth_index(a.nr, a.k);
    if (i < lo || i >= hi) return;
    t = cs[i - lo];
  } else if (lo > 0) {
    return;
  }
  healpix_vector(a, t.x, t.y, out[3 * q], out[3 * q + 1], out[3 * q + 2]);
}

__global__ void k_budget(const Accum* acc, nrt_budget* out, uint64_t* dropped, double emitted,
                         uint64_t spawned, int l_max) {
  if (threadIdx.x != 0) return;
  nrt_budget b;
  b.emitted = emitted;
  b.absorbed = acc->absorbed;
  b.escaped = acc->escaped;
  b.truncated = acc->truncated;
  b.segments = acc->segments;
  b.rays = 0;
  b.splits = 0;
  for (int l = 0; l <= NRT_MAX_LEVEL; ++l) {
    const uint64_t k = l == 0 ? spawned : (l <= l_max ? uint64_t(acc->out_count[l]) : 0);
    b.rays_per_level[l] = k;
    b.rays += k;
    if (l > 0) b.splits += k / 4;
  }
  *out = b;
  if (dropped) *dropped = acc->overflow;
}

__global__ void k_rt_check(const Accum* acc, RtState* rt, unsigned long long threshold,
                           unsigned long long max_iter) {
  if (threadIdx.x != 0 || rt->done) return;
  rt->iters += 1;
  rt->changed = acc->chem_changed;
  rt->overflow |= acc->overflow;
  rt->invalid |= acc->invalid;
  if (rt->invalid || rt->overflow || acc->chem_changed <= threshold || rt->iters >= max_iter)
    rt->done = 1;
}

__global__ void k_rt_reset(RtState* rt) {
  unsigned long long* p = reinterpret_cast<unsigned long long*>(rt);
  for (int i = threadIdx.x; i < int(sizeof(RtState) / 8); i += blockDim.x) p[i] = 0ull;
}

int grid_for(int64_t items, int block, int cap) {
  int64_t g = (items + block - 1) / block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return int(g);
}

}  // namespace

hipError_t launch_prep_fields(const double* n_H, const double* x, double n_th, int64_t ncell,
                              double* a64, Accum* acc, int cus, hipStream_t s) {
  hipLaunchKernelGGL(k_prep, dim3(grid_for(ncell, 256, cus * 16)), dim3(256), 0, s, n_H, x, n_th,
                     ncell, a64, acc);
  return hipGetLastError();
}

hipError_t launch_rt_begin(nrt_ctx* c, const double* x, double* gamma,
                           const unsigned long long* skip, hipStream_t s) {
  const int64_t n = c->lay.cells;
  hipLaunchKernelGGL(k_begin_pass, dim3(grid_for(n, 256, c->cu_count * 16)), dim3(256), 0, s, gamma,
                     n, c->acc, c->n_H, x, c->desc.n_th, c->a64, &c->rt->invalid, skip);
  return hipGetLastError();
}

hipError_t launch_rt_check(const Accum* acc, RtState* rt, unsigned long long threshold,
                           unsigned long long max_iter, hipStream_t s) {
  hipLaunchKernelGGL(k_rt_check, dim3(1), dim3(64), 0, s, acc, rt, threshold, max_iter);
  return hipGetLastError();
}

hipError_t launch_rt_reset(RtState* rt, hipStream_t s) {
  hipLaunchKernelGGL(k_rt_reset, dim3(1), dim3(64), 0, s, rt);
  return hipGetLastError();
}

hipError_t launch_prep(nrt_ctx* c) {
  return launch_prep_fields(c->n_H, c->x, c->desc.n_th, c->lay.cells, c->a64, c->acc,
                            c->cu_count, c->stream);
}

hipError_t launch_spec_stop(const nrt_ctx* c, double* out) {
  const SpecTable t{c->spec_nint, c->spec64, c->spec32};
  // the table ends at an octave boundary: node tau 2^octaves - 1
  const double hi = std::ldexp(1.0, c->spec_nint >> kSpecLog2Sub) - 1.0;
  hipLaunchKernelGGL(k_spec_stop, dim3(1), dim3(64), 0, c->stream, t, c->desc.tau_max, hi, out);
  return hipGetLastError();
}

hipError_t launch_begin_pass(double* gamma, int64_t count, Accum* acc, int cus, hipStream_t s) {
  hipLaunchKernelGGL(k_begin_pass, dim3(grid_for(count, 256, cus * 16)), dim3(256), 0, s, gamma,
                     count, acc, nullptr, nullptr, 0.0, nullptr, nullptr, nullptr);
  return hipGetLastError();
}

hipError_t launch_zero_accum(Accum* acc, hipStream_t s) {
  hipLaunchKernelGGL(k_zero_accum, dim3(1), dim3(256), 0, s, acc);
  return hipGetLastError();
}

namespace {

// The march instantiation for a precision, correction mode, boundary and
// spectrum, and:
//  - the sums of the deposit table: FP64, except in the mixed path's levels 0..4.
//    These set the values around a source (a level-4 ray ends 7.8 cells from it
//    at N_min = 4), and all of them where rays go no deeper (n_min_ray = 0,
//    l_max < 5).  FP64 sums there would be a little faster and a little more
//    exact, but move Gamma by 2e-8 to 3e-8 of itself (its error against 64 bits:
//    6.5e-8 FP32, 4.7e-8 FP64 at 128^3, 7.7e-8 and 7.5e-8 at 256^3), and a path
//    keeps the values that it gave.  What FP32 costs, against FP64 everywhere: an
//    LDS add takes the lanes one by one (3.1 cycles each); open 97^3 676 / 617 us,
//    128^3 10.25 / 10.10 ms, 256^3 12.5 / 11.8, 512^3 7.21 / 6.88, unsplit rays of
//    330 cells 2.79 / 2.43; rays of 5 cells 1.06 / 1.19;
//  - the cell index: 32 bits while n^3 <= 2^32 (n <= 1625), else 64.
using MarchKernel = void (*)(MarchArgs);
constexpr int kFirstWideSumLevel = 5;

template <bool MIXED, bool PERIODIC, bool POLY, typename V, typename Idx>
MarchKernel march_for_corr(int corr) {
  switch (corr) {
    case NRT_CORR_NONE: return k_march<MIXED, NRT_CORR_NONE, PERIODIC, POLY, V, Idx>;
    case NRT_CORR_LINEAR: return k_march<MIXED, NRT_CORR_LINEAR, PERIODIC, POLY, V, Idx>;
    case NRT_CORR_SQUARED: return k_march<MIXED, NRT_CORR_SQUARED, PERIODIC, POLY, V, Idx>;
    case NRT_CORR_NAIVE: return k_march<MIXED, NRT_CORR_NAIVE, PERIODIC, POLY, V, Idx>;
    default: return k_march<MIXED, NRT_CORR_CONSERVATIVE, PERIODIC, POLY, V, Idx>;
  }
}

template <bool MIXED, typename V, typename Idx>
MarchKernel march_for(const nrt_grid_desc& d) {
  if (d.spectrum != NRT_SPEC_MONO)
    return d.periodic ? march_for_corr<MIXED, true, true, V, Idx>(d.corr)
                      : march_for_corr<MIXED, false, true, V, Idx>(d.corr);
  return d.periodic ? march_for_corr<MIXED, true, false, V, Idx>(d.corr)
                    : march_for_corr<MIXED, false, false, V, Idx>(d.corr);
}

bool wide_sums(const nrt_grid_desc& d, int level) {
  return d.precision != NRT_MIXED || level >= kFirstWideSumLevel;
}

MarchKernel march_kernel(const nrt_grid_desc& d, int level) {
  const bool wide = int64_t(d.n) * d.n * d.n > NRT_NARROW_CELLS;
  if (d.precision != NRT_MIXED)
    return wide ? march_for<false, double, int64_t>(d) : march_for<false, double, uint32_t>(d);
  if (!wide_sums(d, level))
    return wide ? march_for<true, float, int64_t>(d) : march_for<true, float, uint32_t>(d);
  return wide ? march_for<true, double, int64_t>(d) : march_for<true, double, uint32_t>(d);
}

}  // namespace

hipError_t march_blocks_per_cu(const nrt_grid_desc& d, int* blocks) {
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, march_kernel(d, kMaxLevel), kBlock, 0);
}

// persistent grid: as many blocks as stay resident, or fewer for small launches
hipError_t launch_march_on(const nrt_grid_desc& d, int cu_count, int resident_per_cu,
                           const nrt_tuning& t, const MarchArgs& args, int64_t rays,
                           hipStream_t st) {
  int per_cu = resident_per_cu > 0 ? resident_per_cu : 2;
  if (t.blocks_per_cu > 0 && t.blocks_per_cu < per_cu) per_cu = t.blocks_per_cu;
  const int blocks = grid_for(rays, kBlock, cu_count * per_cu);
  MarchArgs a = args;
  // Defaults.  A wavefront that refills only once it has drained keeps its 64
  // rays in step: neighbouring pixels at one path length, which share lines of
  // Gamma (5 new ones a step against 10 when it refills at 16 idle lanes; its
  // children are queued side by side, so the next level's runs are bundles
  // again).  Measured, refill at 16 / 64: 1024^3 mixed 351 / 221 ms, 128^3
  // mixed 12.6 / 10.8, FP64 15.7 / 14.2, blackbody 35.7 / 26.8, 256^3 11.5 /
  // 10.4.  Launches with FP32 sums keep the 16 lanes and 128 rays, which set the
  // order of their sums and so their rounding.
  const bool wide = wide_sums(d, a.level);
  a.refill_min = t.refill_min > 0 ? t.refill_min : (wide ? 64 : 16);
  a.claim = t.claim > 0 ? t.claim : (wide ? 256 : 128);
  a.claim_min = t.claim > 0 || !wide ? a.claim : 64;
  hipLaunchKernelGGL(march_kernel(d, a.level), dim3(blocks), dim3(kBlock), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_march(const nrt_ctx* c, const MarchArgs& args, int64_t rays, hipStream_t st) {
  return launch_march_on(c->desc, c->cu_count, c->march_blocks_per_cu, c->tuning, args, rays,
                         st);
}

namespace {
// l0[k] = ndot[k] / 12, the rate of a level-0 ray (a correctly rounded
// division, as on the host); clears the accumulators for a pass
__global__ void k_source_rates(const double* ndot, int64_t m, double* l0, Accum* acc) {
  if (blockIdx.x == 0) clear_accum(acc);
  for (int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; k < m;
       k += int64_t(gridDim.x) * blockDim.x)
    l0[k] = ndot[k] / 12.0;
}
}  // namespace

hipError_t launch_source_rates(const double* ndot, int64_t m, double* l0, Accum* acc,
                               hipStream_t s) {
  hipLaunchKernelGGL(k_source_rates, dim3(grid_for(m, 256, 1024)), dim3(256), 0, s, ndot, m, l0,
                     acc);
  return hipGetLastError();
}

hipError_t launch_budget(const Accum* acc, nrt_budget* out, uint64_t* dropped, double emitted,
                         int64_t spawned, int l_max, hipStream_t s) {
  hipLaunchKernelGGL(k_budget, dim3(1), dim3(64), 0, s, acc, out, dropped, emitted,
                     uint64_t(spawned), l_max);
  return hipGetLastError();
}

hipError_t launch_directions(int levels, int64_t lo, int64_t hi, const double* cos_sin,
                             double* out, hipStream_t s) {
  const int64_t total = dir_table_offset(levels + 1);
  hipLaunchKernelGGL(k_directions, dim3(unsigned((total + 255) / 256)), dim3(256), 0, s, total, lo,
                     hi, reinterpret_cast<const double2*>(cos_sin), out);
  return hipGetLastError();
}

hipError_t launch_healpix(int level, int64_t first, int64_t count, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_healpix, dim3(grid_for(count, 256, 1 << 20)), dim3(256), 0, s, level,
                     first, count, out);
  return hipGetLastError();
}

}  // namespace nrt
