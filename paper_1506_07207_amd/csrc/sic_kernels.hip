// sic_kernels.hip - gfx950 kernels of the simplex-in-cell (SIC) 1D1V step.
//
//   k_tracers  one pass over the tracers: gather + leapfrog move (section 2.3,
//              "gather" with first-order weighting of section 2.4, "move"),
//              and/or the exact segment deposit (section 2.3, eqs. "overlap"
//              and "rho_sum") of the resulting positions.  Workgroups walk
//              a list of work items (by default one item each); one item is
//              a run of 64-tracer chunks of one simulation.  Each workgroup
//              accumulates the item's charge in a private LDS copy of that
//              simulation's mesh and merges it into the global mesh with one
//              atomic per touched cell.
//   k_deposit_faces  the deposit alone (constant segments): per tracer only
//              its cell and segment length; the segments that cross a cell
//              face are queued per wavefront and their face geometry runs 64
//              at a time.
//   k_resident a small simulation (up to 32 chunks) stepped many times in one
//              launch of one workgroup: state in registers, mesh in LDS.
//   k_step     a larger single simulation's step in one launch: every
//              workgroup solves the previous step's charge for itself.
//   k_solve    one workgroup per simulation: finishes the deposit (prefix sum
//              of the covered-run difference array), removes the mean density,
//              integrates Gauss's law for the face fields, averages them to
//              cell centres (identical to the 3-point Poisson equation with a
//              centred-difference field), and writes the field energy and
//              the diagnostics row.
//
// Deposit of one segment.  In mesh units (u = x / dx) a segment [u0, u1]
// covers cells c0 = floor(u0) .. c1 = ceil(u1) - 1.  Its charge q is spread
// with density q / (u1 - u0): the two end cells get their partial overlaps,
// and each fully covered cell in between gets the same amount q / (u1 - u0).
// The covered run is added through a difference array D (+w at its first
// cell, -w after its last) that the solve kernel prefix-sums, so a segment
// costs O(1) however many cells it spans.
//
// Split forms keep positions as (cell, fraction) and deposit int64
// fixed-point charge: the first end cell gets round(q * f0), every covered
// cell round(q / len) and the last end cell the remainder, so each segment
// deposits exactly its fixed-point charge and the mesh is independent of the
// order of the atomics.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "sic_internal.h"

namespace sic {

namespace {

// c reduced by one period either way, for c in [-period, 2 period): of c and
// c + period the smaller as unsigned integers is the one that is not negative,
// and so for c and c - period (four instructions where compares and selects
// take seven).
__device__ __forceinline__ uint32_t wrap_once(int c, uint32_t period) {
  const uint32_t r = min((uint32_t)c, (uint32_t)c + period);
  return min(r, r - period);
}

// Cell index modulo nc for c in [-nc, 2nc); anything else (only reachable
// from non-finite data) is clamped to the last cell so that no access leaves
// the mesh.
__device__ __forceinline__ int wrap_cell(int c, int nc) {
  return (int)min(wrap_once(c, (uint32_t)nc), (uint32_t)nc - 1u);
}

// Periodic reduction of a position into [0, L).  The common case moves at
// most one period, where x - L is exact; a sum that rounds up to L is 0.
__device__ __forceinline__ double wrap_into_box(double x, double L) {
  if (x >= L) {
    x = x - L;
    if (x >= L) x = x - L * floor(x / L);
  } else if (x < 0.0) {
    x = (x >= -L) ? x + L : x - L * floor(x / L);
    if (x < 0.0) x += L;
  }
  return (x >= L) ? 0.0 : x;
}

// ---- split position words ----
//
// U32: the low 32 bits hold the cell, the high 32 bits the fraction of the
// cell as an unsigned integer in units of 2^-32 cell.
// F32: the low 32 bits hold an index on a lattice of 2^kSubBits sub-cells
// per cell (cell = index >> kSubBits), the high 32 bits a float32 offset in
// [0, 1) of a sub-cell.  With 4096 cells at most the index fits 32 bits; the
// float's 24-bit significand then resolves about 2^-44 of a cell, the
// resolution of a float64 position near the top of such a mesh, where a
// float32 offset spanning a whole cell would only resolve 2^-24 of it.
constexpr int kSubBits = 20;
constexpr uint32_t kSubMask = (1u << kSubBits) - 1u;

template <int PREC>
__device__ __forceinline__ int split_cell(uint64_t w) {
  if constexpr (PREC == kSplitF32) return (int)((uint32_t)w >> kSubBits);
  else return (int)(uint32_t)w;
}

// Position within the cell, in [0, 1) cell.
template <int PREC>
__device__ __forceinline__ double split_frac(uint64_t w) {
  if constexpr (PREC == kSplitF32) {
    return ((double)((uint32_t)w & kSubMask) + (double)__uint_as_float((uint32_t)(w >> 32))) * 0x1p-20;
  } else {
    return (double)(uint32_t)(w >> 32) * 0x1p-32;
  }
}

// Word of the point cell + r (r in [0, 1] cell, cell any integer the caller
// has reduced to -nc .. 2nc - 1): the rounding of r to the offset type may
// carry into the next cell.
template <int PREC>
__device__ __forceinline__ uint64_t split_word(int cell, double r, int nc) {
  if constexpr (PREC == kSplitF32) {
    const double ts = r * 0x1p20;  // sub-cells, exact
    double sub = floor(ts);
    float o = (float)(ts - sub);
    if (o >= 1.0f) {
      o = 0.0f;
      sub += 1.0;
    }
    int c = cell;
    if (sub >= 0x1p20) {
      sub -= 0x1p20;
      c += 1;
    }
    c = wrap_cell(c, nc);
    const uint32_t idx = ((uint32_t)c << kSubBits) | ((uint32_t)sub & kSubMask);
    return (uint64_t)idx | ((uint64_t)__float_as_uint(o) << 32);
  } else {
    double sc = rint(r * 4294967296.0);
    int c = cell;
    if (sc >= 4294967296.0) {
      sc = 0.0;
      c += 1;
    }
    return (uint64_t)(uint32_t)wrap_cell(c, nc) | ((uint64_t)(uint32_t)sc << 32);
  }
}

// Position in mesh units of a state word.
template <int PREC>
__device__ __forceinline__ double mesh_pos(uint64_t w, double inv_dx) {
  if constexpr (PREC == kFP64) {
    return __longlong_as_double((long long)w) * inv_dx;
  } else if constexpr (PREC == kSplitF32) {
    // the index with its cell, in sub-cells: one rounding
    return ((double)(uint32_t)w + (double)__uint_as_float((uint32_t)(w >> 32))) * 0x1p-20;
  } else {
    return (double)split_cell<PREC>(w) + split_frac<PREC>(w);
  }
}

// Field at a tracer: linear interpolation between the two cell centres
// around it (first-order weighting), from a field array with one ghost cell on
// each side (E[-1] = E[nc-1], E[nc] = E[0]): no periodic wrap of the two
// indices.  u is the position in mesh units.  The clamp keeps non-finite positions inside the array.
__device__ __forceinline__ double gather_field_ghost(const double *E, double u, int nc) {
  const double g = u - 0.5;
  const double f = floor(g);
  const double s = g - f;
  const int j = min(max((int)f, -1), nc - 1);
  return (1.0 - s) * E[j] + s * E[j + 1];
}

// Split-form word moved by du cells: the position advances by whole cells
// (or, in the F32 form, whole sub-cells) plus a rest that is re-quantised;
// the index wraps periodically.  A non-finite move (a non-finite velocity,
// which the diagnostics flag) leaves the word as it is: a split position has
// no non-finite value.
template <int PREC>
__device__ __forceinline__ uint64_t advance_split(uint64_t w, double du, int nc) {
  // F32 counts in sub-cells, U32 in cells
  constexpr double kUnit = PREC == kSplitF32 ? 0x1p20 : 1.0;
  const double t = (PREC == kSplitF32 ? (double)__uint_as_float((uint32_t)(w >> 32)) : split_frac<PREC>(w)) +
                   du * kUnit;
  if (!(t - t == 0.0)) return w;
  const double k = floor(t);
  const double r = t - k;
  // a step of under 2^30 units converts through a 32-bit integer; longer
  // ones (and their 64-bit conversion) take the rare branch below
  const bool near = fabs(k) < 0x1p30;
  long long carry = 0;
  uint32_t bits;
  if constexpr (PREC == kSplitF32) {
    float o = (float)r;
    if (o >= 1.0f) {
      o = 0.0f;
      carry = 1;
    }
    bits = __float_as_uint(o);
  } else {
    double sc = rint(r * 4294967296.0);
    if (sc >= 4294967296.0) {
      sc = 0.0;
      carry = 1;
    }
    bits = (uint32_t)sc;
  }
  const long long period = (long long)nc << (PREC == kSplitF32 ? kSubBits : 0);
  // a move of less than a period needs one conditional wrap; the (slow,
  // 64-bit) remainder only for longer ones
  bool far = !near;
  long long idx = 0;
  if constexpr (PREC == kSplitU32) {
    // the cell index is below 4096: a near move stays in 32-bit integers
    const uint32_t c = wrap_once((int)(uint32_t)w + (int)(near ? k : 0.0) + (int)carry, (uint32_t)nc);
    far = far || c >= (uint32_t)nc;
    idx = c;
  } else if (nc <= (1 << (30 - kSubBits))) {
    // and so does one of an index below 2^30
    const uint32_t i = wrap_once((int)(uint32_t)w + (int)(near ? k : 0.0) + (int)carry, (uint32_t)period);
    far = far || i >= (uint32_t)period;
    idx = i;
  } else {
    idx = (long long)(uint32_t)w + (long long)(int)(near ? k : 0.0) + carry;
    if (idx >= period) idx -= period;
    else if (idx < 0) idx += period;
    far = far || (unsigned long long)idx >= (unsigned long long)period;
  }
  if (far) {
    idx = ((long long)(uint32_t)w + (long long)k + carry) % period;
    if (idx < 0) idx += period;
  }
  return (uint64_t)(uint32_t)idx | ((uint64_t)bits << 32);
}

// Drift of a state word by dt * v.
template <int PREC>
__device__ __forceinline__ uint64_t drift(uint64_t w, double v, double dt, double L, double inv_dx, int nc) {
  if constexpr (PREC == kFP64) {
    const double x = __longlong_as_double((long long)w);
    return (uint64_t)__double_as_longlong(wrap_into_box(x + dt * v, L));
  } else {
    return advance_split<PREC>(w, (dt * v) * inv_dx, nc);
  }
}

template <class T>
__device__ __forceinline__ void lds_add(T *p, T v) {
  if constexpr (std::is_same<T, double>::value) {
    unsafeAtomicAdd(p, v);
  } else {
    atomicAdd(p, v);
  }
}

// Adds w to cells lo..hi (unwrapped indices, 0 <= hi - lo < nc) of the
// difference array: +w at the first cell, -w after the last.
template <class T>
__device__ __forceinline__ void add_run(T *sD, int lo, int hi, T w, int nc) {
  const int l = wrap_cell(lo, nc);
  const int h = l + min(hi - lo, nc - 1);
  lds_add(sD + l, w);
  if (h + 1 < nc) {
    lds_add(sD + h + 1, (T)(0 - w));
  } else if (h >= nc) {
    lds_add(sD, w);
    lds_add(sD + (h - nc + 1), (T)(0 - w));
  }
}

// 1 / x (x finite, non-zero, normal) by the hardware reciprocal and two
// Newton steps: within an ulp or so of the correctly rounded quotient, at
// about half the instructions of a division.
__device__ __forceinline__ double recip(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  return fma(r, fma(-x, r, 1.0), r);
}

struct Geo {
  double L, half_L, dx, inv_dx, dt;
  int nc;
};

// ---- deposit of constant segments (section 2.3): per segment ----
//
// Used where the tracers are also moved (the fused step): each lane adds its
// segment's end-cell overlaps and covered run directly; the LDS atomics hide
// behind the state the step streams.

// FP64 segment from position a to position b (both in [0, L)).
__device__ __forceinline__ double deposit_fp64(double a, double b, double q, const Geo &g, double *sP,
                                               double *sD) {
  double d = b - a;
  if (d >= g.half_L) d -= g.L;
  else if (d < -g.half_L) d += g.L;
  const double ad = fabs(d);
  if (!(ad <= g.half_L)) return ad;  // non-finite positions: nothing deposited
  if (d == 0.0) {
    // zero-length segment: all of q into the cell owning the point, a point
    // on a face belonging to the lower cell
    const int c = wrap_cell((int)ceil(a / g.dx) - 1, g.nc);
    lds_add(sP + c, q);
    return 0.0;
  }
  const double ua = a * g.inv_dx;
  const double ue = ua + d * g.inv_dx;
  const double u0 = d > 0.0 ? ua : ue;
  const double u1 = d > 0.0 ? ue : ua;
  const double len = u1 - u0;
  const double f0 = floor(u0);
  const int c0 = (int)f0;
  const int c1 = (int)ceil(u1) - 1;
  if (!(len > 0.0) || c1 <= c0) {
    lds_add(sP + wrap_cell(c0, g.nc), q);
    return ad;
  }
  const double w = q / len;
  lds_add(sP + wrap_cell(c0, g.nc), w * ((f0 + 1.0) - u0));
  lds_add(sP + wrap_cell(c1, g.nc), w * (u1 - (double)c1));
  if (c1 - c0 >= 2) add_run(sD, c0 + 1, c1 - 1, w, g.nc);
  return ad;
}

// Split-form segment from word wa at ua to ub (mesh_pos).
template <int PREC>
__device__ __forceinline__ double deposit_split(uint64_t wa, double ua, double ub, long long qf, const Geo &g,
                                                unsigned long long *sP, unsigned long long *sD) {
  const double half_nc = 0.5 * (double)g.nc;
  double du = ub - ua;
  if (du >= half_nc) du -= (double)g.nc;
  else if (du < -half_nc) du += (double)g.nc;
  const double ad = fabs(du) * g.dx;
  if (!(fabs(du) <= half_nc)) return ad;
  if (du == 0.0) {
    const int ca = split_cell<PREC>(wa);
    const int c = wrap_cell(split_frac<PREC>(wa) == 0.0 ? ca - 1 : ca, g.nc);
    lds_add(sP + c, (unsigned long long)qf);
    return 0.0;
  }
  const double ue = ua + du;
  const double u0 = du > 0.0 ? ua : ue;
  const double u1 = du > 0.0 ? ue : ua;
  const double len = u1 - u0;
  const double f0 = floor(u0);
  const int c0 = (int)f0;
  const int c1 = (int)ceil(u1) - 1;
  if (!(len > 0.0) || c1 <= c0) {
    lds_add(sP + wrap_cell(c0, g.nc), (unsigned long long)qf);
    return ad;
  }
  // a correctly rounded quotient is not needed: the shares are rounded to
  // fixed point and the last takes the rest, so the charge is conserved
  // exactly
  const double inv = recip(len);
  const double qd = (double)qf;
  const long long p0 = llrint(qd * (((f0 + 1.0) - u0) * inv));
  long long p1 = qf - p0;
  if (c1 - c0 >= 2) {
    const long long wfix = llrint(qd * inv);
    add_run(sD, c0 + 1, c1 - 1, (unsigned long long)wfix, g.nc);
    p1 -= (long long)(c1 - c0 - 1) * wfix;
  }
  lds_add(sP + wrap_cell(c0, g.nc), (unsigned long long)p0);
  lds_add(sP + wrap_cell(c1, g.nc), (unsigned long long)p1);
  return ad;
}

// ---- deposit of constant segments (section 2.3): face-crossing form ----
//
// Within one 64-tracer chunk let S_t be the charge of the segments before
// segment t.  Walking along the sheet, the charge passed so far at a point of
// segment t is S_t plus the share of q_t before that point (the box function
// is uniform).  The charge of a cell is that cumulative charge where the
// sheet leaves the cell minus where it entered, summed over its visits, so
// every face a segment crosses adds the cumulative charge C at that face to
// the cell being left and subtracts it from the cell being entered.  The two
// terms at a tracer (the end of one segment, the start of the next) fall in
// the same cell and cancel, so a segment inside one cell adds nothing; the
// chunk adds its total charge to the cell where its last segment ends (its
// start contributes -S_0 = 0).  Faces strictly between a segment's first and
// last crossing enclose fully covered cells, which all get q/length (one
// run in the difference array).  The result equals the exact overlap
// deposit; on a dense sheet a wavefront issues LDS atomics only where it
// crosses faces, instead of one or two per tracer.  In fixed point every term
// is an integer and the terms telescope, so each chunk deposits exactly its
// charge.  Used for deposits that do not also move the tracers (the
// deposit-only kernel below), where the per-tracer arithmetic, not the state
// traffic, sets the pace; inside the fused step the per-segment form is
// faster (measured: 8 %).
//
// Cells here are raw: -1 .. nc - 1 before the periodic wrap, a point on a
// face belonging to the lower cell (the W_0 tie rule, which decides where a
// zero-length segment puts its charge): ceil(x / dx) - 1 with the rounded
// quotient.

template <class T>
struct Crossings {
  int lo, hi;  // faces crossed, unwrapped (hi < lo: none)
  T cf, cl;    // cumulative charge at the first and at the last face crossed
  T w;         // charge of each fully covered cell
};

// Faces crossed by the segment from tracer a (cell pa) to tracer b (cell pb),
// the shorter way round, with charge q and chunk charge S before it.
template <int PREC, class T>
__device__ __forceinline__ Crossings<T> face_crossings(uint64_t wa, uint64_t wb, int pa, int pb, T q, T S,
                                                       const Geo &g, double *len_out) {
  Crossings<T> c;
  c.lo = 1;
  c.hi = 0;
  c.cf = c.cl = c.w = (T)0;
  double ua, dm;
  int m = 0;  // periodic image of b relative to a
  if constexpr (PREC == kFP64) {
    const double xa = __longlong_as_double((long long)wa);
    double d = __longlong_as_double((long long)wb) - xa;
    if (d >= g.half_L) {
      d -= g.L;
      m = -1;
    } else if (d < -g.half_L) {
      d += g.L;
      m = 1;
    }
    *len_out = fabs(d);
    if (!(fabs(d) <= g.half_L)) return c;  // non-finite positions
    ua = xa * g.inv_dx;
    dm = d * g.inv_dx;
  } else {
    ua = mesh_pos<PREC>(wa, g.inv_dx);
    const double half_nc = 0.5 * (double)g.nc;
    double du = mesh_pos<PREC>(wb, g.inv_dx) - ua;
    if (du >= half_nc) {
      du -= (double)g.nc;
      m = -1;
    } else if (du < -half_nc) {
      du += (double)g.nc;
      m = 1;
    }
    *len_out = fabs(du) * g.dx;
    if (!(fabs(du) <= half_nc)) return c;
    dm = du;
  }
  const int pbu = pb + m * g.nc;
  if (dm > 0.0) {
    c.lo = pa + 1;  // upward: faces pa+1 .. pb
    c.hi = pbu;
  } else if (dm < 0.0) {
    c.lo = pbu + 1;  // downward: faces pa .. pb+1
    c.hi = pa;
  }
  if (c.hi < c.lo) return c;
  const double len = fabs(dm);
  // length of the segment before its first face, and the charge on it
  const double before = fmin(fmax(dm > 0.0 ? (double)c.lo - ua : ua - (double)c.hi, 0.0), len);
  if constexpr (PREC == kFP64) {
    c.w = q / len;
    c.cf = S + c.w * before;
    c.cl = c.cf + (double)(c.hi - c.lo) * c.w;
  } else {
    const double r = (double)(long long)q / len;
    const long long wfix = llrint(r);
    c.w = (T)wfix;
    c.cf = S + (T)llrint(r * before);
    c.cl = c.cf + (T)((long long)(c.hi - c.lo) * wfix);
  }
  return c;
}

template <class T, class Op>
__device__ __forceinline__ T wave_incl_scan(T v, Op op);
template <class T>
__device__ __forceinline__ T lane_up1(T v);

// Exclusive prefix sum over the wavefront (called by all 64 lanes): the
// inclusive scan moved up one lane.
template <class T>
__device__ __forceinline__ T wave_exclusive_sum(T v) {
  const int lane = threadIdx.x & 63;
  const T prev = lane_up1(wave_incl_scan(v, [](T x, T y) { return x + y; }));
  return lane == 0 ? (T)0 : prev;
}

// ---- piecewise-linear segments (section 2.5) ----
//
// Segment i (tracer i to tracer i+1) carries rho(u) = rho0 + (u - c) g in mesh
// units, rho0 = q / length, c its centroid, g the central difference of the
// neighbouring segments' rho0 over their centroid separation, or 0 at a fold
// corner (centroids not monotone), at an open sheet's end, or when any of the
// three segments has zero length.  Each end cell gets the integral over its
// overlap; the fully covered cells l..h get rho0 + g (j + 1/2 - c), a linear
// ramp A + B (j - l) added through the difference arrays D (constant part)
// and R (second difference of the ramp), so a segment still costs O(1).

// Ramp A + B (j - l) on cells l..h of one period (0 <= l <= h < nc).
template <class T>
__device__ __forceinline__ void add_ramp_nowrap(T *sD, T *sR, int l, int h, T A, T B, int nc) {
  lds_add(sD + l, A);
  if (h + 1 < nc) lds_add(sD + h + 1, (T)(0 - (A + B * (T)(h - l))));
  if (l + 1 <= h) {  // the slope needs a run of two cells or more
    lds_add(sR + l + 1, B);
    if (h + 1 < nc) lds_add(sR + h + 1, (T)(0 - B));
  }
}

// Ramp on unwrapped cells lo..hi (0 <= hi - lo < nc).
template <class T>
__device__ __forceinline__ void add_ramp(T *sD, T *sR, int lo, int hi, T A, T B, int nc) {
  const int l = wrap_cell(lo, nc);
  const int h = l + min(hi - lo, nc - 1);
  if (h < nc) {
    add_ramp_nowrap(sD, sR, l, h, A, B, nc);
  } else {
    add_ramp_nowrap(sD, sR, l, nc - 1, A, B, nc);
    add_ramp_nowrap(sD, sR, 0, h - nc, (T)(A + B * (T)(nc - l)), B, nc);
  }
}

__device__ __forceinline__ double min_image_cells(double d, double half_nc, double nc) {
  if (d >= half_nc) d -= nc;
  else if (d < -half_nc) d += nc;
  return d;
}

// Geometry of a segment in mesh units: start, signed length along the
// shorter way round the box and centroid.
struct SegGeo {
  double u, d, c;
};

// Geometry of the segment from state word wa to wb.  Float64 positions take
// the physical minimum image, as the constant scheme does; split positions
// take it in mesh units.
template <int PREC>
__device__ __forceinline__ SegGeo lin_geo(uint64_t wa, uint64_t wb, const Geo &g) {
  SegGeo s;
  if constexpr (PREC == kFP64) {
    const double xa = __longlong_as_double((long long)wa);
    double d = __longlong_as_double((long long)wb) - xa;
    if (d >= g.half_L) d -= g.L;
    else if (d < -g.half_L) d += g.L;
    s.u = xa * g.inv_dx;
    s.d = d * g.inv_dx;
  } else {
    s.u = mesh_pos<PREC>(wa, g.inv_dx);
    s.d = min_image_cells(mesh_pos<PREC>(wb, g.inv_dx) - s.u, 0.5 * (double)g.nc, (double)g.nc);
  }
  s.c = s.u + 0.5 * s.d;
  return s;
}

// The same of split positions, from their mesh positions.
__device__ __forceinline__ SegGeo lin_geo_mesh(double ua, double ub, const Geo &g) {
  SegGeo s;
  s.u = ua;
  s.d = min_image_cells(ub - ua, 0.5 * (double)g.nc, (double)g.nc);
  s.c = s.u + 0.5 * s.d;
  return s;
}

// Mean density q / length of a segment (q in the accumulator's units), the
// length taken over the extent the deposit integrates so that its pieces add
// up to q; 0 for a zero-length segment.  The quotient by the reciprocal
// (recip): every density, a lane's own and the staged neighbours', comes
// from this one function, so neighbours see the same bits.
__device__ __forceinline__ double lin_density(const SegGeo &s, double q) {
  const double u0 = s.d > 0.0 ? s.u : s.u + s.d;
  const double u1 = s.d > 0.0 ? s.u + s.d : s.u;
  const double len = u1 - u0;
  return len > 0.0 ? q * recip(len) : 0.0;
}

// The density a neighbour's gradient takes from a segment: NaN marks a
// missing segment or one of zero signed length, which drop the gradient.
__device__ __forceinline__ double lin_nb_density(double d, double r) {
  return d != 0.0 ? r : __longlong_as_double(0x7ff8000000000000ll);
}

// Gradient of a segment of signed length d from its neighbours' signed
// lengths and densities (m: the segment before, p: the one after;
// lin_nb_density): the central difference of the densities over the centroid
// separation, 0 at a fold corner (centroids not monotone) or when a neighbour
// is missing or has zero length (density NaN).  Consecutive segments share an
// end, so the centroid before lies (dm_len + d) / 2 behind this one and the
// one after (d + dp_len) / 2 ahead, along the shorter way round the box
// (each length is at most half the box).
__device__ __forceinline__ double lin_gradient(double d, double dm_len, double rm, double dp_len, double rp) {
  // without branches: a wavefront's lanes mostly take the quotient, and the
  // others select 0 (their divisor replaced by 1)
  const double dm = -0.5 * (dm_len + d);
  const double dp = 0.5 * (d + dp_len);
  const bool ok = rm == rm && rp == rp && ((dm < 0.0 && dp > 0.0) || (dm > 0.0 && dp < 0.0));
  const double q = (rp - rm) * recip(ok ? dp - dm : 1.0);
  return ok ? q : 0.0;
}

// A neighbouring segment as the gradient needs it: signed length and density
// (lin_nb_density).
struct LinNb {
  double d, r;
};

// FP64: deposit segment i given its geometry, gradient and density
// r0 = q / length (lin_density; mesh units).
__device__ __forceinline__ void deposit_linear_fp64(double a_phys, const SegGeo &sg, double g, double q, double r0,
                                                    const Geo &geo, double *sP, double *sD, double *sR) {
  if (sg.d == 0.0) {
    const int c = wrap_cell((int)ceil(a_phys / geo.dx) - 1, geo.nc);
    lds_add(sP + c, q);
    return;
  }
  const double u0 = sg.d > 0.0 ? sg.u : sg.u + sg.d;
  const double u1 = sg.d > 0.0 ? sg.u + sg.d : sg.u;
  const double len = u1 - u0;
  const double f0 = floor(u0);
  const int c0 = (int)f0;
  const int c1 = (int)ceil(u1) - 1;
  // a segment inside one cell puts q there; a longer one its first piece
  // (one atomic for both kinds, so a wavefront that holds both issues one)
  const bool multi = (len > 0.0) && c1 > c0;
  const double e0 = f0 + 1.0;
  const double w0 = e0 - u0;
  lds_add(sP + wrap_cell(c0, geo.nc), multi ? w0 * (r0 + g * (0.5 * (u0 + e0) - sg.c)) : q);
  if (multi) {
    const double w1 = u1 - (double)c1;
    lds_add(sP + wrap_cell(c1, geo.nc), w1 * (r0 + g * (0.5 * ((double)c1 + u1) - sg.c)));
    if (c1 - c0 >= 2) {
      const double A = r0 + g * ((double)(c0 + 1) + 0.5 - sg.c);
      add_ramp(sD, sR, c0 + 1, c1 - 1, A, g, geo.nc);
    }
  }
}

// Split form: fixed-point pieces, the last end cell takes the remainder so
// the segment deposits exactly q_fix.
__device__ __forceinline__ void deposit_linear_split(int cell_a, double frac_a, const SegGeo &sg, double g,
                                                     long long qf, double r0, const Geo &geo, unsigned long long *sP,
                                                     unsigned long long *sD, unsigned long long *sR) {
  if (sg.d == 0.0) {
    const int c = wrap_cell(frac_a == 0.0 ? cell_a - 1 : cell_a, geo.nc);
    lds_add(sP + c, (unsigned long long)qf);
    return;
  }
  const double u0 = sg.d > 0.0 ? sg.u : sg.u + sg.d;
  const double u1 = sg.d > 0.0 ? sg.u + sg.d : sg.u;
  const double len = u1 - u0;
  const double f0 = floor(u0);
  const int c0 = (int)f0;
  const int c1 = (int)ceil(u1) - 1;
  // a segment inside one cell puts qf there; a longer one its first piece
  // (one atomic for both kinds)
  const bool multi = (len > 0.0) && c1 > c0;
  const double e0 = f0 + 1.0;
  const long long p0 = multi ? llrint((e0 - u0) * (r0 + g * (0.5 * (u0 + e0) - sg.c))) : qf;
  lds_add(sP + wrap_cell(c0, geo.nc), (unsigned long long)p0);
  if (multi) {
    long long p1 = qf - p0;
    if (c1 - c0 >= 2) {
      const long long n = c1 - c0 - 1;
      const long long A = llrint(r0 + g * ((double)(c0 + 1) + 0.5 - sg.c));
      const long long B = llrint(g);
      add_ramp(sD, sR, c0 + 1, c1 - 1, (unsigned long long)A, (unsigned long long)B, geo.nc);
      p1 -= n * A + B * (n * (n - 1) / 2);
    }
    lds_add(sP + wrap_cell(c1, geo.nc), (unsigned long long)p1);
  }
}

// ---- first-order weighting of segments (section 2.4) ----
//
// Every slice of the box is assigned to the grid points (cell centres) with
// the hat W_1.  With s = u - 1/2 (grid point j at s = j) and r the charge per
// mesh unit, grid point j receives r [H(s1 - j) - H(s0 - j)], H the
// antiderivative of the unit hat.  For a point s = f + t (f = floor(s)), the
// vector H(s - j) over j is 1 up to j = f, less (1 - t)^2 / 2 at f, plus
// t^2 / 2 at f + 1.  With n = f1 - f0 the segment therefore adds
//   f0: a0                 f0 + 1: r - b0 (n >= 1)
//   f0 + 2 .. f1 - 1: r    f1: r - a1 (n >= 2)        f1 + 1: b1 (n >= 1)
// where a = r (1 - t)^2 / 2 and b = r t^2 / 2 at either end; the terms that
// land on one grid point are summed first, so a segment costs as many LDS
// additions as it has distinct grid points, up to four, plus the difference
// array pair for a run of fully covered ones.  Summed terms are written in
// factored form, which keeps a short segment's pieces accurate to rounding of
// its own charge (the plain differences would lose q/length times the
// rounding of O(1) numbers): n = 0 gives f0 q (1 - tm) and f0 + 1 q tm with
// tm = (t0 + t1) / 2 (the hat at the segment's midpoint); n = 1 gives f0 + 1
// r [(1 - t0)(1 + t0) + t1 (2 - t1)] / 2.

__device__ __forceinline__ void deposit_cic_fp64(double u_a, double d_mesh, double q, const Geo &g, double *sP,
                                                 double *sD) {
  const double s0 = (d_mesh > 0.0 ? u_a : u_a + d_mesh) - 0.5;
  const double s1 = (d_mesh > 0.0 ? u_a + d_mesh : u_a) - 0.5;
  const double fl0 = floor(s0);
  const double t0 = s0 - fl0;
  const int f0 = (int)fl0;
  const double fl1 = floor(s1);
  const double t1 = s1 - fl1;
  const int n = (int)fl1 - f0;  // 0 for a point (s1 = s0: t1 = t0, so tm = t0)
  // grid points f0 and f0 + 1 take one addition each in every case; the
  // density (a division) is computed when some lane of the wavefront needs it
  const bool longseg = n >= 1;
  double r = 0.0;
  if (__builtin_amdgcn_ballot_w64(longseg) != 0) r = q / (longseg ? s1 - s0 : 1.0);
  const double hr = 0.5 * r;
  const double tm = 0.5 * (t0 + t1);
  const double a0 = hr * ((1.0 - t0) * (1.0 - t0)), b0 = hr * (t0 * t0);
  lds_add(sP + wrap_cell(f0, g.nc), longseg ? a0 : q * (1.0 - tm));
  lds_add(sP + wrap_cell(f0 + 1, g.nc),
          longseg ? (n == 1 ? hr * ((1.0 - t0) * (1.0 + t0) + t1 * (2.0 - t1)) : r - b0) : q * tm);
  if (longseg) {
    const double a1 = hr * ((1.0 - t1) * (1.0 - t1)), b1 = hr * (t1 * t1);
    lds_add(sP + wrap_cell(f0 + n + 1, g.nc), b1);
    if (n >= 2) {
      lds_add(sP + wrap_cell(f0 + n, g.nc), r - a1);
      if (n >= 3) add_run(sD, f0 + 2, f0 + n - 1, r, g.nc);
    }
  }
}

// Split form: the same terms in fixed-point units; the term at f1 + 1 (at
// f0 + 1 when n = 0) takes the remainder so the segment deposits exactly qf.
__device__ __forceinline__ void deposit_cic_split(double u_a, double d_mesh, long long qf, const Geo &g,
                                                  unsigned long long *sP, unsigned long long *sD) {
  const double qd = (double)qf;
  const double s0 = (d_mesh > 0.0 ? u_a : u_a + d_mesh) - 0.5;
  const double s1 = (d_mesh > 0.0 ? u_a + d_mesh : u_a) - 0.5;
  const double fl0 = floor(s0);
  const double t0 = s0 - fl0;
  const int f0 = (int)fl0;
  if (!(s1 > s0)) {
    const long long p1 = llrint(qd * t0);
    lds_add(sP + wrap_cell(f0, g.nc), (unsigned long long)(qf - p1));
    lds_add(sP + wrap_cell(f0 + 1, g.nc), (unsigned long long)p1);
    return;
  }
  const double fl1 = floor(s1);
  const double t1 = s1 - fl1;
  const int n = (int)fl1 - f0;
  if (n == 0) {
    const long long p0 = llrint(qd * (1.0 - 0.5 * (t0 + t1)));
    lds_add(sP + wrap_cell(f0, g.nc), (unsigned long long)p0);
    lds_add(sP + wrap_cell(f0 + 1, g.nc), (unsigned long long)(qf - p0));
    return;
  }
  const double r = qd / (s1 - s0);
  const double hr = 0.5 * r;
  const double a0 = hr * ((1.0 - t0) * (1.0 - t0)), b0 = hr * (t0 * t0);
  const double a1 = hr * ((1.0 - t1) * (1.0 - t1));
  const long long p0 = llrint(a0);
  const long long p1 = llrint(n == 1 ? hr * ((1.0 - t0) * (1.0 + t0) + t1 * (2.0 - t1)) : r - b0);
  long long rest = qf - p0 - p1;
  lds_add(sP + wrap_cell(f0, g.nc), (unsigned long long)p0);
  lds_add(sP + wrap_cell(f0 + 1, g.nc), (unsigned long long)p1);
  if (n >= 2) {
    const long long pn = llrint(r - a1);
    lds_add(sP + wrap_cell(f0 + n, g.nc), (unsigned long long)pn);
    rest -= pn;
    if (n >= 3) {
      const long long G = llrint(r);
      add_run(sD, f0 + 2, f0 + n - 1, (unsigned long long)G, g.nc);
      rest -= (long long)(n - 2) * G;
    }
  }
  lds_add(sP + wrap_cell(f0 + n + 1, g.nc), (unsigned long long)rest);
}

// A 64-bit value of one lane, broadcast to the wave.
__device__ __forceinline__ uint64_t read_lane64(uint64_t v, int l) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
  return (uint64_t)lo | ((uint64_t)hi << 32);
}

__device__ __forceinline__ double nan_max(double a, double b) {
  // max that propagates NaN (a non-finite segment must reach the flags)
  return (b > a || b != b) ? b : a;
}

// A 4- or 8-byte value moved across lanes by a DPP control (CTRL), written
// in the rows of ROWS; lanes left without a source, and rows not written,
// get 0.  Register moves: no LDS round trip.
template <int CTRL, int ROWS, class T>
__device__ __forceinline__ T dpp_move(T v) {
  static_assert(sizeof(T) == 4 || sizeof(T) == 8, "4- or 8-byte values");
  T r;
  if constexpr (sizeof(T) == 4) {
    int i;
    __builtin_memcpy(&i, &v, 4);
    i = __builtin_amdgcn_update_dpp(0, i, CTRL, ROWS, 0xf, true);
    __builtin_memcpy(&r, &i, 4);
  } else {
    uint64_t u;
    __builtin_memcpy(&u, &v, 8);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWS, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROWS, 0xf, true);
    u = ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
    __builtin_memcpy(&r, &u, 8);
  }
  return r;
}

// Inclusive scan over the wavefront (lane i: v_0 op ... op v_i; all 64
// lanes active): within each 16-lane row by shifts of 1, 2, 4 and 8 lanes,
// then across rows by broadcasting lane 15 into rows 1 and 3 and lane 31
// into rows 2 and 3.  Empty sources contribute 0 (an identity for the sums
// and for the maximum of non-negative values here).
template <class T, class Op>
__device__ __forceinline__ T wave_incl_scan(T v, Op op) {
  v = op(v, dpp_move<0x111, 0xf>(v));  // row_shr:1
  v = op(v, dpp_move<0x112, 0xf>(v));  // row_shr:2
  v = op(v, dpp_move<0x114, 0xf>(v));  // row_shr:4
  v = op(v, dpp_move<0x118, 0xf>(v));  // row_shr:8
  v = op(v, dpp_move<0x142, 0xa>(v));  // row_bcast:15
  v = op(v, dpp_move<0x143, 0xc>(v));  // row_bcast:31
  return v;
}

// Lane 63's value in every lane.
template <class T>
__device__ __forceinline__ T from_lane63(T v) {
  T r;
  if constexpr (sizeof(T) == 4) {
    int i;
    __builtin_memcpy(&i, &v, 4);
    i = __builtin_amdgcn_readlane(i, 63);
    __builtin_memcpy(&r, &i, 4);
  } else {
    uint64_t u;
    __builtin_memcpy(&u, &v, 8);
    u = read_lane64(u, 63);
    __builtin_memcpy(&r, &u, 8);
  }
  return r;
}

// Sum and NaN-propagating maximum over the wavefront, the same bits in every
// lane (all 64 lanes active).
template <class T>
__device__ __forceinline__ T wave_sum(T v) {
  return from_lane63(wave_incl_scan(v, [](T x, T y) { return x + y; }));
}
__device__ __forceinline__ double wave_max(double v) {
  return from_lane63(wave_incl_scan(v, [](double x, double y) { return nan_max(x, y); }));
}

// The value of the next lane (lane_down1) or of the previous one (lane_up1),
// a lane at the wavefront's edge keeping its own: __shfl_down / __shfl_up
// by one lane, as a DPP register move (all 64 lanes active).
template <int CTRL, class T>
__device__ __forceinline__ T dpp_wave_shift(T v) {
  static_assert(sizeof(T) == 4 || sizeof(T) == 8, "4- or 8-byte values");
  T r;
  if constexpr (sizeof(T) == 4) {
    int i;
    __builtin_memcpy(&i, &v, 4);
    i = __builtin_amdgcn_update_dpp(i, i, CTRL, 0xf, 0xf, false);
    __builtin_memcpy(&r, &i, 4);
  } else {
    uint64_t u;
    __builtin_memcpy(&u, &v, 8);
    const int lo0 = (int)(uint32_t)u, hi0 = (int)(uint32_t)(u >> 32);
    const int lo = __builtin_amdgcn_update_dpp(lo0, lo0, CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(hi0, hi0, CTRL, 0xf, 0xf, false);
    u = ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
    __builtin_memcpy(&r, &u, 8);
  }
  return r;
}
template <class T>
__device__ __forceinline__ T lane_down1(T v) {
  return dpp_wave_shift<0x130>(v);  // wave_shl:1
}
template <class T>
__device__ __forceinline__ T lane_up1(T v) {
  return dpp_wave_shift<0x138>(v);  // wave_shr:1
}

}  // namespace

// ---------------------------------------------------------------------------
// Field solve
// ---------------------------------------------------------------------------
namespace {

// Inclusive scan over the 256-thread block of one value per thread, in a
// fixed order.  sWave holds 4 entries.
template <class T>
__device__ __forceinline__ T block_incl_scan(T v, T *sWave) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  v = wave_incl_scan(v, [](T x, T y) { return x + y; });
  if (lane == 63) sWave[wave] = v;
  __syncthreads();
  T base = (T)0;
  for (int w = 0; w < wave; ++w) base += sWave[w];
  __syncthreads();
  return v + base;
}

// The solve's scan and sum over its kSolveThreads threads (four wavefronts,
// mine; a wider workgroup's other wavefronts only pass the barrier), with the
// sums in the order of block_incl_scan.  Each call site passes
// four LDS words of its own, so one barrier per call suffices (nothing
// writes them again before the next solve).
template <class T>
__device__ __forceinline__ T solve_incl_scan(T v, T *slot4, bool mine) {
  const int wave = threadIdx.x >> 6;
  if (mine) {
    v = wave_incl_scan(v, [](T x, T y) { return x + y; });
    if ((threadIdx.x & 63) == 63) slot4[wave] = v;
  }
  __syncthreads();
  // wavefronts 0..wave-1 in order; the zeros added after them change no bits
  T base = (T)0;
  if (mine) {
#pragma unroll
    for (int w = 0; w < 3; ++w) base += (w < wave) ? slot4[w] : (T)0;
  }
  return v + base;
}
template <class T>
__device__ __forceinline__ T solve_sum(T v, T *slot4, bool mine) {
  if (mine) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) slot4[threadIdx.x >> 6] = v;
  }
  __syncthreads();
  return slot4[0] + slot4[1] + slot4[2] + slot4[3];
}

}  // namespace

// The solve of one slot: charge per cell from the P/D (and R) accumulators
// (cleared), mean removal, Gauss's law, cell-centre field, field energy; the
// diagnostics row and the step count.  The accumulators may be the slot's
// global mesh (k_solve) or a workgroup's LDS copy (k_resident, k_step).
// The slot's constants the solve needs, read once by its caller.
struct SlotConst {
  int nc;
  double L, dx, dt, q_unit;
  int64_t mesh_off, hist_off, hist_cap;
};

__device__ __forceinline__ SlotConst slot_const(const InstDesc &I) {
  SlotConst k;
  k.nc = I.n_cells;
  k.L = I.L;
  k.dx = I.dx;
  k.dt = I.dt;
  k.q_unit = I.q_unit;
  k.mesh_off = I.mesh_off;
  k.hist_off = I.hist_off;
  k.hist_cap = I.hist_cap;
  return k;
}

// The slot's point (P) and difference (D) accumulators of this thread's
// cells, summed over their REP copies (rep_stride words apart) in copy
// order and cleared: the first half of the solve, apart so that a caller can
// have these loads in flight with others.  The loads are unconditional (a
// thread past the mesh reads cell 0 and adds zero), so all of them are in
// flight together; the clearing stores follow.
template <int PREC, int CELLS, int REP, class Acc, class T>
__device__ __forceinline__ void solve_take(const SlotConst &kc, Acc *gP, Acc *gD, int64_t rep_stride,
                                           T (&pv)[CELLS], T (&dv)[CELLS]) {
  const int nc = kc.nc;
  const int per = (nc + kSolveThreads - 1) / kSolveThreads;
  const int j0 = threadIdx.x * per;
#pragma unroll
  for (int k = 0; k < CELLS; ++k) {
    pv[k] = (T)0;
    dv[k] = (T)0;
  }
#pragma unroll
  for (int r = 0; r < REP; ++r) {
#pragma unroll
    for (int k = 0; k < CELLS; ++k) {
      const int j = j0 + k;
      const bool own = k < per && j < nc;
      const int64_t at = r * rep_stride + (own ? j : 0);
      const T p = (T)gP[at];
      const T d = (T)gD[at];
      pv[k] += own ? p : (T)0;
      dv[k] += own ? d : (T)0;
    }
  }
#pragma unroll
  for (int r = 0; r < REP; ++r) {
#pragma unroll
    for (int k = 0; k < CELLS; ++k) {
      const int j = j0 + k;
      if (k < per && j < nc) {
        gP[r * rep_stride + j] = (Acc)0;
        gD[r * rep_stride + j] = (Acc)0;
      }
    }
  }
}

// Index of a cell in LDS when each solve thread takes up to 16 consecutive
// ones: a word of padding every 16 keeps the threads of a wavefront, 128 bytes
// apart, off one another's banks.
template <int CELLS>
__device__ __forceinline__ int padded_cell(int j) {
  return CELLS == 16 ? j + (j >> 4) : j;
}

// What the solve leaves for the diagnostics row: this thread's field energy
// sum (threads of the first kSolveThreads; not finite when one of its field
// values is not) and the total charge (every thread).
struct FieldSums {
  double w2, Qtot;
};

// The field of pv, dv (this thread's accumulators from solve_take) and the
// ramps, into sE (LDS, with one ghost cell on each side when ghost is set)
// and into gE and gR (field and density: global memory, or, PADDED, LDS by
// padded_cell) where they are given.  The cells are partitioned over kSolveThreads threads; a wider workgroup's other
// wavefronts only pass the barriers, so the bits are those of a workgroup of
// kSolveThreads.  The field in sE is complete after a barrier following the
// return.
template <int PREC, int CELLS, int REP = 1, bool PADDED = false, class Acc, class T>
__device__ __forceinline__ FieldSums solve_field(const SlotConst &kc, const T (&pv)[CELLS], const T (&dv)[CELLS],
                                                 Acc *gRamp, int64_t ramp_stride, double *sE, bool ghost, double *gE,
                                                 double *gR) {
  using acc_t = typename std::conditional<PREC == kFP64, double, long long>::type;
  static_assert(std::is_same<acc_t, T>::value, "accumulator type");
  // LDS words of the scans and sums, four per call site
  __shared__ acc_t sA[4][4];
  __shared__ double sF[2][4];
  __shared__ double sLastF[kSolveThreads];
  const int tid = threadIdx.x;
  const int nc = kc.nc;
  const double q_unit = kc.q_unit;
  const bool mine = __builtin_amdgcn_readfirstlane(tid >> 6) < kSolveThreads / kChunk;

  // 1. charge per cell: Q_j = P_j + sum_{m <= j} D_m
  const int per = (nc + kSolveThreads - 1) / kSolveThreads;
  const int j0 = tid * per;
  acc_t dsum = (acc_t)0;
#pragma unroll
  for (int k = 0; k < CELLS; ++k) dsum += dv[k];
  const acc_t dbase = solve_incl_scan(dsum, sA[0], mine) - dsum;
  // Linear ramps of piecewise-linear segments: the charge adds the second
  // prefix sum of R (zero for piecewise-constant segments).
  acc_t r2[CELLS];
#pragma unroll
  for (int k = 0; k < CELLS; ++k) r2[k] = (acc_t)0;
  if (gRamp != nullptr) {  // only piecewise-linear segments have ramps; REP copies as P and D
    acc_t rsum = (acc_t)0;
    if (mine) {
#pragma unroll
      for (int r = 0; r < REP; ++r) {
#pragma unroll
        for (int k = 0; k < CELLS; ++k) {
          const int j = j0 + k;
          const bool own = k < per && j < nc;
          const acc_t v = (acc_t)gRamp[r * ramp_stride + (own ? j : 0)];
          r2[k] += own ? v : (acc_t)0;
        }
      }
#pragma unroll
      for (int r = 0; r < REP; ++r) {
#pragma unroll
        for (int k = 0; k < CELLS; ++k) {
          const int j = j0 + k;
          if (k < per && j < nc) gRamp[r * ramp_stride + j] = (Acc)0;
        }
      }
#pragma unroll
      for (int k = 0; k < CELLS; ++k) rsum += r2[k];
    }
    const acc_t base1 = solve_incl_scan(rsum, sA[1], mine) - rsum;
    acc_t s1sum = (acc_t)0;
    if (mine) {
      acc_t run1 = base1;
#pragma unroll
      for (int k = 0; k < CELLS; ++k) {
        run1 += r2[k];
        r2[k] = run1;
        if ((k < per) && (j0 + k < nc)) s1sum += run1;
      }
    }
    const acc_t base2 = solve_incl_scan(s1sum, sA[2], mine) - s1sum;
    if (mine) {
      acc_t run2 = base2;
#pragma unroll
      for (int k = 0; k < CELLS; ++k) {
        if ((k < per) && (j0 + k < nc)) run2 += r2[k];
        r2[k] = run2;
      }
    }
  }
  double Q[CELLS];
  acc_t qsum_acc = (acc_t)0;
  if (mine) {
    acc_t run = dbase;
#pragma unroll
    for (int k = 0; k < CELLS; ++k) {
      run += dv[k];
      const acc_t qa = pv[k] + run + r2[k];
      const bool in = (k < per) && (j0 + k < nc);
      if constexpr (PREC == kFP64) Q[k] = in ? qa : 0.0;
      else Q[k] = in ? (double)qa * q_unit : 0.0;
      if (in) qsum_acc += qa;
    }
  }
  FieldSums out;
  if constexpr (PREC == kFP64) out.Qtot = solve_sum(qsum_acc, sA[3], mine);
  else out.Qtot = (double)solve_sum(qsum_acc, sA[3], mine) * q_unit;

  // 2. Gauss's law on faces: F_{j+1/2} = F_{j-1/2} + (Q_j - Qtot/nc),
  //    F shifted to zero mean; E_j = (F_{j-1/2} + F_{j+1/2}) / 2.
  double qmean = 0.0, rsum = 0.0;
  double F[CELLS];
  if (mine) {
    qmean = out.Qtot / (double)nc;
#pragma unroll
    for (int k = 0; k < CELLS; ++k) {
      const bool in = (k < per) && (j0 + k < nc);
      const double r = in ? (Q[k] - qmean) : 0.0;
      rsum += r;
      F[k] = r;
    }
  }
  const double fbase = solve_incl_scan(rsum, sF[0], mine) - rsum;
  // F's mean and each thread's last face value behind one barrier; the
  // neighbour's value is shifted by the mean after the exchange (the same
  // subtraction, the same bits)
  if (mine) {
    double fsum = 0.0, run = fbase, lastF = 0.0;
#pragma unroll
    for (int k = 0; k < CELLS; ++k) {
      const bool in = (k < per) && (j0 + k < nc);
      run += F[k];
      F[k] = in ? run : 0.0;
      if (in) {
        fsum += F[k];
        lastF = F[k];
      }
    }
    const double fw = wave_sum(fsum);
    if ((tid & 63) == 0) sF[1][tid >> 6] = fw;
    sLastF[tid] = lastF;
  }
  __syncthreads();
  out.w2 = 0.0;
  if (mine) {
    const double fmean = (sF[1][0] + sF[1][1] + sF[1][2] + sF[1][3]) / (double)nc;
#pragma unroll
    for (int k = 0; k < CELLS; ++k)
      if ((k < per) && (j0 + k < nc)) F[k] -= fmean;
    double prevF = (tid == 0) ? sLastF[(nc - 1) / per] - fmean : sLastF[tid - 1] - fmean;
#pragma unroll
    for (int k = 0; k < CELLS; ++k) {
      const int j = j0 + k;
      if ((k < per) && (j < nc)) {
        const double e = 0.5 * (prevF + F[k]);
        prevF = F[k];
        if (sE) {
          sE[j] = e;
          if (ghost) {
            if (j == 0) sE[nc] = e;
            if (j == nc - 1) sE[-1] = e;
          }
        }
        if (gE) {
          const int at = PADDED ? padded_cell<CELLS>(j) : j;
          gE[at] = e;
          gR[at] = (Q[k] - qmean) / kc.dx;
        }
        out.w2 += e * e;
      }
    }
  }
  return out;
}

// Field energy over the workgroup (one barrier; the same bits in every thread).
__device__ __forceinline__ double field_energy(const FieldSums &f, double dx) {
  __shared__ double sW[4];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (wave < kSolveThreads / kChunk) {
    const double w = wave_sum(f.w2);
    if ((threadIdx.x & 63) == 0) sW[wave] = w;
  }
  __syncthreads();
  return 0.5 * dx * (sW[0] + sW[1] + sW[2] + sW[3]);
}

// The sticky flags after a solve.
__device__ __forceinline__ int solve_flags(int solve, int flags0, double L, double W, double ke, double mom,
                                           double ms) {
  int f = 0;
  if (!(W - W == 0.0)) f |= 1;
  // a move with a non-finite velocity (its kinetic energy or momentum)
  if ((solve & kHavePush) && !((ke - ke == 0.0) && (mom - mom == 0.0))) f |= 1;
  if (solve & kHaveDeposit) {
    if (ms != ms) f |= 1;
    else if (ms > 0.45 * L) f |= 2;
  }
  return flags0 | f;
}

// a mod b of non-negative a, positive b: the 64-bit remainder (a long
// instruction sequence) only where the operands need it.
__device__ __forceinline__ int64_t row_of(int64_t a, int64_t b) {
  if ((uint64_t)(a | b) >> 32 == 0) return (int64_t)((uint32_t)a % (uint32_t)b);
  return a % b;
}

// The diagnostics row and the step bookkeeping, by one thread; step0 is the
// slot's step before this solve, flags those after it.
__device__ __forceinline__ void write_row(const SolveArgs &a, int slot, const SlotConst &kc, int64_t step0, int flags,
                                          double W, double Qtot, double ke, double mom, double ms) {
  InstDesc *Ip = a.inst + slot;
  const bool pushed = (a.flags & kHavePush) != 0;
  const int64_t step = pushed ? step0 + 1 : step0;
  Ip->flags = flags;
  DiagRow *H = a.hist + kc.hist_off;
  DiagRow r;
  r.step = step;
  r.t = (double)step * kc.dt;
  r.W_E = W;
  r.KE = __longlong_as_double(0x7ff8000000000000ll);
  r.momentum = r.KE;
  r.total_charge = Qtot;
  r.max_segment = (a.flags & kHaveDeposit) ? ms : r.KE;
  r.flags = flags;
  H[row_of(step, kc.hist_cap)] = r;
  if (pushed && step >= 1) {
    DiagRow *prev = H + row_of(step - 1, kc.hist_cap);
    prev->KE = ke;
    prev->momentum = mom;
  }
  Ip->step = step;
  if ((a.flags & kBatchStep) && pushed && Ip->steps_left > 0) {
    const int64_t left = Ip->steps_left - 1;
    Ip->steps_left = left;
    if (left == 0) {
      Ip->active = 0;
      a.done[slot] = 1;
    }
  }
}

// ---------------------------------------------------------------------------
// Tracer kernel
// ---------------------------------------------------------------------------
// Per-item LDS layout (bytes): P, D (and for linear segments R) accumulators
// and the field E for mesh_cells cells; for tile_cap chunks the item's chunk
// descriptors, the halo copy of the tracer after each chunk (constant
// segments: its state; linear segments: its position word, plus the
// geometry and density of the segment before the chunk and of the one after
// its last segment) and, with per-segment charges, the two charge edges; 48
// doubles for the block reduction.
// ORDER: 0 piecewise-constant segments, 1 piecewise-linear segments (ramp
// array R and three halo copies per chunk), 2 first-order weighting of
// constant segments.  SEG: per-segment charges (a charge word per tracer).
template <class Acc, int ORDER, bool SEG>
__host__ __device__ constexpr size_t tracer_lds_bytes(int mesh_cells, int tile_cap) {
  return (size_t)(2 + (ORDER == 1)) * mesh_cells * sizeof(Acc) + (size_t)(mesh_cells + 2) * sizeof(double) +
         (size_t)tile_cap *
             (sizeof(ChunkDesc) + (ORDER == 1 ? sizeof(uint64_t) + 2 * sizeof(LinNb) : sizeof(double2)) +
              (SEG ? 2 * sizeof(uint64_t) : 0)) +
         48 * sizeof(double);
}

// Charge word -> charge as float64 (split forms: fixed-point units times q_unit).
template <int PREC>
__device__ __forceinline__ double charge_value(uint64_t w, double q_unit) {
  if constexpr (PREC == kFP64) return __longlong_as_double((long long)w);
  else return (double)(long long)w * q_unit;
}

// Mass of a tracer bounded by segments of charge words `left` and `right`:
// half of each.
template <int PREC>
__device__ __forceinline__ double tracer_mass(uint64_t left, uint64_t right, double q_unit) {
  if constexpr (PREC == kFP64) {
    return 0.5 * (__longlong_as_double((long long)left) + __longlong_as_double((long long)right));
  } else {
    return 0.5 * ((double)((long long)left + (long long)right) * q_unit);
  }
}

// The LDS tables of a work item (layout above tracer_lds_bytes).
template <int PREC, int ORDER, bool SEG>
struct ItemLds {
  using acc_t = typename std::conditional<PREC == kFP64, double, unsigned long long>::type;
  acc_t *sP, *sD, *sR;   // sR: linear segments only
  double *sE;            // ghost cells at -1 and nc
  ChunkDesc *sDesc;
  double2 *sHalo;        // orders 0, 2: the tracer after the chunk
  uint64_t *sNextW;      // order 1: the word of the tracer after the chunk
  LinNb *sPrevNb;        // order 1: segment before the chunk
  LinNb *sNextNb;        // order 1: segment after its last one
  uint64_t *sEdge;       // per-segment charges
  double *sRed;          // 3 x 16 waves
  __device__ __forceinline__ ItemLds(unsigned char *smem, int mesh_cells, int tile_cap) {
    constexpr bool kLin = ORDER == 1;
    sP = reinterpret_cast<acc_t *>(smem);
    sD = sP + mesh_cells;
    sR = sD + mesh_cells;
    sE = reinterpret_cast<double *>(sR + (kLin ? mesh_cells : 0)) + 1;
    sDesc = reinterpret_cast<ChunkDesc *>(sE + mesh_cells + 1);
    sHalo = reinterpret_cast<double2 *>(sDesc + tile_cap);
    sNextW = reinterpret_cast<uint64_t *>(sDesc + tile_cap);
    sPrevNb = reinterpret_cast<LinNb *>(sNextW + tile_cap);
    sNextNb = sPrevNb + tile_cap;
    sEdge = kLin ? reinterpret_cast<uint64_t *>(sNextNb + tile_cap) : reinterpret_cast<uint64_t *>(sHalo + tile_cap);
    sRed = reinterpret_cast<double *>(sEdge + (SEG ? 2 * tile_cap : 0));
  }
};

// A halo tracer's word after this step's move (MODE with kPush) or as it is.
template <int PREC, int MODE>
__device__ __forceinline__ uint64_t moved_halo(double2 h, const Geo &g, const double *sE) {
  uint64_t w = (uint64_t)__double_as_longlong(h.x);
  if constexpr ((MODE & kPush) != 0) {
    const double e = gather_field_ghost(sE, mesh_pos<PREC>(w, g.inv_dx), g.nc);
    w = drift<PREC>(w, h.y + g.dt * e, g.dt, g.L, g.inv_dx, g.nc);
  }
  return w;
}

// The segments just outside a chunk, for the gradients of its first and last
// segments (order 1), and the word its last segment ends at: from the
// chunk's own first tracer (own), its partner's first (first; has_first), the
// tracer before it (prev; has_prev) and the one after the partner's first
// (next2; has_next), each moved here (the same functions as the lanes', so
// the same bits).  e0, e1: the charge words of the two segments; q their
// sheet's charge in the accumulator's units.
template <int PREC, int MODE, bool SEG>
__device__ __forceinline__ void stage_linear(const Geo &g, const double *sE, bool has_first, bool has_prev,
                                             bool has_next, double2 own, double2 first, double2 prev, double2 next2,
                                             uint64_t e0, uint64_t e1, double q, uint64_t *wn, LinNb *before,
                                             LinNb *after) {
  auto neighbour = [&](uint64_t wa, uint64_t wb, uint64_t cword) {
    const SegGeo sgn = lin_geo<PREC>(wa, wb, g);
    double qs = q;
    if constexpr (SEG) qs = PREC == kFP64 ? __longlong_as_double((long long)cword) : (double)(long long)cword;
    LinNb nb;
    nb.d = sgn.d;
    nb.r = lin_nb_density(sgn.d, lin_density(sgn, qs));
    return nb;
  };
  LinNb none;
  none.d = 0.0;
  none.r = lin_nb_density(0.0, 0.0);
  *before = none;
  *after = none;
  uint64_t wn1 = 0;
  if (has_first) wn1 = moved_halo<PREC, MODE>(first, g, sE);
  if (has_prev) {
    const uint64_t wpv = moved_halo<PREC, MODE>(prev, g, sE);
    *before = neighbour(wpv, moved_halo<PREC, MODE>(own, g, sE), e0);
  }
  if (has_first && has_next) *after = neighbour(wn1, moved_halo<PREC, MODE>(next2, g, sE), e1);
  *wn = wn1;
}

// Length of the segment between two state words as refinement measures it:
// float64 positions by the physical minimum image, split ones in mesh units.
template <int PREC>
__device__ __forceinline__ double mark_length(uint64_t wa, uint64_t wb, const Geo &g) {
  if constexpr (PREC == kFP64) {
    double d = __longlong_as_double((long long)wb) - __longlong_as_double((long long)wa);
    if (d >= g.half_L) d -= g.L;
    else if (d < -g.half_L) d += g.L;
    return fabs(d);
  } else {
    const double dm = mesh_pos<PREC>(wb, g.inv_dx) - mesh_pos<PREC>(wa, g.inv_dx);
    return fabs(min_image_cells(dm, 0.5 * (double)g.nc, (double)g.nc)) * g.dx;
  }
}

// A chunk's table entry: its descriptor, the charge word of the segment that
// ends at its first tracer (per-segment charges), the word of the tracer
// after it (moved when the step moves) and, for linear segments, the segments
// around it.
struct ChunkTab {
  ChunkDesc d;
  uint64_t edge, next;
  double next_u;  // split forms: the mesh position of next
  LinNb before, after;
};

// The tables of a wavefront's chunks in registers, one chunk per lane: no
// barrier between the wavefronts and no LDS round trip.
template <int PREC, int ORDER, bool SEG>
struct WaveTabs {
  ChunkDesc d;
  int2 lk;                 // order 1
  uint64_t e0, e1;         // per-segment charges
  uint64_t next;           // the moved tracers around the chunk (ChunkTab)
  double next_u;
  LinNb before, after;

  __device__ __forceinline__ void load(const ChunkDesc *chunks, const int2 *links, const uint64_t *cedge, size_t c) {
    d = chunks[c];
    if constexpr (ORDER == 1) lk = links[c];
    if constexpr (SEG) {
      e0 = cedge[2 * c];
      e1 = cedge[2 * c + 1];
    }
  }
  // The halo copies around chunk c, from halos of the chunks from base on.
  struct Halos {
    double2 own, first, prev, next2;  // orders 0, 2: first alone
  };
  __device__ __forceinline__ Halos halos(const double2 *h, size_t c, int base) const {
    Halos r;
    const size_t lc = c - base;
    const size_t pc = d.partner >= 0 ? (size_t)(d.partner - base) : lc;
    if constexpr (ORDER == 1) {
      auto at = [&](int l) { return l >= 0 ? 3 * (size_t)((l >> 2) - base) + (l & 3) : 3 * lc; };
      r.own = h[3 * lc + kHaloFirst];
      r.first = h[3 * pc + kHaloFirst];
      r.prev = h[at(lk.x)];
      r.next2 = h[at(lk.y)];
    } else {
      r.first = h[pc];
    }
    return r;
  }
  __device__ __forceinline__ void move(const Halos &h, const Geo &g, const double *sE) {
    if constexpr (ORDER == 1) {
      stage_linear<PREC, kPush | kDeposit, SEG>(g, sE, d.partner >= 0, lk.x >= 0, lk.y >= 0, h.own, h.first, h.prev,
                                                h.next2, e0, e1, PREC == kFP64 ? d.q : (double)d.q_fix, &next,
                                                &before, &after);
    } else {
      next = moved_halo<PREC, kPush | kDeposit>(h.first, g, sE);
    }
    if constexpr (PREC != kFP64) next_u = mesh_pos<PREC>(next, g.inv_dx);
  }
  // The entry of the wavefront's i-th chunk, from lane i.
  __device__ __forceinline__ ChunkTab entry(int i) const {
    auto f64 = [i](double x) {
      return __longlong_as_double((long long)read_lane64((uint64_t)__double_as_longlong(x), i));
    };
    ChunkTab t;
    t.d.q = f64(d.q);
    t.d.q_fix = PREC == kFP64 || SEG ? 0 : (int64_t)read_lane64((uint64_t)d.q_fix, i);
    t.d.partner = __builtin_amdgcn_readlane(d.partner, i);
    t.d.n_valid = __builtin_amdgcn_readlane(d.n_valid, i);
    t.d.flags = __builtin_amdgcn_readlane(d.flags, i);
    t.edge = SEG ? read_lane64(e0, i) : 0;
    t.next = read_lane64(next, i);  // not read where the form has no use for it
    t.next_u = PREC == kFP64 ? 0.0 : f64(next_u);
    if constexpr (ORDER == 1) {
      t.before.d = f64(before.d);
      t.before.r = f64(before.r);
      t.after.d = f64(after.d);
      t.after.r = f64(after.r);
    }
    return t;
  }
};

// One chunk of a work item: the move (or half kick) and the deposit of its
// segments.  halo_out: orders 0, 2 one copy per chunk, order 1 three.  STORE
// false: the moved state stays in xw and v.
template <int PREC, int MODE, int ORDER, bool SEG, bool STORE = true>
__device__ __forceinline__ void process_chunk(const ItemLds<PREC, ORDER, SEG> &t, const Geo &g, double q_unit,
                                              uint64_t *xs, double *vs, double2 *halo_out, const ChunkTab &tab,
                                              size_t chunk, int lane, uint64_t &xw, double &v, uint64_t cw, double &ke,
                                              double &mom, double &ms, const MarkArgs &mark = MarkArgs()) {
  constexpr bool kLin = ORDER == 1;
  constexpr bool kDep = (MODE & kDeposit) != 0;
  constexpr bool kKick = (MODE & kKickHalf) != 0;
  constexpr bool kField = (MODE & kPush) != 0 || kKick;
  constexpr bool kNeedQ = SEG && (kDep || (MODE & kPush) != 0);
  const ChunkDesc &ch = tab.d;
  const int n_valid = __builtin_amdgcn_readfirstlane(ch.n_valid);
  const bool valid = lane < n_valid;
  const size_t s = chunk * kChunk + lane;
  // Per-segment charges: this lane's segment (cw), the one ending at this
  // tracer (cl) and, for linear segments, the next one (cn).
  uint64_t cl = 0;
  if constexpr (kNeedQ) {
    const uint64_t up = lane_up1(cw);
    cl = lane == 0 ? tab.edge : up;
  }
  if constexpr (kField) {
    // The padding slots of a sheet's last chunk move with the others (they
    // start at rest at 0, and nothing reads them); they have no mass.
    const double e = gather_field_ghost(t.sE, mesh_pos<PREC>(xw, g.inv_dx), g.nc);
    if constexpr (kKick) {
      v = v - (0.5 * g.dt) * e;
      vs[s] = v;
    } else {
      const double vn = v + g.dt * e;
      double qv;
      if constexpr (SEG) {
        qv = tracer_mass<PREC>(cl, cw, q_unit);
      } else {
        // half of each segment the tracer bounds: the ends of an open
        // sheet bound one
        qv = ch.q;
        if (__builtin_amdgcn_readfirstlane((ch.flags & kChunkOpenStart) | (ch.partner & (int)0x80000000)) != 0) {
          const bool end = (lane == 0 && (ch.flags & kChunkOpenStart)) || (lane == n_valid - 1 && ch.partner < 0);
          qv = end ? 0.5 * ch.q : ch.q;
        }
      }
      if (n_valid < kChunk) qv = valid ? qv : 0.0;
      // twice the kinetic energy and momentum: the factor 1/2 is applied
      // to the item's sums (a power of two, so the same bits)
      ke += qv * v * vn;
      mom += qv * (v + vn);
      xw = drift<PREC>(xw, vn, g.dt, g.L, g.inv_dx, g.nc);
      v = vn;
      if constexpr (STORE) {
        __builtin_nontemporal_store(xw, xs + s);
        __builtin_nontemporal_store(v, vs + s);
      }
    }
    const double2 hv2 = make_double2(__longlong_as_double((long long)xw), v);
    if constexpr (kLin) {
      const size_t hb = 3 * chunk;
      if (lane == 0) halo_out[hb + kHaloFirst] = hv2;
      if (lane == 1) halo_out[hb + kHaloSecond] = hv2;
      if (lane == n_valid - 1) halo_out[hb + kHaloLast] = hv2;
    } else {
      if (lane == 0) halo_out[chunk] = hv2;
    }
  }
  // split forms: a lane's mesh position serves its own segment and the one
  // before it
  double ua = 0.0, ub = 0.0;
  if constexpr (kDep && PREC != kFP64) {
    ua = mesh_pos<PREC>(xw, g.inv_dx);
    ub = lane_down1(ua);
    if (lane == n_valid - 1) ub = tab.next_u;
  }
  if constexpr (kDep && kLin) {
    // Every lane computes its own segment's geometry and density; the
    // gradient takes the neighbouring segments' from the lanes next to
    // it (DPP moves), and the first and last lanes take the segments
    // outside the chunk from the staged neighbours.
    const bool last = lane == n_valid - 1;
    const uint64_t dn1 = lane_down1(xw);  // all lanes active: a DPP move reads its neighbour's register
    const uint64_t xp1 = last ? tab.next : dn1;
    const bool has_seg = valid && (!last || ch.partner >= 0);
    SegGeo sg;
    if constexpr (PREC == kFP64) sg = lin_geo<PREC>(xw, xp1, g);
    else sg = lin_geo_mesh(ua, ub, g);
    if (!has_seg) sg.d = 0.0;  // a neighbour without a segment drops the gradient
    double q0 = ch.q;
    long long q0_fix = ch.q_fix;
    if constexpr (SEG) {
      if constexpr (PREC == kFP64) q0 = __longlong_as_double((long long)cw);
      else q0_fix = (long long)cw;
    }
    const double r0 = lin_density(sg, PREC == kFP64 ? q0 : (double)q0_fix);
    const double rv = lin_nb_density(sg.d, r0);
    double dm = lane_up1(sg.d), rm = lane_up1(rv);
    double dp = lane_down1(sg.d), rp = lane_down1(rv);
    if (lane == 0) {
      dm = tab.before.d;
      rm = tab.before.r;
    }
    if (last) {
      dp = tab.after.d;
      rp = tab.after.r;
    }
    if (has_seg) {
      const double grad = lin_gradient(sg.d, dm, rm, dp, rp);
      const double len = fabs(sg.d) * g.dx;
      if (len <= g.half_L) {
        if constexpr (PREC == kFP64) {
          deposit_linear_fp64(__longlong_as_double((long long)xw), sg, grad, q0, r0, g, t.sP, t.sD, t.sR);
        } else {
          deposit_linear_split(split_cell<PREC>(xw), split_frac<PREC>(xw), sg, grad, q0_fix, r0, g, t.sP, t.sD, t.sR);
        }
      }
      ms = nan_max(ms, len);
    }
  }
  if constexpr (kDep && !kLin) {
    uint64_t pw = lane_down1(xw);
    const bool tail = (lane == n_valid - 1);
    bool has_seg = valid;
    if (tail) {
      if (ch.partner < 0) {
        has_seg = false;  // open sheet: the last tracer ends the chain
      } else {
        pw = tab.next;
      }
    }
    if (has_seg) {
      double len;
      double q0 = ch.q;
      long long q0_fix = ch.q_fix;
      if constexpr (SEG) {
        if constexpr (PREC == kFP64) q0 = __longlong_as_double((long long)cw);
        else q0_fix = (long long)cw;
      }
      if constexpr (ORDER == 2) {
        // first-order weighting: geometry in mesh units, minimum image as
        // for the constant scheme
        double dm;
        if constexpr (PREC == kFP64) {
          const double xa = __longlong_as_double((long long)xw);
          double d = __longlong_as_double((long long)pw) - xa;
          if (d >= g.half_L) d -= g.L;
          else if (d < -g.half_L) d += g.L;
          ua = xa * g.inv_dx;
          dm = d * g.inv_dx;
        } else {
          dm = min_image_cells(ub - ua, 0.5 * (double)g.nc, (double)g.nc);
        }
        len = fabs(dm) * g.dx;
        if (len <= g.half_L) {
          if constexpr (PREC == kFP64) deposit_cic_fp64(ua, dm, q0, g, t.sP, t.sD);
          else deposit_cic_split(ua, dm, q0_fix, g, t.sP, t.sD);
        }
      } else {
        if constexpr (PREC == kFP64) {
          len = deposit_fp64(__longlong_as_double((long long)xw), __longlong_as_double((long long)pw), q0, g,
                             t.sP, t.sD);
        } else {
          len = deposit_split<PREC>(xw, ua, ub, q0_fix, g, t.sP, t.sD);
        }
      }
      ms = nan_max(ms, len);
    }
  }
  if constexpr (SEG && MODE == (kPush | kDeposit)) {
    if (mark.cnt != nullptr) {
      // segments to split, by the length that the marking pass takes
      const uint64_t dn = lane_down1(xw);
      const bool tail = lane == n_valid - 1;
      const bool has = valid && !(tail && ch.partner < 0);
      const bool split = has && mark_length<PREC>(xw, tail ? tab.next : dn, g) > mark.l_max;
      const uint64_t lanes = __builtin_amdgcn_ballot_w64(split);
      if (lane == 0) {
        mark.cnt[chunk - mark.chunk_begin] = __builtin_popcountll(lanes);
        mark.mask[chunk - mark.chunk_begin] = lanes;
        // A plain store, the same from every chunk.  (A count would need an
        // atomic on one word, which the marked chunks then wait for in turn:
        // 1.04M tracers, 16000 chunks, took 60 us per step launch, 15 with
        // this; a flag per wavefront, stored once, cost 1 to 7 % of every
        // step with per-segment charges in scalar registers.)
        if (lanes) *mark.any = 1;
      }
    }
  }
}

// Work-item partial sums in a fixed order (deterministic for a fixed item
// decomposition); holds one barrier, after which the item's deposits are
// complete in LDS.  The last wavefront combines the wavefronts' sums: the
// first ones go on to the merge (a small mesh occupies only those).
template <int MODE>
__device__ __forceinline__ void item_partial(double ke, double mom, double ms, double *sRed, Partial *out) {
  constexpr bool kDep = (MODE & kDeposit) != 0;
  constexpr bool kMove = (MODE & kPush) != 0;
  const int lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if constexpr (kMove) {
    ke = wave_sum(ke);
    mom = wave_sum(mom);
  }
  if constexpr (kDep) ms = wave_max(ms);
  if (lane == 0) {
    sRed[wave] = ke;
    sRed[16 + wave] = mom;
    sRed[32 + wave] = ms;
  }
  __syncthreads();
  if (wave == nwaves - 1) {
    const bool in = lane < nwaves;
    const int l = lane & 15;
    if constexpr (kMove) {
      const double k = wave_sum(in ? sRed[l] : 0.0), m = wave_sum(in ? sRed[16 + l] : 0.0);
      if (lane == 0) {
        out->ke = 0.5 * k;
        out->mom = 0.5 * m;
      }
    }
    if constexpr (kDep) {
      const double x = wave_max(in ? sRed[32 + l] : 0.0);
      if (lane == 0) out->maxseg = x;
    }
  }
}

// Adds an item's LDS mesh to the global accumulators (gR: order 1 only), one
// atomic per touched cell.
template <int PREC, int ORDER, bool SEG, class Acc>
__device__ __forceinline__ void merge_mesh(const ItemLds<PREC, ORDER, SEG> &t, Acc *gP, Acc *gD, Acc *gR, int nc) {
  auto add = [](Acc *p, Acc v) {
    if (v != (Acc)0) {
      if constexpr (PREC == kFP64) unsafeAtomicAdd(p, v);
      else atomicAdd(p, v);
    }
  };
  for (int i = threadIdx.x; i < nc; i += blockDim.x) {
    const Acc p = t.sP[i];
    const Acc d = t.sD[i];
    add(gP + i, p);
    add(gD + i, d);
    if constexpr (ORDER == 1) add(gR + i, t.sR[i]);
  }
}

// The set of state arrays that holds a refining simulation's state.
template <class Args>
__device__ __forceinline__ void select_state(Args &a) {
  if (a.sel.state != nullptr && a.sel.state[kRefCur] != 0) {
    a.xs = a.sel.xs;
    a.vs = a.sel.vs;
    a.segq = a.sel.segq;
    a.chunks = a.sel.chunks;
  }
}

// Held to the registers of six wavefronts per SIMD (80), so that three
// workgroups of 512 threads share a compute unit; a few more leave room for
// two (first-order weighting, split U32, per-segment charges, 30.7M tracers at
// 82 registers 301 us, at 80 and 8 bytes of scratch 281; linear segments,
// split U32 272 and 249, FP64 with charges 141 and 133).  Linear segments with
// charges in the split forms take 93: at 80 they spill 64 bytes in the chunk
// loop (310 us, 395 at 80).
template <int PREC, int MODE, int ORDER, bool SEG>
__global__ void __launch_bounds__(1024)
    __attribute__((amdgpu_waves_per_eu(ORDER == 1 && SEG && PREC != kFP64 ? 5 : 6))) k_tracers(TracerArgs a) {
  using acc_t = typename std::conditional<PREC == kFP64, double, unsigned long long>::type;
  if constexpr (SEG) select_state(a);
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr bool kLin = ORDER == 1;
  const ItemLds<PREC, ORDER, SEG> t(smem, a.mesh_cells, a.tile_cap);

  if (a.gate != nullptr && *a.gate <= 0) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nwaves = blockDim.x >> 6;
  const int n_items = *a.n_items;
  constexpr bool kDep = (MODE & kDeposit) != 0;
  constexpr bool kMove = (MODE & kPush) != 0;
  constexpr bool kKick = (MODE & kKickHalf) != 0;
  constexpr bool kField = kMove || kKick;
  constexpr bool kNeedQ = SEG && (kDep || kMove);  // per-segment charges are read
  // chunks whose state is in flight per wavefront (a deposit alone reads 8
  // bytes per tracer and keeps more of them in flight)
  constexpr int kPrefetch = kField ? 3 : 6;

  for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
    const Item item = a.items[it];
    if (item.inst < 0) continue;  // freed slot
    const InstDesc &I = a.inst[item.inst];
    if (a.respect_active && !I.active) continue;
    Geo g;
    g.L = I.L;
    g.half_L = I.half_L;
    g.dx = I.dx;
    g.inv_dx = I.inv_dx;
    g.dt = I.dt;
    g.nc = I.n_cells;
    const int cb = item.chunk_begin;
    const int nch = item.chunk_end - item.chunk_begin;

    // Loads and stores are unconditional (a chunk always has 64 slots; the
    // padding slots of a sheet's last chunk move with the others, see
    // process_chunk), so the only branches around memory operations are uniform.
    // The state is streamed once per step: non-temporal loads and stores
    // keep it from displacing the meshes and tables in the caches.
    auto load_state = [&](int kk, uint64_t &xw, double &v, uint64_t &cw) {
      // past the item's last chunk every lane reads the item's first slot: the
      // loads are still issued, so the count of loads in flight is the same at
      // every stage and the wait before a stage leaves the later ones in flight
      const size_t s = kk < nch ? (size_t)(cb + kk) * kChunk + lane : (size_t)cb * kChunk;
      xw = __builtin_nontemporal_load(a.xs + s);
      if constexpr (kField) v = __builtin_nontemporal_load(a.vs + s);  // a deposit alone needs no velocity
      if constexpr (kNeedQ) cw = a.segq[s];
    };
    // kPrefetch chunks in flight per wavefront, in fixed registers (the
    // loop is fully unrolled over them).  The first ones are issued before
    // the item's tables are staged: they need only the item's chunk range,
    // so their latency overlaps the staging's.
    uint64_t xr[kPrefetch], cr_[kPrefetch];
    double vr[kPrefetch];
#pragma unroll
    for (int j = 0; j < kPrefetch; ++j) {
      xr[j] = cr_[j] = 0;
      vr[j] = 0.0;
      load_state(wave + j * nwaves, xr[j], vr[j], cr_[j]);
      // issue in stage order, as the loop does: the wait before a stage's
      // first use then leaves the later stages' loads in flight
      __builtin_amdgcn_sched_barrier(0);
    }
    // Stage the item's tables in LDS: one pass of global reads per item
    // instead of dependent reads per chunk.
    for (int i = tid; i < g.nc; i += blockDim.x) {
      if constexpr (kDep) {
        t.sP[i] = (acc_t)0;
        t.sD[i] = (acc_t)0;
        if constexpr (kLin) t.sR[i] = (acc_t)0;
      }
      if constexpr (kField) t.sE[i] = a.meshE[I.mesh_off + i];
    }
    if constexpr (kField) {
      if (tid == 0) {
        t.sE[-1] = a.meshE[I.mesh_off + g.nc - 1];
        t.sE[g.nc] = a.meshE[I.mesh_off];
      }
    }
    for (int i = tid; i < nch; i += blockDim.x) {
      t.sDesc[i] = a.chunks[cb + i];
      // the next chunk's halo, read with the descriptor: it is the partner
      // of every chunk but a sheet's last (checked below)
      if constexpr (kDep && !kLin) {
        if (i + 1 < nch) t.sHalo[i] = a.halo_in[cb + i + 1];
      }
      if constexpr (kNeedQ) {
        t.sEdge[2 * i] = a.cedge[2 * (size_t)(cb + i)];
        t.sEdge[2 * i + 1] = a.cedge[2 * (size_t)(cb + i) + 1];
      }
    }
    __syncthreads();
    if constexpr (kDep) {
      // The tracers around each chunk, moved here (once per chunk, one
      // thread) when this step moves, from their state before this step,
      // rather than by a whole wavefront for its last lane.
      for (int i = tid; i < nch; i += blockDim.x) {
        const int pc = t.sDesc[i].partner;
        if constexpr (kLin) {
          const int2 lk = a.links[cb + i];
          auto halo3 = [&](bool has, size_t at) { return has ? a.halo3_in[at] : make_double2(0.0, 0.0); };
          const bool hp = lk.x >= 0, hn = pc >= 0 && lk.y >= 0;
          const double2 own = halo3(hp, 3 * (size_t)(cb + i) + kHaloFirst);
          const double2 first = halo3(pc >= 0, 3 * (size_t)max(pc, 0) + kHaloFirst);
          const double2 prev = halo3(hp, 3 * (size_t)(lk.x >> 2) + (lk.x & 3));
          const double2 next2 = halo3(hn, 3 * (size_t)(lk.y >> 2) + (lk.y & 3));
          stage_linear<PREC, MODE, SEG>(g, t.sE, pc >= 0, hp, hn, own, first, prev, next2,
                                        SEG ? t.sEdge[2 * i] : 0ull, SEG ? t.sEdge[2 * i + 1] : 0ull,
                                        PREC == kFP64 ? t.sDesc[i].q : (double)t.sDesc[i].q_fix, t.sNextW + i,
                                        t.sPrevNb + i, t.sNextNb + i);
        } else if (pc >= 0) {
          double2 h = (pc == cb + i + 1 && i + 1 < nch) ? t.sHalo[i] : a.halo_in[pc];
          const uint64_t w = moved_halo<PREC, MODE>(h, g, t.sE);
          t.sHalo[i] = make_double2(__longlong_as_double((long long)w), mesh_pos<PREC>(w, g.inv_dx));
        }
      }
      __syncthreads();
    }

    // Chunk loop: wave w takes local chunks w, w + nwaves, ...  The loop is
    // unrolled three times with fixed registers per stage, so the state of
    // the next two chunks is in flight while the current one is processed
    // (moving a register whose load is pending would force a wait).
    double ke = 0.0, mom = 0.0, ms = 0.0;
    for (int k = wave; k < nch; k += kPrefetch * nwaves) {
#pragma unroll
      for (int j = 0; j < kPrefetch; ++j) {
        const int kk = k + j * nwaves;
        if (kk < nch) {
          ChunkTab tab;
          tab.d = t.sDesc[kk];
          if constexpr (kNeedQ) tab.edge = t.sEdge[2 * kk];
          if constexpr (kDep && kLin) {
            tab.next = t.sNextW[kk];
            if constexpr (PREC != kFP64) tab.next_u = mesh_pos<PREC>(tab.next, g.inv_dx);
            tab.before = t.sPrevNb[kk];
            tab.after = t.sNextNb[kk];
          } else if constexpr (kDep) {
            const double2 h = t.sHalo[kk];
            tab.next = (uint64_t)__double_as_longlong(h.x);
            tab.next_u = h.y;
          }
          process_chunk<PREC, MODE, ORDER, SEG>(t, g, I.q_unit, a.xs, a.vs, kLin ? a.halo3_out : a.halo_out, tab,
                                                (size_t)(cb + kk), lane, xr[j], vr[j], cr_[j], ke, mom, ms, a.mark);
        }
        load_state(k + (j + kPrefetch) * nwaves, xr[j], vr[j], cr_[j]);
      }
    }

    item_partial<MODE>(ke, mom, ms, t.sRed, a.partials + it);
    if constexpr (kDep) {
      const int64_t roff = I.mesh_off + (int64_t)(it % a.rep) * a.rep_stride;
      merge_mesh<PREC, ORDER, SEG>(t, reinterpret_cast<acc_t *>(a.meshP) + roff,
                                   reinterpret_cast<acc_t *>(a.meshD) + roff,
                                   kLin ? reinterpret_cast<acc_t *>(a.meshR) + roff : (acc_t *)nullptr, g.nc);
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Solve-first step of a single simulation
// ---------------------------------------------------------------------------
// One launch per step: every workgroup first solves the charge that the
// launch before merged (the same arithmetic in all of them, and in k_solve:
// the same bits), then moves and deposits its work item; workgroup 0 also
// writes the diagnostics row of that charge and the step.  Such a step is a
// chain of latencies, not of bytes or operations, so the chain is kept short:
// the simulation's constants and its item's chunk range come with the launch
// (no reads of the item list and the slot's descriptor, each a round trip
// that the next one waits for); the item's descriptors, halos and first
// chunks are in flight during the solve; and every wavefront keeps the tables
// of its own chunks in registers, one chunk per lane, with no barrier and no
// LDS round trip.  Workgroup 0's row: with fewer items than compute units it
// has no item (row_group) and the row holds up none; otherwise it would share
// its compute unit with an item and hold that up by more than the row takes
// at the end of its own (Landau, 256 items: 9.1 us per step with a row
// workgroup, 8.1 without; 20 sheets of 64 tracers, 5 items: 8.1 with, 9.5
// without).
//
// Per step, before (item list and descriptor read in turn, the row first, a
// 64-bit division for the slice to clear; orders 1 and 2 as launch pairs) and
// now: Landau (131072 tracers, 256 cells) 9.3 -> 8.0 us, with linear segments
// 13.7 -> 9.7, first-order weighting on ragged sheets (47000 tracers, 200
// cells, split U32) 11.1 -> 7.2, two-stream (2.1M tracers, 1024 cells, split
// F32) 26 -> 23.  Of the 8.0 us of Landau's, 1.6 are the launch, 1.2 the
// charge, 1.2 the solve, 1.7 moving and depositing one chunk per wavefront
// and 1.2 the merge.
//
// CELLS: cells per solve thread; 0: no solve, for simulations of more items
// than run in one round, whose charge a solve launch solves once.  Their
// workgroups, as many as run at a time, go through all chunks together: the
// wavefronts stream on their own, with no barrier, and the mesh is cleared,
// and merged, once per workgroup (33.5M tracers, 4096 cells: 256
// merges of 8192 additions instead of 2048, on compute units that hold one
// workgroup and had nothing to do meanwhile: 262 -> 216 us, 4.1 -> 5.0 TB/s of
// the state's bytes; a contiguous run for each workgroup instead of all going
// through memory together: 225).
template <int PREC, int ORDER, bool SEG, int CELLS>
__global__ void __launch_bounds__(1024) k_step(StepArgs a) {
  using acc_t = typename std::conditional<PREC == kFP64, double, unsigned long long>::type;
  using sacc_t = typename std::conditional<PREC == kFP64, double, long long>::type;
  constexpr int kMode = kPush | kDeposit;
  constexpr bool kLin = ORDER == 1;
  constexpr int kArrays = kLin ? 3 : 2;
  constexpr bool kSolve = CELLS > 0;
  const int kRep = kSolve ? single_rep(CELLS * kSolveThreads) : single_rep(a.nc);
  constexpr int kPrefetch = 3;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double sRow[5][4];  // workgroup 0: the row's sums by wavefront
  const ItemLds<PREC, ORDER, SEG> t(smem, a.nc, 0);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nt = blockDim.x;
  const int nwaves = nt >> 6;
  const bool row = kSolve && blockIdx.x == 0 && a.acc_in != nullptr;
  Geo g;
  g.L = a.L;
  g.half_L = a.half_L;
  g.dx = a.dx;
  g.inv_dx = a.inv_dx;
  g.dt = a.dt;
  g.nc = a.nc;
  const int nc = a.nc;
  const SlotConst kc = {nc, a.L, a.dx, a.dt, a.q_unit, 0, 0, a.hist_cap};

  // items now and of the launch before (whose partials these are), and of the
  // deposit after that one's refinement
  int n_chunks = a.n_chunks, tile = a.tile, n_items = a.n_items, n_prev = a.n_items, n_ref = 0;
  if constexpr (SEG) {
    if (a.sel.state != nullptr) {
      const int32_t *st = a.sel.state;
      if (st[kRefHalt] != 0) return;
      n_chunks = st[kRefChunks];
      tile = refine_tile(n_chunks, a.tile_fixed);
      n_items = refine_items(n_chunks, a.tile_fixed);
      n_prev = refine_items(st[kRefStepChunks], a.tile_fixed);
      n_ref = st[kRefInserted] > 0 ? n_items : 0;
      select_state(a);
    }
  }
  auto clear_slice = [&]() {
    acc_t *z = reinterpret_cast<acc_t *>(a.acc_zero);
    const int z1 = min(kArrays * kRep * nc, ((int)blockIdx.x + 1) * a.zero_slice);
    for (int i = (int)blockIdx.x * a.zero_slice + tid; i < z1; i += nt) z[i] = (acc_t)0;
  };
  const int it0 = a.row_group ? -1 : 0;  // workgroup 0's item; -1: it has none
  int it = (int)blockIdx.x + it0;
  if (it >= n_items) {  // refining: more workgroups than items so far
    if (a.acc_zero != nullptr) clear_slice();
    return;
  }
  // The wavefront's chunks: c0, c0 + stride, ... below cend.  An item's are
  // consecutive; without the solve the workgroups go through all chunks
  // together.
  const int stride = kSolve ? nwaves : nwaves * (int)gridDim.x;
  int c0 = 0, cend = 0;
  auto range = [&]() {  // a workgroup without an item loads the first one's
    if constexpr (kSolve) {
      const int i = max(it, 0), cb = a.chunk_begin + i * tile;
      c0 = cb + wave;
      cend = cb + min(tile, n_chunks - i * tile);
    } else {
      c0 = a.chunk_begin + (int)blockIdx.x * nwaves + wave;
      cend = a.chunk_begin + a.n_chunks;
    }
  };
  // Lane i holds the tables of the wavefront's i-th chunk from c0 on (an item
  // has at most 64 chunks per wavefront; without the solve, groups of 64).
  WaveTabs<PREC, ORDER, SEG> tabs;
  typename WaveTabs<PREC, ORDER, SEG>::Halos halos;
  auto lane_chunk = [&]() { return (size_t)min(c0 + lane * stride, cend - 1); };
  uint64_t xr[kPrefetch], cr_[kPrefetch];
  double vr[kPrefetch];
  auto load_state = [&](int c, uint64_t &xw, double &v, uint64_t &cw) {
    // past the end every lane reads the last chunk's first slot (k_tracers)
    const size_t s = c < cend ? (size_t)c * kChunk + lane : (size_t)(cend - 1) * kChunk;
    xw = __builtin_nontemporal_load(a.xs + s);
    v = __builtin_nontemporal_load(a.vs + s);
    if constexpr (SEG) cw = a.segq[s];
  };
  auto load_first_states = [&]() {
#pragma unroll
    for (int j = 0; j < kPrefetch; ++j) {
      xr[j] = cr_[j] = 0;
      load_state(c0 + j * stride, xr[j], vr[j], cr_[j]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  range();
  tabs.load(a.chunks, a.links, a.cedge, lane_chunk());
  __builtin_amdgcn_sched_barrier(0);
  FieldSums fs = {0.0, 0.0};
  Partial pr[2];  // the row: the launch before's partials tid and tid + 256
  int64_t step0 = 0;
  int flags0 = 0;
  bool solved = false;
  if constexpr (kSolve) {
    if (a.acc_in != nullptr) {
      solved = true;
      // The charge: cells tid, tid + threads, ... of every array, the copies
      // summed in copy order (as the solve launch sums them) and passed to the
      // solve's threads through the item's still unused LDS mesh (with padding,
      // and the field's room), so that the reads are coalesced and spread over
      // all wavefronts.
      const sacc_t *in = reinterpret_cast<const sacc_t *>(a.acc_in);
      sacc_t *sAcc = reinterpret_cast<sacc_t *>(t.sP);
      constexpr int kCopies = single_rep(CELLS * kSolveThreads);
      sacc_t av[kArrays][kCopies];
      auto load_acc = [&](int j) {
#pragma unroll
        for (int r = 0; r < kCopies; ++r)
#pragma unroll
          for (int k = 0; k < kArrays; ++k) av[k][r] = in[(int64_t)(k * kCopies + r) * nc + j];
      };
      auto sum_acc = [&](int j) {
#pragma unroll
        for (int k = 0; k < kArrays; ++k) {
          sacc_t sum = (sacc_t)0;
#pragma unroll
          for (int r = 0; r < kCopies; ++r) sum += av[k][r];
          sAcc[k * padded_cell<CELLS>(nc) + padded_cell<CELLS>(j)] = sum;
        }
      };
      load_acc(min(tid, nc - 1));
      __builtin_amdgcn_sched_barrier(0);
      halos = tabs.halos(a.halo_in, lane_chunk(), 0);
      load_first_states();
      if (row) {
        step0 = a.sf.inst[0].step;
        flags0 = a.sf.inst[0].flags;
        pr[0] = a.part_in[min(tid, n_prev - 1)];
        pr[1] = a.part_in[min(tid + kSolveThreads, n_prev - 1)];
      }
      if (tid < nc) sum_acc(tid);
      for (int j = tid + nt; j < nc; j += nt) {
        load_acc(j);
        sum_acc(j);
      }
      __syncthreads();
      sacc_t pv[CELLS], dv[CELLS];
      if (wave < kSolveThreads / kChunk) {
        const int per = (nc + kSolveThreads - 1) / kSolveThreads;
#pragma unroll
        for (int k = 0; k < CELLS; ++k) {
          const int j = tid * per + k;
          const bool in_mesh = k < per && j < nc;
          const int at = padded_cell<CELLS>(in_mesh ? j : 0);
          const sacc_t p = sAcc[at], d = sAcc[padded_cell<CELLS>(nc) + at];
          pv[k] = in_mesh ? p : (sacc_t)0;
          dv[k] = in_mesh ? d : (sacc_t)0;
        }
      }
      // the field and the density in global memory are written by the solve
      // launch that ends a run of such steps
      fs = solve_field<PREC, CELLS>(kc, pv, dv, kLin ? sAcc + 2 * (int64_t)nc : (sacc_t *)nullptr, 0, t.sE, true,
                                    (double *)nullptr, (double *)nullptr);
      // The accumulators that the launch before read are cleared, a slice per
      // workgroup (the next launch merges into them).
      clear_slice();
    }
  }
  if (!solved) {
    // the first step of a run (or no solve): the field is in global memory
    halos = tabs.halos(a.halo_in, lane_chunk(), 0);
    load_first_states();
    for (int j = tid; j < nc; j += nt) {
      const double e = a.meshE[j];
      t.sE[j] = e;
      if (j == 0) t.sE[nc] = e;
      if (j == nc - 1) t.sE[-1] = e;
    }
  }
  for (;;) {
    // the solve's threads read the charge from the LDS mesh before its first
    // barrier (linear segments' ramps: before its second, and clear them)
    for (int i = tid; i < nc; i += nt) {
      t.sP[i] = (acc_t)0;
      t.sD[i] = (acc_t)0;
      if constexpr (kLin) t.sR[i] = (acc_t)0;
    }
    __syncthreads();  // the field, the cleared mesh
    double ke = 0.0, mom = 0.0, ms = 0.0;
    if (it >= 0) {
      for (;;) {
        tabs.move(halos, g, t.sE);
        int i = 0;
        const int gend = kSolve ? cend : min(cend, c0 + kChunk * stride);
        for (int k = c0; k < gend; k += kPrefetch * stride) {
#pragma unroll
          for (int j = 0; j < kPrefetch; ++j) {
            const int c = k + j * stride;
            if (c < gend)
              process_chunk<PREC, kMode, ORDER, SEG>(t, g, a.q_unit, a.xs, a.vs, a.halo_out, tabs.entry(i++),
                                                     (size_t)c, lane, xr[j], vr[j], cr_[j], ke, mom, ms, a.mark);
            load_state(c + kPrefetch * stride, xr[j], vr[j], cr_[j]);
          }
        }
        if constexpr (kSolve) break;
        c0 += kChunk * stride;
        if (c0 >= cend) break;
        tabs.load(a.chunks, a.links, a.cedge, lane_chunk());
        halos = tabs.halos(a.halo_in, lane_chunk(), 0);
        load_first_states();
      }
    }
    const bool with_row = kSolve && row && it == it0;
    if (with_row && wave < kSolveThreads / kChunk) {
      // the row's wavefront sums, in the solve launch's order: thread tid
      // sums the items tid, tid + 256, ...
      double pke = 0.0, pmom = 0.0, pms = 0.0;
      auto add = [&](const Partial &p) {
        pke += p.ke;
        pmom += p.mom;
        pms = nan_max(pms, p.maxseg);
      };
      if (tid < n_prev) add(pr[0]);
      if (tid + kSolveThreads < n_prev) add(pr[1]);
      for (int i = tid + 2 * kSolveThreads; i < n_prev; i += kSolveThreads) add(a.part_in[i]);
      double pref = 0.0;
      for (int i = tid; i < n_ref; i += kSolveThreads) pref = nan_max(pref, a.part_ref[i].maxseg);
      const double w = wave_sum(fs.w2), k = wave_sum(pke), m = wave_sum(pmom), x = wave_max(pms), y = wave_max(pref);
      if (lane == 0) {
        sRow[0][wave] = w;
        sRow[1][wave] = k;
        sRow[2][wave] = m;
        sRow[3][wave] = x;
        sRow[4][wave] = y;
      }
    }
    if (it >= 0) item_partial<kMode>(ke, mom, ms, t.sRed, a.part_out + it);
    else __syncthreads();
    if (with_row && tid == nt - 1) {
      const double W = 0.5 * a.dx * (sRow[0][0] + sRow[0][1] + sRow[0][2] + sRow[0][3]);
      const double k = sRow[1][0] + sRow[1][1] + sRow[1][2] + sRow[1][3];
      const double m = sRow[2][0] + sRow[2][1] + sRow[2][2] + sRow[2][3];
      const double x = nan_max(nan_max(sRow[3][0], sRow[3][1]), nan_max(sRow[3][2], sRow[3][3]));
      int flags = solve_flags(a.sf.flags, flags0, a.L, W, k, m, x);
      double longest = x;
      if (n_ref > 0) {  // as k_solve: the row is the refined state's
        longest = nan_max(nan_max(sRow[4][0], sRow[4][1]), nan_max(sRow[4][2], sRow[4][3]));
        flags = solve_flags(a.sf.flags, flags, a.L, W, k, m, longest);
      }
      write_row(a.sf, 0, kc, step0, flags, W, fs.Qtot, k, m, longest);
    }
    if (it < 0) return;
    acc_t *out = reinterpret_cast<acc_t *>(a.acc_out) + (int64_t)(it % kRep) * nc;
    const int64_t arr = (int64_t)kRep * nc;
    merge_mesh<PREC, ORDER, SEG>(t, out, out + arr, out + 2 * arr, nc);
    it += (int)gridDim.x + it0;
    if (it >= n_items) break;
    range();
    tabs.load(a.chunks, a.links, a.cedge, lane_chunk());
    halos = tabs.halos(a.halo_in, lane_chunk(), 0);
    load_first_states();
    __syncthreads();
  }
}

size_t tracer_lds_size(int prec, int order, bool seg, int mesh_cells, int tile_cap) {
  // the accumulators are 8 bytes in every precision
  if (order == 1)
    return seg ? tracer_lds_bytes<double, 1, true>(mesh_cells, tile_cap)
               : tracer_lds_bytes<double, 1, false>(mesh_cells, tile_cap);
  return seg ? tracer_lds_bytes<double, 0, true>(mesh_cells, tile_cap)
             : tracer_lds_bytes<double, 0, false>(mesh_cells, tile_cap);
}

// ---------------------------------------------------------------------------
// Deposit-only kernel (constant segments, face-crossing form)
// ---------------------------------------------------------------------------
// A deposit that does not also move the tracers reads 8 bytes per tracer, so
// its pace is set by the arithmetic per tracer, not by HBM.  On a sheet with
// several tracers per cell most segments cross no cell face: all they need is
// their length (the max-segment diagnostic) and their charge, which the
// chunk's running sum carries to the next crossing.  So the wavefront does
// only that per tracer, and appends every segment whose two ends lie in
// different cells to a per-wavefront ring in LDS; the face geometry of the
// queued segments (a division each) runs 64 at a time, with every lane busy.
// The sum over crossings and chunk ends is the same as in the per-chunk form
// above, term by term.

constexpr int kDepQueue = 64;      // ring entries per wavefront (drained before it would overflow)
constexpr int kDepPrefetch = 6;    // chunks in flight per wavefront

// The word and cell (plus one) of the tracer after a chunk.
struct alignas(16) DepHalo {
  uint64_t w;
  int32_t c;
  int32_t pad;
};

__host__ __device__ constexpr size_t dep_lds_offset_queue(int mesh_cells, int tile_cap) {
  // P, D; descriptors; halos
  return (size_t)2 * mesh_cells * 8 + (size_t)tile_cap * (sizeof(ChunkDesc) + sizeof(DepHalo));
}

// The ring of one wavefront is three arrays (kept apart so that the lanes of
// one queue write or read touch consecutive LDS words): the segment's two
// state words; the cells of its ends (plus one, 16 bits each) and its local
// chunk and lane; with per-segment charges, the chunk's charge before it and
// its own.  24 (40) bytes per entry: a 512-thread workgroup of a 1024-cell
// mesh and 256 chunks per item takes 40 KB, four workgroups per CU.  At the
// end of an item each wavefront's ring holds its segment-length maximum.
template <bool SEG>
__host__ __device__ constexpr size_t dep_lds_bytes(int mesh_cells, int tile_cap, int nwaves) {
  return dep_lds_offset_queue(mesh_cells, tile_cap) + (size_t)nwaves * kDepQueue * (16 + 8 + (SEG ? 16 : 0));
}

// Length of the segment between two state words (minimum image), in the same
// rounding as the per-segment deposit.
template <int PREC>
__device__ __forceinline__ double seg_length(uint64_t wa, uint64_t wb, const Geo &g) {
  // min(|d|, period - |d|) is |d| up to half a period and the other image
  // beyond, and propagates NaN
  if constexpr (PREC == kFP64) {
    const double ad = fabs(__longlong_as_double((long long)wb) - __longlong_as_double((long long)wa));
    return fmin(ad, g.L - ad);
  } else {
    const double nc = (double)g.nc;
    const double ad = fabs(mesh_pos<PREC>(wb, g.inv_dx) - mesh_pos<PREC>(wa, g.inv_dx));
    return fmin(ad, nc - ad) * g.dx;
  }
}

// ceil(x / dx), the raw cell of a tracer plus one (0 .. nc).  x * inv_dx
// is within 2^-50 relative of the rounded quotient, and |u| <= nc, so when
// u's distance to a whole number exceeds tol = (nc + 1) 2^-49 both have the
// same ceiling; otherwise the division decides.
template <int PREC>
__device__ __forceinline__ int point_cell_up(uint64_t w, const Geo &g, double tol, double tol_hi) {
  if constexpr (PREC == kFP64) {
    const double x = __longlong_as_double((long long)w);
    const double u = x * g.inv_dx;
    const double c = ceil(u);
    const double r = c - u;
    if (r > tol && r < tol_hi) return (int)c;
    return (int)ceil(x / g.dx);
  } else {
    return split_frac<PREC>(w) == 0.0 ? split_cell<PREC>(w) : split_cell<PREC>(w) + 1;
  }
}

// Without per-segment charges the kernel is held to 64 VGPRs, so that the
// eight wavefronts of each of four workgroups per CU all fit.
template <int PREC, bool SEG>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(SEG ? 4 : 8)))
k_deposit_faces(TracerArgs a) {
  using acc_t = typename std::conditional<PREC == kFP64, double, unsigned long long>::type;
  extern __shared__ __align__(16) unsigned char smem[];
  if (a.gate != nullptr && *a.gate <= 0) return;
  if constexpr (SEG) select_state(a);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nwaves = blockDim.x >> 6;
  acc_t *sP = reinterpret_cast<acc_t *>(smem);
  acc_t *sD = sP + a.mesh_cells;
  ChunkDesc *sDesc = reinterpret_cast<ChunkDesc *>(sD + a.mesh_cells);
  DepHalo *sHalo = reinterpret_cast<DepHalo *>(sDesc + a.tile_cap);
  ulonglong2 *const qBase = reinterpret_cast<ulonglong2 *>(smem + dep_lds_offset_queue(a.mesh_cells, a.tile_cap));
  ulonglong2 *qW = qBase;
  int2 *qC = reinterpret_cast<int2 *>(qW + nwaves * kDepQueue) + wave * kDepQueue;
  ulonglong2 *qS = reinterpret_cast<ulonglong2 *>(qC + (nwaves - wave) * kDepQueue) + wave * kDepQueue;  // SEG
  qW += wave * kDepQueue;
  const int n_items = *a.n_items;

  // run > 1: a run of consecutive items of one simulation, whose mesh is
  // cleared before the first and merged after the last
  const int it_end = a.run > 1 ? min(n_items, ((int)blockIdx.x + 1) * a.run) : n_items;
  const int it_first = (int)blockIdx.x * a.run, it_step = a.run > 1 ? 1 : gridDim.x;
  for (int it = it_first; it < it_end; it += it_step) {
    const Item item = a.items[it];
    if (item.inst < 0) continue;  // freed slot
    const InstDesc &I = a.inst[item.inst];
    if (a.respect_active && !I.active) continue;
    Geo g;
    g.L = I.L;
    g.half_L = I.half_L;
    g.dx = I.dx;
    g.inv_dx = I.inv_dx;
    g.dt = I.dt;
    g.nc = I.n_cells;
    const int cb = item.chunk_begin;
    const int nch = item.chunk_end - item.chunk_begin;

    if (a.run == 1 || it == it_first) {
      for (int i = tid; i < g.nc; i += blockDim.x) {
        sP[i] = (acc_t)0;
        sD[i] = (acc_t)0;
      }
    }
    // descriptors, and the word and cell of the tracer after each chunk
    for (int i = tid; i < nch; i += blockDim.x) {
      sDesc[i] = a.chunks[cb + i];
      const int pc = a.chunks[cb + i].partner;
      if (pc >= 0) {
        const uint64_t w = (uint64_t)__double_as_longlong(a.halo_in[pc].x);
        sHalo[i].w = w;
        sHalo[i].c = point_cell_up<PREC>(w, g, (double)(g.nc + 1) * 0x1p-49, 1.0 - (double)(g.nc + 1) * 0x1p-49);
      }
    }
    __syncthreads();

    double ms = 0.0;
    bool bad = false;             // a non-finite segment length (reported as NaN)
    int q_head = 0, q_count = 0;  // the wavefront's ring (uniform)

    // The n <= 64 oldest queued segments, one per lane: the faces each
    // crosses, and for the last segment of a chunk the chunk's charge where
    // it ends.
    auto drain = [&](int n) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if (lane < n) {
        const int e = (q_head + lane) & (kDepQueue - 1);
        const ulonglong2 w = qW[e];
        const int2 c = qC[e];
        const int pa = (c.x & 0xffff) - 1;
        const int pb = ((c.x >> 16) & 0xffff) - 1;
        const ChunkDesc &d = sDesc[(c.y >> 6) & 0x3fff];
        const int ln = c.y & 63;
        // the chunk's last segment: its last lane, or the one before for an
        // open sheet's end
        const bool end = ln == (d.partner < 0 ? d.n_valid - 2 : d.n_valid - 1);
        acc_t S, ql;
        if constexpr (SEG) {
          const ulonglong2 sq = qS[e];
          if constexpr (PREC == kFP64) {
            S = __longlong_as_double((long long)sq.x);
            ql = __longlong_as_double((long long)sq.y);
          } else {
            S = sq.x;
            ql = sq.y;
          }
        } else {
          ql = PREC == kFP64 ? (acc_t)d.q : (acc_t)d.q_fix;
          S = ql * (acc_t)ln;
        }
        acc_t eb = (acc_t)0;  // added to the cell where the segment ends
        bool add_b = end;
        if (pa != pb) {
          double len;
          const Crossings<acc_t> cr = face_crossings<PREC, acc_t>(w.x, w.y, pa, pb, ql, S, g, &len);
          if (cr.hi >= cr.lo) {
            lds_add(sP + wrap_cell(pa, g.nc), cr.cf);
            if (cr.hi > cr.lo) add_run(sD, cr.lo, cr.hi - 1, cr.w, g.nc);
            eb = (acc_t)(0 - cr.cl);
            add_b = true;
          }
        }
        if (end) eb += S + ql;
        if (add_b) lds_add(sP + wrap_cell(pb, g.nc), eb);
      }
      q_head = (q_head + n) & (kDepQueue - 1);
      q_count -= n;
      // the entries just read are written again by the next appends
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };

    auto load_state = [&](int kk, uint64_t &xw, uint64_t &cw) {
      const size_t s = kk < nch ? (size_t)(cb + kk) * kChunk + lane : (size_t)cb * kChunk;  // as in k_tracers
      xw = __builtin_nontemporal_load(a.xs + s);
      if constexpr (SEG) cw = a.segq[s];
    };
    const double tol = (double)(g.nc + 1) * 0x1p-49, tol_hi = 1.0 - tol;
    auto process = [&](int kk, uint64_t xw, uint64_t cw) {
      const int n_valid = __builtin_amdgcn_readfirstlane(sDesc[kk].n_valid);
      const bool open_end = __builtin_amdgcn_readfirstlane(sDesc[kk].partner) < 0;
      const int last = open_end ? n_valid - 2 : n_valid - 1;  // lane of the chunk's last segment
      const bool has_seg = lane <= last;
      // the segment's far end: the next lane, or past the chunk the partner's
      // first tracer
      uint64_t xb = lane_down1(xw);
      const int ca = point_cell_up<PREC>(xw, g, tol, tol_hi);
      int cb1 = lane_down1(ca);
      if (!open_end) {
        const bool tail = lane == n_valid - 1;
        const DepHalo h = sHalo[kk];
        xb = tail ? h.w : xb;
        cb1 = tail ? h.c : cb1;
      }
      if (has_seg) {
        const double len = seg_length<PREC>(xw, xb, g);
        ms = fmax(ms, len);
        bad = bad || len != len;
      }
      // queue the segments whose ends lie in different cells, and the
      // chunk's last segment
      const bool rec = has_seg && (ca != cb1 || lane == last);
      acc_t S = (acc_t)0, ql = (acc_t)0;
      if constexpr (SEG) {
        if (has_seg) ql = PREC == kFP64 ? (acc_t)__longlong_as_double((long long)cw) : (acc_t)cw;
        S = wave_exclusive_sum(ql);
      }
      const uint64_t mask = __builtin_amdgcn_ballot_w64(rec);
      if (mask) {
        const int n_new = __builtin_popcountll(mask);
        if (q_count + n_new > kDepQueue) drain(q_count);
        if (rec) {
          const int rank =
              __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
          const int e = (q_head + q_count + rank) & (kDepQueue - 1);
          qW[e] = make_ulonglong2(xw, xb);
          qC[e] = make_int2(ca | (cb1 << 16), (kk << 6) | lane);
          if constexpr (SEG) {
            if constexpr (PREC == kFP64) {
              qS[e] = make_ulonglong2((uint64_t)__double_as_longlong(S), (uint64_t)__double_as_longlong(ql));
            } else {
              qS[e] = make_ulonglong2((uint64_t)S, (uint64_t)ql);
            }
          }
        }
        q_count += n_new;
      }
    };

    uint64_t xr[kDepPrefetch], cr_[kDepPrefetch];
#pragma unroll
    for (int j = 0; j < kDepPrefetch; ++j) {
      xr[j] = cr_[j] = 0;
      load_state(wave + j * nwaves, xr[j], cr_[j]);
      __builtin_amdgcn_sched_barrier(0);  // stage order, as in the loop
    }
    for (int k = wave; k < nch; k += kDepPrefetch * nwaves) {
#pragma unroll
      for (int j = 0; j < kDepPrefetch; ++j) {
        if (k + j * nwaves < nch) process(k + j * nwaves, xr[j], cr_[j]);
        load_state(k + (j + kDepPrefetch) * nwaves, xr[j], cr_[j]);
      }
    }
    if (q_count > 0) drain(q_count);

    if (bad) ms = __longlong_as_double(0x7ff8000000000000ll);
    ms = wave_max(ms);
    if (lane == 0) reinterpret_cast<double *>(qW)[0] = ms;  // the ring is empty now
    __syncthreads();
    if (tid == 0) {
      double x = 0.0;
      for (int w = 0; w < nwaves; ++w) x = nan_max(x, reinterpret_cast<const double *>(qBase + w * kDepQueue)[0]);
      a.partials[it].maxseg = x;
    }
    if (a.run == 1 || it + 1 == it_end) {
      const int64_t roff = I.mesh_off + (int64_t)((a.run > 1 ? (int)blockIdx.x : it) % a.rep) * a.rep_stride;
      acc_t *gP = reinterpret_cast<acc_t *>(a.meshP) + roff;
      acc_t *gD = reinterpret_cast<acc_t *>(a.meshD) + roff;
      for (int i = tid; i < g.nc; i += blockDim.x) {
        const acc_t p = sP[i];
        const acc_t d = sD[i];
        if (p != (acc_t)0) {
          if constexpr (PREC == kFP64) unsafeAtomicAdd(gP + i, p);
          else atomicAdd(gP + i, p);
        }
        if (d != (acc_t)0) {
          if constexpr (PREC == kFP64) unsafeAtomicAdd(gD + i, d);
          else atomicAdd(gD + i, d);
        }
      }
    }
    __syncthreads();
  }
}

// An accumulator summed over its copies, in copy order, into LDS, and cleared;
// consecutive threads take consecutive cells, all copies of 16 rows of them in
// flight together.
template <class T, int REP>
__device__ __forceinline__ void take_lds(T *g, int nc, int64_t rep_stride, T *out) {
  constexpr int kU = 16;
  for (int j0 = threadIdx.x; j0 < nc; j0 += kU * kSolveThreads) {
    T v[kU][REP];
#pragma unroll
    for (int u = 0; u < kU; ++u)
#pragma unroll
      for (int r = 0; r < REP; ++r) v[u][r] = g[r * rep_stride + min(j0 + u * kSolveThreads, nc - 1)];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int j = j0 + u * kSolveThreads;
      if (j < nc) {
        T sum = (T)0;
#pragma unroll
        for (int r = 0; r < REP; ++r) {
          sum += v[u][r];
          g[r * rep_stride + j] = (T)0;
        }
        out[padded_cell<16>(j)] = sum;
      }
    }
  }
}

// CELLS: cells per thread the solve is unrolled for (at least the pool's
// largest mesh over kSolveThreads; the unused ones add exact zeros, so every
// instance gives the same bits).
template <int PREC, int CELLS, int REP>
__global__ void __launch_bounds__(kSolveThreads) k_solve(SolveArgs a) {
  using acc_t = typename std::conditional<PREC == kFP64, double, long long>::type;
  __shared__ double sWd[4];
  if (a.gate != nullptr && *a.gate <= 0) return;
  const int slot = a.slot_list ? a.slot_list[blockIdx.x] : (int)blockIdx.x;
  InstDesc *Ip = a.inst + slot;
  if (!Ip->live) return;
  if (a.respect_active && !Ip->active) return;
  const int tid = threadIdx.x;
  const int2 si = a.slot_items[slot];
  const int item_begin = si.x, item_count = a.n_partials >= 0 ? a.n_partials : si.y;
  const SlotConst kc = slot_const(*Ip);
  acc_t *gP = reinterpret_cast<acc_t *>(a.meshP) + kc.mesh_off;
  acc_t *gD = reinterpret_cast<acc_t *>(a.meshD) + kc.mesh_off;
  acc_t pv[CELLS], dv[CELLS];
  // With 16 cells per thread (128 bytes apart from thread to thread) the
  // accumulators, the field and the density go through LDS, so that global
  // memory is read and written in whole lines (4096 cells, two copies: 26 ->
  // 14 us).
  constexpr bool kLds = CELLS == 16;
  extern __shared__ __align__(16) unsigned char smem[];
  acc_t *sAcc = reinterpret_cast<acc_t *>(smem);
  if constexpr (kLds) {
    take_lds<acc_t, REP>(gP, kc.nc, a.rep_stride, sAcc);
    take_lds<acc_t, REP>(gD, kc.nc, a.rep_stride, sAcc + padded_cell<CELLS>(kc.nc));
  } else {
    solve_take<PREC, CELLS, REP>(kc, gP, gD, a.rep_stride, pv, dv);  // in flight with the partial loads below
  }

  // 1. work-item partials, in item order: each thread sums items tid,
  // tid + 256, ... (loads issued kU at a time), then the wavefront and
  // workgroup sums, all three in one pass
  __shared__ double sMom[4], sMs[4];
  // single simulations (copies) hold thousands of items, a batch's a few each
  constexpr int kU = REP > 1 ? 8 : 4;
  double ke = 0.0, mom = 0.0, ms = 0.0;
  for (int i0 = tid; i0 < item_count; i0 += kU * kSolveThreads) {
    Partial pr[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int i = i0 + u * kSolveThreads;
      if (i < item_count) pr[u] = a.partials[item_begin + i];
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      if (i0 + u * kSolveThreads < item_count) {
        ke += pr[u].ke;
        mom += pr[u].mom;
        ms = nan_max(ms, pr[u].maxseg);
      }
    }
  }
  ke = wave_sum(ke);
  mom = wave_sum(mom);
  ms = wave_max(ms);
  const int wave = tid >> 6;
  if ((tid & 63) == 0) {
    sWd[wave] = ke;
    sMom[wave] = mom;
    sMs[wave] = ms;
  }
  __syncthreads();
  ke = sWd[0] + sWd[1] + sWd[2] + sWd[3];
  mom = sMom[0] + sMom[1] + sMom[2] + sMom[3];
  ms = nan_max(nan_max(sMs[0], sMs[1]), nan_max(sMs[2], sMs[3]));
  acc_t *gRamp = (a.order == 1 && a.meshR) ? reinterpret_cast<acc_t *>(a.meshR) + kc.mesh_off : nullptr;
  FieldSums f;
  if constexpr (kLds) {
    const int per = (kc.nc + kSolveThreads - 1) / kSolveThreads;
#pragma unroll
    for (int k = 0; k < CELLS; ++k) {
      const int j = tid * per + k;
      const bool in = k < per && j < kc.nc;
      const int at = padded_cell<CELLS>(in ? j : 0);
      const acc_t pj = sAcc[at], dj = sAcc[padded_cell<CELLS>(kc.nc) + at];
      pv[k] = in ? pj : (acc_t)0;
      dv[k] = in ? dj : (acc_t)0;
    }
    // the field over the cells' P, the density over their D (the same thread's)
    double *sE = reinterpret_cast<double *>(smem), *sRho = sE + padded_cell<CELLS>(kc.nc);
    __syncthreads();
    f = solve_field<PREC, CELLS, REP, true>(kc, pv, dv, gRamp, a.rep_stride, (double *)nullptr, false, sE, sRho);
    __syncthreads();
    double *gE = a.meshE + kc.mesh_off, *gR = a.meshRho + kc.mesh_off;
    for (int j = tid; j < kc.nc; j += kSolveThreads) {
      gE[j] = sE[padded_cell<CELLS>(j)];
      gR[j] = sRho[padded_cell<CELLS>(j)];
    }
  } else {
    f = solve_field<PREC, CELLS, REP>(kc, pv, dv, gRamp, a.rep_stride, (double *)nullptr, false,
                                      a.meshE + kc.mesh_off, a.meshRho + kc.mesh_off);
  }
  const double W = field_energy(f, kc.dx);
  int flags = Ip->flags;
  if (a.refined != nullptr) {
    // the row is the refined state's; the flags are also those of the state
    // before its refinement
    flags = solve_flags(a.flags, flags, kc.L, W, ke, mom, ms);
    ms = 0.0;
    for (int i = tid; i < a.n_refined; i += kSolveThreads) ms = nan_max(ms, a.refined[i].maxseg);
    ms = wave_max(ms);
    if ((tid & 63) == 0) sMs[wave] = ms;
    __syncthreads();
    ms = nan_max(nan_max(sMs[0], sMs[1]), nan_max(sMs[2], sMs[3]));
  }
  if (tid == 0)
    write_row(a, slot, kc, Ip->step, solve_flags(a.flags, flags, kc.L, W, ke, mom, ms), W, f.Qtot, ke, mom, ms);
  acc_t *z = reinterpret_cast<acc_t *>(a.zero);
  for (int64_t i = tid; i < a.zero_words; i += kSolveThreads) z[i] = (acc_t)0;
}

// ---------------------------------------------------------------------------
// Resident small simulation
// ---------------------------------------------------------------------------
// A simulation of at most kResidentChunks chunks runs many steps in one
// launch of one workgroup: its tracers stay in registers (wavefront w of NW
// owns chunks w, w + NW, ...), the mesh accumulators, the field and the
// chunks' halos in LDS.  The arithmetic is that of the fused step (same move,
// same segment deposit, same solve code), so only the order of the
// floating-point sums of the deposit and of the kinetic-energy and momentum
// diagnostics can differ; the split forms give the same bits.  Such a
// simulation is bound by the latency of one step's chain of dependent
// operations and barriers, so what is not part of the chain is taken out of
// it: the move and the deposit are one pass (every wavefront moves the
// tracers that follow its chunks itself, from the halos of the step before,
// instead of waiting for the others' moves), and one wavefront more holds no
// tracers and reduces and writes the diagnostics rows while the others go on
// with the next step.  Per step (before: two passes, rows in the chain,
// constant segments only): 1024 tracers on 128 cells 4.8 -> 3.0 us, of which
// 1.3 the solve; 1280 tracers, linear segments, 12.2 (launch pairs) -> 5.7.

constexpr int kResidentChunks = 32;  // chunks (2048 tracer slots) a resident launch holds

// The LDS mesh, field and sums (ItemLds), then two sets of halo copies.
template <int ORDER>
__host__ __device__ constexpr size_t resident_halo_offset(int n_cells) {
  return (tracer_lds_bytes<double, ORDER, false>(n_cells, 0) + 15) & ~(size_t)15;
}
template <int ORDER>
__host__ __device__ constexpr size_t resident_lds_bytes(int n_cells) {
  return resident_halo_offset<ORDER>(n_cells) + (size_t)2 * kResidentChunks * (ORDER == 1 ? 3 : 1) * sizeof(double2);
}

// A workgroup barrier that orders LDS only: global stores in flight (the
// diagnostics rows) are not waited for.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int PREC, int ORDER, bool SEG, int CELLS, int NW>
__global__ void __launch_bounds__((NW + 1) * kChunk) k_resident(TracerArgs a, SolveArgs sa, int chunk_begin,
                                                               int n_chunks, int64_t n_steps) {
  using acc_t = typename std::conditional<PREC == kFP64, double, unsigned long long>::type;
  using sacc_t = typename std::conditional<PREC == kFP64, double, long long>::type;
  constexpr bool kLin = ORDER == 1;
  constexpr int kMode = kPush | kDeposit;
  constexpr int kPer = (kResidentChunks + NW - 1) / NW;  // chunks per wavefront
  constexpr int kHalos = kLin ? 3 : 1;        // halo copies per chunk
  constexpr int NT = (NW + 1) * kChunk;
  static_assert(NW * kChunk >= kSolveThreads, "the solve's threads");
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double sW2[kSolveThreads];  // the solve threads' field energy sums
  // the threads' kinetic energy and momentum sums and longest segments
  __shared__ double sPart[3][NW * kChunk];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const InstDesc *Ip = a.inst;
  const int nc = Ip->n_cells;
  const ItemLds<PREC, ORDER, SEG> t(smem, nc, 0);
  double2 *sHalo = reinterpret_cast<double2 *>(smem + resident_halo_offset<ORDER>(nc));  // two sets
  Geo g;
  g.L = Ip->L;
  g.half_L = Ip->half_L;
  g.dx = Ip->dx;
  g.inv_dx = Ip->inv_dx;
  g.dt = Ip->dt;
  g.nc = nc;
  const SlotConst kc = slot_const(*Ip);
  const int64_t step0 = Ip->step;
  int flags = Ip->flags;
  const double2 *gHaloIn = kLin ? a.halo3_in : a.halo_in;
  double2 *gHaloOut = kLin ? a.halo3_out : a.halo_out;

  for (int i = tid; i < nc; i += NT) {
    t.sP[i] = (acc_t)0;
    t.sD[i] = (acc_t)0;
    if constexpr (kLin) t.sR[i] = (acc_t)0;
    const double e = a.meshE[kc.mesh_off + i];
    t.sE[i] = e;
    if (i == 0) t.sE[nc] = e;
    if (i == nc - 1) t.sE[-1] = e;
  }
  for (int i = tid; i < kHalos * n_chunks; i += NT) sHalo[i] = gHaloIn[kHalos * (size_t)chunk_begin + i];
  // the wavefront's chunks, in registers for the whole launch, and their
  // tables, chunk w + i * NW in lane i
  const size_t lane_chunk = (size_t)(chunk_begin + min(wave + lane * NW, n_chunks - 1));
  WaveTabs<PREC, ORDER, SEG> tabs;
  tabs.load(a.chunks, a.links, a.cedge, lane_chunk);
  uint64_t xr[kPer], cwr[kPer];
  double vr[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int c = wave + j * NW;
    xr[j] = cwr[j] = 0;
    vr[j] = 0.0;
    if (wave < NW && c < n_chunks) {
      const size_t sidx = (size_t)(chunk_begin + c) * kChunk + lane;
      xr[j] = a.xs[sidx];
      vr[j] = a.vs[sidx];
      if constexpr (SEG) cwr[j] = a.segq[sidx];
    }
  }
  __syncthreads();

  // the row of the step before (the last wavefront's)
  double rk = 0.0, rm = 0.0, rx = 0.0, rq = 0.0;
  auto finish_row = [&](int64_t step) {
    // in the order of field_energy
    double w[kSolveThreads / kChunk];
#pragma unroll
    for (int i = 0; i < kSolveThreads / kChunk; ++i) w[i] = wave_sum(sW2[i * kChunk + lane]);
    const double W = 0.5 * kc.dx * (w[0] + w[1] + w[2] + w[3]);
    flags = solve_flags(sa.flags, flags, kc.L, W, rk, rm, rx);
    if (lane == 0) write_row(sa, 0, kc, step0 + step, flags, W, rq, rk, rm, rx);
  };

  for (int64_t step = 0; step < n_steps; ++step) {
    const double2 *hin = sHalo + (step & 1) * (kHalos * kResidentChunks);
    double2 *hout = sHalo + ((step & 1) ^ 1) * (kHalos * kResidentChunks);
    if (wave < NW) {
      double ke = 0.0, mom = 0.0, ms = 0.0;
      tabs.move(tabs.halos(hin, lane_chunk, chunk_begin), g, t.sE);
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        const int c = wave + j * NW;
        if (c < n_chunks)
          process_chunk<PREC, kMode, ORDER, SEG, false>(t, g, kc.q_unit, nullptr, nullptr, hout, tabs.entry(j),
                                                        (size_t)c, lane, xr[j], vr[j], cwr[j], ke, mom, ms);
      }
      sPart[0][tid] = ke;
      sPart[1][tid] = mom;
      sPart[2][tid] = ms;
    } else if (step > 0) {
      finish_row(step - 1);
    }
    lds_barrier();  // the deposit is complete
    if (wave == NW) {
      rk = rm = rx = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        rk += sPart[0][w * kChunk + lane];
        rm += sPart[1][w * kChunk + lane];
        rx = nan_max(rx, sPart[2][w * kChunk + lane]);
      }
      rk = 0.5 * wave_sum(rk);
      rm = 0.5 * wave_sum(rm);
      rx = wave_max(rx);
    }
    // solve (clears the accumulators, leaves the field in LDS; in global
    // memory too after the last step)
    sacc_t pv[CELLS], dv[CELLS];
    if (wave < kSolveThreads / kChunk) solve_take<PREC, CELLS, 1>(kc, t.sP, t.sD, 0, pv, dv);
    const bool last = step == n_steps - 1;
    const FieldSums f = solve_field<PREC, CELLS>(kc, pv, dv, kLin ? t.sR : (acc_t *)nullptr, 0, t.sE, true,
                                                 last ? sa.meshE + kc.mesh_off : (double *)nullptr,
                                                 last ? sa.meshRho + kc.mesh_off : (double *)nullptr);
    rq = f.Qtot;
    if (tid < kSolveThreads) sW2[tid] = f.w2;
    lds_barrier();  // the field is complete
  }
  if (wave == NW) finish_row(n_steps - 1);

  // state and halos back to global memory
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int c = wave + j * NW;
    if (wave < NW && c < n_chunks) {
      const size_t sidx = (size_t)(chunk_begin + c) * kChunk + lane;
      a.xs[sidx] = xr[j];
      a.vs[sidx] = vr[j];
    }
  }
  const double2 *hend = sHalo + (n_steps & 1) * (kHalos * kResidentChunks);
  for (int i = tid; i < kHalos * n_chunks; i += NT) gHaloOut[kHalos * (size_t)chunk_begin + i] = hend[i];
}

// ---------------------------------------------------------------------------
// Ingest / extract / utilities
// ---------------------------------------------------------------------------
template <int PREC>
__global__ void __launch_bounds__(256) k_ingest(IngestArgs a) {
  const int cl = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (cl >= a.n_chunks) return;
  const int lane = threadIdx.x & 63;
  const int c = a.chunk_begin + cl;
  const ChunkDesc ch = a.chunks[c];
  const InstDesc &I = a.inst[ch.inst];
  const size_t s = (size_t)c * kChunk + lane;
  uint64_t w = 0, cw = 0;
  double v = 0.0;
  if (lane < ch.n_valid) {
    const int64_t src = a.chunk_in_off[cl] + lane;
    v = a.v_in[src];
    if (a.w_in) {
      w = a.w_in[src];  // a state word of this pool (re-layout)
    } else {
      const double x = wrap_into_box(a.x_in[src], I.L);
      if constexpr (PREC == kFP64) {
        w = (uint64_t)__double_as_longlong(x);
      } else {
        const double u = x * I.inv_dx;
        const double f = floor(u);
        w = split_word<PREC>((int)f, u - f, I.n_cells);
      }
    }
    if (a.segq) {
      if (a.cw_in) {
        cw = a.cw_in[src];
      } else if (a.c_in) {
        if constexpr (PREC == kFP64) cw = (uint64_t)__double_as_longlong(a.c_in[src]);
        else cw = (uint64_t)llrint(a.c_in[src] * a.q_scale);
      } else {
        if constexpr (PREC == kFP64) cw = (uint64_t)__double_as_longlong(ch.q);
        else cw = (uint64_t)ch.q_fix;
      }
      if (lane == ch.n_valid - 1 && ch.partner < 0) cw = 0;  // an open sheet's last tracer starts no segment
    }
  }
  a.xs[s] = w;
  a.vs[s] = v;
  if (a.segq) a.segq[s] = cw;
  const double2 hv = make_double2(__longlong_as_double((long long)w), v);
  if (lane == 0) a.halo[c] = hv;
  if (a.halo3) {
    if (lane == 0) a.halo3[3 * (size_t)c + kHaloFirst] = hv;
    if (lane == 1) a.halo3[3 * (size_t)c + kHaloSecond] = hv;
    if (lane == ch.n_valid - 1) a.halo3[3 * (size_t)c + kHaloLast] = hv;
  }
}

template <int PREC>
__global__ void __launch_bounds__(256) k_extract(ExtractArgs a) {
  const int cl = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (cl >= a.n_chunks) return;
  const int lane = threadIdx.x & 63;
  const int c = a.chunk_begin + cl;
  const ChunkDesc ch = a.chunks[c];
  if (lane >= ch.n_valid) return;
  const InstDesc &I = a.inst[ch.inst];
  if (a.step_out != nullptr && cl == 0 && lane == 0) *a.step_out = I.step;
  const size_t s = (size_t)c * kChunk + lane;
  const int64_t dst = a.chunk_in_off[cl] + lane;
  const uint64_t w = a.xs[s];
  double x;
  if constexpr (PREC == kFP64) {
    x = __longlong_as_double((long long)w);
  } else {
    x = mesh_pos<PREC>(w, I.inv_dx) * I.dx;
  }
  a.x_out[dst] = x;
  a.v_out[dst] = a.vs[s];
  if (a.c_out) a.c_out[dst] = charge_value<PREC>(a.segq[s], I.q_unit);
}

// Charge edges of a chunk range (one thread per chunk): the charge of the
// segment ending at the chunk's first tracer and of the segment starting at
// its partner tracer.
__global__ void __launch_bounds__(256) k_charge_edges(const ChunkDesc *chunks, const int64_t *prev_slot,
                                                      const uint64_t *segq, uint64_t *cedge, int32_t chunk_begin,
                                                      int32_t n_chunks) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_chunks) return;
  const int c = chunk_begin + i;
  const int64_t pv = prev_slot[c];
  const int32_t pc = chunks[c].partner;
  cedge[2 * (size_t)c] = pv >= 0 ? segq[pv] : 0ull;
  cedge[2 * (size_t)c + 1] = pc >= 0 ? segq[(size_t)pc * kChunk] : 0ull;
}

// Refinement, one wavefront per chunk.  Each valid lane looks at its segment
// (to the next tracer, or for the last lane to the partner tracer; none at
// an open sheet's end) and marks it when its minimum-image length exceeds
// l_max.
template <int PREC>
__device__ __forceinline__ bool refine_segment(const uint64_t *xs, const double *vs, const ChunkDesc &ch,
                                               const InstDesc &I, int lane, uint64_t w, uint64_t &wn, double &vn,
                                               double &du, double l_max) {
  bool has = lane < ch.n_valid;
  if (lane == ch.n_valid - 1) {
    if (ch.partner >= 0) {
      wn = xs[(size_t)ch.partner * kChunk];
      vn = vs[(size_t)ch.partner * kChunk];
    } else {
      has = false;
    }
  }
  if (!has) return false;
  double len;
  if constexpr (PREC == kFP64) {
    const double xa = __longlong_as_double((long long)w);
    double d = __longlong_as_double((long long)wn) - xa;
    if (d >= I.half_L) d -= I.L;
    else if (d < -I.half_L) d += I.L;
    du = d;
    len = fabs(d);
  } else {
    const double ua = mesh_pos<PREC>(w, I.inv_dx);
    const double dm = min_image_cells(mesh_pos<PREC>(wn, I.inv_dx) - ua, 0.5 * (double)I.n_cells, (double)I.n_cells);
    du = dm;
    len = fabs(dm) * I.dx;
  }
  return len > l_max;
}

// The centre of a split segment and the charges of its halves (fixed point:
// they differ by at most one unit and sum exactly).
template <int PREC>
__device__ __forceinline__ void refine_split(uint64_t w, uint64_t cq, double du, const InstDesc &I, uint64_t *wm,
                                             uint64_t *c0, uint64_t *c1) {
  if constexpr (PREC == kFP64) {
    const double h = 0.5 * __longlong_as_double((long long)cq);
    *c0 = *c1 = (uint64_t)__double_as_longlong(h);
    const double xa = __longlong_as_double((long long)w);
    *wm = (uint64_t)__double_as_longlong(wrap_into_box(xa + 0.5 * du, I.L));
  } else {
    const long long q = (long long)cq;
    const long long q1 = q >> 1;
    *c0 = (uint64_t)(q - q1);
    *c1 = (uint64_t)q1;
    *wm = advance_split<PREC>(w, 0.5 * du, I.n_cells);
  }
}

template <int PREC>
__global__ void __launch_bounds__(256) k_refine_mark(RefineArgs a) {
  const int cl = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (cl >= a.n_chunks) return;  // uniform per wavefront
  const int lane = threadIdx.x & 63;
  const int c = a.chunk_begin + cl;
  const ChunkDesc ch = a.chunks[c];
  const InstDesc &I = a.inst[ch.inst];
  const size_t s = (size_t)c * kChunk + lane;
  const uint64_t w = a.xs[s];
  uint64_t wn = lane_down1(w);
  double vn = 0.0, du = 0.0;
  const bool flag = refine_segment<PREC>(a.xs, a.vs, ch, I, lane, w, wn, vn, du, a.l_max);
  const uint64_t mask = __ballot(flag);
  if (lane == 0) {
    a.cnt[cl] = __popcll(mask);
    a.mask[cl] = mask;
  }
}

// Writes the chunk's tracers to the flat output, each marked one followed by
// the centre of its segment: mean velocity, and the charge split in halves
// (fixed point: the halves differ by at most one unit and sum exactly).
template <int PREC>
__global__ void __launch_bounds__(256) k_refine_scatter(RefineArgs a) {
  const int cl = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (cl >= a.n_chunks) return;  // uniform per wavefront
  const int lane = threadIdx.x & 63;
  const int c = a.chunk_begin + cl;
  const ChunkDesc ch = a.chunks[c];
  const InstDesc &I = a.inst[ch.inst];
  const size_t s = (size_t)c * kChunk + lane;
  const uint64_t w = a.xs[s];
  const double v = a.vs[s];
  const uint64_t cq = a.segq[s];
  uint64_t wn = lane_down1(w);
  double vn = lane_down1(v);
  double du = 0.0;
  refine_segment<PREC>(a.xs, a.vs, ch, I, lane, w, wn, vn, du, a.l_max);
  // the marking pass decided (the host sized the output from its counts)
  const uint64_t mask = a.mask[cl];
  const bool flag = ((mask >> lane) & 1ull) != 0;
  if (lane >= ch.n_valid) return;
  const int64_t out = a.out_off[cl] + lane + __popcll(mask & ((1ull << lane) - 1ull));
  uint64_t c0 = cq;
  if (flag) {
    uint64_t c1, wm;
    refine_split<PREC>(w, cq, du, I, &wm, &c0, &c1);
    a.w_out[out + 1] = wm;
    a.v_out[out + 1] = 0.5 * (v + vn);
    a.c_out[out + 1] = c1;
  }
  a.w_out[out] = w;
  a.v_out[out] = v;
  a.c_out[out] = c0;
}

// A refinement pass on the device (one simulation, whose step marked its
// segments; the host's layout building done on the device, so that refining
// steps need no round trip).  The plan, one workgroup: every chunk's first
// tracer's index in the new order (the old tracers plus the inserted ones,
// sheet-major), each sheet's new tracer count, its first chunk in the new
// layout and its first index, and the capacity check.  A step that marked
// nothing (most, before the sheets fold) ends it at once.  A pass that would
// exceed the capacity inserts nothing and halts the simulation (inactive; the
// host reports it).
__global__ void __launch_bounds__(1024) k_refine_plan(RefinePassArgs a) {
  __shared__ long long sW[16];
  __shared__ long long sTk[16];
  __shared__ long long sTot[2];
  __shared__ int sOver;
  const int tid = threadIdx.x;
  const int nth = blockDim.x;
  int32_t *st = a.state;
  const int halted = st[kRefHalt], marks = st[kRefMarks], n = st[kRefChunks];
  const int cur = st[kRefCur];
  const ChunkDesc *chunks = cur ? a.chunks[1] : a.chunks[0];
  // a chunk and a sheet per thread, in flight with the state words (both sets'
  // descriptors: which one is current is among them)
  const int cap = min(a.chunk_cap, nth);
  int my_cnt = 0, my_nv0 = 0, my_nv1 = 0, my_nt = 0;
  if (tid < cap) {
    my_cnt = a.cnt[tid];
    my_nv0 = a.chunks[0][a.chunk_begin + tid].n_valid;
    my_nv1 = a.chunks[1][a.chunk_begin + tid].n_valid;
  }
  if (tid < a.n_sheets) my_nt = a.nt[tid];
  __syncthreads();
  if (tid == 0) {
    sOver = 0;
    st[kRefMarks] = 0;
    if (!halted) {
      st[kRefSteps] += 1;
      st[kRefStepChunks] = n;
    }
    if (halted || marks == 0) st[kRefInserted] = 0;
  }
  if (halted || marks == 0) return;
  if (n <= nth && a.n_sheets <= nth) {
    // up to 1024 chunks and sheets: one of each per thread, scans of 32-bit
    // integers (at most 128 tracers per old chunk) and offsets in LDS instead
    // of a walk over the chunks and reads back from memory (8 -> 5 us)
    __shared__ int sOff[1025];
    __shared__ int sS[3][16];
    const int lane = tid & 63, wave = tid >> 6, nw = nth >> 6;
    auto scan = [&](int v, int *s16) {
      const int i = wave_incl_scan(v, [](int x, int y) { return x + y; });
      if (lane == 63) s16[wave] = i;
      __syncthreads();
      int base = 0;
      for (int w = 0; w < nw; ++w) base += w < wave ? s16[w] : 0;
      return base + i;
    };
    const int S = a.n_sheets;
    const int v = tid < n ? (cur ? my_nv1 : my_nv0) + my_cnt : 0;
    const int end = scan(v, sS[0]);
    if (tid == 0) sOff[0] = 0;
    sOff[tid + 1] = end;
    if (tid < n) a.out_off[tid] = end - v;
    const int och = tid < S ? (my_nt + kChunk - 1) / kChunk : 0;
    const int f1 = scan(och, sS[1]), f0 = f1 - och;  // its barrier: sOff
    const int o0 = tid < S ? sOff[f0] : 0, nn = tid < S ? sOff[f1] - o0 : 0;
    const int nch = (nn + kChunk - 1) / kChunk;
    const int l1 = scan(nch, sS[2]);
    int64_t *first2 = a.work + S, *flat0 = a.work + 2 * S + 1, *first1 = a.work + 3 * S + 1;
    if (tid < S) {
      a.work[tid] = nn;
      first2[tid] = l1 - nch;
      flat0[tid] = o0;
      first1[tid] = f0;
    }
    if (tid == S - 1) {
      first2[S] = l1;
      first1[S] = f1;
      if (sOff[n] > a.max_tracers || l1 > a.chunk_cap) {
        st[kRefHalt] = 1;
        st[kRefInserted] = 0;
        a.inst[a.slot].active = 0;
      } else {
        st[kRefInserted] = 1;
        st[kRefChunks] = l1;
        st[kRefCur] ^= 1;
      }
    }
    return;
  }
  // Each wavefront takes a contiguous range of chunks and walks it 64 chunks
  // (one per lane, coalesced) at a time, kB groups of loads in flight
  // together: a wavefront scan gives each chunk its offset within the range
  // (written to out_off), the ranges' totals are scanned across the
  // wavefronts, and a second coalesced pass adds each range's base.
  const int lane = tid & 63, wave = tid >> 6, nw = nth >> 6;
  const int per_w = (n + nw - 1) / nw;
  const int w0 = min(n, wave * per_w), w1 = min(n, w0 + per_w);
  constexpr int kB = 4;
  long long run_v = 0, run_k = 0;  // the range so far (every lane)
  for (int gb = w0; gb < w1; gb += kB * 64) {
    long long kv[kB], vv[kB];
#pragma unroll
    for (int u = 0; u < kB; ++u) {
      const int c = gb + u * 64 + lane;
      const int cc = min(c, w1 - 1);
      const long long k = a.cnt[cc];
      const long long v = (long long)chunks[a.chunk_begin + cc].n_valid + k;
      kv[u] = c < w1 ? k : 0;
      vv[u] = c < w1 ? v : 0;
    }
#pragma unroll
    for (int u = 0; u < kB; ++u) {
      const int c = gb + u * 64 + lane;
      const long long iv = wave_incl_scan(vv[u], [](long long x, long long y) { return x + y; });
      const long long ik = wave_incl_scan(kv[u], [](long long x, long long y) { return x + y; });
      if (c < w1) a.out_off[c] = run_v + iv - vv[u];
      run_v += from_lane63(iv);
      run_k += from_lane63(ik);
    }
  }
  if (lane == 0) {
    sW[wave] = run_v;
    sTk[wave] = run_k;
  }
  __syncthreads();
  long long base_v = 0, tot_v = 0, tot_k = 0;
  for (int w = 0; w < nw; ++w) {
    if (w < wave) base_v += sW[w];
    tot_v += sW[w];
    tot_k += sTk[w];
  }
#pragma unroll 4
  for (int c = w0 + lane; c < w1; c += 64) a.out_off[c] += base_v;
  if (tid == 0) {
    sTot[0] = tot_v;
    sTot[1] = tot_k;
  }
  __syncthreads();
  const long long carry = sTot[0], inserted = sTot[1];
  const long long total_new = carry;
  const int S = a.n_sheets;
  int64_t *newnt = a.work;
  int64_t *first2 = a.work + S;  // S + 1 entries
  int64_t *flat0 = a.work + 2 * S + 1;
  int64_t *first1 = a.work + 3 * S + 1;  // S + 1 entries
  long long old_first = 0, new_first = 0;
  for (int base = 0; base < S; base += nth) {
    const int s = base + tid;
    long long och = 0, nch = 0, nn = 0, o0 = 0;
    if (s < S) och = ((long long)a.nt[s] + kChunk - 1) / kChunk;
    const long long io = block_incl_scan(och, sW);
    if (s < S) {
      const long long f0 = old_first + io - och, f1 = old_first + io;  // old chunks of sheet s
      o0 = a.out_off[f0];
      const long long o1 = f1 < n ? a.out_off[f1] : total_new;
      nn = o1 - o0;
      nch = (nn + kChunk - 1) / kChunk;
      if (nn > 0x7fffffffll) sOver = 1;
    }
    const long long in2 = block_incl_scan(nch, sW);
    if (s < S) {
      newnt[s] = nn;
      first2[s] = new_first + in2 - nch;
      flat0[s] = o0;
      first1[s] = old_first + io - och;
    }
    if (tid == nth - 1) {
      sTot[0] = io;
      sTot[1] = in2;
    }
    __syncthreads();
    old_first += sTot[0];
    new_first += sTot[1];
    __syncthreads();
  }
  if (tid == 0) {
    first2[S] = new_first;
    first1[S] = old_first;
    const bool over = sOver != 0 || total_new > a.max_tracers || new_first > a.chunk_cap;
    if (over) {
      st[kRefHalt] = 1;
      st[kRefInserted] = 0;
      a.inst[a.slot].active = 0;
    } else {
      st[kRefInserted] = (int32_t)(inserted < 0x7fffffffll ? inserted : 0x7fffffffll);
      st[kRefChunks] = (int32_t)new_first;
      st[kRefCur] ^= 1;
    }
  }
}

// The planned pass: every old chunk's wavefront writes its tracers, and the
// centre tracer after each marked one, to their slots in the other set of
// state arrays, with the halo copies and charge edges that they are (one
// launch and one pass over the tracers; a flat staging array, a re-ingest
// from it and a pass for the edges took three launches and two).  A thread
// per new chunk writes its descriptor, its links and its work item; the
// accumulators of the unrefined deposit are cleared for the refined one.
template <int PREC>
__global__ void __launch_bounds__(256) k_refine_rebuild(RefinePassArgs a) {
  const int32_t *st = a.state;
  if (st[kRefInserted] <= 0) return;
  const int to = st[kRefCur], from = to ^ 1;  // the plan made the new set current
  const int n1 = st[kRefStepChunks], n2 = st[kRefChunks];
  const int S = a.n_sheets;
  const int64_t *newnt = a.work;
  const int64_t *first2 = a.work + S;
  const int64_t *flat0 = a.work + 2 * S + 1;
  const int64_t *first1 = a.work + 3 * S + 1;
  const InstDesc &I = a.inst[a.slot];
  auto sheet_of = [S](const int64_t *first, int c) {  // the sheet holding chunk c: last s with first[s] <= c
    int lo = 0, hi = S - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (first[mid] <= c) lo = mid;
      else hi = mid - 1;
    }
    return lo;
  };
  const uint64_t *xs = from ? a.xs[1] : a.xs[0];
  const double *vs = from ? a.vs[1] : a.vs[0];
  const uint64_t *segq = from ? a.segq[1] : a.segq[0];
  const ChunkDesc *chunks = from ? a.chunks[1] : a.chunks[0];
  uint64_t *xo = to ? a.xs[1] : a.xs[0];
  double *vo = to ? a.vs[1] : a.vs[0];
  uint64_t *co = to ? a.segq[1] : a.segq[0];
  ChunkDesc *chunks_out = to ? a.chunks[1] : a.chunks[0];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)));
  const int nwaves = gridDim.x * (blockDim.x >> 6);
  for (int cl = wave; cl < n1; cl += nwaves) {
    const int sh = sheet_of(first1, cl);
    const int64_t n = newnt[sh], f0 = flat0[sh];
    const int64_t base = a.chunk_begin + first2[sh];  // the sheet's first chunk
    const int64_t last = base + (n - 1) / kChunk;     // and its last one
    const bool closed = a.closed[sh] != 0;
    const ChunkDesc ch = chunks[a.chunk_begin + cl];
    const size_t s = (size_t)(a.chunk_begin + cl) * kChunk + lane;
    const uint64_t w = xs[s], cq = segq[s];
    const double v = vs[s];
    uint64_t wn = lane_down1(w);
    double vn = lane_down1(v), du = 0.0;
    refine_segment<PREC>(xs, vs, ch, I, lane, w, wn, vn, du, 0.0);
    const uint64_t mask = a.mask[cl];
    // tracer r of the sheet
    auto place = [&](int64_t r, uint64_t pw, double pv, uint64_t pc) {
      const int64_t c = base + (r >> 6);
      const int l = (int)(r & 63);
      const size_t at = (size_t)base * kChunk + (size_t)r;
      xo[at] = pw;
      vo[at] = pv;
      co[at] = pc;
      const double2 h = make_double2(__longlong_as_double((long long)pw), pv);
      const bool end = r == n - 1;
      if (a.order == 1) {
        if (l == 0) a.halo[3 * c + kHaloFirst] = h;
        if (l == 1) a.halo[3 * c + kHaloSecond] = h;
        if (l == 63 || end) a.halo[3 * c + kHaloLast] = h;
      } else if (l == 0) {
        a.halo[c] = h;
      }
      // its segment starts at the partner of the chunk before it, and ends at
      // the first tracer of the chunk after it
      if (l == 0 && (r > 0 || closed)) a.cedge[2 * (r > 0 ? c - 1 : last) + 1] = pc;
      if (end) a.cedge[2 * base] = closed ? pc : 0ull;
      else if (l == 63) a.cedge[2 * (c + 1)] = pc;
      if (end && !closed) a.cedge[2 * last + 1] = 0ull;
    };
    if (lane < ch.n_valid) {
      const bool flag = ((mask >> lane) & 1ull) != 0;
      const int64_t r = a.out_off[cl] - f0 + lane + __popcll(mask & ((1ull << lane) - 1ull));
      uint64_t c0 = cq;
      if (flag) {
        uint64_t c1, wm;
        refine_split<PREC>(w, cq, du, I, &wm, &c0, &c1);
        place(r + 1, wm, 0.5 * (v + vn), c1);
      }
      place(r, w, v, c0);
    }
    if (cl + 1 == first1[sh + 1]) {  // the sheet's last old chunk clears the padding of its last new one
      const int64_t r = n + lane;
      if (r < (last - base + 1) * kChunk) {
        const size_t at = (size_t)base * kChunk + (size_t)r;
        xo[at] = 0;
        vo[at] = 0.0;
        co[at] = 0;
      }
    }
  }
  const int tid = blockIdx.x * blockDim.x + threadIdx.x, nt = gridDim.x * blockDim.x;
  auto n_valid_of = [](long long n, long long k) { return (int32_t)min((long long)kChunk, n - k * kChunk); };
  for (int c = tid; c < n2; c += nt) {
    const int sh = sheet_of(first2, c);
    const long long k = c - first2[sh];
    const long long n = newnt[sh];
    const long long nch = (n + kChunk - 1) / kChunk;
    const int32_t first = a.chunk_begin + (int32_t)first2[sh];
    const bool cl = a.closed[sh] != 0;
    ChunkDesc d;
    d.q = a.q[sh];
    d.q_fix = a.fixed ? (int64_t)llrint(a.q[sh] * a.q_scale) : 0;
    d.n_valid = n_valid_of(n, k);
    d.inst = a.slot;
    d.flags = (k == 0 && !cl) ? kChunkOpenStart : 0;
    d.partner = (k + 1 < nch) ? (int32_t)(first + k + 1) : (cl ? first : -1);
    chunks_out[first + k] = d;
    if (a.links) {
      int2 lk = make_int2(-1, -1);
      if (!cl || n >= 3) {
        if (k > 0) lk.x = (int32_t)(((first + k - 1) << 2) | kHaloLast);
        else if (cl) lk.x = (int32_t)(((first + nch - 1) << 2) | kHaloLast);
        if (d.partner >= 0) {
          const long long pk = d.partner - first;
          if (n_valid_of(n, pk) >= 2) {
            lk.y = (d.partner << 2) | kHaloSecond;
          } else {
            const int32_t pp = (pk + 1 < nch) ? (int32_t)(first + pk + 1) : (cl ? first : -1);
            if (pp >= 0) lk.y = (pp << 2) | kHaloFirst;
          }
        }
      }
      a.links[first + k] = lk;
    }
  }
  const int tile = refine_tile(n2, a.tile_fixed), n_items = refine_items(n2, a.tile_fixed);
  for (int c = tid; c < n_items; c += nt) {
    Item it;
    it.inst = a.slot;
    it.chunk_begin = a.chunk_begin + c * tile;
    it.chunk_end = a.chunk_begin + min(n2, (c + 1) * tile);
    it.pad = 0;
    a.items[a.item_begin + c] = it;
  }
  for (int sh = tid; sh < S; sh += nt) a.nt[sh] = (int32_t)newnt[sh];
  uint64_t *z = reinterpret_cast<uint64_t *>(a.acc_zero);
  if (z != nullptr)
    for (int64_t i = tid; i < a.acc_words; i += nt) z[i] = 0;
  if (tid == 0) {
    a.slot_items[a.slot].y = n_items;
    *a.n_items = a.item_begin + n_items;
  }
}

template <int PREC>
__global__ void __launch_bounds__(256) k_zero_mesh(void *meshP, void *meshD, void *meshR, InstDesc *inst,
                                                   const int32_t *slot_list, int rep, int64_t rep_stride,
                                                   int64_t step) {
  using acc_t = typename std::conditional<PREC == kFP64, double, long long>::type;
  const int slot = slot_list ? slot_list[blockIdx.x] : (int)blockIdx.x;
  const InstDesc &I = inst[slot];
  if (step >= 0 && threadIdx.x == 0) inst[slot].step = step;
  for (int r = 0; r < rep; ++r) {
    const int64_t off = I.mesh_off + r * rep_stride;
    acc_t *P = reinterpret_cast<acc_t *>(meshP) + off;
    acc_t *D = reinterpret_cast<acc_t *>(meshD) + off;
    acc_t *R = meshR ? reinterpret_cast<acc_t *>(meshR) + off : nullptr;
    for (int j = threadIdx.x; j < I.n_cells; j += blockDim.x) {
      P[j] = (acc_t)0;
      D[j] = (acc_t)0;
      if (R) R[j] = (acc_t)0;
    }
  }
}

// The reads of a diagnostics call in one launch, to host memory: a call then
// waits for the stream once, where a copy per item waited for each (one step
// and its diagnostics on 50 cells: six waits of 10 to 15 us).
__global__ void __launch_bounds__(256) k_export(ExportArgs a) {
  const int tid = blockIdx.x * blockDim.x + threadIdx.x, nt = gridDim.x * blockDim.x;
  const InstDesc &I = *a.inst;
  const int64_t step = I.step, cap = I.hist_cap;
  const uint64_t *src = reinterpret_cast<const uint64_t *>(a.inst);
  uint64_t *out = reinterpret_cast<uint64_t *>(a.out);
  constexpr int kRowWords = sizeof(DiagRow) / 8;
  static_assert(sizeof(InstDesc) <= kExportRow && kExportRow + sizeof(DiagRow) <= kExportMesh, "export layout");
  for (int i = tid; i < (int)(sizeof(InstDesc) / 8); i += nt) out[i] = src[i];
  const uint64_t *newest = reinterpret_cast<const uint64_t *>(a.hist + row_of(step, cap));
  for (int i = tid; i < kRowWords; i += nt) out[kExportRow / 8 + i] = newest[i];
  out += kExportMesh / 8;
  if (a.rho != nullptr) {
    double *m = reinterpret_cast<double *>(out);
    for (int i = tid; i < a.nc; i += nt) {
      m[i] = a.rho[i];
      m[a.nc + i] = a.E[i];
    }
    out += 2 * a.nc;
  }
  const int64_t avail = min(step + 1 - min(step, a.hist_from), cap);
  int64_t rows = min(avail, a.rows);
  if (rows > a.max_rows) rows = 0;  // the caller copies them
  for (int64_t i = tid; i < rows * kRowWords; i += nt) {
    const DiagRow *r = a.hist + row_of(step + 1 - rows + i / kRowWords, cap);
    out[i] = reinterpret_cast<const uint64_t *>(r)[i % kRowWords];
  }
}

// Streaming copy for the bandwidth calibration: per iteration each lane has
// kCopyUnroll 16-byte loads in flight before it stores them; loads and stores
// are non-temporal (the array streams through once), and the workgroups
// stride over the array together.
typedef double f64x2 __attribute__((ext_vector_type(2)));
constexpr int kCopyUnroll = 4;

__global__ void __launch_bounds__(256) k_copy(const f64x2 *__restrict__ src, f64x2 *__restrict__ dst, int64_t n2) {
  const int64_t bd = blockDim.x;
  const int64_t per_iter = (int64_t)gridDim.x * bd * kCopyUnroll;
  int64_t i = (int64_t)blockIdx.x * bd * kCopyUnroll + threadIdx.x;
  for (; i + (kCopyUnroll - 1) * bd < n2; i += per_iter) {
    f64x2 r[kCopyUnroll];
#pragma unroll
    for (int u = 0; u < kCopyUnroll; ++u) r[u] = __builtin_nontemporal_load(src + i + u * bd);
#pragma unroll
    for (int u = 0; u < kCopyUnroll; ++u) __builtin_nontemporal_store(r[u], dst + i + u * bd);
  }
  for (int u = 0; u < kCopyUnroll; ++u) {
    if (i + u * bd < n2) dst[i + u * bd] = src[i + u * bd];
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
constexpr size_t kLdsMax = 160 * 1024;  // per workgroup on gfx950

// Raises a kernel's dynamic LDS limit to bytes, the most that a launch of it
// asks for, before its first launch on a device (devices: those done).  The
// limit belongs to the kernel, which all simulations and threads share: set to
// one launch's size it would refuse a larger launch of another thread.
static hipError_t allow_lds(const void *f, size_t bytes, std::atomic<uint64_t> &devices) {
  int device = 0;
  hipError_t e = hipGetDevice(&device);
  if (e != hipSuccess) return e;
  const uint64_t bit = 1ull << (device & 63);
  if (devices.load() & bit) return hipSuccess;
  e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess) devices.fetch_or(bit);
  return e;
}

// The deposit-only launch of constant segments: its own LDS layout (no field,
// a ring per wavefront), with the workgroup narrowed until it fits.
template <int PREC, bool SEG>
static hipError_t deposit_faces(const TracerArgs &a, int grid, int block, hipStream_t st) {
  static std::atomic<uint64_t> devices{0};
  const hipError_t e = allow_lds((const void *)k_deposit_faces<PREC, SEG>, kLdsMax, devices);
  if (e != hipSuccess) return e;
  size_t lds = dep_lds_bytes<SEG>(a.mesh_cells, a.tile_cap, block / kChunk);
  while (lds > kLdsMax && block > kChunk) {
    block /= 2;
    lds = dep_lds_bytes<SEG>(a.mesh_cells, a.tile_cap, block / kChunk);
  }
  if (lds > kLdsMax) return hipErrorInvalidValue;
  TracerArgs b = a;
  if (grid <= kComputeUnits) b.run = 1;  // fewer than run at a time in any case
  if (b.run > 1) {
    // a.run items per workgroup at most, fewer while workgroups are left that
    // would run at the same time
    int per_cu = 1;
    const hipError_t e =
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)k_deposit_faces<PREC, SEG>, block, lds);
    if (e != hipSuccess) return e;
    // where the LDS mesh leaves a compute unit one or two workgroups, they
    // have little to do while one of them clears or merges (33.5M tracers, one
    // item at a time and in runs: 2048 cells 111 and 107 us, 2500 116 and 111,
    // 3000 155 and 137, 4096 192 and 170); four overlap one another, and one
    // item at a time spreads better (67M tracers, 1024 cells: 138 us, 143 in
    // runs of four)
    const int resident = std::max(1, per_cu) * kComputeUnits;
    b.run = per_cu > 2 ? 1 : std::max(1, std::min(b.run, (grid + resident - 1) / resident));
    // Of two workgroups per compute unit, runs that leave many of the places
    // empty lose more than they save: 600 items in 300 pairs (2048 cells, with
    // charges) 38 -> 42 us, 698 in 349 (3000 cells) 50 -> 52 to 57; 820 in 410
    // 50 -> 44, with charges 58 -> 53 but 1639 in runs of four 96 -> 101.
    if (per_cu == 2 && (SEG ? 10 : 4) * grid < (SEG ? 9 : 3) * resident * b.run) b.run = 1;
    grid = (grid + b.run - 1) / b.run;
  }
  hipLaunchKernelGGL((k_deposit_faces<PREC, SEG>), dim3(grid), dim3(block), lds, st, b);
  return hipGetLastError();
}

template <int PREC, int ORDER, bool SEG>
static hipError_t tracers_prec(int mode, const TracerArgs &a, int grid, int block, size_t lds, hipStream_t st) {
  switch (mode) {
    case kDeposit:
      if constexpr (ORDER == 0) {
        return deposit_faces<PREC, SEG>(a, grid, block, st);
      } else {
        hipLaunchKernelGGL((k_tracers<PREC, kDeposit, ORDER, SEG>), dim3(grid), dim3(block), lds, st, a);
      }
      break;
    case kPush:
      hipLaunchKernelGGL((k_tracers<PREC, kPush, ORDER, SEG>), dim3(grid), dim3(block), lds, st, a);
      break;
    case kPush | kDeposit:
      hipLaunchKernelGGL((k_tracers<PREC, kPush | kDeposit, ORDER, SEG>), dim3(grid), dim3(block), lds, st, a);
      break;
    case kKickHalf:
      hipLaunchKernelGGL((k_tracers<PREC, kKickHalf, ORDER, SEG>), dim3(grid), dim3(block), lds, st, a);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

constexpr int kMaxItemChunks = 256;  // of a tracer launch's work item

template <int PREC, int ORDER, bool SEG>
static hipError_t set_lds_limit() {
  static std::atomic<uint64_t> devices[4];
  constexpr size_t bytes = tracer_lds_bytes<double, ORDER, SEG>(kMaxCells, kMaxItemChunks);
  static_assert(bytes <= kLdsMax, "the largest item's tables");
  const void *fns[] = {(const void *)k_tracers<PREC, kPush, ORDER, SEG>,
                       (const void *)k_tracers<PREC, kPush | kDeposit, ORDER, SEG>,
                       (const void *)k_tracers<PREC, kKickHalf, ORDER, SEG>};
  for (int i = 0; i < 3; ++i) {
    const hipError_t e = allow_lds(fns[i], bytes, devices[i]);
    if (e != hipSuccess) return e;
  }
  if constexpr (ORDER != 0) return allow_lds((const void *)k_tracers<PREC, kDeposit, ORDER, SEG>, bytes, devices[3]);
  return hipSuccess;
}

// Dispatch of a runtime (precision, order, per-segment charges) triple to a
// template instance.
template <template <int, int, bool> class F, class... Args>
static hipError_t dispatch(int prec, int order, bool seg, Args &&...args) {
#define SIC_CASE(P, O)                                                                    \
  if (prec == P && order == O)                                                            \
    return seg ? F<P, O, true>::run(args...) : F<P, O, false>::run(args...);
  SIC_CASE(kFP64, 0) SIC_CASE(kFP64, 1) SIC_CASE(kFP64, 2)
  SIC_CASE(kSplitF32, 0) SIC_CASE(kSplitF32, 1) SIC_CASE(kSplitF32, 2)
  SIC_CASE(kSplitU32, 0) SIC_CASE(kSplitU32, 1) SIC_CASE(kSplitU32, 2)
#undef SIC_CASE
  return hipErrorInvalidValue;
}

template <int PREC, int ORDER, bool SEG>
struct LaunchTracers {
  static hipError_t run(int mode, const TracerArgs &a, int grid, int block, size_t lds, hipStream_t st) {
    return tracers_prec<PREC, ORDER, SEG>(mode, a, grid, block, lds, st);
  }
};

template <int PREC, int ORDER, bool SEG>
struct SetLdsLimit {
  static hipError_t run() { return set_lds_limit<PREC, ORDER, SEG>(); }
};

int set_tracer_lds_limit(int prec, int order, bool seg) { return (int)dispatch<SetLdsLimit>(prec, order, seg); }

// Solve-first steps (single simulations).
template <int PREC, int ORDER, bool SEG, int CELLS>
static hipError_t step_launch(const StepArgs &a, int grid, int block, size_t lds, hipStream_t st) {
  // (not the whole 160 KB: the solve's static LDS takes part of it)
  static std::atomic<uint64_t> devices{0};
  const hipError_t e = allow_lds((const void *)k_step<PREC, ORDER, SEG, CELLS>,
                                 tracer_lds_bytes<double, ORDER, SEG>(CELLS * kSolveThreads, 0), devices);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_step<PREC, ORDER, SEG, CELLS>), dim3(grid), dim3(block), lds, st, a);
  return hipGetLastError();
}

// The step of linear segments is built for meshes of up to 1024 cells: with
// 16 cells per thread its solve's three arrays do not fit 128 registers.
bool step_supported(int order, int max_cells) {
  return max_cells >= 1 && max_cells <= (order == 1 ? 4 * kSolveThreads : kMaxCells);
}

template <int PREC, int ORDER, bool SEG>
struct LaunchStep {
  static hipError_t run(const StepArgs &a, int grid, int block, size_t lds, hipStream_t st) {
    const int per = (a.nc + kSolveThreads - 1) / kSolveThreads;
    if (per <= 1) return step_launch<PREC, ORDER, SEG, 1>(a, grid, block, lds, st);
    if (per <= 4) return step_launch<PREC, ORDER, SEG, 4>(a, grid, block, lds, st);
    if constexpr (ORDER != 1) return step_launch<PREC, ORDER, SEG, 16>(a, grid, block, lds, st);
    return hipErrorInvalidValue;
  }
};

template <int PREC, int ORDER, bool SEG>
struct LaunchRun {
  static hipError_t run(const StepArgs &a, int block, size_t lds, hipStream_t st, int *grid) {
    // as many workgroups as run at a time
    int per_cu = 1;
    const void *f = (const void *)k_step<PREC, ORDER, SEG, 0>;
    static std::atomic<uint64_t> devices{0};
    hipError_t e = allow_lds(f, tracer_lds_bytes<double, ORDER, SEG>(kMaxCells, 0), devices);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, block, lds);
    if (e != hipSuccess) return e;
    StepArgs b = a;
    const int n = std::max(1, std::min(*grid, std::max(1, per_cu) * kComputeUnits));
    b.n_items = n;
    *grid = n;
    hipLaunchKernelGGL((k_step<PREC, ORDER, SEG, 0>), dim3(n), dim3(block), lds, st, b);
    return hipGetLastError();
  }
};

int launch_run(int prec, int order, bool seg, const StepArgs &a, int block, void *stream, int *grid) {
  if (a.nc < 1 || a.nc > kMaxCells || block < kChunk || block > 1024 || a.n_chunks < 1 || *grid < 1 ||
      a.acc_in != nullptr || a.acc_zero != nullptr || a.sel.state != nullptr)
    return (int)hipErrorInvalidValue;
  const size_t lds = tracer_lds_size(prec, order, seg, a.nc, 0);
  return (int)dispatch<LaunchRun>(prec, order, seg, a, block, lds, (hipStream_t)stream, grid);
}

int launch_step(int prec, int order, bool seg, const StepArgs &a, int grid, int block, void *stream) {
  // a wavefront stages at most 64 chunks of an item: a.tile <= block
  if (!step_supported(order, a.nc) || block < kSolveThreads || a.tile < 1 || a.tile > block || a.n_items < 1 ||
      grid < 1 || grid > a.n_items || (a.sel.state != nullptr && !seg))
    return (int)hipErrorInvalidValue;
  // the chunks' tables are in registers: the mesh, the field and the sums only
  const size_t lds = tracer_lds_size(prec, order, seg, a.nc, 0);
  StepArgs b = a;
  b.row_group = grid < kComputeUnits ? 1 : 0;
  grid += b.row_group;
  const int words = (order == 1 ? 3 : 2) * single_rep(a.nc) * a.nc;
  b.zero_slice = (words + grid - 1) / grid;
  return (int)dispatch<LaunchStep>(prec, order, seg, b, grid, block, lds, (hipStream_t)stream);
}

int launch_tracers(int prec, int mode, int order, bool seg, const TracerArgs &a, int grid, int block, size_t lds,
                   void *stream) {
  if (grid <= 0) return 0;
  return (int)dispatch<LaunchTracers>(prec, order, seg, mode, a, grid, block, lds, (hipStream_t)stream);
}

// Meshes of up to 1024 cells run the resident kernel with 12 wavefronts of
// up to three chunks each and one for the rows (a pass of 100 steps of 32
// chunks on 128 cells: 619 us; 8 wavefronts 692, 11 674, 15 651; of one chunk:
// 424, and 409 with 8); larger ones, whose solve holds 16 cells per thread in
// registers, with four (us per step, with the rows in the chain before and now:
// 64 tracers on 1100, 2048 and 4096 cells 4.9, 6.1, 10.7 and 3.9, 5.3, 10.2;
// 2 x 1000 tracers 12.0, 13.1, 17.9 and 8.3, 9.7, 14.6; as solve-first launches
// the last one takes 17.7) and, with a third array, not with linear segments.
template <int PREC, int ORDER, bool SEG, int CELLS>
static hipError_t resident_launch(const TracerArgs &a, const SolveArgs &sa, int chunk_begin, int n_chunks,
                                  int n_cells, int64_t n_steps, hipStream_t st) {
  constexpr int NW = CELLS <= 4 ? 12 : kSolveThreads / kChunk;
  const size_t lds = resident_lds_bytes<ORDER>(n_cells);
  static std::atomic<uint64_t> devices{0};
  const hipError_t e = allow_lds((const void *)k_resident<PREC, ORDER, SEG, CELLS, NW>,
                                 resident_lds_bytes<ORDER>(CELLS * kSolveThreads), devices);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_resident<PREC, ORDER, SEG, CELLS, NW>), dim3(1), dim3((NW + 1) * kChunk), lds, st, a, sa,
                     chunk_begin, n_chunks, n_steps);
  return hipGetLastError();
}

// Cells per solve thread the kernels are built for: 1, 4 or 16.
static int solve_cells(int max_cells) { return kSolveCells[solve_class(max_cells)] / kSolveThreads; }

template <int PREC, int ORDER, bool SEG>
struct LaunchResident {
  static hipError_t run(const TracerArgs &a, const SolveArgs &sa, int chunk_begin, int n_chunks, int n_cells,
                        int64_t n_steps, hipStream_t st) {
    switch (solve_cells(n_cells)) {
      case 1: return resident_launch<PREC, ORDER, SEG, 1>(a, sa, chunk_begin, n_chunks, n_cells, n_steps, st);
      case 4: return resident_launch<PREC, ORDER, SEG, 4>(a, sa, chunk_begin, n_chunks, n_cells, n_steps, st);
      default:
        if constexpr (ORDER != 1)
          return resident_launch<PREC, ORDER, SEG, 16>(a, sa, chunk_begin, n_chunks, n_cells, n_steps, st);
        return hipErrorInvalidValue;
    }
  }
};

bool resident_supported(int order, int n_chunks, int n_cells) {
  return n_chunks >= 1 && n_chunks <= kResidentChunks && step_supported(order, n_cells);
}

int launch_resident(int prec, int order, bool seg, const TracerArgs &a, const SolveArgs &sa, int chunk_begin,
                    int n_chunks, int n_cells, int64_t n_steps, void *stream) {
  if (n_steps <= 0) return 0;
  if (!resident_supported(order, n_chunks, n_cells)) return (int)hipErrorInvalidValue;
  return (int)dispatch<LaunchResident>(prec, order, seg, a, sa, chunk_begin, n_chunks, n_cells, n_steps,
                                       (hipStream_t)stream);
}

template <int PREC, int CELLS, int REP>
static hipError_t solve_launch(const SolveArgs &a, int n_blocks, hipStream_t st) {
  // 16 cells per thread: the accumulators of the largest mesh in LDS, padded
  // (68 KB beside the static LDS)
  constexpr size_t lds = CELLS == 16 ? 2 * sizeof(double) * (CELLS + 1) * kSolveThreads : 0;
  if constexpr (lds > 0) {
    static std::atomic<uint64_t> devices{0};
    const hipError_t e = allow_lds((const void *)k_solve<PREC, CELLS, REP>, lds, devices);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_solve<PREC, CELLS, REP>), dim3(n_blocks), dim3(kSolveThreads), lds, st, a);
  return hipGetLastError();
}

template <int CELLS, int REP>
static hipError_t solve_cells_launch(int prec, const SolveArgs &a, int n_blocks, hipStream_t st) {
  switch (prec) {
    case kFP64: return solve_launch<kFP64, CELLS, REP>(a, n_blocks, st);
    case kSplitF32: return solve_launch<kSplitF32, CELLS, REP>(a, n_blocks, st);
    case kSplitU32: return solve_launch<kSplitU32, CELLS, REP>(a, n_blocks, st);
    default: return hipErrorInvalidValue;
  }
}

template <int REP>
static hipError_t solve_rep_launch(int prec, const SolveArgs &a, int n_blocks, int max_cells, hipStream_t st) {
  switch (solve_cells(max_cells)) {
    case 1: return solve_cells_launch<1, REP>(prec, a, n_blocks, st);
    case 4: return solve_cells_launch<4, REP>(prec, a, n_blocks, st);
    default: return solve_cells_launch<16, REP>(prec, a, n_blocks, st);
  }
}

int launch_solve(int prec, const SolveArgs &a, int n_blocks, int max_cells, void *stream) {
  hipStream_t st = (hipStream_t)stream;
  if (n_blocks <= 0) return 0;
  if (max_cells < 1 || max_cells > kMaxCells) return (int)hipErrorInvalidValue;
  if (a.rep == 1) return (int)solve_rep_launch<1>(prec, a, n_blocks, max_cells, st);
  if (a.rep == 2) return (int)solve_rep_launch<2>(prec, a, n_blocks, max_cells, st);
  if (a.rep == kSmallMeshRep && max_cells <= kSolveThreads)
    return (int)solve_cells_launch<1, kSmallMeshRep>(prec, a, n_blocks, st);
  return (int)hipErrorInvalidValue;
}

int launch_ingest(int prec, const IngestArgs &a, void *stream) {
  hipStream_t st = (hipStream_t)stream;
  const int grid = (a.n_chunks + 3) / 4;
  if (grid <= 0) return 0;
  switch (prec) {
    case kFP64: hipLaunchKernelGGL(k_ingest<kFP64>, dim3(grid), dim3(256), 0, st, a); break;
    case kSplitF32: hipLaunchKernelGGL(k_ingest<kSplitF32>, dim3(grid), dim3(256), 0, st, a); break;
    case kSplitU32: hipLaunchKernelGGL(k_ingest<kSplitU32>, dim3(grid), dim3(256), 0, st, a); break;
    default: return (int)hipErrorInvalidValue;
  }
  return (int)hipGetLastError();
}

int launch_extract(int prec, const ExtractArgs &a, void *stream) {
  hipStream_t st = (hipStream_t)stream;
  const int grid = (a.n_chunks + 3) / 4;
  if (grid <= 0) return 0;
  switch (prec) {
    case kFP64: hipLaunchKernelGGL(k_extract<kFP64>, dim3(grid), dim3(256), 0, st, a); break;
    case kSplitF32: hipLaunchKernelGGL(k_extract<kSplitF32>, dim3(grid), dim3(256), 0, st, a); break;
    case kSplitU32: hipLaunchKernelGGL(k_extract<kSplitU32>, dim3(grid), dim3(256), 0, st, a); break;
    default: return (int)hipErrorInvalidValue;
  }
  return (int)hipGetLastError();
}

int launch_export(const ExportArgs &a, void *stream) {
  // most of the room for rows is often unused: a thread for every four words
  // that there may be
  const int64_t words = std::max<int64_t>(2 * a.nc, 8 * std::min(a.rows, a.max_rows));
  const int grid = (int)std::min<int64_t>(8, words / 1024 + 1);  // at least one: the descriptor and the row
  hipLaunchKernelGGL(k_export, dim3(grid), dim3(256), 0, (hipStream_t)stream, a);
  return (int)hipGetLastError();
}

int launch_zero_mesh(int prec, void *meshP, void *meshD, void *meshR, InstDesc *inst,
                     const int32_t *slot_list, int n_blocks, int rep, int64_t rep_stride, void *stream,
                     int64_t step) {
  hipStream_t st = (hipStream_t)stream;
  if (n_blocks <= 0) return 0;
  if (rep < 1) return (int)hipErrorInvalidValue;
  if (prec == kFP64)
    hipLaunchKernelGGL(k_zero_mesh<kFP64>, dim3(n_blocks), dim3(256), 0, st, meshP, meshD, meshR, inst, slot_list,
                       rep, rep_stride, step);
  else
    hipLaunchKernelGGL(k_zero_mesh<kSplitF32>, dim3(n_blocks), dim3(256), 0, st, meshP, meshD, meshR, inst,
                       slot_list, rep, rep_stride, step);
  return (int)hipGetLastError();
}

int launch_charge_edges(const ChunkDesc *chunks, const int64_t *prev_slot, const uint64_t *segq, uint64_t *cedge,
                        int32_t chunk_begin, int32_t n_chunks, void *stream) {
  if (n_chunks <= 0) return 0;
  hipLaunchKernelGGL(k_charge_edges, dim3((n_chunks + 255) / 256), dim3(256), 0, (hipStream_t)stream, chunks,
                     prev_slot, segq, cedge, chunk_begin, n_chunks);
  return (int)hipGetLastError();
}

int launch_refine_mark(int prec, const RefineArgs &a, void *stream) {
  hipStream_t st = (hipStream_t)stream;
  const int grid = (a.n_chunks + 3) / 4;
  if (grid <= 0) return 0;
  switch (prec) {
    case kFP64: hipLaunchKernelGGL(k_refine_mark<kFP64>, dim3(grid), dim3(256), 0, st, a); break;
    case kSplitF32: hipLaunchKernelGGL(k_refine_mark<kSplitF32>, dim3(grid), dim3(256), 0, st, a); break;
    case kSplitU32: hipLaunchKernelGGL(k_refine_mark<kSplitU32>, dim3(grid), dim3(256), 0, st, a); break;
    default: return (int)hipErrorInvalidValue;
  }
  return (int)hipGetLastError();
}

int launch_refine_scatter(int prec, const RefineArgs &a, void *stream) {
  hipStream_t st = (hipStream_t)stream;
  const int grid = (a.n_chunks + 3) / 4;
  if (grid <= 0) return 0;
  switch (prec) {
    case kFP64: hipLaunchKernelGGL(k_refine_scatter<kFP64>, dim3(grid), dim3(256), 0, st, a); break;
    case kSplitF32: hipLaunchKernelGGL(k_refine_scatter<kSplitF32>, dim3(grid), dim3(256), 0, st, a); break;
    case kSplitU32: hipLaunchKernelGGL(k_refine_scatter<kSplitU32>, dim3(grid), dim3(256), 0, st, a); break;
    default: return (int)hipErrorInvalidValue;
  }
  return (int)hipGetLastError();
}

int launch_refine_plan(const RefinePassArgs &a, void *stream) {
  hipLaunchKernelGGL(k_refine_plan, dim3(1), dim3(1024), 0, (hipStream_t)stream, a);
  return (int)hipGetLastError();
}

int launch_refine_rebuild(int prec, const RefinePassArgs &a, void *stream) {
  hipStream_t st = (hipStream_t)stream;
  // the capacity at a wavefront per chunk, up to two workgroups per compute
  // unit (a simulation holds far fewer chunks than its capacity for most of a
  // run, and a launch pays for the workgroups that find nothing to do)
  const int grid = std::max(1, std::min((a.chunk_cap + 3) / 4, 2 * kComputeUnits));
  switch (prec) {
    case kFP64: hipLaunchKernelGGL(k_refine_rebuild<kFP64>, dim3(grid), dim3(256), 0, st, a); break;
    case kSplitF32: hipLaunchKernelGGL(k_refine_rebuild<kSplitF32>, dim3(grid), dim3(256), 0, st, a); break;
    case kSplitU32: hipLaunchKernelGGL(k_refine_rebuild<kSplitU32>, dim3(grid), dim3(256), 0, st, a); break;
    default: return (int)hipErrorInvalidValue;
  }
  return (int)hipGetLastError();
}

int launch_copy_bench(const double *src, double *dst, int64_t n, int grid, void *stream) {
  const int64_t n2 = n / 2;
  hipLaunchKernelGGL(k_copy, dim3(grid), dim3(256), 0, (hipStream_t)stream, (const f64x2 *)src, (f64x2 *)dst, n2);
  return (int)hipGetLastError();
}

}  // namespace sic
