// HIP kernels (gfx950) of the peridynamic grain-aggregate step.
//
// Layout in HBM
//   u      : two buffers of double4 (x, y, z, w); w carries the node's packed
//            grain-local lattice index (10 bits per axis) in its low 32 bits
//            and its grain id in the high 32 bits, so one 32-byte gather per
//            bond brings both the neighbour displacement and its lattice offset.
//   v, a   : SoA FP64, touched only by the owning lane.
//   bonds  : sliced-ELL (SELL-64) CSR.  Slice s = nodes [64 s, 64 s + 64) (one
//            wavefront); entry k of lane l sits at colE[slice_off[s] + 64 k + l],
//            so the column loads of a wavefront are one coalesced 256-byte read.
//            A column word is node_j | class << node_bits, class = index of the
//            lattice offset in the horizon stencil.  Bond memory lives in the
//            word itself: a bond that breaks is rewritten to node_i with the
//            zero-force class, which is also what padding entries hold, so the
//            step kernel needs no separate broken-flag reads.  On large meshes
//            the slice path's steps read, and break bonds in, a second set of
//            rows, in which the lanes of a slice hold the same class at the same
//            entry (k_align); the column words follow when something else reads
//            them (k_lined_to_cols).
//
// Each lane owns one node and evaluates its row in order (gather formulation,
// Sec. 3.1 eq. (peri-damage) with nodal quadrature, Sec. 6.1): no atomics, so
// results are bitwise reproducible run to run.

#include <hip/hip_ext.h>

#include <algorithm>
#include <utility>

#include "pd_internal.h"

namespace pdk {

// Workgroups are dispatched round-robin over the 8 XCDs of the MI355X; map them
// so each XCD walks one contiguous range of slices (its L2 then holds that
// range's neighbourhood instead of every eighth slice of the whole mesh).
__device__ __forceinline__ int64_t xcd_remap(int64_t b, int64_t nb) {
  const int64_t x = b & 7, q = nb >> 3, r = nb & 7;
  return x * q + (x < r ? x : r) + (b >> 3);
}

// the halt word, read the same by every lane of the launch
__device__ __forceinline__ bool halted(const uint32_t* halt) {
  return __builtin_amdgcn_readfirstlane(__hip_atomic_load(halt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) != 0u;
}

__device__ __forceinline__ int unpack_x(int p) { return p & 1023; }
__device__ __forceinline__ int unpack_y(int p) { return (p >> 10) & 1023; }
__device__ __forceinline__ int unpack_z(int p) { return (p >> 20) & 1023; }
__device__ __forceinline__ int packed_ijk(double w) { return (int)(__double_as_longlong(w) & 0xffffffffll); }
__device__ __forceinline__ int packed_grain(double w) { return (int)(__double_as_longlong(w) >> 32); }

// reference position origin + h*ijk evaluated exactly as the input lays it out
__device__ __forceinline__ double lattice_pos(double origin, double h, int idx) {
  return __dadd_rn(origin, __dmul_rn(h, (double)idx));
}

// 1/sqrt(x) to full double precision: hardware estimate refined by one
// Newton step with the cubic term, r (1 + e/2 + 3e^2/8), e = 1 - x r^2.
__device__ __forceinline__ double rsqrt_full(double x) {
  double r = __builtin_amdgcn_rsq(x);
  const double t = x * r;
  const double e = fma(-t, r, 1.0);
  double c = 0.375;
  asm volatile("" : "+s"(c));  // (made here: hoisted out of a bond loop it would hold two vector registers)
  return fma(r * e, fma(c, e, 0.5), r);
}

// 1/x to full double precision: hardware estimate refined by r (1 + e + e^2),
// e = 1 - x r.
__device__ __forceinline__ double rcp_full(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

// ---------------------------------------------------------------------------
// bond family (Sec. 3.1) and bond removal (Sec. 6.3)
// ---------------------------------------------------------------------------

constexpr int64_t kUnbounded = ((int64_t)1) << 50;

// The notch plane cuts the segment A->B strictly inside (0 < t < 1) exactly
// when the plane function changes sign between the endpoints; the crossing
// point A + t (B - A), t = fA / (fA - fB), is tested against the bounds with
// everything multiplied by the positive denominator.
__device__ bool notch_cuts(const CutDev& c, const int64_t A[3], const int64_t B[3]) {
  const int64_t fa = c.plane[0] * A[0] + c.plane[1] * A[1] + c.plane[2] * A[2] + c.plane[3];
  const int64_t fb = c.plane[0] * B[0] + c.plane[1] * B[1] + c.plane[2] * B[2] + c.plane[3];
  if (fa == 0 || fb == 0 || ((fa < 0) == (fb < 0))) return false;
  int64_t num = fa, den = fa - fb;
  if (den < 0) {
    num = -num;
    den = -den;
  }
  for (int q = 0; q < 3; ++q) {
    const int64_t qs = A[q] * den + num * (B[q] - A[q]);
    if (c.lo[q] > -kUnbounded && qs < c.lo[q] * den) return false;
    if (c.hi[q] < kUnbounded && qs > c.hi[q] * den) return false;
  }
  return true;
}

__device__ __forceinline__ int64_t sq_dist(const int64_t A[3], const int64_t C[3]) {
  const int64_t a = A[0] - C[0], b = A[1] - C[1], d = A[2] - C[2];
  return a * a + b * b + d * d;
}

// closest point of segment A->B to the centre, all in integers
__device__ bool chord_cuts(const CutDev& c, const int64_t A[3], const int64_t B[3]) {
  int64_t D[3], W[3];
  for (int q = 0; q < 3; ++q) {
    D[q] = B[q] - A[q];
    W[q] = c.c[q] - A[q];
  }
  const int64_t dd = D[0] * D[0] + D[1] * D[1] + D[2] * D[2];
  const int64_t wd = W[0] * D[0] + W[1] * D[1] + W[2] * D[2];
  if (wd <= 0) return sq_dist(A, c.c) < c.r2;
  if (wd >= dd) return sq_dist(B, c.c) < c.r2;
  const int64_t ww = W[0] * W[0] + W[1] * W[1] + W[2] * W[2];
  return ww * dd - wd * wd < c.r2 * dd;
}

__device__ bool cut_between(const CutDev* cuts, const int32_t* cut_begin, int g, int pi, int pj) {
  const int c0 = cut_begin[g], c1 = cut_begin[g + 1];
  if (c0 == c1) return false;
  const int64_t A[3] = {2 * (int64_t)unpack_x(pi), 2 * (int64_t)unpack_y(pi), 2 * (int64_t)unpack_z(pi)};
  const int64_t B[3] = {2 * (int64_t)unpack_x(pj), 2 * (int64_t)unpack_y(pj), 2 * (int64_t)unpack_z(pj)};
  for (int k = c0; k < c1; ++k) {
    const CutDev& c = cuts[k];
    if (c.kind == 0 && notch_cuts(c, A, B)) return true;
    if (c.kind == 1 && (sq_dist(A, c.c) < c.r2 || sq_dist(B, c.c) < c.r2)) return true;
    if (c.kind == 2 && chord_cuts(c, A, B)) return true;
  }
  return false;
}

__device__ __forceinline__ bool bond_cut(const BuildArgs& b, int g, int pi, int pj) {
  return cut_between(b.cuts, b.cut_begin, g, pi, pj);
}

// node index at lattice point ijk + d of grain g, or -1
__device__ __forceinline__ int lookup(const BuildArgs& b, int g, int p, int s) {
  const int dx = (s & 255) - 8, dy = ((s >> 8) & 255) - 8, dz = ((s >> 16) & 255) - 8;
  const int lx = unpack_x(p) - b.gmap_lo[3 * g] + dx;
  const int ly = unpack_y(p) - b.gmap_lo[3 * g + 1] + dy;
  const int lz = unpack_z(p) - b.gmap_lo[3 * g + 2] + dz;
  const int ex = b.gmap_dim[3 * g], ey = b.gmap_dim[3 * g + 1], ez = b.gmap_dim[3 * g + 2];
  if (lx < 0 || ly < 0 || lz < 0 || lx >= ex || ly >= ey || lz >= ez) return -1;
  return b.gmap[b.gmap_off[g] + ((int64_t)lx * ey + ly) * ez + lz];
}

__global__ void k_map_fill(BuildArgs b) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= b.n) return;
  const double w = b.u[i].w;
  const int p = packed_ijk(w), g = packed_grain(w);
  const int lx = unpack_x(p) - b.gmap_lo[3 * g];
  const int ly = unpack_y(p) - b.gmap_lo[3 * g + 1];
  const int lz = unpack_z(p) - b.gmap_lo[3 * g + 2];
  const int ey = b.gmap_dim[3 * g + 1], ez = b.gmap_dim[3 * g + 2];
  b.gmap[b.gmap_off[g] + ((int64_t)lx * ey + ly) * ez + lz] = (int32_t)i;
}

__global__ void k_bond_count(BuildArgs b) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= b.n) return;
  const double w = b.u[i].w;
  const int p = packed_ijk(w), g = packed_grain(w);
  int cnt = 0;
  for (int k = 0; k < b.n_stencil; ++k) {
    const int j = lookup(b, g, p, b.stencil[k]);
    if (j < 0) continue;
    if (bond_cut(b, g, p, packed_ijk(b.u[j].w))) continue;
    ++cnt;
  }
  b.rowlen[i] = cnt;
}

// padded slot count (64 * widest row) of every slice
__global__ void k_slice_width(BuildArgs b) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= b.nslices) return;
  int w = 0;
  for (int l = 0; l < kWave; ++l) {
    const int64_t i = s * kWave + l;
    if (i < b.n) w = max(w, b.rowlen[i]);
  }
  w = (w + kUnroll - 1) / kUnroll * kUnroll;
  b.slice_off[s] = (int64_t)w * kWave;
}

// one wavefront per slice: write the row (stencil order), sort it ascending,
// pad it with the node itself and write the slice's padding masks
__global__ __launch_bounds__(kBlock) void k_bond_fill(BuildArgs b) {
  const int lane = threadIdx.x & 63;
  const int64_t s = (int64_t)blockIdx.x * kSlicesPerBlock + (threadIdx.x >> 6);
  if (s >= b.nslices) return;  // whole wavefront leaves together
  const int64_t i = s * kWave + lane;
  const bool valid = i < b.n;
  const int64_t off = b.slice_off[s];
  const int W = (int)((b.slice_off[s + 1] - off) / kWave);
  uint32_t* col = b.colE + off + lane;
  uint32_t* orig = b.colOrig + off + lane;
  const uint32_t node_mask = (1u << b.node_bits) - 1u;
  int len = 0;
  if (valid) {
    const double w = b.u[i].w;
    const int p = packed_ijk(w), g = packed_grain(w);
    for (int k = 0; k < b.n_stencil; ++k) {
      const int j = lookup(b, g, p, b.stencil[k]);
      if (j < 0) continue;
      if (bond_cut(b, g, p, packed_ijk(b.u[j].w))) continue;
      col[(int64_t)len * kWave] = (uint32_t)j | ((uint32_t)k << b.node_bits);
      ++len;
    }
    // insertion sort on the node index (rows come out nearly sorted)
    for (int k = 1; k < len; ++k) {
      const uint32_t x = col[(int64_t)k * kWave];
      int q = k - 1;
      while (q >= 0 && (col[(int64_t)q * kWave] & node_mask) > (x & node_mask)) {
        col[(int64_t)(q + 1) * kWave] = col[(int64_t)q * kWave];
        --q;
      }
      col[(int64_t)(q + 1) * kWave] = x;
    }
    for (int k = len; k < W; ++k) col[(int64_t)k * kWave] = (uint32_t)i | b.sentinel_hi;
  } else {
    for (int k = 0; k < W; ++k) col[(int64_t)k * kWave] = b.sentinel_hi;
  }
  for (int k = 0; k < W; ++k) orig[(int64_t)k * kWave] = col[(int64_t)k * kWave];
}

// Lined rows: the lanes of a slice hold the same class of the same stencil table at
// the same entry, and a lane that has no such bond a word with kBroken.  Each row keeps
// its order, so a node's sum is the same.  In the compact rows the lanes of nodes near a
// grain's surface run ahead of the others; lined up, the bond constants of an entry are
// the same for the wavefront and come through scalar loads, and the neighbours of nodes
// consecutive on a lattice line are consecutive.
// One wavefront per slice merges its rows: the entry at hand is the first (table, axis
// order, class) that any lane has next, classes ranked as rows of that order list them.
// Where that takes more than half as many entries again as the widest row has, the
// slice has no lined rows and keeps to the compact ones: grains of different tables or
// axis orders meet in it (twice the entries; the longest wavefront then decides a
// launch), or its nodes are in no lattice order.
template <bool FILL>
__global__ __launch_bounds__(kBlock) void k_align(AlignArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t s = (int64_t)blockIdx.x * kSlicesPerBlock + (threadIdx.x >> 6);
  if (s >= a.nslices) return;  // whole wavefront leaves together
  const int64_t i = s * kWave + lane;
  const bool valid = i < a.n;
  const int len = valid ? a.rowlen[i] : 0;
  const int64_t so = a.slice_off[s];
  const int wide = (int)((a.slice_off[s + 1] - so) / kWave);
  const int limit = wide + wide / 2;
  const uint32_t* orig = a.colOrig + so + lane;
  const uint32_t* live = a.colE + so + lane;
  const int g = valid ? packed_grain(a.u[i].w) : 0;
  const uint32_t table = (uint32_t)a.grains[g].cls * (uint32_t)(a.n_stencil + 1);
  const int order = a.axis_order[g];
  const int32_t* rank = a.axis_rank + order * a.n_stencil;
  const uint32_t first = (uint32_t)(a.grains[g].cls * 6 + order) * (uint32_t)a.n_stencil;
  const uint32_t none = (uint32_t)(s * kWave) | kBroken;
  const uint32_t node_mask = (1u << a.node_bits) - 1u;
  uint32_t* out = nullptr;
  int32_t* row = nullptr;
  int W = 0;
  if (FILL) {
    const int64_t o = a.off[s];
    W = (int)((a.off[s + 1] - o) / kWave);
    if (W == 0) return;
    out = a.lined + o + lane;
    row = a.row + o / kWave;
  }
  int k = 0, p = 0;
  uint32_t w = 0u, wn = 0u, l = 0u, ln = 0u;  // entries k and k + 1 as built and as they are now
  auto entry = [&](int q, uint32_t& o, uint32_t& e) {
    if (q >= len) return;
    o = orig[(int64_t)q * kWave];
    if (FILL) e = live[(int64_t)q * kWave];
  };
  entry(0, w, l);
  entry(1, wn, ln);
  for (;; ++p) {
    const uint32_t key = k < len ? first + (uint32_t)rank[w >> a.node_bits] : 0xffffffffu;
    uint32_t m = key;
    for (int o = 32; o > 0; o >>= 1) m = min(m, (uint32_t)__shfl_xor((int)m, o, kWave));
    if (m == 0xffffffffu || p >= (FILL ? W : limit + 1)) break;
    const bool take = key == m;
    if (FILL) {
      // a lane without this bond names the neighbour of the nearest lane that has it (a
      // lower one if there is), whose cache line is fetched anyway
      const uint64_t has = __ballot(take);
      const uint64_t below = has & ((1ull << lane) - 1ull);
      const int src = take ? lane : below ? 63 - __clzll((long long)below) : __ffsll((unsigned long long)has) - 1;
      const uint32_t j = (uint32_t)__shfl((int)(w & node_mask), src, kWave);
      out[(int64_t)p * kWave] = take && l == w ? j : j | kBroken;
      if (take) row[p] = (int32_t)((table + (w >> a.node_bits)) * (uint32_t)sizeof(StencilC));  // (all the same)
      // (entries of several tables share a class's mask, zero before)
      const uint64_t intact = __ballot(take && l == w);
      if (lane == __ffsll((unsigned long long)has) - 1)
        atomicOr((unsigned long long*)(a.live + s * a.n_stencil + (w >> a.node_bits)), (unsigned long long)intact);
    }
    if (take) {
      ++k;
      w = wn;
      l = ln;
      entry(k + 1, wn, ln);
    }
  }
  if (FILL) {
    for (; p < W; ++p) {
      out[(int64_t)p * kWave] = none;
      if (lane == 0) row[p] = 0;
    }
  } else if (lane == 0) {
    a.off[s] = p > limit ? 0 : (int64_t)((p + kBatch - 1) / kBatch * kBatch) * kWave;
  }
}

// the column words of the slices in which a bond of the lined rows broke: an entry whose
// lane bit is clear becomes a broken one
__global__ void k_lined_to_cols(AlignArgs a) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const int64_t s = i / kWave, lane = i % kWave;
  if (!a.news[s]) return;
  const int wide = (int)((a.slice_off[s + 1] - a.slice_off[s]) / kWave);
  const uint64_t* live = a.live + s * a.n_stencil;
  for (int k = 0; k < wide; k += kUnroll) {  // (padding has the class after the last)
    const int64_t at = a.slice_off[s] + (int64_t)k * kWave + lane;
    uint32_t c[kUnroll];
    uint64_t m[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) c[u] = a.colOrig[at + u * kWave] >> a.node_bits;
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) m[u] = live[c[u] < (uint32_t)a.n_stencil ? c[u] : 0u];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
      if (c[u] < (uint32_t)a.n_stencil && !((m[u] >> lane) & 1ull)) a.colE[at + u * kWave] = (uint32_t)i | a.sentinel_hi;
  }
  a.news[s] = 0;  // (by every lane of the slice's wavefront, which has read it)
}

// ---------------------------------------------------------------------------
// the fused step: bond force + break + damage, contact, walls, velocity Verlet
// ---------------------------------------------------------------------------

// contact distance exactly as p_j - p_i = (X_j - X_i) + (u_j - u_i), no contraction
__device__ __forceinline__ double contact_d2(double xj, double xi, double uj, double ui, double yj,
                                             double yi, double vj, double vi, double zj, double zi,
                                             double wj, double wi, double& dx, double& dy,
                                             double& dz) {
  dx = __dadd_rn(__dsub_rn(xj, xi), __dsub_rn(uj, ui));
  dy = __dadd_rn(__dsub_rn(yj, yi), __dsub_rn(vj, vi));
  dz = __dadd_rn(__dsub_rn(zj, zi), __dsub_rn(wj, wi));
  return __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)), __dmul_rn(dz, dz));
}

__device__ __forceinline__ double wave_sum(double x) {
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, kWave);
  return x;
}

#ifndef PD_STEP_WAVES_PER_EU
#define PD_STEP_WAVES_PER_EU 4
#endif

// g = 1 - (1 + x)^(-1/2) = x q(x).  For |x| <= kShortRange (stretches up to 0.27%, beyond the
// critical stretch of sand at the sizes meshed here, 0.17%) q is a polynomial of degree 6
// (coefficients from csrc/bond_series.py, constant term exactly 1/2, relative error about
// 1e-18).  Up to kWideRange the same polynomial's value, by then off by up to 9e-9, is
// corrected once (g_corrected); beyond, the exact form.
constexpr double kShortRange = 0.0055, kWideRange = 0.08;
// The non-trivial coefficients, highest degree first.  The tile kernel holds them in
// scalar registers, with the same arithmetic either way: as
// literals the compiler rebuilds each 64-bit constant with two moves per use.
struct PolyS {
  double c[6];
};
constexpr PolyS kPolyS{{0x1.ad0525d77783ap-3, -0x1.ce05735c7b7b0p-3, 0x1.f7fffffae5b32p-3, -0x1.17fffffd4c6e0p-2,
                         0x1.400000000000ap-2, -0x1.800000000000bp-2}};
__device__ __forceinline__ double q_short(double x, const PolyS& P) {
  double p = fma(P.c[0], x, P.c[1]);
#pragma unroll
  for (int k = 2; k < 6; ++k) p = fma(p, x, P.c[k]);
  return fma(p, x, 0.5);
}
__device__ __forceinline__ PolyS poly_in_registers() {
  PolyS P = kPolyS;
  asm volatile("" : "+v"(P.c[0]));  // (an instruction reads one scalar pair: c1, in the first)
#pragma unroll
  for (int k = 1; k < 6; ++k) asm volatile("" : "+s"(P.c[k]));
  return P;
}
// One Newton step of r = 1 - g towards (1 + x)^(-1/2): with e = 1 - (1 + x) r^2, r (1 + e/2).
// e = (2 g - x) + g (2 x - g - x g), whose first difference is exact, so that g comes out
// right to half a unit in the last place (the error left, 3/8 e^2, is 5e-18 of g at |x| =
// 0.08).  Six operations and no constants to make, where a polynomial of degree 8 (up to
// 0.02) took nine and sixteen scalar moves, 122 times over in the tile kernel: what a
// strained body fetched did not fit the instruction cache.  Random displacements of 0.6% of
// a spacing, 274,130 nodes: tiles 87 us a step instead of 117, lined rows 84 instead of
// 118; compact rows (48,900 nodes) 43 instead of 59; calm bodies as before.
__device__ __forceinline__ double g_corrected(double x, double q) {
  double g = x * q;
  asm volatile("" : "+v"(g));  // (keeps this where it is rarely taken, out of the straight code)
  const double e = fma(g, fma(-x, g, fma(2.0, x, -g)), fma(2.0, g, -x));
  return fma(e, fma(0.5, g, -0.5), g);
}

// The exact form, x / (w + sqrt(w)) with w = 1 + x taken as |y|^2 / |xi|^2: right to 6e-16
// also where a bond is compressed to a fraction of its length and 1 + x would cancel.
__device__ __forceinline__ double g_exact(double x, double yx, double yy, double yz, double inv) {
  const double w = fma(yx, yx, fma(yy, yy, yz * yz)) * inv;
  return x * rcp_full(fma(w, rsqrt_full(w), w));
}

// The fused step of one workgroup: SPB slices (one wavefront each) starting at
// slice slice_base + SPB * blk.  s_st holds the stencil tables in LDS.
// Regularised Coulomb friction (Sec. 3.3) added to f: t is the tangential
// velocity of the node relative to its partner, mu_fr = mu times the repulsive
// force density of the pair.  Slip when |t| exceeds the threshold mu_fr dt / rho:
// magnitude mu_fr against t; otherwise stick, -(rho / dt) t, which would stop t
// in one step.  The two branches agree at the threshold.
__device__ __forceinline__ void stick_slip(double mu_fr, double rho, double dt, double tx, double ty,
                                           double tz, double& fx, double& fy, double& fz) {
  const double vt = sqrt(tx * tx + ty * ty + tz * tz);
  const double k = vt > mu_fr * dt / rho ? mu_fr / vt : rho / dt;
  fx = fma(-k, tx, fx);
  fy = fma(-k, ty, fy);
  fz = fma(-k, tz, fz);
}

// ---- several walls at a corner (Sec. 4.1.1) ----
// Area and first moments (v, w) of {v > b, w > c, v^2 + w^2 < r^2}: for a
// given v the region spans w in (max(c, -s), s), s = sqrt(r^2 - v^2), which
// integrates in closed form over the pieces of the v axis where the lower end
// is c (|v| < e = sqrt(r^2 - c^2)) or -s.  Differences of squares are taken
// as (r - x)(r + x): with a fused multiply-add r*r - x*x at x = r leaves the
// rounding error of x*x, whose square root would enter at 1e-8 relative.
__device__ __forceinline__ double disk_f0(double r, double x) {
  const double q = fmax((r - x) * (r + x), 0.0);
  return 0.5 * (x * sqrt(q) + r * r * asin(fmin(1.0, fmax(-1.0, x / r))));
}
__device__ __forceinline__ double disk_f1(double r, double x) {
  const double q = fmax((r - x) * (r + x), 0.0);
  return -q * sqrt(q) * (1.0 / 3.0);
}
__device__ void disk_cut(double r, double b, double c, double& A, double& Mv, double& Mw) {
  A = Mv = Mw = 0.0;
  if (!(r > 0.0) || b >= r || c >= r) return;
  const double v0 = fmax(b, -r);
  const bool lower_c = c > -r;  // the bound w > c cuts the disk
  const double e = lower_c ? sqrt(fmax((r - c) * (r + c), 0.0)) : r;
  // piece |v| < e with lower end c (when the bound cuts), pieces e <= |v| < r with -s
  for (int k = 0; k < 3; ++k) {
    double x0, x1;
    bool with_c;
    if (!lower_c) {
      if (k != 1) continue;
      x0 = -r, x1 = r, with_c = false;
    } else if (k == 1) {
      x0 = -e, x1 = e, with_c = true;
    } else {
      if (c >= 0.0) continue;  // there -s > c: nothing outside |v| < e
      x0 = k == 0 ? -r : e, x1 = k == 0 ? -e : r, with_c = false;
    }
    x0 = fmax(x0, v0);
    if (!(x1 > x0)) continue;
    const double dA = disk_f0(r, x1) - disk_f0(r, x0), dM = disk_f1(r, x1) - disk_f1(r, x0);
    if (with_c) {
      A += dA - c * (x1 - x0);
      Mv += dM - 0.5 * c * ((x1 - x0) * (x1 + x0));
      Mw += 0.5 * ((r - c) * (r + c) * (x1 - x0) - (x1 * x1 * x1 - x0 * x0 * x0) * (1.0 / 3.0));
    } else {
      A += 2.0 * dA;
      Mv += 2.0 * dM;
    }
  }
}

// Volume and centroid (along u, v, w) of {|x| < R, u > a, v > b, w > c}
// (c = -inf: two planes).  Slices u = R cos(phi) are integrated over phi, split
// where a slice changes shape, each piece by Gauss-Legendre on a cosine map of
// the piece (gl: nodes and weights on [0, pi]), which makes the end-point
// power laws of the slice area smooth.
__device__ void corner_region(const double* gl, int ngl, double R, double a, double b, double c, double& V,
                              double& cu, double& cv, double& cw) {
  double acc0 = 0.0, acc1 = 0.0, acc2 = 0.0, acc3 = 0.0;
  const double u0 = fmax(a, -R);
  double cuts[8];
  int nc = 0;
  cuts[nc++] = u0;
  const double rr[3] = {fabs(b), fabs(c), sqrt(b * b + c * c)};
  for (int k = 0; k < 3; ++k) {
    if (!(rr[k] < R)) continue;
    const double uk = sqrt((R - rr[k]) * (R + rr[k]));
    if (uk > u0 && uk < R) cuts[nc++] = uk;
    if (-uk > u0 && -uk < R) cuts[nc++] = -uk;
  }
  cuts[nc++] = R;
  for (int i = 1; i < nc; ++i)
    for (int j = i; j > 0 && cuts[j] < cuts[j - 1]; --j) {
      const double t = cuts[j];
      cuts[j] = cuts[j - 1];
      cuts[j - 1] = t;
    }
  for (int k = 0; k + 1 < nc; ++k) {
    if (!(cuts[k + 1] > cuts[k])) continue;
    const double p0 = acos(fmin(1.0, fmax(-1.0, cuts[k + 1] / R)));
    const double p1 = acos(fmin(1.0, fmax(-1.0, cuts[k] / R)));
    const double mid = 0.5 * (p0 + p1), half = 0.5 * (p1 - p0);
    for (int q = 0; q < ngl; ++q) {
      const double th = gl[q], w = gl[ngl + q];
      const double ph = mid - half * cos(th);
      const double sp = sin(ph), u = R * cos(ph);
      const double jw = w * half * sin(th) * R * sp;
      double A, Mv, Mw;
      disk_cut(R * sp, b, c, A, Mv, Mw);
      acc0 += jw * A;
      acc1 += jw * u * A;
      acc2 += jw * Mv;
      acc3 += jw * Mw;
    }
  }
  V = acc0;
  const double inv = acc0 > 0.0 ? 1.0 / acc0 : 0.0;
  cu = acc1 * inv;
  cv = acc2 * inv;
  cw = acc3 * inv;
}

// Inclusion-exclusion over the walls the node touches (at most three taken,
// in wall order): pairs of orthogonal walls subtract, an orthogonal triple
// adds, each term -K_n (R_c - |c - p|) |S| (c - p)/|c - p| over the part S of
// the contact ball beyond all of its walls.  Wall l takes each term's
// component along its normal: corr[k] for the wall index hw[k].
__device__ void wall_corner_terms(const StepArgs& A, double Kn, const double* hd, const int* hw, int nh,
                                  double* corr) {
  bool orth[3][3];
  for (int x = 0; x < nh; ++x)
    for (int y = 0; y < nh; ++y) {
      const double* na = A.walls[hw[x]].n;
      const double* nb = A.walls[hw[y]].n;
      orth[x][y] = fabs(na[0] * nb[0] + na[1] * nb[1] + na[2] * nb[2]) < 1e-12;
    }
  // the three pairs (x, y) and, with three walls, the triple
  const int terms = nh == 3 ? 4 : 1;
  for (int t = 0; t < terms; ++t) {
    int m[3] = {0, 1, -1};
    if (t == 1) m[0] = 0, m[1] = 2;
    if (t == 2) m[0] = 1, m[1] = 2;
    if (t == 3) m[2] = 2;
    const bool triple = m[2] >= 0;
    if (!orth[m[0]][m[1]] || (triple && (!orth[m[0]][2] || !orth[m[1]][2]))) continue;
    double V, cu, cv, cw;
    corner_region(A.corner_gl, A.corner_ngl, A.Rc, hd[m[0]], hd[m[1]], triple ? hd[2] : -INFINITY, V, cu, cv, cw);
    if (!(V > 0.0)) continue;
    const double cen[3] = {cu, cv, cw};
    double cp[3] = {0.0, 0.0, 0.0};  // c - p along the outward directions -n_l
    for (int k = 0; k < (triple ? 3 : 2); ++k)
      for (int q = 0; q < 3; ++q) cp[q] -= cen[k] * A.walls[hw[m[k]]].n[q];
    const double ell = sqrt(cp[0] * cp[0] + cp[1] * cp[1] + cp[2] * cp[2]);
    if (!(ell > 0.0)) continue;
    const double f = (triple ? 1.0 : -1.0) * -Kn * (A.Rc - ell) * V / ell;
    for (int k = 0; k < (triple ? 3 : 2); ++k) {
      const double* nl = A.walls[hw[m[k]]].n;
      corr[m[k]] += f * (cp[0] * nl[0] + cp[1] * nl[1] + cp[2] * nl[2]);
    }
  }
}

// Corner corrections of every node for this evaluation: nodes touching two or
// three walls get corner_w = count | wall indices << 8 (k + 1) and their
// corrections in corner_c; the others 0.  force_only: walls at the offsets of
// the last evaluation.
__global__ void k_wall_corners(StepArgs A, int force_only) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= A.n || (!force_only && halted(A.halt))) return;
  const double4 ui = A.ucur[i];
  const GrainC* G = A.grains + packed_grain(ui.w);
  const int p = packed_ijk(ui.w);
  const double px = lattice_pos(G->origin[0], G->h, unpack_x(p)) + ui.x;
  const double py = lattice_pos(G->origin[1], G->h, unpack_y(p)) + ui.y;
  const double pz = lattice_pos(G->origin[2], G->h, unpack_z(p)) + ui.z;
  int hw[3];
  double hd[3];
  int nh = 0;
  for (int w = 0; w < A.n_walls && nh < 3; ++w) {
    const WallDev* Wd = A.walls + w;
    const bool in = px >= Wd->lo[0] && px <= Wd->hi[0] && py >= Wd->lo[1] && py <= Wd->hi[1] &&
                    pz >= Wd->lo[2] && pz <= Wd->hi[2];
    const double o = force_only ? Wd->off_used : Wd->off;
    const double d = Wd->n[0] * px + Wd->n[1] * py + Wd->n[2] * pz - o;
    if (in && d < A.Rc && d > -A.Rc) {
      hw[nh] = w;
      hd[nh] = d;
      ++nh;
    }
  }
  uint32_t pw = 0u;
  if (nh >= 2) {
    double corr[3] = {0.0, 0.0, 0.0};
    wall_corner_terms(A, A.Kn[G->mat * A.n_mat + G->mat], hd, hw, nh, corr);
    pw = (uint32_t)nh;
    for (int k = 0; k < nh; ++k) {
      pw |= (uint32_t)hw[k] << (8 * (k + 1));
      A.corner_c[3 * i + k] = corr[k];
    }
  }
  A.corner_w[i] = pw;
}

// Everything after the bond sum for the node of this lane: contact with other
// grains, damping and friction (Secs. 3.2-3.4), rigid walls (Sec. 4.1) with the
// wavefront's reaction partial in wall_partial column col (written when col_ok),
// and velocity Verlet (Sec. 6.2).  Every lane of the wavefront takes part (the
// wall partials are wavefront sums); lanes without a node pass valid = false.
// The node's velocity and previous acceleration, read by the Verlet update.
struct NodeVA {
  double vx, vy, vz, ax, ay, az;
};
__device__ __forceinline__ NodeVA load_va(const StepArgs& A, int64_t i, bool valid) {
  NodeVA r{0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  if (valid) {
    r.vx = A.v[i];
    r.vy = A.v[A.n + i];
    r.vz = A.v[2 * A.n + i];
    r.ax = A.a[i];
    r.ay = A.a[A.n + i];
    r.az = A.a[2 * A.n + i];
  }
  return r;
}

// Is the bond from node i to node j (same grain) intact after this evaluation's
// breaks?  The node's built entries are sorted by neighbour index, so a binary
// search finds j's entry; a pair with no entry (outside the horizon, or cut)
// has no bond.  The bond memory is the live column word on the compact rows
// (path = kInCols) and, on the tiled path, the node's lane bit in the lane mask of
// its class in the grain's axis order path (the tile kernel stores a class's
// mask as soon as a bond of it breaks, before any node's tail).
constexpr int kInCols = -1, kInLined = -2;
__device__ __forceinline__ bool bond_intact(const StepArgs& A, int64_t i, int j, int path) {
  const uint32_t node_mask = (1u << A.node_bits) - 1u;
  const int64_t base = A.slice_off[i >> 6] + (i & 63);
  int lo = 0, hi = A.rowlen[i] - 1;
  while (lo <= hi) {
    const int mid = (lo + hi) >> 1;
    const int64_t at = base + ((int64_t)mid << 6);
    const uint32_t wo = A.colOrig[at];
    const int jm = (int)(wo & node_mask);
    if (jm < j) {
      lo = mid + 1;
    } else if (jm > j) {
      hi = mid - 1;
    } else {
      if (path < 0) return A.colE[at] == wo;
      const int b = A.ctob[path * A.n_stencil + (int)(wo >> A.node_bits)];
      const int32_t sl = A.slot[i];
      return ((A.lmask[(int64_t)(sl >> 6) * kTileClasses + b] >> (sl & 63)) & 1ull) != 0ull;
    }
  }
  return false;
}

// The same for a slice with lined rows: the lattice offset from pi to pj (packed) names the
// class, whose lane mask of intact bonds the slice keeps.  (The bond loop takes breaks
// from the masks by atomics; the load is one as well, past the first-level cache.)
__device__ __forceinline__ bool bond_intact_lined(const StepArgs& A, int64_t i, int pi, int pj) {
  const int m = A.m, w = 2 * m + 1;
  const int x = unpack_x(pj) - unpack_x(pi) + m, y = unpack_y(pj) - unpack_y(pi) + m, z = unpack_z(pj) - unpack_z(pi) + m;
  if (min(min(x, y), z) < 0 || max(max(x, y), z) >= w) return false;
  const int k = A.offset_class[(x * w + y) * w + z];
  if (k < 0) return false;
  const uint64_t live = __hip_atomic_load(A.lined_live + (i >> 6) * A.n_stencil + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return (live >> (i & 63)) & 1ull;
}

// Repulsion of node j on node i when closer than R_c (Sec. 3.2), with normal
// damping (Sec. 3.4) and stick-slip friction (Sec. 3.3): between grains, and
// between nodes of one grain without an intact bond (Sec. 5, where c_w / R_c
// is the same K_n; self-contact needs R_c below the lattice spacing, so the
// repulsive-only bond of pairs shorter than R_c never arises).
// uj and Xj are the partner's displacement and reference position.
template <bool EXTRA>
__device__ __forceinline__ void contact_pair(const StepArgs& A, int64_t i, int j, bool listed, const double4& uj,
                                             const double4& Xj, const double4& Xi, const double4& ui,
                                             const double4& vhi, int mi, double rho_i, bool damp, bool fric,
                                             int path, double& fx, double& fy, double& fz) {
  double yx, yy, yz;
  const double d2 = contact_d2(Xj.x, Xi.x, uj.x, ui.x, Xj.y, Xi.y, uj.y, ui.y, Xj.z, Xi.z, uj.z, ui.z, yx, yy, yz);
  if (listed && d2 < A.Rc2 && d2 > 0.0) {
    // a node of the same grain repels only while no intact bond joins the two
    if (EXTRA && A.self_contact && packed_grain(uj.w) == packed_grain(ui.w) &&
        (path == kInLined ? bond_intact_lined(A, i, packed_ijk(ui.w), packed_ijk(uj.w)) : bond_intact(A, i, j, path)))
      return;
    // where all grains are alike their constants are kernel arguments, not loads
    // behind the partner's
    double Kn = A.one.Kn, Vj = A.one.V;
    if (!A.alike) {
      const GrainC* Gj = A.grains + packed_grain(uj.w);
      Kn = A.Kn[mi * A.n_mat + Gj->mat];
      Vj = Gj->V;
    }
    const double d = sqrt(d2);
    const double rep = Kn * (A.Rc - d) * Vj;
    double coef = -rep / d;
    double4 vhj = make_double4(0.0, 0.0, 0.0, 0.0);
    if (damp || fric) vhj = A.vh_cur[j];
    const double wx = vhi.x - vhj.x, wy = vhi.y - vhj.y, wz = vhi.z - vhj.z;
    if (damp) {
      // -beta (w . e) e V_j, w = velocity of i relative to j, e = y / d
      const double w = wx * yx + wy * yy + wz * yz;
      coef -= A.beta * Vj * w / d2;
    }
    fx = fma(coef, yx, fx);
    fy = fma(coef, yy, fy);
    fz = fma(coef, yz, fz);
    if (fric) {
      // tangential part of w against the repulsive force density rep
      const double inv_d = 1.0 / d;
      const double ex = yx * inv_d, ey = yy * inv_d, ez = yz * inv_d;
      const double wn = wx * ex + wy * ey + wz * ez;
      stick_slip(A.mu * rep, rho_i, A.dt, wx - wn * ex, wy - wn * ey, wz - wn * ez, fx, fy, fz);
    }
  }
}

// x / rho with r the rounded reciprocal of rho: the product corrected by its
// residual, which rounds as the division does but for rare last places, in three
// operations instead of a dozen (finite x)
__device__ __forceinline__ double over_rho(double x, double rho, double r) {
  const double q = x * r;
  return fma(fma(-rho, q, x), r, q);
}

// A wall's fields for one evaluation: through the constant address space (scalar
// loads, all walls' in flight together) in kernels during which no wall changes,
// else as ordinary loads.
struct WallIn {
  double n[3], off, rate, lo[3], hi[3];
};
template <bool SCALAR, bool USED>
__device__ __forceinline__ WallIn wall_in(const WallDev* walls, int w) {
  WallIn r;
  auto take = [&](auto* W) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      r.n[q] = W->n[q];
      r.lo[q] = W->lo[q];
      r.hi[q] = W->hi[q];
    }
    r.off = USED ? W->off_used : W->off;
    r.rate = USED ? W->rate_used : W->rate;
  };
  if constexpr (SCALAR) take((const __attribute__((address_space(4))) WallDev*)(walls + w));
  else take(walls + w);
  return r;
}

// EXTRA = false compiles out self-contact and the wall-corner corrections (the
// tiled kernel's variant for runs with neither); SCALAR_WALLS: see wall_in; SPLIT
// also writes the split copy of u.
// Bound by the latency of its dependent loads, so none of them sits behind a
// branch that another one could have been issued before (the compiler waits for
// every outstanding load where branches join).
template <int MODE, bool EXTRA, bool SCALAR_WALLS, bool SPLIT>
__device__ __forceinline__ void node_tail(const StepArgs& A, int64_t i, bool valid, const double4& ui,
                                          const GrainC* G, int ix, int iy, int iz, double fx, double fy,
                                          double fz, int nbroke, bool col_ok, int64_t col, const NodeVA& va,
                                          int path) {
  const int lane = threadIdx.x & 63;
  // mid-step velocity of this node for the normal damping (Sec. 3.4) and
  // stick-slip friction (Sec. 3.3) laws
  const bool damp = A.beta > 0.0, fric = A.mu > 0.0, vdep = damp || fric;
  const int64_t il = valid ? i : 0;
  double4 vhi = make_double4(0.0, 0.0, 0.0, 0.0);
  if (vdep) vhi = A.vh_cur[il];
  const double ox = G->origin[0], oy = G->origin[1], oz = G->origin[2];
  GrainOne own = A.one;
  int mi = 0;
  if (!A.alike) {
    mi = G->mat;
    own = GrainOne{G->h, G->V, G->rho, G->inv_rho, A.Kn[mi * A.n_mat + mi]};
  }

  // ---- repulsive contact with the candidates: nodes of other grains and, with
  // self-contact, of the same grain (Secs. 3.2, 5) ----
  if (A.cand_ptr != nullptr) {
    // rows past the capacity were not stored (the rebuild flagged it)
    const int32_t c0 = (int32_t)min((int64_t)A.cand_ptr[il], A.cand_capacity);
    const int32_t c1 = valid ? (int32_t)min((int64_t)A.cand_ptr[il + 1], A.cand_capacity) : c0;
    if (c1 > c0) {
      // keep the candidate gathers here: hoisted above the bond loop they
      // would hold their registers through it
      asm volatile("" ::: "memory");
      const double4 Xi = A.X4[i];
      // kContactBatch candidates at a time: their u and reference positions, and
      // the next batch's indices, are all in flight before the first pair is
      // evaluated (past the row's end its last candidate is read again); the
      // pairs are still added in row order
      int jn[kContactBatch];
#pragma unroll
      for (int k = 0; k < kContactBatch; ++k) jn[k] = A.cand[c0 + k < c1 ? c0 + k : c1 - 1];
      for (int32_t e = c0; e < c1; e += kContactBatch) {
        int jj[kContactBatch];
        double4 uj[kContactBatch], Xj[kContactBatch];
#pragma unroll
        for (int k = 0; k < kContactBatch; ++k) {
          jj[k] = jn[k];
          uj[k] = A.ucur[jj[k]];
          const double* xp = reinterpret_cast<const double*>(A.X4 + jj[k]);
          Xj[k] = make_double4(xp[0], xp[1], xp[2], 0.0);
        }
#pragma unroll
        for (int k = 0; k < kContactBatch; ++k) {
          const int32_t en = e + kContactBatch + k;
          jn[k] = A.cand[en < c1 ? en : c1 - 1];
        }
#pragma unroll
        for (int k = 0; k < kContactBatch; ++k)
          contact_pair<EXTRA>(A, i, jj[k], e + k < c1, uj[k], Xj[k], Xi, ui, vhi, mi, own.rho, damp, fric, path, fx,
                              fy, fz);
      }
    }
  }

  // ---- several walls at a corner (Sec. 4.1.1): the corrections of the normal
  // magnitudes that k_wall_corners left for this node (at most three walls) ----
  const uint32_t corner_pw = (EXTRA && A.wall_corners && valid) ? A.corner_w[i] : 0u;

  // ---- rigid walls: spherical-cap law (Sec. 4.1), walls summed.  One partial per
  // slice (wavefront) and wall it touches, component-major, and a byte that says
  // which: the finalize sums them in slice order, whatever the workgroup size or
  // launch split ----
  const double px = lattice_pos(ox, own.h, ix) + ui.x;
  const double py = lattice_pos(oy, own.h, iy) + ui.y;
  const double pz = lattice_pos(oz, own.h, iz) + ui.z;
  uint32_t touched = 0u;
  for (int w = 0; w < A.n_walls; ++w) {
    const WallIn Wd = wall_in<SCALAR_WALLS, MODE == MODE_FORCE_ONLY>(A.walls, w);
    const double d = Wd.n[0] * px + Wd.n[1] * py + Wd.n[2] * pz - Wd.off;
    const bool in = valid & (px >= Wd.lo[0]) & (px <= Wd.hi[0]) & (py >= Wd.lo[1]) & (py <= Wd.hi[1]) &
                    (pz >= Wd.lo[2]) & (pz <= Wd.hi[2]) & (d < A.Rc);
    if (__ballot(in) == 0ull) continue;
    bool hit = false;
    double mag = 0.0, ftx = 0.0, fty = 0.0, ftz = 0.0;  // normal magnitude, friction
    if (in) {
      if (d <= -A.Rc) {
        if (MODE != MODE_FORCE_ONLY) atomicOr(A.status, ST_PENETRATION);
      } else {
        // cap of the contact ball beyond the wall: height Rc - d, volume
        // (pi/3)(Rc-d)^2(2Rc+d); its centroid lies 3(Rc+d)^2/(4(2Rc+d)) from p
        const double H = A.Rc - d, q = 2.0 * A.Rc + d;
        const double vol = (M_PI / 3.0) * H * H * q;
        const double ell = 0.75 * (A.Rc + d) * (A.Rc + d) / q;
        const double rep = own.Kn * (A.Rc - ell) * vol;
        mag = rep;
        if (EXTRA) {
#pragma unroll
          for (int k = 0; k < 3; ++k)
            if ((int)(corner_pw & 3u) > k && (int)((corner_pw >> (8 * (k + 1))) & 255u) == w)
              mag += A.corner_c[3 * i + k];
        }
        if (damp) {
          // damping against the wall: relative normal velocity v . n - wall rate
          const double vn = Wd.n[0] * vhi.x + Wd.n[1] * vhi.y + Wd.n[2] * vhi.z;
          mag -= A.beta * (vn - Wd.rate) * vol;
        }
        if (fric) {
          // the wall moves along its normal only: friction sees v's tangential part
          const double wx = vhi.x - Wd.rate * Wd.n[0], wy = vhi.y - Wd.rate * Wd.n[1],
                       wz = vhi.z - Wd.rate * Wd.n[2];
          const double wn = wx * Wd.n[0] + wy * Wd.n[1] + wz * Wd.n[2];
          stick_slip(A.mu * rep, own.rho, A.dt, wx - wn * Wd.n[0], wy - wn * Wd.n[1],
                     wz - wn * Wd.n[2], ftx, fty, ftz);
        }
        hit = true;
      }
    }
    if (hit) {
      fx = fma(mag, Wd.n[0], fx) + ftx;
      fy = fma(mag, Wd.n[1], fy) + fty;
      fz = fma(mag, Wd.n[2], fz) + ftz;
    }
    if (MODE != MODE_FORCE_ONLY && __ballot(hit) != 0ull) {
      const double vm = hit ? own.V * mag : 0.0, vf = hit ? own.V : 0.0;
      const double r0 = wave_sum(fma(vf, ftx, vm * Wd.n[0]));
      const double r1 = wave_sum(fma(vf, fty, vm * Wd.n[1]));
      const double r2 = wave_sum(fma(vf, ftz, vm * Wd.n[2]));
      touched |= 1u << w;
      if (lane == 0 && col_ok) {
        A.wall_partial[(int64_t)(3 * w) * A.partial_stride + col] = r0;
        A.wall_partial[(int64_t)(3 * w + 1) * A.partial_stride + col] = r1;
        A.wall_partial[(int64_t)(3 * w + 2) * A.partial_stride + col] = r2;
      }
    }
  }
  if (MODE != MODE_FORCE_ONLY && A.n_walls > 0 && lane == 0 && col_ok) A.wall_touched[col] = (uint8_t)touched;

  // ---- velocity Verlet (Sec. 6.2) and stores ----
  if (MODE == MODE_FORCE_ONLY) {
    if (valid) {
      A.Fout[i] = fx;
      A.Fout[A.n + i] = fy;
      A.Fout[2 * A.n + i] = fz;
    }
  } else {
    const bool bad = valid && !(isfinite(fx) && isfinite(fy) && isfinite(fz));
    const double dt = A.dt, hdt = 0.5 * dt, hdt2 = 0.5 * dt * dt;
    double anx = over_rho(fx, own.rho, own.inv_rho) + A.g[0];
    double any = over_rho(fy, own.rho, own.inv_rho) + A.g[1];
    double anz = over_rho(fz, own.rho, own.inv_rho) + A.g[2];
    if (__ballot(bad) != 0ull) {
      if (bad) {
        atomicOr(A.status, ST_NAN);
        anx = fx / own.rho + A.g[0];
        any = fy / own.rho + A.g[1];
        anz = fz / own.rho + A.g[2];
      }
    }
    const bool fixed = A.fixed != nullptr && A.fixed[il] != 0;
    if (valid) {
      if (fixed) anx = any = anz = 0.0;
      double vx = va.vx, vy = va.vy, vz = va.vz;
      if (MODE == MODE_STEP) {
        vx = fixed ? 0.0 : fma(hdt, va.ax + anx, vx);
        vy = fixed ? 0.0 : fma(hdt, va.ay + any, vy);
        vz = fixed ? 0.0 : fma(hdt, va.az + anz, vz);
      } else if (fixed) {
        vx = vy = vz = 0.0;
      }
      A.v[i] = vx;
      A.v[A.n + i] = vy;
      A.v[2 * A.n + i] = vz;
      A.a[i] = anx;
      A.a[A.n + i] = any;
      A.a[2 * A.n + i] = anz;
      // positions of the next step: u + dt v + dt^2/2 a
      double4 un = ui;
      if (!fixed) {
        un.x = fma(hdt2, anx, fma(dt, vx, ui.x));
        un.y = fma(hdt2, any, fma(dt, vy, ui.y));
        un.z = fma(hdt2, anz, fma(dt, vz, ui.z));
      }
      A.unext[i] = un;
      if (SPLIT) {
        A.uxy_next[i] = make_double2(un.x, un.y);
        A.uz_next[i] = un.z;
      }
      if (vdep) {
        // the next evaluation's damping and friction see v_{n+1} + dt/2 a_{n+1}
        A.vh_next[i] = fixed ? make_double4(0.0, 0.0, 0.0, 0.0)
                             : make_double4(fma(hdt, anx, vx), fma(hdt, any, vy), fma(hdt, anz, vz), 0.0);
      }
      if (nbroke) A.intact[i] -= nbroke;
    }
  }
}

// The bond sum of a slice over the compact rows, their tables in LDS.
template <int MODE, bool ABS, int DEPTH>
__device__ __forceinline__ void bonds_compact(const StepArgs& A, const StencilC* s_st, int64_t slice, bool slice_ok,
                                              int64_t i, int lane, bool valid, const double4& ui, const GrainC* G,
                                              double& fx, double& fy, double& fz, int& nbroke) {
  const double thr_x = G->thr_x, lo_x = G->lo_x;
  const uint32_t node_mask = (1u << A.node_bits) - 1u;
  const int node_bits = A.node_bits;

  // ---- peridynamic bonds with bond memory ----
  // A row is taken kBatch entries at a time (slice widths are multiples of it), as
  // a pipeline: while batch b computes, the neighbours of the next DEPTH - 1
  // batches are being gathered and the column words of as many more are being
  // read.  A gather's latency is then hidden behind other wavefronts' and its
  // own wavefront's arithmetic.  Uneven aggregate of 125,000 nodes: 43 us a launch,
  // 69 us with 8 entries gathered and then computed; 8,338 nodes (one wavefront a
  // SIMD): 23 us against 40 (27 with the rare forms in line: nothing hides a taken branch).  The loads are issued without a branch (past the
  // row's end the last batch is read again).  Broken bonds and padding carry the
  // zero-force class and point at the node itself, so every entry is evaluated
  // the same way.
  //
  // Bond law (Sec. 3.1): the force on i is c s V_j y/|y|, y = xi + eta, and
  //   c V s / |y| = (c V / |xi|) g,   g = 1 - |xi|/|y| = 1 - (1 + x)^(-1/2),
  //   x = (|y|^2 - |xi|^2) / |xi|^2,   |y|^2 - |xi|^2 = eta . (2 xi + eta).
  // g comes from a polynomial, corrected past kShortRange, when |x| <= kWideRange (no
  // square root or division), else from g = (|y|^2 - |xi|^2) / (|y| (|y| + |xi|)), over
  // |xi|^2; no form subtracts nearly equal numbers.  The bond breaks when s > s0, which is x >
  // (1 + s0)^2 - 1.  The form is chosen per lane, so any grouping of bonds (the
  // tiled path) computes the same values.
  int64_t off = 0;
  int W = 0;
  if (slice_ok) {
    off = A.slice_off[slice];
    W = (int)((A.slice_off[slice + 1] - off) >> 6);
  }
  uint32_t* cp = A.colE + off + lane;
  const char* ubase = reinterpret_cast<const char*>(A.ucur);
  const char* tbase = reinterpret_cast<const char*>(s_st) +
                      (uint32_t)G->cls * (uint32_t)(A.n_stencil + 1) * (uint32_t)sizeof(StencilC);
  const uint32_t mine = (uint32_t)(valid ? i : 0) | A.sentinel_hi;
  constexpr int CR = 2 * DEPTH;  // batches of column words held
  uint32_t cw[CR][kBatch];
  double ux[DEPTH][kBatch], uy[DEPTH][kBatch], uz[DEPTH][kBatch];
  const int nb = W / kBatch;
  const PolyS P = poly_in_registers();
  auto columns = [&](int b, uint32_t (&c)[kBatch]) {
    const uint32_t* q = cp + (b < nb ? b : nb - 1) * (kBatch * kWave);
#pragma unroll
    for (int u = 0; u < kBatch; ++u) c[u] = q[u * kWave];
  };
  auto gather = [&](const uint32_t (&c)[kBatch], int r) {
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const double* q = reinterpret_cast<const double*>(ubase + ((c[u] & node_mask) << 5));
      ux[r][u] = q[0];
      uy[r][u] = q[1];
      uz[r][u] = q[2];
    }
  };
  auto row_of = [&](uint32_t c) {
    return *reinterpret_cast<const StencilC*>(tbase + (c >> node_bits) * (uint32_t)sizeof(StencilC));
  };
  auto batch = [&](int b, uint32_t (&c)[kBatch], int r) {
    StencilC S = row_of(c[0]);
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      StencilC Sn = S;
      if (u + 1 < kBatch) Sn = row_of(c[u + 1]);
      const double ex = ux[r][u] - ui.x, ey = uy[r][u] - ui.y, ez = uz[r][u] - ui.z;
      const double yx = S.hx + ex, yy = S.hy + ey, yz = S.hz + ez;  // y = xi + eta
      // |y|^2 - |xi|^2 = eta . (2 xi + eta)
      const double d = fma(ex, fma(2.0, S.hx, ex), fma(ey, fma(2.0, S.hy, ey), ez * fma(2.0, S.hz, ez)));
      const double x = d * S.inv_l0sq;
      bool over = x > thr_x;
      if (ABS) over = over || x < lo_x;
      const double q = q_short(x, P);
      double coef = (S.civ * x) * q;
      const bool far = !(fabs(x) <= kShortRange);
      if (__builtin_expect(__ballot(far) != 0ull, 0)) {
        const bool exact = !(fabs(x) <= kWideRange);
        double g = g_corrected(x, q);
        if (__builtin_expect(__ballot(exact) != 0ull, 0)) g = exact ? g_exact(x, yx, yy, yz, S.inv_l0sq) : g;
        coef = far ? S.civ * g : coef;
      }
      coef = over ? 0.0 : coef;
      fx = fma(coef, yx, fx);
      fy = fma(coef, yy, fy);
      fz = fma(coef, yz, fz);
      if (__builtin_expect(MODE != MODE_FORCE_ONLY && __ballot(over && valid) != 0ull, 0)) {
        if (over && valid) {
          cp[(b * kBatch + u) * kWave] = mine;  // the bond stays broken from now on
          ++nbroke;
        }
      }
      S = Sn;
      // materialise the running sums: left alone, the compiler sinks every entry's
      // additions to the end and keeps all of their terms in registers
      asm volatile("" : "+v"(fx), "+v"(fy), "+v"(fz));
    }
  };
  if (W > 0) {
#pragma unroll
    for (int b = 0; b < CR - 1; ++b) columns(b, cw[b]);
#pragma unroll
    for (int b = 0; b < DEPTH - 1; ++b) gather(cw[b], b);
    for (int b0 = 0; b0 < nb; b0 += CR) {
#pragma unroll
      for (int r = 0; r < CR; ++r) {
        if (b0 + r >= nb) break;
        columns(b0 + r + CR - 1, cw[(r + CR - 1) % CR]);
        gather(cw[(r + DEPTH - 1) % CR], (r + DEPTH - 1) % DEPTH);
        batch(b0 + r, cw[r], r % DEPTH);
      }
    }
  }
}

// f += coef y on the lanes of the scalar mask m, which needs no selection of coef:
// lanes whose bond is gone (or breaks) are switched off for the three additions
__device__ __forceinline__ void add_on_lanes(uint64_t m, double coef, double yx, double yy, double yz, double& fx,
                                             double& fy, double& fz) {
  uint64_t saved;
  asm volatile(
      "s_and_saveexec_b64 %3, %4\n\t"
      "v_fma_f64 %0, %5, %6, %0\n\t"
      "v_fma_f64 %1, %5, %7, %1\n\t"
      "v_fma_f64 %2, %5, %8, %2\n\t"
      "s_mov_b64 exec, %3"
      : "+v"(fx), "+v"(fy), "+v"(fz), "=&s"(saved)
      : "s"(m), "v"(coef), "v"(yx), "v"(yy), "v"(yz)
      : "scc");
}

// Tables read through the constant address space: they are the same for the
// whole wavefront (and change in no launch that reads them), so these become
// scalar loads.
typedef const __attribute__((address_space(4))) StencilC* TileTab;
typedef int Rows4 __attribute__((ext_vector_type(4)));
static_assert(kBatch == 4, "a batch's table rows come with one load");

__device__ __forceinline__ bool lined_up(const StepArgs& A, int64_t slice) {
  return A.lined_off[slice + 1] != A.lined_off[slice];
}

// The bond sum of a slice over its lined rows: the arithmetic and the order of
// bonds_compact, with the entry's constants in scalar registers (an entry ahead) and
// its live lanes in a lane mask.  Pipelined like it.  The vector cache bounds it, at one
// 64-byte line a cycle: 60 lines an entry, 102 over compact rows (u as (x, y) and z, so
// that a line holds four and eight nodes instead of two: 66 instead of 78; lanes
// without the bond reading a neighbour's line: 60 instead of 66).  523,690 nodes in 125
// spheres: 149 us a launch instead of 204.
// A break is one store and, for the wavefront, one atomic on the class's mask; the compact
// rows follow when something reads them.  Written to both by the step, through a search of
// the compact row, the breaks of a collision at 50 m/s (274,130 nodes) took a step from 110
// to 170 us (compact rows 121, now 92 to 101).
template <int MODE, bool ABS, int DEPTH>
__device__ __forceinline__ void bonds_lined(const StepArgs& A, int64_t slice, int64_t i, int lane, bool valid,
                                            const double4& ui, const GrainC* G, double& fx, double& fy,
                                            double& fz, int& nbroke) {
  const int64_t off = A.lined_off[slice];
  const int W = (int)((A.lined_off[slice + 1] - off) >> 6);
  const int nb = W / kBatch;
  const double thr_x = G->thr_x, lo_x = G->lo_x;
  uint32_t* cp = A.lined + off + lane;
  const int32_t* rows = A.lined_row + (off >> 6);
  const char* xybase = reinterpret_cast<const char*>(A.uxy);
  const char* zbase = reinterpret_cast<const char*>(A.uz);
  const char* tbase = reinterpret_cast<const char*>(A.stencil);
  const uint64_t mine = __ballot(valid);
  constexpr int CR = 2 * DEPTH;  // batches of column words held
  uint32_t cw[CR][kBatch];
  double ux[DEPTH][kBatch], uy[DEPTH][kBatch], uz[DEPTH][kBatch];
  const PolyS P = poly_in_registers();
  auto columns = [&](int b, uint32_t (&c)[kBatch]) {
    const uint32_t* q = cp + (b < nb ? b : nb - 1) * (kBatch * kWave);
#pragma unroll
    for (int u = 0; u < kBatch; ++u) c[u] = q[u * kWave];
  };
  auto gather = [&](const uint32_t (&c)[kBatch], int r) {
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const double2 q = *reinterpret_cast<const double2*>(xybase + (c[u] << 4));  // (drops the flags)
      ux[r][u] = q.x;
      uy[r][u] = q.y;
      uz[r][u] = *reinterpret_cast<const double*>(zbase + (c[u] << 3));
    }
  };
  struct RowK {
    double hx, hy, hz, inv, civ;
  };
  // the places of the first 128 entries' table rows, across the lanes (every wait for a
  // scalar load is a wait for all of them, and these would miss the caches)
  const int32_t r0 = rows[lane < W ? lane : W - 1], r1 = rows[lane + kWave < W ? lane + kWave : W - 1];
  auto list = [&](int b) {
    if (b < 2 * kWave / kBatch) {
      const int32_t r = b < kWave / kBatch ? r0 : r1;
      const int l = b % (kWave / kBatch) * kBatch;
      return Rows4{__builtin_amdgcn_readlane(r, l), __builtin_amdgcn_readlane(r, l + 1),
                   __builtin_amdgcn_readlane(r, l + 2), __builtin_amdgcn_readlane(r, l + 3)};
    }
    const int32_t* p = rows + (b < nb ? b : nb - 1) * kBatch;
    asm volatile("" : "+s"(p));  // (keeps the load here)
    return *(const __attribute__((address_space(4))) Rows4*)p;
  };
  auto row_at = [&](int at) {
    const char* p = tbase + at;
    asm volatile("" : "+s"(p));  // (keeps the loads here)
    const TileTab t = (TileTab)p;
    return RowK{t->hx, t->hy, t->hz, t->inv_l0sq, t->civ};
  };
  Rows4 rc, rn = list(0);
  RowK S = row_at(rn[0]);
  auto batch = [&](int b, const uint32_t (&c)[kBatch], int r) {
    rc = rn;
    rn = list(b + 1);
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const double ex = ux[r][u] - ui.x, ey = uy[r][u] - ui.y, ez = uz[r][u] - ui.z;
      const double yx = S.hx + ex, yy = S.hy + ey, yz = S.hz + ez;  // y = xi + eta
      // |y|^2 - |xi|^2 = eta . (2 xi + eta)
      const double d = fma(ex, fma(2.0, S.hx, ex), fma(ey, fma(2.0, S.hy, ey), ez * fma(2.0, S.hz, ez)));
      const double x = d * S.inv;
      bool over = x > thr_x;
      if (ABS) over = over || x < lo_x;
      const double inv = S.inv, civ = S.civ, cx = civ * x;
      S = row_at(u + 1 < kBatch ? rc[(u + 1) % kBatch] : rn[0]);
      const double q = q_short(x, P);
      double coef = cx * q;
      const uint64_t live = __ballot((int32_t)c[u] >= 0);
      const bool far = !(fabs(x) <= kShortRange);
      if (__builtin_expect((__ballot(far) & live) != 0ull, 0)) {
        const bool exact = !(fabs(x) <= kWideRange);
        double g = g_corrected(x, q);
        if (__builtin_expect((__ballot(exact) & live) != 0ull, 0)) g = exact ? g_exact(x, yx, yy, yz, inv) : g;
        coef = far ? civ * g : coef;
      }
      const uint64_t ov = __ballot(over);
      add_on_lanes(live & ~ov, coef, yx, yy, yz, fx, fy, fz);
      if (__builtin_expect(MODE != MODE_FORCE_ONLY && (live & ov & mine) != 0ull, 0)) {
        if (over && valid && (int32_t)c[u] >= 0) {
          cp[(b * kBatch + u) * kWave] = c[u] | kBroken;  // the bond stays broken from now on
          ++nbroke;
        }
        // and in its class's mask, by atomics: lanes of another table share it
        const uint32_t k = (uint32_t)rc[u] / (uint32_t)sizeof(StencilC) % (uint32_t)(A.n_stencil + 1);
        if (lane == 0) {
          __hip_atomic_fetch_and(A.lined_live + slice * A.n_stencil + k, ~(live & ov & mine), __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
          A.lined_news[slice] = 1;
        }
      }
    }
  };
#pragma unroll
  for (int b = 0; b < CR - 1; ++b) columns(b, cw[b]);
#pragma unroll
  for (int b = 0; b < DEPTH - 1; ++b) gather(cw[b], b);
  for (int b0 = 0; b0 < nb; b0 += CR) {
#pragma unroll
    for (int r = 0; r < CR; ++r) {
      if (b0 + r >= nb) break;
      columns(b0 + r + CR - 1, cw[(r + CR - 1) % CR]);
      gather(cw[(r + DEPTH - 1) % CR], (r + DEPTH - 1) % DEPTH);
      batch(b0 + r, cw[r], r % DEPTH);
    }
  }
}

template <int MODE, bool ABS, int SPB, int DEPTH, bool SCALAR_WALLS, bool LINED>
__device__ __forceinline__ void step_body(const StepArgs& A, const StencilC* s_st, int64_t blk) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  const int64_t slice = A.slice_base + blk * SPB + wid;
  const bool slice_ok = slice < A.slice_end;
  const int64_t i = slice * kWave + lane;
  const bool valid = slice_ok && i >= A.node_lo && i < A.node_hi;

  double4 ui = make_double4(0.0, 0.0, 0.0, 0.0);
  if (valid) ui = A.ucur[i];
  const int pi = packed_ijk(ui.w);
  const GrainC* G = A.grains + (valid ? packed_grain(ui.w) : 0);
  double fx = 0.0, fy = 0.0, fz = 0.0;
  int nbroke = 0;
  const bool lined = LINED && slice_ok && lined_up(A, slice);
  if (lined)
    bonds_lined<MODE, ABS, DEPTH>(A, slice, i, lane, valid, ui, G, fx, fy, fz, nbroke);
  else
    bonds_compact<MODE, ABS, DEPTH>(A, s_st, slice, slice_ok, i, lane, valid, ui, G, fx, fy, fz, nbroke);
  node_tail<MODE, true, SCALAR_WALLS, LINED>(A, i, valid, ui, G, unpack_x(pi), unpack_y(pi), unpack_z(pi), fx, fy, fz, nbroke,
                                      slice_ok, A.partial_base + (slice - A.slice_base), load_va(A, i, valid),
                                      lined ? kInLined : kInCols);
}

__device__ __forceinline__ void stage_stencil(const StepArgs& A, StencilC* s_st) {
  const int rows = A.n_classes * (A.n_stencil + 1);
  for (int k = threadIdx.x; k < rows; k += blockDim.x) s_st[k] = A.stencil[k];
  __syncthreads();
}

// DEPTH 2 in 128 registers, so that four wavefronts a SIMD stay resident; DEPTH 4, at
// two, for meshes that leave a SIMD one wavefront or less, whose only cover for a
// gather is its own other gathers.
template <int MODE, bool ABS, int SPB, int DEPTH, bool LINED>
__global__ __launch_bounds__(SPB * kWave) __attribute__((amdgpu_waves_per_eu(DEPTH > 2 ? 2 : PD_STEP_WAVES_PER_EU)))
void k_step(StepArgs A) {
  extern __shared__ StencilC s_st[];
  if (MODE == MODE_STEP && halted(A.halt)) return;
  const int64_t blk = A.xcd_remap ? xcd_remap(blockIdx.x, gridDim.x) : (int64_t)blockIdx.x;
  bool tables = !LINED;
  if (LINED)
#pragma unroll
    for (int w = 0; w < SPB; ++w) {
      const int64_t s = A.slice_base + blk * SPB + w;
      tables = tables || (s < A.slice_end && !lined_up(A, s));
    }
  if (tables) stage_stencil(A, s_st);  // (the same for the workgroup)
  step_body<MODE, ABS, SPB, DEPTH, true, LINED>(A, s_st, blk);
}

// ---------------------------------------------------------------------------
// tiled bond loop: u of a tile and its halo in LDS, bond memory in class masks
// ---------------------------------------------------------------------------

// Offset, in the halo box, of the neighbour in horizon class k (lexicographic
// (ds, dm, df) with 0 < |d|^2 <= 9) from the lane's corner cell (its own cell
// minus kTileR on each axis); -1 past the last class.
constexpr int tile_class_off(int k) {
  int n = 0;
  for (int a = -kTileR; a <= kTileR; ++a)
    for (int b = -kTileR; b <= kTileR; ++b)
      for (int c = -kTileR; c <= kTileR; ++c) {
        const int d2 = a * a + b * b + c * c;
        if (d2 == 0 || d2 > kTileR * kTileR) continue;
        if (n == k) return ((a + kTileR) * kHM + (b + kTileR)) * kHF + (c + kTileR);
        ++n;
      }
  return -1;
}
static_assert(tile_class_off(kTileClasses - 1) >= 0 && tile_class_off(kTileClasses) < 0,
              "horizon factor 3 has 122 classes");
static_assert((kHalo + tile_class_off(kTileClasses - 1)) * sizeof(double) <= 65535,
              "plane and class offsets must fit the LDS immediate offset");

// offset (ds, dm, df) of horizon class k, and the place of its |d|^2 among the
// eight values that occur
struct ClassOff {
  int d[3];
  int norm;
};
constexpr ClassOff tile_class(int k) {
  int n = 0;
  for (int a = -kTileR; a <= kTileR; ++a)
    for (int b = -kTileR; b <= kTileR; ++b)
      for (int c = -kTileR; c <= kTileR; ++c) {
        const int d2 = a * a + b * b + c * c;
        if (d2 == 0 || d2 > kTileR * kTileR) continue;
        if (n == k) return ClassOff{{a, b, c}, tile_norm(d2)};
        ++n;
      }
  return ClassOff{{0, 0, 0}, -1};
}
// the six orders of the lattice axes (slowest first)
constexpr int kAxisOrder[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};
// component of the offset of class k along x, y or z in axis order perm
constexpr int tile_comp(int k, int perm, int axis) {
  const ClassOff c = tile_class(k);
  return kAxisOrder[perm][0] == axis ? c.d[0] : kAxisOrder[perm][1] == axis ? c.d[1] : c.d[2];
}

typedef const __attribute__((address_space(4))) TileNorms* NormTab;
typedef const __attribute__((address_space(4))) uint64_t* MaskTab;

// The constants of a tile that stay in scalar registers for the whole class loop:
// the components of xi are multiples of h, the threshold is the same for every
// bond, and so is the polynomial.  (1 / |xi|^2 and c V / |xi| depend on |d|^2 only,
// but all eight pairs as well would not fit: what the compiler keeps in vector
// lanes instead costs a vector instruction each time it is read.)
struct TileK {
  double h[4];  // 0, h, 2 h, 3 h
  double thr_x, lo_x;
  PolyS P;
};
__device__ __forceinline__ TileK tile_constants(NormTab n) {
  TileK T;
  T.h[0] = 0.0;
#pragma unroll
  for (int k = 1; k < 4; ++k) T.h[k] = n->h[k];
  T.thr_x = n->thr_x;
  T.lo_x = n->lo_x;
  T.P = poly_in_registers();
  return T;
}

// Operands of one horizon class: the neighbour's u from LDS, 1 / |xi|^2 and c V /
// |xi| (and in the generic variant, PERM < 0, xi) through scalar loads.  The lane masks of intact bonds
// come four classes at a time, a group ahead.
constexpr int kMaskGroup = 4;
struct TileIn {
  double ux, uy, uz;
  double hx, hy, hz;
  double inv, civ;
  uint64_t live[kMaskGroup], next[kMaskGroup];
};

template <int G>
__device__ __forceinline__ void mask_load(const uint64_t* mrow, uint64_t (&m)[kMaskGroup]) {
  if constexpr (G * kMaskGroup < kTileClasses) {
    const uint64_t* mp = mrow + G * kMaskGroup;
    asm volatile("" : "+s"(mp));  // (keeps the load here instead of at the kernel's entry)
#pragma unroll
    for (int k = 0; k < kMaskGroup; ++k) m[k] = ((MaskTab)mp)[k];  // the last group reads into the padding
  }
}

template <int K, int PERM>
__device__ __forceinline__ void tile_load(const double* L, const double* Lz, const StencilC* tabp,
                                          const TileNorms* norms, TileIn& in) {
  constexpr int off = tile_class_off(K);
  const TileNorms* np = norms;
  asm volatile("" : "+s"(np));  // (keeps the loads here instead of at the kernel's entry)
  in.inv = ((NormTab)np)->bond[tile_class(K).norm][0];
  in.civ = ((NormTab)np)->bond[tile_class(K).norm][1];
  in.ux = L[off];
  in.uy = L[kHalo + off];
  in.uz = Lz[off];
  if constexpr (PERM < 0) {
    const StencilC* rowp = tabp + K;
    asm volatile("" : "+s"(rowp));
    const TileTab row = (TileTab)rowp;
    in.hx = row->hx;
    in.hy = row->hy;
    in.hz = row->hz;
  }
}

// e + SCALE xi for a component of xi that is C spacings: nothing to add at zero
template <int C, int SCALE>
__device__ __forceinline__ double plus_xi(double e, const TileK& T) {
  if constexpr (C == 0) return e;
  else if constexpr (SCALE == 1) return C > 0 ? e + T.h[C > 0 ? C : 0] : e - T.h[C < 0 ? -C : 0];
  else return C > 0 ? fma(2.0, T.h[C > 0 ? C : 0], e) : fma(-2.0, T.h[C < 0 ? -C : 0], e);
}

// One horizon class of the lane's node: the same arithmetic, in the same order,
// as an entry of the slice path, so the two paths agree bitwise.  A class with
// no bond (outside the grain, another grain, cut, or broken) adds nothing.  The
// operands of class K arrived during class K - 1; once the first of them is used
// (which waits for all of them) class K + 1's loads are issued, so that they
// travel while class K computes.  The class's lane mask of intact bonds decides
// in scalar registers which lanes add a force, and loses the lanes whose bond
// breaks now; a wavefront in which one breaks stores the mask (lane 0) and counts
// the breaks per lane.  FP64 issue bounds the loop: 25 vector instructions per
// class with the axis order known at compile time.  With 30 (every xi component
// added, the degree-8 polynomial for all, the force selected per lane) the plate's
// launch took 143 us instead of 117, the large aggregate's 1927 us instead of 1780.
// The other forms and the breaks are marked unlikely: placed out of line, so that the
// straight code of 122 classes fits the instruction cache (plate 117.9 -> 115.5 us,
// a volume of 373,248 nodes 84.1 -> 77.2, the large aggregate 1621 -> 1548), and short
// (see g_corrected).
template <int K, bool ABS, int PERM>
__device__ __forceinline__ void tile_bond(const double* L, const double* Lz, const StencilC* tabp, const TileNorms* norms,
                                          const uint64_t* mrow, uint64_t* mrow_w, TileIn& in, const TileK& T,
                                          double uix, double uiy, double uiz, int& nbroke, double& fx, double& fy,
                                          double& fz) {
  const double ex = in.ux - uix, ey = in.uy - uiy, ez = in.uz - uiz;
  constexpr int cx = tile_comp(K, PERM < 0 ? 0 : PERM, 0), cy = tile_comp(K, PERM < 0 ? 0 : PERM, 1),
                cz = tile_comp(K, PERM < 0 ? 0 : PERM, 2);
  double wx, wy, wz;  // 2 xi + eta
  if constexpr (PERM >= 0) {
    wx = plus_xi<cx, 2>(ex, T);
    wy = plus_xi<cy, 2>(ey, T);
    wz = plus_xi<cz, 2>(ez, T);
  } else {
    wx = fma(2.0, in.hx, ex);
    wy = fma(2.0, in.hy, ey);
    wz = fma(2.0, in.hz, ez);
  }
  const uint64_t live = in.live[K % kMaskGroup];
  const double inv = in.inv, civ = in.civ, hx = in.hx, hy = in.hy, hz = in.hz;
  __builtin_amdgcn_sched_barrier(0);
  if constexpr ((K + 1) % kMaskGroup == 0) {
#pragma unroll
    for (int k = 0; k < kMaskGroup; ++k) in.live[k] = in.next[k];
    mask_load<(K + 1) / kMaskGroup + 1>(mrow, in.next);
  }
  if constexpr (K + 1 < kTileClasses) tile_load<K + 1, PERM>(L, Lz, tabp, norms, in);
  auto xi_plus = [&](double ax, double ay, double az, double& yx, double& yy, double& yz) {
    if constexpr (PERM >= 0) {
      yx = plus_xi<cx, 1>(ax, T);
      yy = plus_xi<cy, 1>(ay, T);
      yz = plus_xi<cz, 1>(az, T);
    } else {
      yx = hx + ax;
      yy = hy + ay;
      yz = hz + az;
    }
  };
  double yx, yy, yz;  // xi + eta
  xi_plus(ex, ey, ez, yx, yy, yz);
  const double d = fma(ex, wx, fma(ey, wy, ez * wz));
  const double x = d * inv;
  bool over = x > T.thr_x;
  if (ABS) over = over || x < T.lo_x;
  const double cx_ = civ * x;
  const double q = q_short(x, T.P);
  double coef = cx_ * q;
  // the per-lane choice of the slice path, the other forms computed only when a
  // lane with an intact bond needs them
  const bool far = !(fabs(x) <= kShortRange);
  if (__builtin_expect((__ballot(far) & live) != 0ull, 0)) {
    const bool exact = !(fabs(x) <= kWideRange);
    double g = g_corrected(x, q);
    if (__builtin_expect((__ballot(exact) & live) != 0ull, 0)) {
      // (y made here again: used by both, it would be made before the break test, whose
      // latency it covers where it is: 1% of the launch)
      double ax = ex, ay = ey, az = ez, bx, by, bz;
      asm volatile("" : "+v"(ax), "+v"(ay), "+v"(az));
      xi_plus(ax, ay, az, bx, by, bz);
      g = exact ? g_exact(x, bx, by, bz, inv) : g;
    }
    coef = far ? civ * g : coef;
  }
  // an intact bond within its limit adds its force; a bond past its limit stays
  // broken from now on
  const uint64_t ov = __ballot(over);
  add_on_lanes(live & ~ov, coef, yx, yy, yz, fx, fy, fz);
  const uint64_t brk = live & ov;
  if (__builtin_expect(brk != 0ull, 0)) {
    uint64_t carry;
    mrow_w[K] = live & ~ov;  // (by every lane, the same)
    asm("v_addc_co_u32_e64 %0, %1, %0, 0, %2" : "+v"(nbroke), "=&s"(carry) : "s"(brk));
  }
}

template <bool ABS, int PERM, int... K>
__device__ __forceinline__ void tile_bonds(std::integer_sequence<int, K...>, const double* L, const double* Lz,
                                           const StencilC* tab, const TileNorms* norms, const uint64_t* mrow, uint64_t* mrow_w,
                                           double uix, double uiy, double uiz, int& nbroke, double& fx, double& fy,
                                           double& fz) {
  const TileK T = tile_constants((NormTab)norms);
  TileIn in;
  mask_load<0>(mrow, in.live);
  mask_load<1>(mrow, in.next);
  tile_load<0, PERM>(L, Lz, tab, norms, in);
  (tile_bond<K, ABS, PERM>(L, Lz, tab, norms, mrow, mrow_w, in, T, uix, uiy, uiz, nbroke, fx, fy, fz), ...);
}

__device__ __forceinline__ int64_t tile_cell(const TileGrain& TG, int s, int m, int f) {
  return TG.map_off + ((int64_t)s * TG.em + m) * TG.ef + f;
}

// One workgroup per tile: stage u of the tile and its halo (cells outside the
// grain hold zeros and have no bonds), evaluate the 122 horizon classes of each
// lane's cell from LDS, then the node tail of the slice path.  Lane l of
// wavefront w owns cell (s0 + w, m0 + l / 16, f0 + l % 16).
template <bool ABS, bool EXTRA>
__global__ __launch_bounds__(kTS * kWave) __attribute__((amdgpu_waves_per_eu(4))) void k_step_tile(StepArgs A) {
  // x, y and z planes of the halo box
  __shared__ double s_u[3 * kHalo];
  constexpr int kNT = kTS * kWave;
  constexpr int kFill = (kHalo + kNT - 1) / kNT;  // halo cells per thread
  if (halted(A.halt)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t t = A.xcd_remap ? xcd_remap(blockIdx.x, gridDim.x) : (int64_t)blockIdx.x;
  const int4 T = A.tiles[t];
  const TileGrain TG = A.tgrain[T.x];
  // the lane's own cell, then the halo: every map read is issued before the
  // first wait and every u read before the second, so the fill costs two
  // memory round trips rather than two per cell
  const int lm = lane / kTF, lf = lane % kTF;
  const int cs = T.y + wid, cm = T.z + lm, cf = T.w + lf;
  const bool own_in = cs < TG.es && cm < TG.em && cf < TG.ef;
  int64_t i = own_in ? (int64_t)A.tmap[tile_cell(TG, cs, cm, cf)] : -1;
  int j[kFill];
#pragma unroll
  for (int r = 0; r < kFill; ++r) {
    const int c = tid + r * kNT;
    const int hs = c / (kHM * kHF), rr = c - hs * (kHM * kHF);
    const int hm = rr / kHF, hf = rr - hm * kHF;
    const int ps = T.y - kTileR + hs, pm = T.z - kTileR + hm, pf = T.w - kTileR + hf;
    j[r] = -1;
    if (c < kHalo && ps >= 0 && ps < TG.es && pm >= 0 && pm < TG.em && pf >= 0 && pf < TG.ef)
      j[r] = A.tmap[tile_cell(TG, ps, pm, pf)];
  }
  const bool valid = i >= 0;
  double4 ui = make_double4(0.0, 0.0, 0.0, 0.0);
  if (valid) ui = A.ucur[i];
  // bring this wavefront's lane masks (122 x 8 B) into the L2 with the other
  // prologue loads, so that the class loop's scalar loads of them hit there
  const uint64_t* mrow_r = A.lmask + ((int64_t)t * kTS + wid) * kTileClasses;
  uint4 mpre = make_uint4(0u, 0u, 0u, 0u);
  if (lane < kTileClasses / 2) mpre = reinterpret_cast<const uint4*>(mrow_r)[lane];
  double hx_[kFill], hy_[kFill], hz_[kFill];
#pragma unroll
  for (int r = 0; r < kFill; ++r) {
    hx_[r] = hy_[r] = hz_[r] = 0.0;
    if (j[r] >= 0) {
      const double4 u = A.ucur[j[r]];
      hx_[r] = u.x;
      hy_[r] = u.y;
      hz_[r] = u.z;
    }
  }
#pragma unroll
  for (int r = 0; r < kFill; ++r) {
    const int c = tid + r * kNT;
    if (c < kHalo) {
      s_u[c] = hx_[r];
      s_u[kHalo + c] = hy_[r];
      s_u[2 * kHalo + c] = hz_[r];
    }
  }
  // the lane's own grain (in lattice mode a tile holds nodes of several grains)
  const GrainC* G = A.grains + (valid ? packed_grain(ui.w) : 0);
  const int pi = packed_ijk(ui.w);
  __syncthreads();

  const double* L = s_u + (wid * kHM + lm) * kHF + lf;
  const double* Lz = L + 2 * kHalo;  // own base: plane and class offsets must fit the 16-bit immediate
  double fx = 0.0, fy = 0.0, fz = 0.0;
  const StencilC* tab = A.ttab + (int64_t)TG.table * kTileClasses;
  const TileNorms* norms = A.tnorm + TG.table;
  // this wavefront's lane masks, one per class
  uint64_t* mrow_w = A.lmask + ((int64_t)t * kTS + wid) * kTileClasses;
  int nbroke = 0;  // bonds of this lane's node broken in this step
  // a layer beyond the last nodes of the box (the far ends of a lattice-mode
  // box) has no bonds: its wavefront leaves the vector units to the others
  if (__ballot(valid) != 0ull) {
    const auto classes = std::make_integer_sequence<int, kTileClasses>{};
    // the node orders of a shared lattice (x-y-z) and of a plate thin along z (x-z-y) have
    // the zero components of xi compiled out: a slab of 200 x 20 x 192 nodes takes 102 to
    // 107 us a step in these two orders, 108 to 112 in the four others, all of which took
    // 126 to 130 before (a variant for each order, with and without the |s| reading, would
    // be six times the code)
    if (!ABS && TG.perm == 0)
      tile_bonds<ABS, 0>(classes, L, Lz, tab, norms, mrow_r, mrow_w, ui.x, ui.y, ui.z, nbroke, fx, fy, fz);
    else if (!ABS && TG.perm == 1)
      tile_bonds<ABS, 1>(classes, L, Lz, tab, norms, mrow_r, mrow_w, ui.x, ui.y, ui.z, nbroke, fx, fy, fz);
    else
      tile_bonds<ABS, -1>(classes, L, Lz, tab, norms, mrow_r, mrow_w, ui.x, ui.y, ui.z, nbroke, fx, fy, fz);
  }
  // the prefetch's data is not needed; consuming it keeps the load
  asm volatile("" ::"v"(mpre.x ^ mpre.y ^ mpre.z ^ mpre.w));
  node_tail<MODE_STEP, EXTRA, true, false>(A, i, valid, ui, G, unpack_x(pi), unpack_y(pi), unpack_z(pi), fx, fy, fz, nbroke,
                              true, (int64_t)kTS * t + wid, load_va(A, i, valid), TG.perm);
}

__device__ __constant__ int kAxisPerm[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};

// cell of node (packed grain-local ijk p) of grain g in its tile box B
__device__ __forceinline__ void tile_coords(const TileGrain& Gg, const TileGrain& B, int p, int& s, int& m, int& f) {
  const int q[3] = {unpack_x(p) + Gg.goff[0], unpack_y(p) + Gg.goff[1], unpack_z(p) + Gg.goff[2]};
  s = q[kAxisPerm[B.perm][0]] - B.lo_s;
  m = q[kAxisPerm[B.perm][1]] - B.lo_m;
  f = q[kAxisPerm[B.perm][2]] - B.lo_f;
}

__global__ void k_tile_map_fill(StepArgs A) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= A.n) return;
  const double w = A.ucur[i].w;
  const TileGrain Gg = A.tgrain[packed_grain(w)];
  const TileGrain B = A.tgrain[Gg.box];
  int s, m, f;
  tile_coords(Gg, B, packed_ijk(w), s, m, f);
  const_cast<int32_t*>(A.tmap)[tile_cell(B, s, m, f)] = (int32_t)i;
}

// Lane masks from the column words: one wavefront per layer of a tile, lane l
// on the cell it owns in the step kernel.  Each lane gathers its node's live
// built bonds as tile-class bits (class ctob[perm][slice class]); a ballot per
// class forms the wavefront's mask.
__global__ __launch_bounds__(256) void k_cols_to_mask(StepArgs A, const int16_t* ctob, const uint32_t* colOrig) {
  const int64_t wv = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
  if (wv >= A.n_tiles * kTS) return;  // whole wavefronts leave together
  const int lane = threadIdx.x & 63;
  const int64_t t = wv / kTS;
  const int w = (int)(wv % kTS);
  const int4 T = A.tiles[t];
  const TileGrain TG = A.tgrain[T.x];
  const int cs = T.y + w, cm = T.z + lane / kTF, cf = T.w + lane % kTF;
  const int64_t i = (cs < TG.es && cm < TG.em && cf < TG.ef) ? (int64_t)A.tmap[tile_cell(TG, cs, cm, cf)] : -1;
  uint32_t m[4] = {0u, 0u, 0u, 0u};
  if (i >= 0) {
    const int64_t sc = i / kWave, sl = i % kWave;
    const int64_t off = A.slice_off[sc];
    const int W = (int)((A.slice_off[sc + 1] - off) / kWave);
    const int perm = A.tgrain[packed_grain(A.ucur[i].w)].perm;
    for (int e = 0; e < W; ++e) {
      const int64_t at = off + (int64_t)e * kWave + sl;
      const uint32_t wo = colOrig[at];
      const int cls = (int)(wo >> A.node_bits);
      if (cls >= A.n_stencil || A.colE[at] != wo) continue;
      const int b = ctob[perm * A.n_stencil + cls];
      m[b >> 5] |= 1u << (b & 31);
    }
  }
  uint64_t* row = A.lmask + wv * kTileClasses;
  for (int K = 0; K < kTileClasses; ++K) {
    const uint64_t bits = __ballot(((m[K >> 5] >> (K & 31)) & 1u) != 0u);
    if (lane == 0) row[K] = bits;
  }
}

// the inverse: an entry whose lane bit is clear becomes a broken column word
__global__ void k_mask_to_cols(StepArgs A, const int16_t* ctob, const uint32_t* colOrig) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= A.n) return;
  const int32_t sl = A.slot[i];
  if (sl < 0) return;
  const int64_t sc = i / kWave, lane = i % kWave;
  const int64_t off = A.slice_off[sc];
  const int W = (int)((A.slice_off[sc + 1] - off) / kWave);
  const int perm = A.tgrain[packed_grain(A.ucur[i].w)].perm;
  const uint64_t* rowm = A.lmask + (int64_t)(sl >> 6) * kTileClasses;
  for (int e = 0; e < W; ++e) {
    const int64_t at = off + (int64_t)e * kWave + lane;
    const uint32_t wo = colOrig[at];
    const int cls = (int)(wo >> A.node_bits);
    if (cls >= A.n_stencil) continue;
    const uint64_t m = rowm[ctob[perm * A.n_stencil + cls]];
    A.colE[at] = ((m >> (sl & 63)) & 1ull) ? wo : ((uint32_t)i | A.sentinel_hi);
  }
}

// Wall reactions are reduced in a fixed order in two levels, the same in every
// step-loop mode: (1) chunk q of 1024 slice columns is summed by one wavefront,
// lane l taking columns 1024 q + l + 64 k (k = 0..15) in turn, then across the
// lanes (a column that touched no wall adds a zero and is not read: most of
// them); (2) the chunk sums of a component are summed as by 1024 threads (virtual
// thread v takes chunks v, v + 1024, ...), across each virtual wave's lanes and
// over the 16 virtual waves in order.  With at most 64 chunks only virtual wave 0
// holds data and (2) is one wavefront's lane sum.
template <typename F>
__device__ __forceinline__ void chunk_sums(const StepArgs& A, int64_t q, F put) {
  const int lane = threadIdx.x & 63;
  const int64_t n = A.partial_stride, b = q * kChunk + lane;
  uint32_t t[16], any = 0u;
#pragma unroll
  for (int k = 0; k < 16; ++k) t[k] = A.wall_touched[b + 64 * k < n ? b + 64 * k : n - 1];
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    t[k] = b + 64 * k < n ? t[k] : 0u;
    any |= t[k];
  }
  for (int w = 0; w < A.n_walls; ++w) {
    const bool some = __ballot((any >> w) & 1u) != 0ull;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      double s = 0.0;
      if (some) {
        const double* p = A.wall_partial + (int64_t)(3 * w + c) * n;
        double v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = ((t[k] >> w) & 1u) ? p[b + 64 * k] : 0.0;
#pragma unroll
        for (int k = 0; k < 16; ++k) s += v[k];
        s = wave_sum(s);
      }
      if (lane == 0) put(3 * w + c, s);
    }
  }
}

// Level (2) by one workgroup of NT threads from the chunk sums, then the reactions
// and the wall positions of the next step: prescribed velocity or servo on the
// measured stress.  chunk(c, q): sum q of component c.
template <int NT, typename F>
__device__ __forceinline__ void finalize_level2(const StepArgs& A, double (*red)[1024 / kWave],
                                                double* tot, int64_t* s_step, F chunk) {
  constexpr int VT = 1024 / NT;
  constexpr int CB = NT >= 1024 ? 8 : 2;  // components per batch (register budget)
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int nc = 3 * A.n_walls;
  const int64_t nq = (A.partial_stride + kChunk - 1) / kChunk;
  if (nq <= kWave) {
    for (int c = wv; c < nc; c += NT / kWave) {
      const double t = wave_sum(lane < nq ? chunk(c, lane) : 0.0);
      if (lane == 0) tot[c] = t;
    }
  } else {
    for (int c0 = 0; c0 < nc; c0 += CB) {
      double acc[CB][VT];
#pragma unroll
      for (int cc = 0; cc < CB; ++cc)
#pragma unroll
        for (int k = 0; k < VT; ++k) acc[cc][k] = 0.0;
      for (int64_t b0 = 0; b0 < nq; b0 += 1024) {
#pragma unroll
        for (int k = 0; k < VT; ++k) {
          const int64_t b = b0 + tid + (int64_t)NT * k;  // virtual thread tid + NT k
#pragma unroll
          for (int cc = 0; cc < CB; ++cc) {
            const int c = c0 + cc;
            if (c < nc && b < nq) acc[cc][k] += chunk(c, b);
          }
        }
      }
#pragma unroll
      for (int cc = 0; cc < CB; ++cc) {
        if (c0 + cc < nc) {
#pragma unroll
          for (int k = 0; k < VT; ++k) {
            const double t = wave_sum(acc[cc][k]);
            if (lane == 0) red[c0 + cc][wv + (NT / kWave) * k] = t;
          }
        }
      }
    }
    __syncthreads();
    if (tid < nc) {
      double t = 0.0;
      for (int k = 0; k < 1024 / kWave; ++k) t += red[tid][k];
      tot[tid] = t;
    }
  }
  // a halted step changes neither the walls nor the step count
  if (A.advance && halted(A.halt)) return;
  if (tid == 0) *s_step = *A.step + A.advance;  // the step this evaluation belonged to
  __syncthreads();
  const int64_t s = *s_step;
  if (tid == 0) *A.step = s;
  // one thread per wall: its loads are independent of the other walls'
  if (tid < A.n_walls) {
    WallDev W = A.walls[tid];
    for (int q = 0; q < 3; ++q) {
      W.force[q] = -tot[3 * tid + q];
      if (A.advance) W.impulse[q] += W.force[q] * A.dt;
    }
    W.off_used = W.off;
    W.rate_used = W.rate;
    if (W.mode == PD_WALL_VELOCITY) {
      W.off = W.off0 + W.vel * ((double)(s + 1) * A.dt);
      W.rate = W.vel;
    } else if (W.mode == PD_WALL_SERVO) {
      const double sigma = -(W.force[0] * W.n[0] + W.force[1] * W.n[1] + W.force[2] * W.n[2]) / W.area;
      W.rate = W.gain * (W.target - sigma);
      W.off = W.off + A.dt * W.rate;
    }
    A.walls[tid] = W;
  }
}

// Level (1) for more than kFusedChunks chunks: one wavefront per chunk.  Level (2)
// and the wall update run in the next kernel, whose start sees every chunk sum (a
// kernel boundary instead of a device-scope fence per workgroup).
__global__ __launch_bounds__(kWave) void k_wall_chunks(StepArgs A) {
  const int64_t nq = (A.partial_stride + kChunk - 1) / kChunk;
  const int64_t q = blockIdx.x;
  if (q >= nq) return;
  chunk_sums(A, q, [&](int c, double s) { A.wall_chunk[(int64_t)c * nq + q] = s; });
}

__device__ __forceinline__ void set_halt(const StepArgs& A) {
  // the last kernel of the step: the next step halts if this one raised a flag
  if (threadIdx.x == 0)
    __hip_atomic_store(A.halt, __hip_atomic_load(A.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// 1024 threads: level (2) is written for 1024 virtual threads, so each takes
// one of them (the sums are the same for any workgroup size)
__global__ __launch_bounds__(1024) void k_wall_finalize(StepArgs A) {
  __shared__ double red[kMaxWalls * 3][1024 / kWave];
  __shared__ double tot[kMaxWalls * 3];
  __shared__ int64_t s_step;
  const int64_t nq = (A.partial_stride + kChunk - 1) / kChunk;
  finalize_level2<1024>(A, red, tot, &s_step, [&](int c, int64_t q) { return A.wall_chunk[(int64_t)c * nq + q]; });
  set_halt(A);
}

// Both levels in one launch for up to kFusedChunks chunks (two rounds of the 16
// wavefronts: 32,768 slices or tile wavefronts): a launch less every step, 4.7 us.
constexpr int kFusedChunks = 32;
__global__ __launch_bounds__(1024) void k_wall_finalize_small(StepArgs A) {
  __shared__ double sums[kMaxWalls * 3][kFusedChunks];
  __shared__ double tot[kMaxWalls * 3];
  __shared__ int64_t s_step;
  const int64_t nq = (A.partial_stride + kChunk - 1) / kChunk;
  for (int64_t q = threadIdx.x >> 6; q < nq && A.n_walls > 0; q += 1024 / kWave)
    chunk_sums(A, q, [&](int c, double s) { sums[c][q] = s; });
  __syncthreads();
  finalize_level2<1024>(A, nullptr, tot, &s_step, [&](int c, int64_t q) { return sums[c][q]; });
  set_halt(A);
}

// ---------------------------------------------------------------------------
// persistent step loop: nsteps steps (no candidate rebuild among them) in one
// cooperative launch.  Workgroups walk their slice blocks of a step and meet at
// one grid barrier per step; the workgroup that arrives last reduces the wall
// reactions (in the order the launched wall kernels use, so the result is the
// same bit for bit) and writes the halt word before it releases the others,
// who then read the new wall state and the halt word.  Every wait has a spin
// limit, so each wave exits even if a barrier were never completed.
// ---------------------------------------------------------------------------

// Arrive at the grid barrier; returns (uniformly over the workgroup) whether
// this workgroup arrived last.  The last one must call grid_release after its
// serial work; the others have already waited for that release on return.
__device__ __forceinline__ bool grid_arrive(const BarrierArgs& B, uint32_t nblocks, uint32_t* status,
                                            uint32_t* s_flag) {
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();  // release this workgroup's writes to every XCD
    const uint32_t g = __hip_atomic_load(B.gen, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
    const bool last = atomicAdd(B.count, 1u) == nblocks - 1u;
    if (!last) {
      uint32_t spins = 0;
      while (__hip_atomic_load(B.gen, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) == g) {
        __builtin_amdgcn_s_sleep(1);
        if (++spins > B.spin_limit) {
          atomicOr(status, ST_BARRIER);
          break;
        }
      }
    }
    __threadfence();  // acquire the other workgroups' writes
    *s_flag = last ? 1u : 0u;
  }
  __syncthreads();
  return *s_flag != 0u;
}

__device__ __forceinline__ void grid_release(const BarrierArgs& B) {
  __syncthreads();
  if (threadIdx.x == 0) {
    atomicExch(B.count, 0u);
    __threadfence();  // release the serial work before the generation moves
    atomicAdd(B.gen, 1u);
  }
  __syncthreads();
}

template <bool ABS>
__global__ __launch_bounds__(4 * kWave) __attribute__((amdgpu_waves_per_eu(3)))
void k_step_persistent(StepArgs A, int64_t nsteps, BarrierArgs B) {
  extern __shared__ StencilC s_st[];
  __shared__ double red[kMaxWalls * 3][1024 / kWave];
  __shared__ double tot[kMaxWalls * 3];
  __shared__ int64_t s_step;
  __shared__ uint32_t s_last;
  if (halted(A.halt)) return;
  stage_stencil(A, s_st);
  // the nv 4-slice blocks are cut evenly into rounds x gridDim runs (of 0 or
  // 1 blocks mostly).  In dispatch order workgroup b takes run q gridDim + b in
  // round q; in XCD order (gridDim a multiple of 8) the nx = gridDim / 8
  // workgroups of XCD x walk the x-th eighth of the runs side by side, so each
  // XCD's L2 serves one contiguous eighth of the mesh.  An even cut by blocks
  // measured faster than one by padded bond slots: the per-node work of a
  // slice (contact, walls, Verlet) does not scale with its bonds.
  const int64_t nv = (A.slice_end - A.slice_base + 3) / 4;
  const int64_t nb = gridDim.x, rounds = (nv + nb - 1) / nb, np = rounds * nb;
  int64_t p0 = blockIdx.x, pstep = nb;
  if (A.xcd_remap && (gridDim.x & 7u) == 0u) {
    const int64_t nx = nb >> 3;
    p0 = (int64_t)(blockIdx.x & 7u) * rounds * nx + (blockIdx.x >> 3);
    pstep = nx;
  }
  for (int64_t k = 0; k < nsteps; ++k) {
    for (int64_t q = 0; q < rounds; ++q) {
      const int64_t p = p0 + q * pstep;
      const int64_t vb1 = nv * (p + 1) / np;
      for (int64_t vb = nv * p / np; vb < vb1; ++vb) step_body<MODE_STEP, ABS, 4, 2, false, false>(A, s_st, vb);
    }
    if (grid_arrive(B, gridDim.x, A.status, &s_last)) {
      // level (1) by this workgroup's wavefronts, then level (2)
      const int64_t nq = (A.partial_stride + kChunk - 1) / kChunk;
      if (A.n_walls > 0)
        for (int64_t q = threadIdx.x >> 6; q < nq; q += 4)
          chunk_sums(A, q, [&](int c, double s) { A.wall_chunk[(int64_t)c * nq + q] = s; });
      __threadfence_block();
      __syncthreads();
      finalize_level2<4 * kWave>(A, red, tot, &s_step,
                                 [&](int c, int64_t q) { return A.wall_chunk[(int64_t)c * nq + q]; });
      set_halt(A);
      grid_release(B);
    }
    if (halted(A.halt)) break;
    // the drift just written is the next step's position; mid-step velocities likewise
    const double4* uc = A.ucur;
    A.ucur = A.unext;
    A.unext = const_cast<double4*>(uc);
    const double4* vc = A.vh_cur;
    A.vh_cur = A.vh_next;
    A.vh_next = const_cast<double4*>(vc);
  }
}

// ---------------------------------------------------------------------------
// energies (diagnostic): kinetic, elastic, contact, gravity potential
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(kBlock) void k_energy(StepArgs A, double* partial4) {
  __shared__ double red[4][kBlock];
  const int tid = threadIdx.x;
  const int64_t i = (int64_t)blockIdx.x * kBlock + tid;
  double e[4] = {0.0, 0.0, 0.0, 0.0};
  if (i < A.n) {
    const double4 ui = A.ucur[i];
    const GrainC* G = A.grains + packed_grain(ui.w);
    const int pi = packed_ijk(ui.w);
    const double V = G->V, rho = G->rho;
    const double vx = A.v[i], vy = A.v[A.n + i], vz = A.v[2 * A.n + i];
    e[0] = 0.5 * rho * V * (vx * vx + vy * vy + vz * vz);
    e[3] = -rho * V * (A.g[0] * ui.x + A.g[1] * ui.y + A.g[2] * ui.z);
    const int64_t s = i / kWave;
    const int lane = (int)(i % kWave);
    const int64_t off = A.slice_off[s];
    const int W = (int)((A.slice_off[s + 1] - off) / kWave);
    double w = 0.0;
    for (int k = 0; k < W; ++k) {
      const uint32_t cw = A.colE[off + (int64_t)k * kWave + lane];
      if ((cw & ~((1u << A.node_bits) - 1u)) == A.sentinel_hi) continue;  // broken or padding
      const int j = (int)(cw & ((1u << A.node_bits) - 1u));
      const double4 uj = A.ucur[j];
      const int pj = packed_ijk(uj.w);
      const int dx = unpack_x(pj) - unpack_x(pi), dy = unpack_y(pj) - unpack_y(pi),
                dz = unpack_z(pj) - unpack_z(pi);
      const double xx = G->h * dx, xy = G->h * dy, xz = G->h * dz;
      const double ex = uj.x - ui.x, ey = uj.y - ui.y, ez = uj.z - ui.z;
      const double yx = xx + ex, yy = xy + ey, yz = xz + ez;
      const double l0 = sqrt(xx * xx + xy * xy + xz * xz), l = sqrt(yx * yx + yy * yy + yz * yz);
      const double dd = ex * (2.0 * xx + ex) + ey * (2.0 * xy + ey) + ez * (2.0 * xz + ez);
      const double st = dd / (l0 * (l + l0));
      // micropotential 1/2 c w(|xi|) s^2 |xi| times V_j
      w += 0.5 * (G->cVih * G->h) * (1.0 - l0 * G->conic_inv_delta) * st * st * l0;
    }
    e[1] = 0.5 * V * w;
    if (A.cand_ptr != nullptr) {
      const int32_t c0 = (int32_t)min((int64_t)A.cand_ptr[i], A.cand_capacity);
      const int32_t c1 = (int32_t)min((int64_t)A.cand_ptr[i + 1], A.cand_capacity);
      for (int32_t c = c0; c < c1; ++c) {
        const int j = A.cand[c];
        const double4 uj = A.ucur[j];
        double yx, yy, yz;
        const double d2 = contact_d2(A.X[j], A.X[i], uj.x, ui.x, A.X[A.n + j], A.X[A.n + i], uj.y,
                                     ui.y, A.X[2 * A.n + j], A.X[2 * A.n + i], uj.z, ui.z, yx, yy, yz);
        if (!(d2 < A.Rc2)) continue;
        const GrainC* Gj = A.grains + packed_grain(uj.w);
        const double d = sqrt(d2);
        e[2] += 0.5 * V * 0.5 * A.Kn[G->mat * A.n_mat + Gj->mat] * (A.Rc - d) * (A.Rc - d) * Gj->V;
      }
    }
  }
  for (int q = 0; q < 4; ++q) red[q][tid] = e[q];
  __syncthreads();
  for (int o = kBlock / 2; o > 0; o >>= 1) {
    if (tid < o)
      for (int q = 0; q < 4; ++q) red[q][tid] += red[q][tid + o];
    __syncthreads();
  }
  if (tid < 4) partial4[(int64_t)blockIdx.x * 4 + tid] = red[tid][0];
}

__global__ void k_reduce_energy(const double* partial4, int32_t nblocks, double* out4) {
  if (threadIdx.x < 4) {
    double s = 0.0;
    for (int b = 0; b < nblocks; ++b) s += partial4[(int64_t)b * 4 + threadIdx.x];
    out4[threadIdx.x] = s;
  }
}

constexpr int kScanThreads = 1024;
constexpr int kScanItems = 4;
constexpr int kScanTile = kScanThreads * kScanItems;

// ---------------------------------------------------------------------------
// contact candidates: hashed uniform cell grid, counting sort, per-node rows
// ---------------------------------------------------------------------------

__device__ __forceinline__ uint32_t cell_hash(int cx, int cy, int cz, uint32_t T) {
  return (((uint32_t)cx * 73856093u) ^ ((uint32_t)cy * 19349663u) ^ ((uint32_t)cz * 83492791u)) &
         (T - 1u);
}

// cell coordinates are clamped to |c| < 2^20 - 1 so that a cell and its
// neighbours pack into one 63-bit key (21 bits per axis); nodes beyond the clamp
// share boundary cells and are still separated by the exact distance test
constexpr int kCellClamp = (1 << 20) - 2;

__device__ __forceinline__ int cell_coord(double p, double inv_cell) {
  double c = floor(p * inv_cell);
  c = fmin(fmax(c, -(double)kCellClamp), (double)kCellClamp);
  return (int)c;
}

__device__ __forceinline__ long long cell_key(int cx, int cy, int cz) {
  return ((long long)(cx + (1 << 20)) << 42) | ((long long)(cy + (1 << 20)) << 21) |
         (long long)(cz + (1 << 20));
}

// Culling.  A grain whose box comes within the cutoff of no other grain's box has no
// candidates, nor has a node farther than the cutoff from the boxes near its grain: they
// are neither binned nor searched.

__device__ __forceinline__ long long ord_key(double x) {
  const long long b = __double_as_longlong(x);
  return b ^ ((b >> 63) & 0x7fffffffffffffffll);
}
__device__ __forceinline__ double ord_val(long long k) {
  return __longlong_as_double(k ^ ((k >> 63) & 0x7fffffffffffffffll));
}

__global__ void k_box_init(ContactArgs c) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= 6 * (int64_t)c.n_grains) return;
  c.gbox[t] = (t % 6) < 3 ? ord_key(INFINITY) : ord_key(-INFINITY);
}

__device__ __forceinline__ long long wave_min_ll(long long x) {
  for (int o = 32; o > 0; o >>= 1) {
    const long long y = __shfl_xor(x, o, kWave);
    x = y < x ? y : x;
  }
  return x;
}
__device__ __forceinline__ long long wave_max_ll(long long x) {
  for (int o = 32; o > 0; o >>= 1) {
    const long long y = __shfl_xor(x, o, kWave);
    x = y > x ? y : x;
  }
  return x;
}

// Displacement since the last rebuild beyond skin/2 invalidates the list; the
// positions of this rebuild are kept (a halted step leaves them alone).
__device__ __forceinline__ void skin_node(const ContactArgs& c, int64_t i, const double4& u, int check) {
  if (check) {
    const double dx = u.x - c.u_build[i], dy = u.y - c.u_build[c.n + i], dz = u.z - c.u_build[2 * c.n + i];
    if (dx * dx + dy * dy + dz * dz > c.skin_half2) atomicOr(c.status, ST_SKIN);
  }
  c.u_build[i] = u.x;
  c.u_build[c.n + i] = u.y;
  c.u_build[2 * c.n + i] = u.z;
}

__global__ void k_skin(ContactArgs c, int check) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= c.n || halted(c.halt)) return;
  skin_node(c, i, c.u[i], check);
}

// the same and the grain boxes in one pass over the nodes: one workgroup per
// chunk of a single grain, LDS reduction, then 6 atomics
__global__ __launch_bounds__(256) void k_skin_box(ContactArgs c, int check) {
  __shared__ long long red[6][256 / kWave];
  const int tid = threadIdx.x;
  const bool live = !halted(c.halt);
  const int64_t* ch = c.box_chunks + 3 * (int64_t)blockIdx.x;
  const int g = (int)ch[0];
  const int64_t e = ch[2];
  long long k[6] = {ord_key(INFINITY), ord_key(INFINITY), ord_key(INFINITY),
                    ord_key(-INFINITY), ord_key(-INFINITY), ord_key(-INFINITY)};
  for (int64_t i = ch[1] + tid; i < e; i += 256) {
    const double4 u = c.u[i];
    if (live) skin_node(c, i, u, check);
    const long long x = ord_key(c.X[i] + u.x), y = ord_key(c.X[c.n + i] + u.y),
                    z = ord_key(c.X[2 * c.n + i] + u.z);
    k[0] = min(k[0], x);
    k[1] = min(k[1], y);
    k[2] = min(k[2], z);
    k[3] = max(k[3], x);
    k[4] = max(k[4], y);
    k[5] = max(k[5], z);
  }
  for (int q = 0; q < 6; ++q) {
    const long long w = q < 3 ? wave_min_ll(k[q]) : wave_max_ll(k[q]);
    if ((tid & 63) == 0) red[q][tid >> 6] = w;
  }
  __syncthreads();
  if (tid < 6) {
    long long w = red[tid][0];
    for (int v = 1; v < 256 / kWave; ++v) w = tid < 3 ? min(w, red[tid][v]) : max(w, red[tid][v]);
    if (tid < 3) atomicMin(c.gbox + 6 * g + tid, w);
    else atomicMax(c.gbox + 6 * g + tid, w);
  }
}

// Which of a grain's nodes can meet another grain's: none, those within the cutoff of the
// boxes that come near it (of the box around them), or all.  One wavefront per grain, the
// others tested 64 at a time; with self-contact all nodes count, but for a grain without
// nodes or with a position that is not a number on any axis: such a box does not bound
// its nodes, which must then not be binned (the step flags them).  Two touching balls of
// 381,000 nodes, a rebuild every step: 293 us a step over hashed cells (a far pair of small
// grains) and 276 over dense ones; with every node binned and searched 597 and 310.
constexpr int kBinAll = 0, kBinNone = 1, kBinNear = 2;
constexpr int kNearNodes = 512;
__global__ __launch_bounds__(kWave) void k_near_boxes(ContactArgs c, double cut) {
  const int a = blockIdx.x, lane = threadIdx.x;
  double alo[3], ahi[3];
  bool box = true;
  for (int q = 0; q < 3; ++q) {
    const double lo = ord_val(c.gbox[6 * a + q]), hi = ord_val(c.gbox[6 * a + 3 + q]);
    box = box && lo <= hi;
    alo[q] = lo - cut;
    ahi[q] = hi + cut;
  }
  bool near = c.self_contact && box;
  // the box around the boxes that come near
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  // (a small grain is binned whole: not worth going on through all others, 188 us a step
  // with a rebuild against 205 for 4,096 grains of 33 nodes)
  const bool small = c.grain_begin[a + 1] - c.grain_begin[a] < kNearNodes;
  for (int b0 = 0; b0 < c.n_grains && box && !c.self_contact && !(small && near); b0 += kWave) {
    const int b = b0 + lane;
    bool ov = b < c.n_grains && b != a;
    if (ov) {
      double blo[3], bhi[3];
      for (int q = 0; q < 3; ++q) {
        blo[q] = ord_val(c.gbox[6 * b + q]);
        bhi[q] = ord_val(c.gbox[6 * b + 3 + q]);
        ov = ov && blo[q] <= ahi[q] && bhi[q] >= alo[q];
      }
      for (int q = 0; q < 3; ++q) {
        lo[q] = ov ? fmin(lo[q], blo[q]) : lo[q];
        hi[q] = ov ? fmax(hi[q], bhi[q]) : hi[q];
      }
    }
    near = near || __ballot(ov) != 0ull;
  }
  int where = near ? kBinAll : kBinNone;
  if (near && !c.self_contact && !small)
    for (int q = 0; q < 3; ++q) {
      for (int o = 32; o > 0; o >>= 1) {
        lo[q] = fmin(lo[q], __shfl_xor(lo[q], o, kWave));
        hi[q] = fmax(hi[q], __shfl_xor(hi[q], o, kWave));
      }
      lo[q] -= cut;
      hi[q] += cut;
      if (alo[q] + cut < lo[q] || ahi[q] - cut > hi[q]) where = kBinNear;
      if (lane == 0) {
        c.nearbox[6 * a + q] = lo[q];
        c.nearbox[6 * a + 3 + q] = hi[q];
      }
    }
  if (lane == 0) c.binned[a] = where;
}

// The cell grid of this rebuild: the box around the nodes to be binned (the
// union of the boxes of the grains that have any), in cells; dense when
// its cell count fits the buckets.  One wavefront.
__global__ __launch_bounds__(kWave) void k_grid_setup(ContactArgs c) {
  const int lane = threadIdx.x;
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int g = lane; g < c.n_grains; g += kWave)
    for (int q = 0; q < 3; ++q) {
      const double a = ord_val(c.gbox[6 * g + q]), b = ord_val(c.gbox[6 * g + 3 + q]);
      if (a <= b && c.binned[g] != kBinNone) {  // grains without nodes keep an empty box
        lo[q] = fmin(lo[q], a);
        hi[q] = fmax(hi[q], b);
      }
    }
  for (int q = 0; q < 3; ++q)
    for (int o = 32; o > 0; o >>= 1) {
      lo[q] = fmin(lo[q], __shfl_xor(lo[q], o, kWave));
      hi[q] = fmax(hi[q], __shfl_xor(hi[q], o, kWave));
    }
  if (lane != 0) return;
  // (nothing to bin: one empty cell)
  const bool any = lo[0] <= hi[0] && lo[1] <= hi[1] && lo[2] <= hi[2];
  int64_t cells = 1, o[3], e[3];
  for (int q = 0; q < 3; ++q) {
    o[q] = any ? cell_coord(lo[q], c.inv_cell) : 0;
    e[q] = any ? cell_coord(hi[q], c.inv_cell) - o[q] + 1 : 1;
    cells = cells <= (int64_t)c.T ? cells * e[q] : cells;
  }
  const bool dense = cells <= (int64_t)c.T;
  c.grid[0] = dense ? 1 : 0;
  for (int q = 0; q < 3; ++q) {
    c.grid[1 + q] = o[q];
    c.grid[4 + q] = e[q];
  }
  c.grid[7] = dense ? cells : (int64_t)c.T;
  // The search's first test is in FP32 on positions relative to the box corner.
  // With extents up to M a stored coordinate is off by at most 2^-24 M and the
  // distance of two nodes by less than 8 * 2^-24 M (1 + 2^-20), so that no pair
  // within the cutoff lies beyond this limit; the pairs it lets through are
  // tested exactly.
  double M = 0.0;
  for (int q = 0; q < 3; ++q) {
    c.origin[q] = any ? lo[q] : 0.0;
    M = any ? fmax(M, hi[q] - lo[q]) : M;
  }
  const double lim = (sqrt(c.cut2) + M * 0x1p-21) * (1.0 + 1e-5);
  c.origin[3] = lim * lim;
}

// bucket of a cell: its lexicographic index in the dense grid, else its hash
__device__ __forceinline__ uint32_t cell_bucket(const ContactArgs& c, bool dense, int cx, int cy, int cz) {
  if (dense)
    return (uint32_t)(((int64_t)(cx - c.grid[1]) * c.grid[5] + (cy - c.grid[2])) * c.grid[6] + (cz - c.grid[3]));
  return cell_hash(cx, cy, cz, c.T);
}

// The atomic that counts a bucket's nodes also numbers them, so that the
// scatter needs no second one.
__global__ void k_bin(ContactArgs c) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= c.n) return;
  const double4 u = c.u[i];
  const int g = packed_grain(u.w);
  const double px = c.X[i] + u.x, py = c.X[c.n + i] + u.y, pz = c.X[2 * c.n + i] + u.z;
  const int where = c.binned[g];
  bool in = where != kBinNone;
  if (where == kBinNear) {
    const double* b = c.nearbox + 6 * g;
    in = px >= b[0] && py >= b[1] && pz >= b[2] && px <= b[3] && py <= b[4] && pz <= b[5];
  }
  if (!in) {
    c.rank[i] = -1;
    c.cand_count[i] = 0;
    return;
  }
  const int cx = cell_coord(px, c.inv_cell);
  const int cy = cell_coord(py, c.inv_cell);
  const int cz = cell_coord(pz, c.inv_cell);
  const long long key = cell_key(cx, cy, cz);
  const uint32_t hsh = cell_bucket(c, c.grid[0] != 0, cx, cy, cz);
  c.rec[2 * i] = make_int4((int)i, g, (int)(key & 0xffffffffll), (int)(key >> 32));
  c.rec[2 * i + 1] = make_int4(__float_as_int((float)(px - c.origin[0])), __float_as_int((float)(py - c.origin[1])),
                               __float_as_int((float)(pz - c.origin[2])), (int)i);
  c.cellh[i] = hsh;
  c.rank[i] = atomicAdd(c.bucket_count + hsh, 1);
}

// first record of bucket b (b up to the number of buckets in use): the scan
// leaves block-local sums and the sums before each block
__device__ __forceinline__ int bucket_begin(const ContactArgs& c, int64_t b) {
  return c.bucket_start[b] + c.bucket_top[b / kScanTile];
}

__global__ void k_scatter(ContactArgs c) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= c.n) return;
  const int r = c.rank[i];
  if (r < 0) return;
  const int at = bucket_begin(c, c.cellh[i]) + r;
  c.srec[at] = c.rec[2 * i];
  c.spos[at] = c.rec[2 * i + 1];
}

// What a bucket holds: kTagEmpty, the grain of all its nodes, or kTagMixed.  Most
// cells around a node hold nothing but its own grain; a 4-byte tag then stands
// for all their records.  (One entry more at either end, so that the search can
// read the three cells of a z-run as one.)
constexpr int kTagEmpty = -1, kTagMixed = -2;
__global__ __launch_bounds__(256) void k_tag(ContactArgs c) {
  const uint32_t nb = (uint32_t)c.grid[7];
  for (uint32_t b = blockIdx.x * 256 + threadIdx.x; b < nb; b += gridDim.x * 256) {
    int e = bucket_begin(c, b);
    const int e1 = bucket_begin(c, b + 1);
    int tag = kTagEmpty;
    if (e < e1) {
      tag = c.srec[e].y;
      while (++e < e1)
        if (c.srec[e].y != tag) {
          tag = kTagMixed;
          break;
        }
    }
    c.celltag[b + 1] = tag;
  }
}

// Search: the cells around a node that hold another grain's nodes.  Each workgroup
// first reads the tags around its records and keeps the nodes with such a cell (in
// a dense aggregate of 1000 grains, about half), then gives each of those a thread.
// In a dense grid a z-run of three cells is one range of records, cut to the cells
// that count.  Bound by the rate at which the vector cache serves 64 lanes' own
// addresses, so a record is one 16-byte load (FP32 position and node; its grain is
// told from the node's range), kRecs of them in flight; the nodes of other grains
// (with self-contact, all but itself) that may lie within the cutoff go to a row in
// LDS and are tested exactly in a second pass over it, kNear at a time, into the
// node's fixed-width scratch row.  Threads walk the binned nodes in bucket order,
// so neighbouring lanes read the same runs.  Counts beyond the scratch row's width
// raise the overflow flag.  Large aggregate (9.26 million nodes, cutoff 1.45 h):
// 0.95 ms; one thread per node over every record of the 27 cells, 32 bytes of u and
// of X each, took 1.89 ms.
constexpr int kRecs = 6, kNear = 6;
constexpr int kNearRow = 24;  // entries of a thread's row in LDS; a fuller one is tested record by record

// the exact test of the cnt nodes j(0), j(1), ...: out(node) for each within the cutoff
template <typename J, typename F>
__device__ __forceinline__ void near_nodes(const ContactArgs& c, const double4& ui, const double4& Xi, int cnt, J j,
                                           F out) {
  for (int q = 0; q < cnt; q += kNear) {
    int jj[kNear];
    double4 uj[kNear], Xj[kNear];
#pragma unroll
    for (int k = 0; k < kNear; ++k) jj[k] = j(q + k < cnt ? q + k : cnt - 1);
#pragma unroll
    for (int k = 0; k < kNear; ++k) {
      uj[k] = c.u[jj[k]];
      const double* xp = reinterpret_cast<const double*>(c.X4 + jj[k]);
      Xj[k] = make_double4(xp[0], xp[1], xp[2], 0.0);
    }
#pragma unroll
    for (int k = 0; k < kNear; ++k) {
      double yx, yy, yz;
      const double d2 = contact_d2(Xj[k].x, Xi.x, uj[k].x, ui.x, Xj[k].y, Xi.y, uj[k].y, ui.y, Xj[k].z, Xi.z, uj[k].z,
                                   ui.z, yx, yy, yz);
      if (q + k < cnt && d2 < c.cut2) out(jj[k]);
    }
  }
}

// the cell of a record
__device__ __forceinline__ void record_cell(const int4& r, int& cx, int& cy, int& cz) {
  const long long key = ((long long)r.w << 32) | (long long)(uint32_t)r.z;
  cx = (int)((key >> 42) & 0x1fffff) - (1 << 20);
  cy = (int)((key >> 21) & 0x1fffff) - (1 << 20);
  cz = (int)(key & 0x1fffff) - (1 << 20);
}

// Every record that may be a candidate of record me, run by run: f(node) for each
// that passes the FP32 test.  cells: bit 3 d + q of a dense grid's run d, cell z +
// q - 1, says that the cell may hold one.
template <typename F>
__device__ __forceinline__ void search_runs(const ContactArgs& c, const int4& me, const int4& pi, float lim2,
                                            uint32_t cells, F f) {
  int cx, cy, cz;
  record_cell(me, cx, cy, cz);
  // the nodes that do not count: those of the node's own grain, with
  // self-contact only itself (whether a pair is bonded is decided at the force,
  // from the bond memory)
  const uint32_t skip0 = c.self_contact ? (uint32_t)me.x : (uint32_t)c.grain_begin[me.y];
  const uint32_t skipn = c.self_contact ? 1u : (uint32_t)c.grain_begin[me.y + 1] - skip0;
  const float x = __int_as_float(pi.x), y = __int_as_float(pi.y), z = __int_as_float(pi.z);
  auto range = [&](int e, int e1, auto keyed, int klo, int khi) {
    for (; e < e1; e += kRecs) {
      int4 p[kRecs], r[kRecs];
#pragma unroll
      for (int k = 0; k < kRecs; ++k) {
        const int at = e + k < e1 ? e + k : e1 - 1;
        p[k] = c.spos[at];
        if (keyed) r[k] = c.srec[at];
      }
#pragma unroll
      for (int k = 0; k < kRecs; ++k) {
        const float dx = __int_as_float(p[k].x) - x, dy = __int_as_float(p[k].y) - y, dz = __int_as_float(p[k].z) - z;
        bool ok = e + k < e1 && (uint32_t)p[k].w - skip0 >= skipn && !(dx * dx + dy * dy + dz * dz > lim2);
        if (keyed) ok = ok && r[k].z == klo && r[k].w == khi;  // else another cell in the same bucket
        if (ok) f(p[k].w);
      }
    }
  };
  if (c.grid[0]) {
    const int ey = (int)c.grid[5], ez = (int)c.grid[6];
    const int lx = cx - (int)c.grid[1], ly = cy - (int)c.grid[2], lz = cz - (int)c.grid[3];
    const uint32_t b0 = ((uint32_t)lx * ey + ly) * ez + lz;
    int e0[9], e1[9];
#pragma unroll
    for (int d = 0; d < 9; ++d) {
      const uint32_t m = (cells >> (3 * d)) & 7u;
      // (a run without a bit is empty; its bounds are read from the node's own cell)
      const uint32_t b = m ? b0 + (uint32_t)((d / 3 - 1) * ey + (d % 3 - 1)) * ez : b0;
      e0[d] = bucket_begin(c, m ? b + (uint32_t)(__ffs(m) - 2) : b);
      e1[d] = m ? bucket_begin(c, b + (uint32_t)(31 - __clz(m))) : e0[d];
    }
#pragma unroll
    for (int d = 0; d < 9; ++d) range(e0[d], e1[d], std::false_type{}, 0, 0);
  } else {
    const int own = c.self_contact ? kTagEmpty : me.y;
    for (int d = 0; d < kCellDirs; ++d) {
      const int nx = cx + d % 3 - 1, ny = cy + (d / 3) % 3 - 1, nz = cz + d / 9 - 1;
      const long long nkey = cell_key(nx, ny, nz);
      const uint32_t b = cell_hash(nx, ny, nz, c.T);
      const int t = c.celltag[b + 1];
      if (t == kTagEmpty || t == own) continue;
      range(bucket_begin(c, b), bucket_begin(c, (int64_t)b + 1), std::true_type{}, (int)(nkey & 0xffffffffll),
            (int)(nkey >> 32));
    }
  }
}

// near: this thread's row in LDS, entries 256 apart
__device__ __forceinline__ void search_node(const ContactArgs& c, int e0, uint32_t cells, int* near) {
  const int4 me = c.srec[e0], pi = c.spos[e0];
  const float lim2 = __double2float_ru(c.origin[3]);
  const int64_t i = me.x;
  int32_t* row = c.cand_scratch + i * (int64_t)c.scratch_w;
  const double4 ui = c.u[i], Xi = c.X4[i];
  int cnt = 0, kept = 0;
  auto keep = [&](int j) {
    if (kept < c.scratch_w) row[kept] = j;
    ++kept;
  };
  search_runs(c, me, pi, lim2, cells, [&](int j) {
    if (cnt < kNearRow) near[256 * cnt] = j;
    ++cnt;
  });
  if (cnt <= kNearRow) {
    near_nodes(c, ui, Xi, cnt, [&](int k) { return near[256 * k]; }, keep);
  } else {
    search_runs(c, me, pi, lim2, cells, [&](int j) { near_nodes(c, ui, Xi, 1, [&](int) { return j; }, keep); });
  }
  if (kept > c.scratch_w) {
    atomicOr(c.status, ST_CAND_OVERFLOW);
    kept = c.scratch_w;
  }
  c.cand_count[i] = kept;
}

// per: records of a workgroup / 256.  More of them fill its wavefronts better
// with the nodes that are left to search, fewer leave more workgroups.
constexpr int kSearchPer = 4;
__global__ __launch_bounds__(256) void k_cand_search(ContactArgs c, int per) {
  __shared__ uint2 list[256 * kSearchPer];
  __shared__ int near[kNearRow * 256];
  __shared__ int listed;
  const int total = bucket_begin(c, c.grid[7]);
  const int64_t r0 = (int64_t)blockIdx.x * 256 * per;
  if (r0 >= total) return;
  if (threadIdx.x == 0) listed = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const bool dense = c.grid[0] != 0;
  const int ex = (int)c.grid[4], ey = (int)c.grid[5], ez = (int)c.grid[6];
  for (int k = 0; k < per; ++k) {
    const int64_t e0 = r0 + k * 256 + threadIdx.x;
    bool search = e0 < total;
    uint32_t cells = 0u;
    if (search && dense) {
      const int4 me = c.srec[e0];
      const int own = c.self_contact ? kTagEmpty : me.y;
      int cx, cy, cz;
      record_cell(me, cx, cy, cz);
      const int lx = cx - (int)c.grid[1], ly = cy - (int)c.grid[2], lz = cz - (int)c.grid[3];
      const uint32_t b0 = ((uint32_t)lx * ey + ly) * ez + lz;
      int tag[9][3];
#pragma unroll
      for (int d = 0; d < 9; ++d) {  // (no branch: all nine loads at once)
        const int nx = lx + d / 3 - 1, ny = ly + d % 3 - 1;
        const bool in = nx >= 0 && ny >= 0 && nx < ex && ny < ey;
        __builtin_memcpy(tag[d], c.celltag + (in ? ((uint32_t)nx * ey + ny) * ez + lz : b0), sizeof tag[d]);
        if (!in) tag[d][0] = tag[d][1] = tag[d][2] = kTagEmpty;
      }
#pragma unroll
      for (int d = 0; d < 9; ++d)
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          const bool in = (q != 0 || lz > 0) && (q != 2 || lz + 1 < ez);
          cells |= (in && tag[d][q] != kTagEmpty && tag[d][q] != own ? 1u : 0u) << (3 * d + q);
        }
      search = cells != 0u;
      if (!search) c.cand_count[me.x] = 0;
    }
    const uint64_t m = __ballot(search);
    if (m) {
      int at = 0;
      if (lane == __ffsll((unsigned long long)m) - 1) at = atomicAdd(&listed, __popcll(m));
      at = __shfl(at, __ffsll((unsigned long long)m) - 1, kWave) + __popcll(m & ((1ull << lane) - 1ull));
      if (search) list[at] = make_uint2((uint32_t)e0, cells);
    }
  }
  __syncthreads();
  const int n = listed;
  for (int q = threadIdx.x; q < n; q += 256) search_node(c, (int)list[q].x, list[q].y, near + threadIdx.x);
}

// ascending order of N values in registers (Batcher's odd-even merge network)
template <int N>
__device__ __forceinline__ void sort_network(int (&v)[N]) {
#pragma unroll
  for (int p = 1; p < N; p *= 2)
#pragma unroll
    for (int k = p; k >= 1; k /= 2)
#pragma unroll
      for (int j = k % p; j <= N - 1 - k; j += 2 * k)
#pragma unroll
        for (int i = 0; i < k; ++i)
          if (i + j + k < N && (i + j) / (2 * p) == (i + j + k) / (2 * p)) {
            const int lo = min(v[i + j], v[i + j + k]), hi = max(v[i + j], v[i + j + k]);
            v[i + j] = lo;
            v[i + j + k] = hi;
          }
}

// scratch row -> CSR row (ascending; rows past the total capacity are cut and
// flagged).  Rows of up to kSortRow candidates, nearly all of them, are read
// with every load in flight and sorted in registers; longer ones by insertion.
constexpr int kSortRow = 16;
__global__ __launch_bounds__(256) void k_cand_compact(ContactArgs c) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i > c.n) return;
  const int64_t base = c.cand_count[i] + c.cand_top[i / kScanTile];
  c.cand_ptr[i] = (int32_t)base;
  if (i == c.n) {
    if (base > c.capacity) atomicOr(c.status, ST_CAND_OVERFLOW);
    return;
  }
  const int cnt = (int)(c.cand_count[i + 1] + c.cand_top[(i + 1) / kScanTile] - base);
  if (cnt == 0) return;
  const int32_t* row = c.cand_scratch + i * (int64_t)c.scratch_w;
  const int64_t end = base + cnt < c.capacity ? base + cnt : c.capacity;
  if (cnt <= kSortRow && end == base + cnt) {
    int v[kSortRow];
#pragma unroll
    for (int k = 0; k < kSortRow; ++k) v[k] = row[k < cnt ? k : cnt - 1];
#pragma unroll
    for (int k = 0; k < kSortRow; ++k) v[k] = k < cnt ? v[k] : INT32_MAX;
    sort_network(v);
#pragma unroll
    for (int k = 0; k < kSortRow; ++k)
      if (k < cnt) c.cand[base + k] = v[k];
    return;
  }
  for (int64_t a = base; a < end; ++a) {
    const int32_t x = row[a - base];
    int64_t q = a - 1;
    while (q >= base && c.cand[q] > x) {
      c.cand[q + 1] = c.cand[q];
      --q;
    }
    c.cand[q + 1] = x;
  }
}

__global__ void k_fill_u4(double4* u4, const double* u, const int32_t* ijk, const int64_t* grain_of,
                          int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int64_t w = (int64_t)(uint32_t)(ijk[i] | (ijk[n + i] << 10) | (ijk[2 * n + i] << 20)) |
                    (grain_of[i] << 32);
  u4[i] = make_double4(u[i], u[n + i], u[2 * n + i], __longlong_as_double(w));
}

// ---------------------------------------------------------------------------
// exclusive scans (3 passes: block-local, block sums, add)
// ---------------------------------------------------------------------------

template <typename T>
__device__ T block_inclusive_scan(T x, T* s) {
  const int tid = threadIdx.x;
  s[tid] = x;
  __syncthreads();
  for (int o = 1; o < kScanThreads; o <<= 1) {
    const T t = tid >= o ? s[tid - o] : T(0);
    __syncthreads();
    s[tid] += t;
    __syncthreads();
  }
  return s[tid];
}

template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_scan_local(const T* in, T* out, int64_t n,
                                                             T* block_sums) {
  __shared__ T s[kScanThreads];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  T v[kScanItems];
  T tot = 0;
  for (int k = 0; k < kScanItems; ++k) {
    v[k] = base + k < n ? in[base + k] : T(0);
    tot += v[k];
  }
  const T inc = block_inclusive_scan(tot, s);
  T run = inc - tot;
  for (int k = 0; k < kScanItems; ++k) {
    if (base + k < n) out[base + k] = run;
    run += v[k];
  }
  if (threadIdx.x == kScanThreads - 1) block_sums[blockIdx.x] = inc;
}

template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_scan_top(T* block_sums, int64_t nb, T* total) {
  __shared__ T s[kScanThreads];
  T carry = 0;
  for (int64_t c = 0; c < nb; c += kScanThreads) {
    const int64_t idx = c + threadIdx.x;
    const T x = idx < nb ? block_sums[idx] : T(0);
    const T inc = block_inclusive_scan(x, s);
    if (idx < nb) block_sums[idx] = carry + inc - x;
    const T chunk = s[kScanThreads - 1];
    __syncthreads();
    carry += chunk;
  }
  if (threadIdx.x == 0) *total = carry;
}

// The rebuild's two scans, over n values that only the device knows: the same
// two passes, without the third - readers add the block's sum themselves.
// Buckets (n = those in use, one more value as the end): the counts are cleared
// as they are read, so they are zero when the next rebuild bins.  Candidate
// counts: in place, the value past the last node is the end.
template <bool BUCKETS>
__global__ __launch_bounds__(kScanThreads) void k_scan_rebuild(ContactArgs c) {
  __shared__ int32_t s[kScanThreads];
  const int64_t n = BUCKETS ? c.grid[7] : c.n;
  const int64_t tile0 = (int64_t)blockIdx.x * kScanTile;
  if (tile0 > n) return;
  const int64_t base = tile0 + (int64_t)threadIdx.x * kScanItems;
  int32_t* in = BUCKETS ? c.bucket_count : c.cand_count;
  int32_t* out = BUCKETS ? c.bucket_start : c.cand_count;
  int32_t v[kScanItems], tot = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) v[k] = in[base + k < n ? base + k : n - 1];
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    v[k] = base + k < n ? v[k] : 0;
    tot += v[k];
  }
  const int32_t inc = block_inclusive_scan(tot, s);
  int32_t run = inc - tot;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (base + k <= n) out[base + k] = run;
    if (BUCKETS && base + k < n) in[base + k] = 0;
    run += v[k];
  }
  if (threadIdx.x == kScanThreads - 1) (BUCKETS ? c.bucket_top : c.cand_top)[blockIdx.x] = inc;
}

template <bool BUCKETS>
__global__ __launch_bounds__(kScanThreads) void k_scan_rebuild_top(ContactArgs c) {
  __shared__ int32_t s[kScanThreads];
  const int64_t nb = (BUCKETS ? c.grid[7] : c.n) / kScanTile + 1;
  int32_t* sums = BUCKETS ? c.bucket_top : c.cand_top;
  int32_t carry = 0;
  for (int64_t b = 0; b < nb; b += kScanThreads) {
    const int64_t idx = b + threadIdx.x;
    const int32_t x = idx < nb ? sums[idx] : 0;
    const int32_t inc = block_inclusive_scan(x, s);
    if (idx < nb) sums[idx] = carry + inc - x;
    const int32_t chunk = s[kScanThreads - 1];
    __syncthreads();
    carry += chunk;
  }
}

template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_scan_add(T* out, int64_t n, const T* block_sums) {
  const T add = block_sums[blockIdx.x];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  for (int k = 0; k < kScanItems; ++k)
    if (base + k < n) out[base + k] += add;
}

__global__ void k_pack_x4(const double* X, double4* X4, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) X4[i] = make_double4(X[i], X[n + i], X[2 * n + i], 0.0);
}

// the fields of pd_get that are not stored the way they are handed out, made on
// the device (56 bytes of u and 16 of counts per node at copy rate; taken through
// host memory, u of 9.26 million nodes cost about 80 ms)
__global__ void k_unpack_u(const double4* u4, double* out, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double4 u = u4[i];
  out[i] = u.x;
  out[n + i] = u.y;
  out[2 * n + i] = u.z;
}

__global__ void k_split_u(const double4* u4, double2* uxy, double* uz, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double4 u = u4[i];
  uxy[i] = make_double2(u.x, u.y);
  uz[i] = u.z;
}

__global__ void k_damage(const int32_t* intact, const int32_t* initial, double* out, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int32_t n0 = initial[i];
  out[i] = n0 > 0 ? 1.0 - (double)intact[i] / (double)n0 : 0.0;
}

hipError_t launch_unpack_u(const double4* u4, double* out, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_unpack_u, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, u4, out, n);
  return hipGetLastError();
}

hipError_t launch_split_u(const double4* u4, double2* uxy, double* uz, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_split_u, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, u4, uxy, uz, n);
  return hipGetLastError();
}

hipError_t launch_damage(const int32_t* intact, const int32_t* initial, double* out, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_damage, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, intact, initial, out, n);
  return hipGetLastError();
}

__global__ void k_fill_i32_kernel(int32_t* p, int32_t v, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_i32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}

hipError_t launch_pack_x4(const double* X, double4* X4, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_pack_x4, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, X, X4, n);
  return hipGetLastError();
}

template <typename T>
__global__ void k_set_value(T* p, T v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}

int64_t scan_scratch_elems(int64_t n) { return (n + kScanTile - 1) / kScanTile + 1; }

template <typename T>
static hipError_t scan_impl(const T* in, T* out, int64_t n, T* scratch, hipStream_t s) {
  if (n <= 0) {
    hipLaunchKernelGGL(k_set_value<T>, dim3(1), dim3(64), 0, s, out, T(0));
    return hipGetLastError();
  }
  const int64_t nb = (n + kScanTile - 1) / kScanTile;
  hipLaunchKernelGGL(k_scan_local<T>, dim3((unsigned)nb), dim3(kScanThreads), 0, s, in, out, n, scratch);
  hipLaunchKernelGGL(k_scan_top<T>, dim3(1), dim3(kScanThreads), 0, s, scratch, nb, out + n);
  hipLaunchKernelGGL(k_scan_add<T>, dim3((unsigned)nb), dim3(kScanThreads), 0, s, out, n,
                     (const T*)scratch);
  return hipGetLastError();
}

hipError_t scan_i64(const int64_t* in, int64_t* out, int64_t n, int64_t* scratch, hipStream_t s) {
  return scan_impl<int64_t>(in, out, n, scratch, s);
}
// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

static inline unsigned grid_for(int64_t n, int threads) {
  return (unsigned)((n + threads - 1) / threads);
}

hipError_t launch_map_fill(const BuildArgs& b, hipStream_t s) {
  if (b.n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_map_fill, dim3(grid_for(b.n, 256)), dim3(256), 0, s, b);
  return hipGetLastError();
}
hipError_t launch_bond_count(const BuildArgs& b, hipStream_t s) {
  if (b.n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_bond_count, dim3(grid_for(b.n, 256)), dim3(256), 0, s, b);
  return hipGetLastError();
}
hipError_t launch_slice_width(const BuildArgs& b, hipStream_t s) {
  if (b.nslices == 0) return hipSuccess;
  hipLaunchKernelGGL(k_slice_width, dim3(grid_for(b.nslices, 256)), dim3(256), 0, s, b);
  return hipGetLastError();
}
hipError_t launch_bond_fill(const BuildArgs& b, hipStream_t s) {
  if (b.nslices == 0) return hipSuccess;
  hipLaunchKernelGGL(k_bond_fill, dim3(grid_for(b.nslices, kSlicesPerBlock)), dim3(kBlock), 0, s, b);
  return hipGetLastError();
}

hipError_t launch_align_width(const AlignArgs& a, hipStream_t s) {
  if (a.nslices == 0) return hipSuccess;
  hipLaunchKernelGGL(k_align<false>, dim3(grid_for(a.nslices, kSlicesPerBlock)), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_align_fill(const AlignArgs& a, hipStream_t s) {
  if (a.nslices == 0) return hipSuccess;
  hipLaunchKernelGGL(k_align<true>, dim3(grid_for(a.nslices, kSlicesPerBlock)), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_lined_to_cols(const AlignArgs& a, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_lined_to_cols, dim3(grid_for(a.n, 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

int32_t step_blocks_spb(int64_t nslices, int slices_per_block) {
  return (int32_t)grid_for(nslices, slices_per_block);
}
int32_t step_grid_blocks(int64_t nslices) { return step_blocks_spb(nslices, kSlicesPerBlock); }

hipError_t launch_wall_finalize(const StepArgs& a, hipStream_t s) {
  const int64_t nq = (a.partial_stride + kChunk - 1) / kChunk;
  if (nq <= kFusedChunks) {
    hipLaunchKernelGGL(k_wall_finalize_small, dim3(1), dim3(1024), 0, s, a);
    return hipGetLastError();
  }
  if (a.n_walls > 0) hipLaunchKernelGGL(k_wall_chunks, dim3((unsigned)nq), dim3(kWave), 0, s, a);
  hipLaunchKernelGGL(k_wall_finalize, dim3(1), dim3(1024), 0, s, a);
  return hipGetLastError();
}

static size_t step_lds(const StepArgs& a) {
  return sizeof(StencilC) * (size_t)(a.n_stencil + 1) * (size_t)a.n_classes;
}

template <int MODE, int SPB, int DEPTH, bool LINED>
static void launch_step_d(const StepArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const int32_t nb = step_blocks_spb(a.slice_end - a.slice_base, SPB);
  if (nb == 0) return;
  void (*kern)(StepArgs) = a.abs_stretch ? k_step<MODE, true, SPB, DEPTH, LINED> : k_step<MODE, false, SPB, DEPTH, LINED>;
  // with events, the launch itself records them around the kernel
  if (e0 || e1) hipExtLaunchKernelGGL(kern, dim3(nb), dim3(SPB * kWave), step_lds(a), s, e0, e1, 0, a);
  else hipLaunchKernelGGL(kern, dim3(nb), dim3(SPB * kWave), step_lds(a), s, a);
}

// the deep pipeline up to one slice for each of the chip's 1024 SIMDs (with two
// each, 125,000 nodes, it took 46 us against 43)
constexpr int64_t kDeepSlices = 1024;
template <int MODE, int SPB>
static void launch_step_t(const StepArgs& a, hipStream_t s, hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr) {
  const bool deep = a.slice_end - a.slice_base <= kDeepSlices;
  if constexpr (MODE == MODE_STEP) {
    if (a.lined) return launch_step_d<MODE, SPB, 2, true>(a, s, e0, e1);
    // (so few slices never run eight to a workgroup, see launch_step_spb)
    if constexpr (SPB < 8)
      if (deep) return launch_step_d<MODE, SPB, 4, false>(a, s, e0, e1);
  }
  launch_step_d<MODE, SPB, 2, false>(a, s, e0, e1);
}

hipError_t launch_step(const StepArgs& a, int mode, hipStream_t s) {
  if (mode == MODE_FIRST) launch_step_t<MODE_FIRST, kSlicesPerBlock>(a, s);
  else if (mode == MODE_STEP) launch_step_t<MODE_STEP, kSlicesPerBlock>(a, s);
  else launch_step_t<MODE_FORCE_ONLY, kSlicesPerBlock>(a, s);
  return hipGetLastError();
}

// A mesh with fewer workgroups than compute units is spread out: the wavefronts of a
// workgroup share one vector cache while others stand idle (131 slices: 21.6 us
// a launch with one each, 23.0 with four; even from 1,964 slices on).
// The wall partials are per slice, so the results do not depend on it.
constexpr int64_t kCUs = 256;
hipError_t launch_step_spb(const StepArgs& a, int slices_per_block, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const int64_t slices = a.slice_end - a.slice_base;
  while (slices_per_block > 1 && slices_per_block <= 8 && (slices - 1) / slices_per_block < kCUs - 1)
    slices_per_block /= 2;
  switch (slices_per_block) {
    case 1: launch_step_t<MODE_STEP, 1>(a, s, e0, e1); break;
    case 2: launch_step_t<MODE_STEP, 2>(a, s, e0, e1); break;
    case 4: launch_step_t<MODE_STEP, 4>(a, s, e0, e1); break;
    case 8: launch_step_t<MODE_STEP, 8>(a, s, e0, e1); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

int32_t persistent_max_blocks(const StepArgs& a) {
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  const void* fn = a.abs_stretch ? reinterpret_cast<const void*>(&k_step_persistent<true>)
                                 : reinterpret_cast<const void*>(&k_step_persistent<false>);
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 4 * kWave, step_lds(a)) != hipSuccess)
    return 0;
  return per_cu * cus;
}

hipError_t launch_step_persistent(const StepArgs& a, int64_t nsteps, int32_t nblocks, const BarrierArgs& b,
                                  hipStream_t s) {
  if (nsteps <= 0) return hipSuccess;
  if (step_blocks_spb(a.slice_end - a.slice_base, 4) == 0) return hipSuccess;
  StepArgs aa = a;
  BarrierArgs bb = b;
  void* args[] = {&aa, &nsteps, &bb};
  const void* fn = a.abs_stretch ? reinterpret_cast<const void*>(&k_step_persistent<true>)
                                 : reinterpret_cast<const void*>(&k_step_persistent<false>);
  // a cooperative launch fails rather than start more workgroups than can be
  // resident at once, which the grid barrier relies on
  return hipLaunchCooperativeKernel(fn, dim3((unsigned)nblocks), dim3(4 * kWave), args,
                                    (unsigned)step_lds(a), s);
}

// early-rebuild watch, before an evaluation between cadence rebuilds: a node
// beyond skin/2 of where the list was built may have a partner within R_c
// that the list lacks.  The flag halts this step and the ones after it (the
// step kernel and the wall pass see the halt word), so the host can rebuild
// the list at these positions and go on from the same step.
__global__ void k_skin_watch(ContactArgs c, uint32_t* halt) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= c.n || halted(c.halt)) return;
  const double4 u = c.u[i];
  const double dx = u.x - c.u_build[i], dy = u.y - c.u_build[c.n + i], dz = u.z - c.u_build[2 * c.n + i];
  if (dx * dx + dy * dy + dz * dz > c.skin_half2) {
    atomicOr(c.status, ST_REBUILD);
    atomicOr(halt, ST_REBUILD);
  }
}

hipError_t launch_skin_watch(const ContactArgs& c, uint32_t* halt, hipStream_t s) {
  if (c.n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_skin_watch, dim3(grid_for(c.n, 256)), dim3(256), 0, s, c, halt);
  return hipGetLastError();
}

hipError_t launch_contact_rebuild(const ContactArgs& c, int check_skin, hipStream_t s) {
  if (c.n == 0) return hipSuccess;
  const unsigned g = grid_for(c.n, 256);
  if (c.n_grains == 1 && !c.self_contact) {  // nothing can touch: only the positions of the rebuild are kept
    hipLaunchKernelGGL(k_skin, dim3(g), dim3(256), 0, s, c, check_skin);
    return hipGetLastError();
  }
  // boxes inflated by the cutoff, and by more than positions are rounded (p = X + u, at up to
  // 1e9 cutoffs from the origin)
  const double cut = sqrt(c.cut2) * (1.0 + 1e-6) + 1e-300;
  const unsigned gg = (unsigned)c.n_grains;
  hipLaunchKernelGGL(k_box_init, dim3(grid_for(6 * (int64_t)c.n_grains, 256)), dim3(256), 0, s, c);
  hipLaunchKernelGGL(k_skin_box, dim3((unsigned)c.n_box_chunks), dim3(256), 0, s, c, check_skin);
  hipLaunchKernelGGL(k_near_boxes, dim3(gg), dim3(kWave), 0, s, c, cut);
  hipLaunchKernelGGL(k_grid_setup, dim3(1), dim3(kWave), 0, s, c);
  hipLaunchKernelGGL(k_bin, dim3(g), dim3(256), 0, s, c);
  hipLaunchKernelGGL(k_scan_rebuild<true>, dim3((unsigned)((int64_t)c.T / kScanTile + 1)), dim3(kScanThreads), 0, s, c);
  hipLaunchKernelGGL(k_scan_rebuild_top<true>, dim3(1), dim3(kScanThreads), 0, s, c);
  hipLaunchKernelGGL(k_scatter, dim3(g), dim3(256), 0, s, c);
  hipLaunchKernelGGL(k_tag, dim3(std::min(grid_for((int64_t)c.T, 256), 8192u)), dim3(256), 0, s, c);
  // four records a thread once that still leaves every CU eight wavefronts a SIMD
  const int per = c.n >= (int64_t)256 * kSearchPer * 2048 ? kSearchPer : 1;
  hipLaunchKernelGGL(k_cand_search, dim3(grid_for(c.n, 256 * per)), dim3(256), 0, s, c, per);
  hipLaunchKernelGGL(k_scan_rebuild<false>, dim3((unsigned)(c.n / kScanTile + 1)), dim3(kScanThreads), 0, s, c);
  hipLaunchKernelGGL(k_scan_rebuild_top<false>, dim3(1), dim3(kScanThreads), 0, s, c);
  hipLaunchKernelGGL(k_cand_compact, dim3(grid_for(c.n + 1, 256)), dim3(256), 0, s, c);
  return hipGetLastError();
}

hipError_t launch_energy(const StepArgs& a, double* partial4, int32_t nblocks, hipStream_t s) {
  if (nblocks == 0) return hipSuccess;
  hipLaunchKernelGGL(k_energy, dim3(nblocks), dim3(kBlock), 0, s, a, partial4);
  return hipGetLastError();
}

hipError_t launch_reduce_energy(const double* partial4, int32_t nblocks, double* out4,
                                hipStream_t s) {
  hipLaunchKernelGGL(k_reduce_energy, dim3(1), dim3(64), 0, s, partial4, nblocks, out4);
  return hipGetLastError();
}

template <bool ABS, bool EXTRA>
void launch_tile_variant(const StepArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const dim3 grid((unsigned)a.n_tiles), block(kTS * kWave);
  void (*kern)(StepArgs) = k_step_tile<ABS, EXTRA>;
  if (e0 || e1) hipExtLaunchKernelGGL(kern, grid, block, 0, s, e0, e1, 0, a);
  else hipLaunchKernelGGL(kern, grid, block, 0, s, a);
}

hipError_t launch_step_tile(const StepArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (a.n_tiles == 0) return hipSuccess;
  const bool extra = a.self_contact || a.wall_corners;
  if (a.abs_stretch) {
    if (extra) launch_tile_variant<true, true>(a, s, e0, e1);
    else launch_tile_variant<true, false>(a, s, e0, e1);
  } else {
    if (extra) launch_tile_variant<false, true>(a, s, e0, e1);
    else launch_tile_variant<false, false>(a, s, e0, e1);
  }
  return hipGetLastError();
}

hipError_t launch_tile_map_fill(const StepArgs& a, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_tile_map_fill, dim3(grid_for(a.n, 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_cols_to_mask(const StepArgs& a, const int16_t* ctob, const uint32_t* colOrig, hipStream_t s) {
  if (a.n_tiles == 0) return hipSuccess;
  hipLaunchKernelGGL(k_cols_to_mask, dim3(grid_for(a.n_tiles * kTS * kWave, 256)), dim3(256), 0, s, a, ctob, colOrig);
  return hipGetLastError();
}

hipError_t launch_mask_to_cols(const StepArgs& a, const int16_t* ctob, const uint32_t* colOrig, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_mask_to_cols, dim3(grid_for(a.n, 256)), dim3(256), 0, s, a, ctob, colOrig);
  return hipGetLastError();
}

hipError_t launch_wall_corners(const StepArgs& a, int force_only, hipStream_t s) {
  if (a.n == 0 || !a.wall_corners) return hipSuccess;
  hipLaunchKernelGGL(k_wall_corners, dim3(grid_for(a.n, 256)), dim3(256), 0, s, a, force_only);
  return hipGetLastError();
}

hipError_t launch_fill_u4(double4* u4, const double* u, const int32_t* ijk, const int64_t* grain_of,
                          int64_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_u4, dim3(grid_for(n, 256)), dim3(256), 0, s, u4, u, ijk, grain_of, n);
  return hipGetLastError();
}

}  // namespace pdk
