// libnep: HIP kernels and C ABI for one NEP loss-and-gradient evaluation on
// MI355X (gfx950).  The declarations and contracts are in include/nep.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "../../include/nep.h"
#include "nep_kernels.h"

namespace nep {

// =============================================================== neighbors
// The lists of an atom i hold the (j, s) of its own structure that pass the
// float64 predicate of Eq. 2, evaluated without fused multiply-add, in canonical
// order: j ascending, then the shifts in code order.  Where a cell may hold
// several images of j within rc, the per-axis test |(x_j - x_i) + s L| < rc
// keeps the candidate shifts and each is tested.
//
// IEEE double product and sum with one rounding each.  The library is built
// with floating-point contraction, and d^2 = (dx dx + dy dy) + dz dz of the
// predicate must not become fused multiply-adds (a pair within an ulp of rc
// can change sides), so the squares and their sums are single instructions
// the compiler cannot merge.
__device__ __forceinline__ double mul_d(double a, double b) {
  double r;
  asm("v_mul_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double add_d(double a, double b) {
  double r;
  asm("v_add_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double dist2_d(double dx, double dy, double dz) {
  return add_d(add_d(mul_d(dx, dx), mul_d(dy, dy)), mul_d(dz, dz));
}

__device__ __forceinline__ unsigned axis_candidates(double d0, double L, double rc) {
  unsigned m = 0;
  if (fabs(__dadd_rn(d0, -L)) < rc) m |= 1u;
  if (fabs(d0) < rc) m |= 2u;
  if (fabs(__dadd_rn(d0, L)) < rc) m |= 4u;
  return m;
}

// One atom per group of 8 lanes; lane s scans the s-th contiguous eighth of
// the atom's structure, so concatenating the lanes' entries in lane order
// keeps the canonical (j, code) order.
//
// Fast decision.  When every cell edge is at least 2(rc + delta) and at most
// kNbrFastL, at most one image of j lies within rc + delta, and the single
// precision minimum image finds it.  Its squared distance is then within
// 3e-3 A^2 of the float64 value, far inside the margins of the shell
// |r - rc| < delta = 0.01 A (at least 0.0199 A^2 for rc >= 1 A), so pairs
// outside the shell are decided in single precision and only pairs in the
// shell, and every pair of smaller or larger cells, take the float64 test.
//
// Positions of the atoms j that a block's 32 atoms scan are staged in LDS in
// tiles of kNbrTile atoms; every lane of the block walks the same tiles.
constexpr int kNbrThreads = 256;   // threads per block
constexpr int kNbrAPB = kNbrThreads / 8;   // atoms per block
constexpr int kNbrTile = 1024;
constexpr int kNbrBuf = 24;   // entries buffered per lane (angular mask: 32 bits), plus a scratch slot
constexpr float kNbrDelta = 0.01f;
constexpr float kNbrFastL = 512.0f;

struct ScanCtx {
  int i;
  double xi, yi, zi, Lx, Ly, Lz, xy, xz, yz, rcR, rcR2, rcA2;
  float xf, yf, zf, Lxf, Lyf, Lzf, xyf, xzf, yzf, ilx, ily, ilz;
  float inR2, outR2, inA2, outA2;
  bool fast;
};

// a tile of positions in LDS holding atoms [base, base + kNbrTile)
struct PosTile {
  const float* x;
  const float* y;
  const float* z;
  int base;
};

// LDS written by one lane and read by another lane of the same wavefront: a
// wavefront's LDS instructions complete in issue order, so it is enough that
// the compiler keeps every memory access on its side of this point.
__device__ __forceinline__ void lds_lane_exchange() { asm volatile("" ::: "memory"); }
// Block barrier that orders LDS only: __syncthreads would also wait for the
// wavefront's outstanding global stores.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// A value the compiler cannot see through.  The float64 paths below run for
// few candidates of the single-image scan; taking their inputs through this
// keeps their conversions inside the branch instead of being computed ahead
// of the test for every candidate.
__device__ __forceinline__ int opaque_int(int v) {
  asm volatile("" : "+v"(v));
  return v;
}
__device__ __forceinline__ float opaque_float(float v) {
  asm volatile("" : "+v"(v));
  return v;
}

// float64 predicate of Eq. 2 for the pair (i, j) over the candidate shifts;
// calls emit(j, code, is_angular) in ascending code order
template <class Emit>
__device__ __forceinline__ void exact_pair(const ScanCtx& c, const PosTile& t, int j, Emit& emit) {
  const int q = opaque_int(j - t.base);
  const double x0 = __dadd_rn((double)t.x[q], -c.xi);
  const unsigned mx = axis_candidates(x0, c.Lx, c.rcR);
  if (!mx) return;
  const double y0 = __dadd_rn((double)t.y[q], -c.yi);
  const unsigned my = axis_candidates(y0, c.Ly, c.rcR);
  if (!my) return;
  const double z0 = __dadd_rn((double)t.z[q], -c.zi);
  const unsigned mz = axis_candidates(z0, c.Lz, c.rcR);
  if (!mz) return;
  for (unsigned bx = mx; bx; bx &= bx - 1u) {
    const int sx = __builtin_ctz(bx);
    const double dx = sx == 1 ? x0 : __dadd_rn(x0, sx == 0 ? -c.Lx : c.Lx);
    const double dx2 = mul_d(dx, dx);
    for (unsigned by = my; by; by &= by - 1u) {
      const int sy = __builtin_ctz(by);
      const double dy = sy == 1 ? y0 : __dadd_rn(y0, sy == 0 ? -c.Ly : c.Ly);
      const double dxy = add_d(dx2, mul_d(dy, dy));
      for (unsigned bz = mz; bz; bz &= bz - 1u) {
        const int sz = __builtin_ctz(bz);
        const int code = 9 * sx + 3 * sy + sz;
        const double dz = sz == 1 ? z0 : __dadd_rn(z0, sz == 0 ? -c.Lz : c.Lz);
        const double d2 = add_d(dxy, mul_d(dz, dz));
        if (d2 < c.rcR2 && !(j == c.i && code == 13)) emit(j, code, d2 < c.rcA2);
      }
    }
  }
}

// The same predicate in a triclinic cell with edge vectors a = (Lx, 0, 0),
// b = (xy, Ly, 0), c = (xz, yz, Lz): d = (x_j - x_i) + sa a + sb b + sc c with
// each component summed left to right, dx = ((x0 + sa Lx) + sb xy) + sc xz,
// dy = (y0 + sb Ly) + sc yz, dz = z0 + sc Lz (the products are exact).  dz
// prunes sc, dy prunes (sb, sc), then dx is formed per surviving shift.
template <class Emit>
__device__ __forceinline__ void exact_pair_tri(const ScanCtx& c, const PosTile& t, int j, Emit& emit) {
  const int q = opaque_int(j - t.base);
  const double z0 = __dadd_rn((double)t.z[q], -c.zi);
  const unsigned mz = axis_candidates(z0, c.Lz, c.rcR);
  if (!mz) return;
  const double y0 = __dadd_rn((double)t.y[q], -c.yi);
  double dyv[9], dzv[3];
#pragma unroll
  for (int sc = 0; sc < 3; ++sc) dzv[sc] = sc == 1 ? z0 : __dadd_rn(z0, sc == 0 ? -c.Lz : c.Lz);
  unsigned myz = 0;
#pragma unroll
  for (int sb = 0; sb < 3; ++sb) {
    const double yb = sb == 1 ? y0 : __dadd_rn(y0, sb == 0 ? -c.Ly : c.Ly);
#pragma unroll
    for (int sc = 0; sc < 3; ++sc) {
      const double dy = sc == 1 ? yb : __dadd_rn(yb, sc == 0 ? -c.yz : c.yz);
      dyv[3 * sb + sc] = dy;
      myz |= (((mz >> sc) & 1u) && fabs(dy) < c.rcR) ? (1u << (3 * sb + sc)) : 0u;
    }
  }
  if (!myz) return;
  const double x0 = __dadd_rn((double)t.x[q], -c.xi);
#pragma unroll
  for (int sa = 0; sa < 3; ++sa) {
    const double xa = sa == 1 ? x0 : __dadd_rn(x0, sa == 0 ? -c.Lx : c.Lx);
#pragma unroll
    for (int sb = 0; sb < 3; ++sb) {
      const double xb = sb == 1 ? xa : __dadd_rn(xa, sb == 0 ? -c.xy : c.xy);
#pragma unroll
      for (int sc = 0; sc < 3; ++sc) {
        if (!((myz >> (3 * sb + sc)) & 1u)) continue;
        const double dx = sc == 1 ? xb : __dadd_rn(xb, sc == 0 ? -c.xz : c.xz);
        const double dy = dyv[3 * sb + sc], dz = dzv[sc];
        const double d2 = dist2_d(dx, dy, dz);
        const int code = 9 * sa + 3 * sb + sc;
        if (d2 < c.rcR2 && !(j == c.i && code == 13)) emit(j, code, d2 < c.rcA2);
      }
    }
  }
}

template <bool kTri, class Emit>
__device__ __forceinline__ void exact_any(const ScanCtx& c, const PosTile& t, int j, Emit& emit) {
  if constexpr (kTri)
    exact_pair_tri(c, t, j, emit);
  else
    exact_pair(c, t, j, emit);
}

// Single-precision minimum image: e = x_j - x_i minus the lattice vector
// H k, k the rounded fractional coordinates of e (H upper triangular, so
// f_c = e_z / Lz, f_b = (e_y - yz f_c) / Ly, f_a = (e_x - xy f_b - xz f_c) / Lx).
// In an orthorhombic cell this is the per-axis rounding.
template <bool kTri>
__device__ __forceinline__ void min_image(const ScanCtx& c, float& ex, float& ey, float& ez, float& kx, float& ky,
                                          float& kz) {
  if constexpr (kTri) {
    const float fc = ez * c.ilz;
    const float fb = (ey - c.yzf * fc) * c.ily;
    const float fa = (ex - c.xyf * fb - c.xzf * fc) * c.ilx;
    kx = rintf(fa);
    ky = rintf(fb);
    kz = rintf(fc);
    ex = ex - c.Lxf * kx - c.xyf * ky - c.xzf * kz;
    ey = ey - c.Lyf * ky - c.yzf * kz;
    ez -= c.Lzf * kz;
  } else {
    kx = rintf(ex * c.ilx);
    ky = rintf(ey * c.ily);
    kz = rintf(ez * c.ilz);
    ex -= c.Lxf * kx;
    ey -= c.Lyf * ky;
    ez -= c.Lzf * kz;
  }
}

// float64 squared length of the image s = -k of j, in the predicate's order
// (the products k L are exact, k being 0 or +-1, so contracting them is harmless)
template <bool kTri>
__device__ __forceinline__ double image_d2(const ScanCtx& c, float px, float py, float pz, float kx, float ky,
                                           float kz) {
  double dx = __dadd_rn(__dadd_rn((double)px, -c.xi), -(double)kx * c.Lx);
  double dy = __dadd_rn(__dadd_rn((double)py, -c.yi), -(double)ky * c.Ly);
  const double dz = __dadd_rn(__dadd_rn((double)pz, -c.zi), -(double)kz * c.Lz);
  if constexpr (kTri) {
    dx = __dadd_rn(__dadd_rn(dx, -(double)ky * c.xy), -(double)kz * c.xz);
    dy = __dadd_rn(dy, -(double)kz * c.yz);
  }
  return dist2_d(dx, dy, dz);
}

template <bool kTri, class Emit>
__device__ __forceinline__ void scan_range(const ScanCtx& c, const PosTile& t, int jb, int je, Emit& emit) {
  for (int j = jb; j < je; ++j) {
    if (c.fast) {
      const int q = j - t.base;
      const float px = t.x[q], py = t.y[q], pz = t.z[q];
      float ex = px - c.xf, ey = py - c.yf, ez = pz - c.zf, kx, ky, kz;
      min_image<kTri>(c, ex, ey, ez, kx, ky, kz);
      const float r2 = ex * ex + ey * ey + ez * ez;
      if (r2 >= c.outR2) continue;
      if (r2 < c.inR2 && fabsf(kx) <= 1.f && fabsf(ky) <= 1.f && fabsf(kz) <= 1.f) {
        // shift s = -k on each axis; code 9(sx+1) + 3(sy+1) + (sz+1)
        const int code = 9 * (1 - (int)kx) + 3 * (1 - (int)ky) + (1 - (int)kz);
        if (j == c.i && code == 13) continue;
        bool ang = r2 < c.inA2;
        if (!ang && r2 < c.outA2) ang = image_d2<kTri>(c, px, py, pz, kx, ky, kz) < c.rcA2;
        emit(j, code, ang);
        continue;
      }
    }
    exact_any<kTri>(c, t, j, emit);
  }
}

// The buffered decision of one candidate j at (px, py, pz).  Outside the
// shell it is made without branches: the entry is written to the lane's next
// buffer slot and the count only advances when the pair is inside, so a
// later entry overwrites a rejected one (slot kNbrBuf takes the writes once
// the buffer is full).  Pairs in the shell branch to the float64 predicate.
template <bool kTri, class Keep>
__device__ __forceinline__ void keep_one(const ScanCtx& c, const PosTile& t, int j, float px, float py, float pz,
                                         uint32_t* buf, int& nR, int& nA, uint32_t& angmask, Keep& keep) {
  float ex = px - c.xf, ey = py - c.yf, ez = pz - c.zf, kx, ky, kz;
  min_image<kTri>(c, ex, ey, ez, kx, ky, kz);
  const float r2 = ex * ex + ey * ey + ez * ez;
  // k is 0 or +-1 for positions inside the cell (the position flag's
  // condition), so the shift s = -k always has a code
  const int code = 13 - (int)fmaf(9.f, kx, fmaf(3.f, ky, kz));
  const bool decided = r2 < c.inR2;
  const bool in = decided & ((j != c.i) | (code != 13));   // bitwise: no branch per candidate
  bool ang = r2 < c.inA2;
  buf[kNbrThreads * min(nR, kNbrBuf)] = ((uint32_t)j << 5) | (uint32_t)(code & 31);
  if (in && !ang && r2 < c.outA2)
    ang = image_d2<kTri>(c, opaque_float(px), opaque_float(py), opaque_float(pz), kx, ky, kz) < c.rcA2;
  angmask |= (in && ang && nR < kNbrBuf) ? (1u << nR) : 0u;
  nR += in ? 1 : 0;
  nA += (in && ang) ? 1 : 0;
  if (!decided && r2 < c.outR2) exact_any<kTri>(c, t, j, keep);
}

// The buffered scan of the single pass over [jb, je); cells too small or too
// large for the single-image test take the float64 predicate for every pair.
template <bool kTri, class Keep>
__device__ __forceinline__ void scan_keep(const ScanCtx& c, const PosTile& t, int jb, int je, uint32_t* buf,
                                          int& nR, int& nA, uint32_t& angmask, Keep& keep) {
  // one loop per case: a shared loop let the float64 coordinate differences
  // of the exact path be computed ahead of the test for every candidate
  if (!c.fast) {
    for (int j = jb; j < je; ++j) exact_any<kTri>(c, t, j, keep);
    return;
  }
  for (int j = jb; j < je; ++j) {
    const int q = j - t.base;
    keep_one<kTri>(c, t, j, t.x[q], t.y[q], t.z[q], buf, nR, nA, angmask, keep);
  }
}

// Triclinic cells.  Every neighbor lies among the 27 images when the
// positions' fractional coordinates are in [0, 1) and each perpendicular
// width of the cell is at least rc: the fractional coordinates of a vector
// shorter than rc are then below 1 in magnitude.  Positions are accepted with
// fractional coordinates in [-kFracTol, 1 + kFracTol) and widths from
// rc / (1 - 2 kFracTol) up, which keeps the same bound.  The single-image fast
// decision needs each width at least 2 (rc + delta): an image within
// rc + delta then has fractional coordinates of magnitude below 1/2 by a
// margin of delta / (2 (rc + delta)), so the rounded fractional coordinates
// select it.
constexpr double kFracTol = 1e-5;

struct CellCheck {
  bool box_ok, pos_ok, fast_ok;
};

// perpendicular widths V / |b x c|, V / |c x a|, V / |a x b| of the cell
__device__ __forceinline__ void cell_widths(const ScanCtx& c, double& ha, double& hb, double& hc) {
  const double bc_x = c.Ly * c.Lz, bc_y = -c.xy * c.Lz, bc_z = c.xy * c.yz - c.Ly * c.xz;
  const double V = c.Lx * c.Ly * c.Lz;
  ha = fabs(V) / sqrt(bc_x * bc_x + bc_y * bc_y + bc_z * bc_z);
  hb = fabs(c.Ly * c.Lz) / sqrt(c.Lz * c.Lz + c.yz * c.yz);
  hc = fabs(c.Lz);
}

template <bool kTri>
__device__ __forceinline__ CellCheck check_cell(const ScanCtx& c, float rcR, float rcA) {
  CellCheck k;
  const float wide = 2.0f * (rcR + kNbrDelta);
  const bool small = c.Lxf <= kNbrFastL && c.Lyf <= kNbrFastL && c.Lzf <= kNbrFastL && rcA >= 1.0f;
  const bool tilted = kTri && (c.xyf != 0.f || c.xzf != 0.f || c.yzf != 0.f);
  if (!tilted) {
    k.pos_ok = c.xf >= 0.f && c.xf < c.Lxf && c.yf >= 0.f && c.yf < c.Lyf && c.zf >= 0.f && c.zf < c.Lzf;
    k.box_ok = c.Lxf >= rcR && c.Lyf >= rcR && c.Lzf >= rcR;
    k.fast_ok = c.Lxf >= wide && c.Lyf >= wide && c.Lzf >= wide && small;
    return k;
  }
  double ha, hb, hc;
  cell_widths(c, ha, hb, hc);
  const double hmin = fmin(ha, fmin(hb, hc));
  k.box_ok = c.Lxf > 0.f && c.Lyf > 0.f && c.Lzf > 0.f && hmin * (1.0 - 2.0 * kFracTol) >= (double)rcR;
  const double fc = c.zi / c.Lz;
  const double fb = (c.yi - c.yz * fc) / c.Ly;
  const double fa = (c.xi - c.xy * fb - c.xz * fc) / c.Lx;
  k.pos_ok = fa >= -kFracTol && fa < 1.0 + kFracTol && fb >= -kFracTol && fb < 1.0 + kFracTol &&
             fc >= -kFracTol && fc < 1.0 + kFracTol;
  k.fast_ok = hmin >= (double)wide && small && fabsf(c.xyf) <= kNbrFastL && fabsf(c.xzf) <= kNbrFastL &&
              fabsf(c.yzf) <= kNbrFastL;
  return k;
}

// The scan context of atom i of structure st at (x, y, z): cell, cutoffs and
// the shell bounds of the single-precision decision.
template <bool kTri>
__device__ __forceinline__ CellCheck init_ctx(const NbrArgs& a, int st, int i, float x, float y, float z,
                                              ScanCtx& c) {
  c.i = i;
  c.Lxf = a.box[3 * st];
  c.Lyf = a.box[3 * st + 1];
  c.Lzf = a.box[3 * st + 2];
  c.xyf = kTri ? a.tilt[3 * st] : 0.f;
  c.xzf = kTri ? a.tilt[3 * st + 1] : 0.f;
  c.yzf = kTri ? a.tilt[3 * st + 2] : 0.f;
  c.xf = x;
  c.yf = y;
  c.zf = z;
  c.xi = c.xf;
  c.yi = c.yf;
  c.zi = c.zf;
  c.Lx = c.Lxf;
  c.Ly = c.Lyf;
  c.Lz = c.Lzf;
  c.xy = c.xyf;
  c.xz = c.xzf;
  c.yz = c.yzf;
  const CellCheck ck = check_cell<kTri>(c, a.rcR, a.rcA);
  c.rcR = (double)a.rcR;
  c.rcR2 = c.rcR * c.rcR;  // exact: a float squared in double
  c.rcA2 = (double)a.rcA * (double)a.rcA;
  c.ilx = 1.0f / c.Lxf;
  c.ily = 1.0f / c.Lyf;
  c.ilz = 1.0f / c.Lzf;
  c.fast = ck.fast_ok;
  c.inR2 = (a.rcR - kNbrDelta) * (a.rcR - kNbrDelta);
  c.outR2 = (a.rcR + kNbrDelta) * (a.rcR + kNbrDelta);
  c.inA2 = (a.rcA - kNbrDelta) * (a.rcA - kNbrDelta);
  c.outA2 = (a.rcA + kNbrDelta) * (a.rcA + kNbrDelta);
  return ck;
}

// Candidates of the single-image scan: bit b of mask[c] tells whether atom
// jb + 32 c + b of [jb, je) (at most 128) may lie within rc + delta, its
// single-precision distance being below that bound.  In an orthorhombic cell
// the nearest image along an axis is min(|e|, L - |e|).  Atom j is at tile
// slot j - t.base; up to 7 slots past the range are read and masked off.
constexpr int kNbrMasks = 4;
template <bool kTri>
__device__ __forceinline__ void scan_hits(const ScanCtx& c, const PosTile& t, int jb, int je,
                                          uint32_t (&mask)[kNbrMasks]) {
#pragma unroll
  for (int k = 0; k < kNbrMasks; ++k) {
    uint32_t m = 0;
    const int n = min(je - jb - 32 * k, 32);   // candidates of this mask
    const int q0 = jb + 32 * k - t.base;
    for (int b = 0; b < n; b += 8) {
      uint32_t m8 = 0;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int q = q0 + b + u;
        float ex = t.x[q] - c.xf, ey = t.y[q] - c.yf, ez = t.z[q] - c.zf;
        if constexpr (kTri) {
          float kx, ky, kz;
          min_image<true>(c, ex, ey, ez, kx, ky, kz);
        } else {
          ex = fminf(fabsf(ex), fabsf(c.Lxf - fabsf(ex)));
          ey = fminf(fabsf(ey), fabsf(c.Lyf - fabsf(ey)));
          ez = fminf(fabsf(ez), fabsf(c.Lzf - fabsf(ez)));
        }
        m8 |= (ex * ex + ey * ey + ez * ez < c.outR2) ? (1u << u) : 0u;
      }
      m |= m8 << b;
    }
    mask[k] = n >= 32 ? m : (n > 0 ? m & ((1u << n) - 1u) : 0u);
  }
}

// Lists of atom c.i from its T hits, tile slots in canonical order at
// slot k in buf[kNbrThreads (k / 8) + k % 8] (buf: the first of the atom's 8
// lane columns).  Lane s takes entries s, s + 8, ...; a ballot over the
// atom's lanes gives each kept entry its place, so 8 consecutive entries are
// stored together.
template <bool kTri>
__device__ __forceinline__ void write_hits(const NbrArgs& a, const ScanCtx& c, const PosTile& t, const uint32_t* buf,
                                           int T, int s, int& totR, int& totA) {
  const size_t col = (size_t)c.i;
  const int sh = threadIdx.x & 24;
  const bool up = threadIdx.x & 32;
  const uint32_t below = (1u << s) - 1u;
  int nR = 0, nA = 0;
  for (int k0 = 0; k0 < T; k0 += 8) {
    const bool on = k0 + s < T;
    const int q = on ? (int)buf[kNbrThreads * (k0 >> 3) + s] : c.i - t.base;
    const int j = t.base + q;
    const float px = t.x[q], py = t.y[q], pz = t.z[q];
    float ex = px - c.xf, ey = py - c.yf, ez = pz - c.zf, kx, ky, kz;
    min_image<kTri>(c, ex, ey, ez, kx, ky, kz);
    const float r2 = ex * ex + ey * ey + ez * ez;
    const int code = 13 - (int)fmaf(9.f, kx, fmaf(3.f, ky, kz));
    bool in = on & ((j != c.i) | (code != 13));
    bool ang = r2 < c.inA2;
    // inside either shell the float64 predicate decides
    const bool shR = r2 >= c.inR2, shA = !ang && r2 < c.outA2;
    if (in && (shR || shA)) {
      const double d2 = image_d2<kTri>(c, px, py, pz, kx, ky, kz);
      if (shR) in = d2 < c.rcR2;
      if (shA) ang = d2 < c.rcA2;
    }
    ang = ang && in;
    const unsigned long long bR = __ballot(in), bA = __ballot(ang);
    const uint32_t mR = ((up ? (uint32_t)(bR >> 32) : (uint32_t)bR) >> sh) & 255u;
    const uint32_t mA = ((up ? (uint32_t)(bA >> 32) : (uint32_t)bA) >> sh) & 255u;
    const uint32_t e = ((uint32_t)j << 5) | (uint32_t)(code & 31);
    const int oR = nR + __popc(mR & below), oA = nA + __popc(mA & below);
    if (in && oR < a.capR) a.idxR[col * a.capR + oR] = e;
    if (ang && oA < a.capA) a.idxA[col * a.capA + oA] = e;
    nR += __popc(mR);
    nA += __popc(mA);
  }
  totR = nR;
  totA = nA;
}

// Cell-list search of large structures.  A structure of at least
// kCellMinAtoms atoms whose cell takes the single-image decision is cut into
// na x nb x nc bins along its edge vectors, each bin at least rc + kCellPad
// thick across (perpendicular width over the bin count), at least 3 bins per
// axis and no more bins than atoms.  An atom's bin comes from its
// single-precision fractional coordinates; their error, and the accepted
// positions up to 1e-5 outside the cell, move an atom by under 0.006 A for
// cells up to kNbrFastL (twice that is below kCellPad), so two atoms in bins
// that are not adjacent along some axis lie more than rc apart in every
// image.  Each atom then meets as
// candidates exactly the atoms of its 27 surrounding bins and takes the same
// per-candidate decision as the all-pairs scan, so its entries are the same.
// Within rc + delta every j has one image at most (each width is at least
// 2 (rc + delta)), so an entry's rank among the atom's entries by (j, code)
// is its canonical slot.
//
// Bins of structure n have the ids atom_offset[n] + bin (< atom_offset[n+1]);
// the bins are counted, scanned into start offsets, and the binned atoms
// placed bin by bin as (x, y, z, j).  An atom with more hits than its LDS row
// holds is left to the all-pairs kernel (acell[i] = -1), which runs afterwards.
constexpr int kCellMinAtoms = 1024;     // default smallest structure searched through cell lists
constexpr int kCellMinAtomsLo = 64;     // smallest value a tuning may set
constexpr double kCellPad = 0.05;
constexpr int kScanChunk = 2048;   // bin ids per block of the offset scan

// bins per axis of structure st, (0, 0, 0, 0) for the all-pairs search
template <bool kTri>
__device__ int4 cell_grid(const NbrArgs& a, int st) {
  const int4 none = make_int4(0, 0, 0, 0);
  const int n = a.aoff[st + 1] - a.aoff[st];
  if (n < a.cell_min) return none;
  ScanCtx c;
  if (!init_ctx<kTri>(a, st, a.aoff[st], 0.f, 0.f, 0.f, c).fast_ok) return none;
  double ha, hb, hc;
  cell_widths(c, ha, hb, hc);
  // the single-image cells are at most kNbrFastL wide and rc >= 1 A: at most
  // 512 bins per axis
  const double w = (double)a.rcR + kCellPad;
  int na = (int)(ha / w), nb = (int)(hb / w), nc = (int)(hc / w);
  while ((long long)na * nb * nc > n) {
    if (na >= nb && na >= nc)
      --na;
    else if (nb >= nc)
      --nb;
    else
      --nc;
  }
  if (na < 3 || nb < 3 || nc < 3) return none;
  return make_int4(na, nb, nc, na * nb * nc);
}

// zeroes the bin counts and sets every structure's bins
template <bool kTri>
__global__ __launch_bounds__(256) void k_cell_setup(NbrArgs a) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t < a.N) a.cell[t] = 0;
  if (t < a.S) a.grid[t] = cell_grid<kTri>(a, t);
}

// bin of each atom of a binned structure and its slot in the bin
template <bool kTri>
__global__ __launch_bounds__(256) void k_cell_bin(NbrArgs a) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= a.N) return;
  int lo = 0, hi = a.S;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (a.aoff[mid] <= i) lo = mid; else hi = mid;
  }
  const int st = lo;
  a.astruct[i] = st;
  const int4 g = a.grid[st];
  int bin = -1, slot = 0;
  if (g.w > 0) {
    const float x = a.pos[i], y = a.pos[a.N + i], z = a.pos[2 * a.N + i];
    float fa, fb, fc;
    if constexpr (kTri) {
      const float xy = a.tilt[3 * st], xz = a.tilt[3 * st + 1], yz = a.tilt[3 * st + 2];
      fc = z / a.box[3 * st + 2];
      fb = (y - yz * fc) / a.box[3 * st + 1];
      fa = (x - xy * fb - xz * fc) / a.box[3 * st];
    } else {
      fa = x / a.box[3 * st];
      fb = y / a.box[3 * st + 1];
      fc = z / a.box[3 * st + 2];
    }
    // clamped in float (a NaN goes to bin 0; the position flag reports it)
    const int ia = (int)fminf(fmaxf(floorf(fa * (float)g.x), 0.f), (float)(g.x - 1));
    const int ib = (int)fminf(fmaxf(floorf(fb * (float)g.y), 0.f), (float)(g.y - 1));
    const int ic = (int)fminf(fmaxf(floorf(fc * (float)g.z), 0.f), (float)(g.z - 1));
    bin = a.aoff[st] + (ia * g.y + ib) * g.z + ic;
    slot = atomicAdd(&a.cell[bin], 1);
  }
  a.acell[i] = bin;
  a.aslot[i] = slot;
}

// exclusive prefix over 256 threads; returns the block total
__device__ __forceinline__ int block_exclusive_scan(int v, int& excl, int* red) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int inc = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int u = __shfl_up(inc, d, 64);
    if (lane >= d) inc += u;
  }
  if (lane == 63) red[w] = inc;
  __syncthreads();
  int before = 0, total = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    before += q < w ? red[q] : 0;
    total += red[q];
  }
  __syncthreads();
  excl = before + inc - v;
  return total;
}

// per chunk of kScanChunk bin ids: the sum of the counts
__global__ __launch_bounds__(256) void k_cell_part(int n, const int* __restrict__ cnt, int* __restrict__ part) {
  __shared__ int red[4];
  const int b = blockIdx.x * kScanChunk + threadIdx.x * 8;
  int v = 0;
#pragma unroll
  for (int q = 0; q < 8; ++q) v += b + q < n ? cnt[b + q] : 0;
  int excl;
  const int tot = block_exclusive_scan(v, excl, red);
  if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// counts -> start offsets over [0, n), and the total at [n].  Up to
// kScanDirect chunks every block sums the counts before its own (at most 30,720
// loads by the last block) instead of reading the sums of k_cell_part, whose
// launch took 4 us.
constexpr int kScanDirect = 16;
__global__ __launch_bounds__(256) void k_cell_start(int n, const int* __restrict__ cnt, const int* __restrict__ part,
                                                    int* __restrict__ start) {
  __shared__ int red[4];
  int off = 0;
  if ((int)gridDim.x <= kScanDirect) {
    const int4* c4 = reinterpret_cast<const int4*>(cnt);   // whole chunks of counts
    const int n4 = (int)blockIdx.x * (kScanChunk / 4);
#pragma unroll 4
    for (int q = threadIdx.x; q < n4; q += 256) {
      const int4 v = c4[q];
      off += (v.x + v.y) + (v.z + v.w);
    }
  } else {
    for (int q = threadIdx.x; q < (int)blockIdx.x; q += 256) off += part[q];
  }
  int excl;
  off = block_exclusive_scan(off, excl, red);
  const int b = blockIdx.x * kScanChunk + threadIdx.x * 8;
  int v[8], sum = 0;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    v[q] = b + q < n ? cnt[b + q] : 0;
    sum += v[q];
  }
  const int tot = block_exclusive_scan(sum, excl, red);
  int run = off + excl;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    if (b + q < n) start[b + q] = run;
    run += v[q];
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) start[n] = off + tot;
}

// binned atoms bin by bin as (x, y, z, j)
__global__ __launch_bounds__(256) void k_cell_place(NbrArgs a) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= a.N) return;
  const int bin = a.acell[i];
  if (bin < 0) return;
  a.cpos[a.start[bin] + a.aslot[i]] =
      make_float4(a.pos[i], a.pos[a.N + i], a.pos[2 * a.N + i], __int_as_float(i));
}

// Lists of the binned atoms, 8 lanes per atom.  Blocks take the atoms in bin
// order, so a block's atoms share most of their candidates.
//
// The 27 bins are 9 rows of three consecutive bins: lane s takes row s and all
// lanes share row 8, so the bounds of every row are one set of loads and the
// candidates of a row contiguous loads, eight in flight a lane.  As in the
// all-pairs scan a first part only tests the distance; its hits, gathered in
// the atom's LDS row, are decided 8 at a time, and the kept entries ranked by
// (j, code) against the row, four to an LDS read.  (The candidates of one row
// after another, each decided in full, were a chain of about 20 dependent
// loads, and the ranking one LDS read per comparison: 33 us for 9261 atoms,
// where a SIMD has one wavefront, now 14; 41 us for 27000 atoms, now 26.)
constexpr int kCellHits = 8 * kNbrBuf;        // hits an atom may have
constexpr int kCellRow = kCellHits + 4;       // LDS words of its row, padded to whole 16-byte reads

// Stores the m entries of an LDS row (padded with 0xFFFFFFFF to a multiple of
// 4) into list at their ranks below cap; lane s of 8 takes entries s, s + 8, ...
__device__ __forceinline__ void store_ranked(const uint32_t* row, int m, int s, uint32_t* __restrict__ list, int cap) {
  for (int g = 0; g < m; g += 32) {
    uint32_t e[4];
    int rank[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      e[u] = row[min(g + 8 * u + s, m - 1)];
      rank[u] = 0;
    }
    for (int q = 0; q < m; q += 4) {
      const uint4 v = *reinterpret_cast<const uint4*>(row + q);
#pragma unroll
      for (int u = 0; u < 4; ++u)
        rank[u] += (v.x < e[u] ? 1 : 0) + (v.y < e[u] ? 1 : 0) + (v.z < e[u] ? 1 : 0) + (v.w < e[u] ? 1 : 0);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (g + 8 * u + s < m && rank[u] < cap) list[rank[u]] = e[u];
  }
}

template <bool kTri>
__global__ __launch_bounds__(kNbrThreads) void k_cell_neighbors(NbrArgs a) {
  __shared__ __align__(16) uint32_t rows[2][kNbrAPB * kCellRow];   // hits, then entries; angular entries
  // the first ceil(M / 32) blocks work, renumbered over the XCDs among themselves
  const int M = a.start[a.N], nbw = (M + kNbrAPB - 1) / kNbrAPB;
  if ((int)blockIdx.x >= nbw) return;
  const int b0 = xcd_block_of(blockIdx.x, nbw) * kNbrAPB;
  const int s = threadIdx.x & 7;
  const int al = (int)(threadIdx.x >> 3), k = b0 + al;
  const bool live = k < M;
  const float4 me = a.cpos[min(k, M - 1)];
  const int i = __float_as_int(me.w);
  const int st = a.astruct[i];
  const int4 g = a.grid[st];
  ScanCtx c;
  init_ctx<kTri>(a, st, i, me.x, me.y, me.z, c);   // single-image decision: c.fast holds
  const int base = a.aoff[st];
  const int loc = a.acell[i] - base;
  const int kc = loc % g.z, kb = (loc / g.z) % g.y, ka = loc / (g.y * g.z);
  // bins kc-1, kc, kc+1 of a row are consecutive ids, split in two runs when
  // the row wraps
  // (kc = 0: [0, 1] and [nc-1]; kc = nc-1: [0] and [nc-2, nc-1]; else [kc-1, kc+1])
  const bool edge = kc == 0 || kc == g.z - 1;
  const int r0lo = edge ? 0 : kc - 1, r0hi = kc == 0 ? 1 : (edge ? 0 : kc + 1);
  const int r1lo = kc == 0 ? g.z - 1 : g.z - 2, r1hi = g.z - 1;
  struct Row {
    int q0, n0, q1, n;   // first run [q0, q0 + n0), second from q1, n in both
  };
  auto row_of = [&](int r) {
    const int da = r / 3 - 1, db = r % 3 - 1;
    const int xa = ka + da < 0 ? g.x - 1 : (ka + da == g.x ? 0 : ka + da);
    const int yb = kb + db < 0 ? g.y - 1 : (kb + db == g.y ? 0 : kb + db);
    const int* cs = a.start + base + (xa * g.y + yb) * g.z;
    Row w;
    w.q0 = cs[r0lo];
    w.n0 = cs[r0hi + 1] - w.q0;
    w.q1 = cs[edge ? r1lo : r0lo];
    w.n = w.n0 + (edge ? cs[edge ? r1hi + 1 : r0lo] - w.q1 : 0);
    if (!live) w.n0 = w.n = 0;
    return w;
  };
  const Row own = row_of(s), shared = row_of(8);
  uint32_t* hit = rows[0] + al * kCellRow;
  uint32_t* ang_row = rows[1] + al * kCellRow;
  int T = 0;   // hits of the atom; those past kCellHits are counted only
  // this lane's candidates first, first + step, ... of a row, 64 at a time
  auto scan = [&](const Row& w, int first, int step) {
    const int n = (w.n - first + step - 1) / step;
    auto slot = [&](int t) {
      const int x = first + t * step;
      return x < w.n0 ? w.q0 + x : w.q1 + (x - w.n0);
    };
    for (int t0 = 0; __any(t0 < n); t0 += 64) {
      uint32_t mask[2] = {0, 0};
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        for (int b = 0; b < 32; b += 8) {
          const int t1 = t0 + 32 * h + b;
          if (!__any(t1 < n)) break;
          float4 p[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) p[u] = a.cpos[min(slot(max(min(t1 + u, n - 1), 0)), M - 1)];
          uint32_t m8 = 0;
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            float ex = p[u].x - c.xf, ey = p[u].y - c.yf, ez = p[u].z - c.zf;
            if constexpr (kTri) {
              float kx, ky, kz;
              min_image<true>(c, ex, ey, ez, kx, ky, kz);
            } else {
              ex = fminf(fabsf(ex), fabsf(c.Lxf - fabsf(ex)));
              ey = fminf(fabsf(ey), fabsf(c.Lyf - fabsf(ey)));
              ez = fminf(fabsf(ez), fabsf(c.Lzf - fabsf(ez)));
            }
            m8 |= (t1 + u < n && ex * ex + ey * ey + ez * ez < c.outR2) ? (1u << u) : 0u;
          }
          mask[h] |= m8 << b;
        }
      }
      const int cnt = __popc(mask[0]) + __popc(mask[1]);
      int w0 = cnt;
#pragma unroll
      for (int d = 1; d < 8; d <<= 1) {
        const int u = __shfl_up(w0, d, 8);
        if (s >= d) w0 += u;
      }
      const int tot = __shfl(w0, 7, 8);
      w0 += T - cnt;
#pragma unroll
      for (int h = 0; h < 2; ++h)
        for (uint32_t m = mask[h]; m; m &= m - 1u, ++w0)
          if (w0 < kCellHits) hit[w0] = (uint32_t)slot(t0 + 32 * h + __builtin_ctz(m));
      T += tot;
    }
  };
  scan(own, 0, 1);
  scan(shared, s, 8);
  lds_lane_exchange();
  const bool spill = T > kCellHits;
  if (spill) T = 0;
  // the hits, 8 at a time; entry u of the row is written after hit u is read
  const int sh = threadIdx.x & 24;
  const bool up = threadIdx.x & 32;
  const uint32_t below = (1u << s) - 1u;
  int nR = 0, nA = 0;
  float4 pn = me;
  if (s < T) pn = a.cpos[hit[s]];
  for (int k0 = 0; __any(k0 < T); k0 += 8) {
    const bool on = k0 + s < T;
    const float4 p = pn;
    if (k0 + 8 + s < T) pn = a.cpos[hit[k0 + 8 + s]];
    const int j = __float_as_int(p.w);
    float ex = p.x - c.xf, ey = p.y - c.yf, ez = p.z - c.zf, kx, ky, kz;
    min_image<kTri>(c, ex, ey, ez, kx, ky, kz);
    const float r2 = ex * ex + ey * ey + ez * ez;
    const int code = 13 - (int)fmaf(9.f, kx, fmaf(3.f, ky, kz));
    bool in = on & ((j != i) | (code != 13));
    bool ang = r2 < c.inA2;
    // inside either shell the float64 predicate decides
    const bool shR = r2 >= c.inR2, shA = !ang && r2 < c.outA2;
    if (in && (shR || shA)) {
      const double d2 = image_d2<kTri>(c, p.x, p.y, p.z, kx, ky, kz);
      if (shR) in = d2 < c.rcR2;
      if (shA) ang = d2 < c.rcA2;
    }
    ang = ang && in;
    const unsigned long long bR = __ballot(in), bA = __ballot(ang);
    const uint32_t mR = ((up ? (uint32_t)(bR >> 32) : (uint32_t)bR) >> sh) & 255u;
    const uint32_t mA = ((up ? (uint32_t)(bA >> 32) : (uint32_t)bA) >> sh) & 255u;
    const uint32_t e = ((uint32_t)j << 5) | (uint32_t)(code & 31);
    lds_lane_exchange();
    if (in) hit[nR + __popc(mR & below)] = e;
    if (ang) ang_row[nA + __popc(mA & below)] = e;
    lds_lane_exchange();
    nR += __popc(mR);
    nA += __popc(mA);
  }
  if (s < 4) {
    hit[nR + s] = 0xFFFFFFFFu;
    ang_row[nA + s] = 0xFFFFFFFFu;
  }
  lds_lane_exchange();
  if (!live) return;
  if (spill) {
    if (s == 0) a.acell[i] = -1;
    return;
  }
  store_ranked(hit, nR, s, a.idxR + (size_t)i * a.capR, a.capR);
  store_ranked(ang_row, nA, s, a.idxA + (size_t)i * a.capA, a.capA);
  if (s == 0) {
    a.cntR[i] = nR;
    a.cntA[i] = nA;   // an overflow is flagged by the all-pairs launch that follows
  }
}

// Position of the key in a sorted row holding m valid entries (of cap), -1
// if absent.  The last entry of every run of 8 (four independent loads at a
// time) picks the run, then the run's 8 entries (two 16-byte loads) give the
// position.  Entries past m are treated as larger than any key.
__device__ __forceinline__ int row_find(const uint32_t* __restrict__ row, int m, int cap, uint32_t key) {
  const int nrun = (m + 7) >> 3;
  int below = 0;
  for (int r0 = 0; r0 < nrun; r0 += 4) {
    uint32_t last[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      // unconditional loads from inside the row, then the mask
      const int q = 8 * (r0 + u) + 7;
      const uint32_t x = row[min(q, cap - 1)];
      last[u] = (r0 + u < nrun && q < m) ? x : 0xFFFFFFFFu;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) below += (r0 + u < nrun && last[u] < key) ? 1 : 0;
  }
  int pos = -1;
  if (below < nrun) {
    const int b = 8 * below;   // the key, if present, lies in entries b .. b + 7
    uint32_t v[8];
    if (b + 8 <= cap && (((uintptr_t)(row + b)) & 15) == 0) {
      const uint4 x = *reinterpret_cast<const uint4*>(row + b);
      const uint4 y = *reinterpret_cast<const uint4*>(row + b + 4);
      v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
      v[4] = y.x; v[5] = y.y; v[6] = y.z; v[7] = y.w;
    } else {
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = b + u < cap ? row[b + u] : 0xFFFFFFFFu;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (b + u < m && v[u] == key) pos = b + u;
  }
  return pos;
}

// ============================================================ species order
// Atoms are laid out chunk by chunk (kOrdChunk atoms of the batch each), in a
// chunk by (species, angular neighbor count descending), with ties in atom
// order: every block of the per-atom kernels holds one species, and a
// wavefront's 8 atoms have similar pair counts, so their pair loops end
// together.  A chunk is sorted by one block in one launch (a counting sort
// over the whole batch took three), its atoms stay close in memory, and the
// layout is deterministic.  The key of atom i is
// t * kOrdBuckets + (kOrdBuckets - 1 - min(nA_i, kOrdBuckets - 1)).
//
// Chunk c starts at position c * order_stride(T); its species segments start on
// multiples of kSegAlign positions and the rest holds -1.
constexpr int kOrdChunk = 2048;
constexpr int kOrdBuckets = 64;
constexpr int kOrdMaxT = 4;    // species of the compiled shapes
constexpr int kSegAlign = 32;  // species segments start on multiples of the atoms per block
__host__ __device__ constexpr int order_stride(int T) { return kOrdChunk + T * kSegAlign; }
// Positions that chunk c writes: its own and, by the last one, the rest of the
// array, whose size is rounded up past the chunks (-1 there: the kernels of
// degrees l > 4 read every position).
__device__ __forceinline__ int order_len(int c, int nch, int T, int Npad) {
  return c + 1 < nch ? order_stride(T) : Npad - c * order_stride(T);
}

__device__ __forceinline__ int order_key(int t, int T, int nA) {
  if (t < 0 || t >= T) return -1;
  return t * kOrdBuckets + (kOrdBuckets - 1 - min(max(nA, 0), kOrdBuckets - 1));
}

struct OrderArgs {
  int N, Npad, T, nch;   // Npad: positions of the array, at least those of the chunks
  const int* type;
  const int* cntA;
  int* seg;     // [nch][T][2] species segment start and count
  int* order;   // [Npad]
  int* blist;   // [nch][order_blocks(T)] blocks of 32 positions, most pairs first, -1: none
};

// blocks of 32 positions of a chunk
__host__ __device__ constexpr int order_blocks(int T) { return order_stride(T) / kSegAlign; }

// Block of 32 positions that launch index b of a per-atom kernel takes, -1 for
// none: every chunk's block of most pairs first, then every chunk's next one.
// Blocks of 9 to 12 pairs an atom take two 64-pair rounds per wavefront; started
// last they left a tail of 30 us on a 130 us adjoint.
__host__ __device__ inline int order_grid(int nch, int T) { return nch * order_blocks(T); }
__device__ __forceinline__ int launch_block(const int* __restrict__ blist, int nch, int T, int b) {
  return blist[(b % nch) * order_blocks(T) + b / nch];
}

// Order of a batch of up to kTypeOrderAtoms atoms: species segments with their
// atoms in atom order, without the pair counts.  So few atoms leave most SIMDs
// with one wavefront of 2 or 4 atoms, which have nothing to balance, and the
// order then needs no launch after the neighbor build (5 us of a 58 us step of
// 544 atoms): extra blocks of the build form it, 256 threads a chunk.
constexpr int kTypeOrderAtoms = 8192;
constexpr int kTypeOrdLds = (kOrdChunk / kWave + 1) * kOrdMaxT + kOrdChunk + order_stride(kOrdMaxT);   // ints
__device__ __forceinline__ void type_order(const OrderArgs& a, int c, int* lds) {
  constexpr int NV = kOrdChunk / kWave;
  int* cnt = lds;                            // [NV][kOrdMaxT] atoms of 64 by species, then those before them
  int* tot = cnt + NV * kOrdMaxT;            // [kOrdMaxT]
  int* key = tot + kOrdMaxT;                 // [kOrdChunk] 64 species + rank among the 64, -1: not placed
  int* ord = key + kOrdChunk;                // [stride]
  const int T = a.T, stride = order_stride(T);
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  const int n = min(a.N - c * kOrdChunk, kOrdChunk), len = order_len(c, a.nch, T, a.Npad);
  const int* type = a.type + c * kOrdChunk;
  // loops of the chunk's own atoms, not unrolled: a block runs this once, with
  // a cold instruction cache
  int next = type[min((int)threadIdx.x, n - 1)];
  for (int q = threadIdx.x; q < stride; q += 256) ord[q] = -1;
#pragma unroll 1
  for (int q = threadIdx.x; q - lane < n; q += 256) {
    const int t = q < n && next >= 0 && next < T ? next : -1;
    next = type[min(q + 256, n - 1)];
    int k = -1;
#pragma unroll
    for (int u = 0; u < kOrdMaxT; ++u) {
      const unsigned long long m = __ballot(t == u);
      if (t == u) k = kWave * u + __popcll(m & ((1ull << lane) - 1ull));
      if (lane == u) cnt[q / kWave * kOrdMaxT + u] = __popcll(m);
    }
    key[q] = k;
  }
  __syncthreads();
  if (wid < kOrdMaxT) {   // wavefront u scans species u
    const int v = lane < (n + kWave - 1) / kWave ? cnt[lane * kOrdMaxT + wid] : 0;
    int inc = v;
#pragma unroll
    for (int d = 1; d < NV; d <<= 1) {
      const int x = __shfl_up(inc, d, kWave);
      if (lane >= d) inc += x;
    }
    if (lane < NV) cnt[lane * kOrdMaxT + wid] = inc - v;
    if (lane == NV - 1) tot[wid] = inc;
  }
  __syncthreads();
  int start[kOrdMaxT], at = 0;
#pragma unroll
  for (int u = 0; u < kOrdMaxT; ++u) {
    const int m = tot[u];
    start[u] = at;
    at += (m + kSegAlign - 1) / kSegAlign * kSegAlign;
    if (u < T && (int)threadIdx.x == u) {
      a.seg[2 * (c * T + u)] = c * stride + start[u];
      a.seg[2 * (c * T + u) + 1] = m;
    }
  }
#pragma unroll 1
  for (int q = threadIdx.x; q < n; q += 256) {
    const int k = key[q];
    if (k < 0) continue;
    const int t = k / kWave;
    const int s0 = t == 0 ? start[0] : (t == 1 ? start[1] : (t == 2 ? start[2] : start[3]));
    ord[s0 + cnt[q / kWave * kOrdMaxT + t] + k % kWave] = c * kOrdChunk + q;
  }
  __syncthreads();
#pragma unroll 1
  for (int q = threadIdx.x; q < len; q += 256) a.order[(size_t)c * stride + q] = q < stride ? ord[q] : -1;
  const int nb = order_blocks(T);
  for (int q = threadIdx.x; q < nb; q += 256)
    a.blist[c * nb + q] = ord[q * kSegAlign] >= 0 ? (c * stride) / kSegAlign + q : -1;
}

// LDS of order_body (ints): counts per 64 atoms and key, key offsets, the
// chunk's positions, species counts
constexpr int kOrdLds = (kOrdChunk / kWave + 1) * kOrdMaxT * kOrdBuckets + order_stride(kOrdMaxT) + 8;

// Chunk c with NT threads, which take its atoms NT at a time.  Rank of an atom
// among the atoms of its key: lanes before it in its wavefront (one ballot per
// key bit; a loop over the distinct keys took 15 rounds), then the groups of
// 64 before it.
template <int NT>
__device__ __forceinline__ void order_body(const OrderArgs& a, int c, int* lds) {
  constexpr int NR = kOrdChunk / NT, NWR = NT / kWave, NV = kOrdChunk / kWave;
  static_assert(NWR >= kOrdMaxT, "a wavefront per species");
  const int T = a.T, K = T * kOrdBuckets, stride = order_stride(T);
  int* wcnt = lds;                 // [NV][K] counts, then counts before the group
  int* off = wcnt + NV * K;        // [K] key totals, then starts in the species segment
  int* ord = off + K;              // [stride]
  int* cnt = ord + stride;         // [T]
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  for (int q = threadIdx.x; q < NV * K; q += NT) wcnt[q] = 0;
  for (int q = threadIdx.x; q < stride; q += NT) ord[q] = -1;
  __syncthreads();
  int key[NR], rank[NR];
  const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int i = c * kOrdChunk + r * NT + threadIdx.x;
    key[r] = i < a.N ? order_key(a.type[i], T, a.cntA[i]) : -1;
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int vw = r * NWR + wid;
    unsigned long long m = __ballot(key[r] >= 0);   // lanes of this lane's key
#pragma unroll
    for (int bit = 0; (1 << bit) < kOrdMaxT * kOrdBuckets; ++bit) {
      const unsigned long long b = __ballot((key[r] >> bit) & 1);
      m &= (key[r] >> bit) & 1 ? b : ~b;
    }
    rank[r] = __popcll(m & below);
    if (key[r] >= 0 && rank[r] == 0) wcnt[vw * K + key[r]] = __popcll(m);
  }
  __syncthreads();
  for (int q = threadIdx.x; q < K; q += NT) {
    int v[NV], run = 0;
#pragma unroll
    for (int w = 0; w < NV; ++w) v[w] = wcnt[w * K + q];
#pragma unroll
    for (int w = 0; w < NV; ++w) {
      wcnt[w * K + q] = run;
      run += v[w];
    }
    off[q] = run;
  }
  __syncthreads();
  if (wid < T) {   // wavefront t scans the buckets of species t
    const int v = off[wid * kOrdBuckets + lane];
    int inc = v;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const int u = __shfl_up(inc, d, kWave);
      if (lane >= d) inc += u;
    }
    off[wid * kOrdBuckets + lane] = inc - v;
    if (lane == kWave - 1) cnt[wid] = inc;
  }
  __syncthreads();
  int start[kOrdMaxT], at = 0;
#pragma unroll
  for (int t = 0; t < kOrdMaxT; ++t) {
    start[t] = at;
    if (t < T) at += (cnt[t] + kSegAlign - 1) / kSegAlign * kSegAlign;
  }
#pragma unroll
  for (int t = 0; t < kOrdMaxT; ++t)
    if (t < T && (int)threadIdx.x == t) {
      a.seg[2 * (c * T + t)] = c * stride + start[t];
      a.seg[2 * (c * T + t) + 1] = cnt[t];
    }
#pragma unroll
  for (int r = 0; r < NR; ++r)
    if (key[r] >= 0) {
      const int t = key[r] / kOrdBuckets;
      int s0 = 0;
#pragma unroll
      for (int u = 1; u < kOrdMaxT; ++u) s0 = t == u ? start[u] : s0;
      ord[s0 + off[key[r]] + wcnt[(r * NWR + wid) * K + key[r]] + rank[r]] = c * kOrdChunk + r * NT + threadIdx.x;
    }
  __syncthreads();
  const int len = order_len(c, a.nch, T, a.Npad);
  for (int q = threadIdx.x; q < len; q += NT) a.order[(size_t)c * stride + q] = q < stride ? ord[q] : -1;
  // blocks by their first atom's pair count (its largest), descending; up to 4
  // chunks give every block a CU of its own, so their order does not matter
  // (and sorting them took 2 us of a 180-atom MD step)
  const int nb = order_blocks(T);
  if (a.nch <= 4) {
    for (int q = threadIdx.x; q < nb; q += NT)
      a.blist[c * nb + q] = ord[q * kSegAlign] >= 0 ? (c * stride) / kSegAlign + q : -1;
    __syncthreads();
    return;
  }
  int* place = wcnt + nb;
  for (int q = threadIdx.x; q < nb; q += NT) {
    wcnt[q] = ord[q * kSegAlign] >= 0 ? a.cntA[ord[q * kSegAlign]] : -1;
    place[q] = 0;
  }
  __syncthreads();
  // a block's place: the blocks before it, a share of them per thread
  constexpr int PT = NT / 128 > 0 ? NT / 128 : 1;
  static_assert(order_blocks(kOrdMaxT) <= 128, "a thread group per share");
  if ((int)threadIdx.x % 128 < nb) {
    const int q = threadIdx.x % 128, v = wcnt[q];
    int r = 0;
    for (int o = threadIdx.x / 128; o < nb; o += PT) {
      const int x = wcnt[o];
      r += x > v || (x == v && o < q) ? 1 : 0;
    }
    atomicAdd(&place[q], r);
  }
  __syncthreads();
  for (int q = threadIdx.x; q < nb; q += NT)
    a.blist[c * nb + place[q]] = wcnt[q] >= 0 ? (c * stride) / kSegAlign + q : -1;
  __syncthreads();
}

__device__ __forceinline__ void collect_flags(const FlagArgs& f, int* lds) {
  if (threadIdx.x == 0) lds[0] = 0;
  __syncthreads();
  int v = 0;
  for (int q = threadIdx.x; q < f.n; q += blockDim.x) v |= f.bflags[q];
  if (v) atomicOr(&lds[0], v);
  __syncthreads();
  if (threadIdx.x == 0) {
    if (f.step) {
      const int st = f.step[0];
      f.flags[0] = lds[0] | (st < 1 ? FL_STEP : 0);
      f.cur[0] = st;
      f.step[0] = st + 1;
    } else if (lds[0]) {
      atomicOr(f.flags, lds[0]);
    }
  }
  __syncthreads();
}

__global__ __launch_bounds__(1024) void k_order(OrderArgs a, FlagArgs f) {
  __shared__ int lds[kOrdLds];
  if (blockIdx.x == 0) collect_flags(f, lds);
  order_body<1024>(a, blockIdx.x, lds);
}

// ========================================================== list building
// kCells: the cell search ran before and wrote the lists of the atoms with
// acell[i] >= 0.  The first nblk blocks build lists; any more form the species
// order of a small batch, a chunk each.
template <bool kTri, bool kCells>
__global__ __launch_bounds__(kNbrThreads) void k_neighbors(NbrArgs a, int nblk, OrderArgs og) {
  // 8 slots past the tile: scan_hits reads candidates eight at a time
  __shared__ float tx[kNbrTile + 8], ty[kNbrTile + 8], tz[kNbrTile + 8];
  __shared__ __align__(16) uint32_t nbuf[kNbrThreads * (kNbrBuf + 1)];
  __shared__ int jr[2];
  static_assert(kTypeOrdLds <= kNbrThreads * (kNbrBuf + 1), "the order's words fit the entry buffers");
  if ((int)blockIdx.x >= nblk) {
    type_order(og, blockIdx.x - nblk, reinterpret_cast<int*>(nbuf));
    return;
  }
  const int s = threadIdx.x & 7;
  const int b0 = xcd_block_of(blockIdx.x, nblk) * kNbrAPB;
  const int i = b0 + (threadIdx.x >> 3);
  const bool live = i < a.N;
  const int ic = live ? i : a.N - 1;
  // structure of the block's first atom (scalar search), then forward from it:
  // step by step, and by halves where more than the block's 32 lie between, as
  // only empty ones can (a run of 50000 took 4.8 ms step by step, now 26 us)
  const cptr<int> aoff = as_const(a.aoff);
  int lo = 0, hi = a.S;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (aoff[mid] <= min(b0, a.N - 1)) lo = mid; else hi = mid;
  }
  for (int k = 0; lo + 1 < a.S && a.aoff[lo + 1] <= ic; ++k) {
    ++lo;
    if (k < kNbrAPB) continue;
    hi = a.S;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (a.aoff[mid] <= ic) lo = mid; else hi = mid;
    }
  }
  const int st = lo;
  const int a0 = max(a.aoff[st], 0), a1 = min(a.aoff[st + 1], a.N);
  // the block's atoms are consecutive, so their structures cover [jr[0], jr[1])
  if (threadIdx.x == 0) jr[0] = a0;
  if (i == min(b0 + kNbrAPB - 1, a.N - 1) && s == 0) jr[1] = a1;
  ScanCtx c;
  const CellCheck ck = init_ctx<kTri>(a, st, ic, a.pos[ic], a.pos[a.N + ic], a.pos[2 * a.N + ic], c);
  int fl = 0;
  if (!ck.pos_ok) fl |= FL_POS;
  bool ok = live;
  if (!ck.box_ok) {
    fl |= FL_BOX;
    ok = false;
  }
  if (live && s == 0) {
    a.astruct[i] = st;
    const int ti = a.type[i];
    if (ti < 0 || ti >= a.T) fl |= FL_TYPE;
  }
  // atoms whose lists the cell search wrote (it leaves acell[i] >= 0)
  const bool mine = live && !(kCells && a.acell[ic] >= 0);
  const int len = ok && mine ? a1 - a0 : 0;
  const int jb = a0 + (len * s) / 8, je = a0 + (len * (s + 1)) / 8;
  // after the cell search, a block with no atom left to scan walks no tiles
  bool any = true;
  if constexpr (kCells)
    any = __syncthreads_or(len > 0);
  else
    __syncthreads();
  const int jlo = jr[0], jhi = any ? jr[1] : jr[0];
  // walks the tiles of [jlo, jhi); this lane scans [b, e) of each
  auto sweep = [&](int b, int e, auto&& scan) {
    for (int t0 = jlo; t0 < jhi; t0 += kNbrTile) {
      const int tn = min(kNbrTile, jhi - t0);
      for (int q = threadIdx.x; q < tn; q += kNbrThreads) {
        tx[q] = a.pos[t0 + q];
        ty[q] = a.pos[a.N + t0 + q];
        tz[q] = a.pos[2 * a.N + t0 + q];
      }
      __syncthreads();
      const PosTile t{tx, ty, tz, t0};
      scan(t, max(b, t0), min(e, t0 + tn));
      __syncthreads();
    }
  };
  // one scan: each lane keeps its entries in an LDS buffer (angular
  // membership as a bit mask), and after the 8-lane prefix copies them to
  // their slots; a lane with more than kNbrBuf entries makes the whole block
  // rescan and write directly
  uint32_t* mybuf = nbuf + threadIdx.x;   // slot u at mybuf[kNbrThreads u]
  int nR = 0, nA = 0;
  uint32_t angmask = 0;
  auto keep = [&](int j, int code, bool ang) {
    if (nR < kNbrBuf) {
      mybuf[kNbrThreads * nR] = ((uint32_t)j << 5) | (uint32_t)code;
      angmask |= ang ? (1u << nR) : 0u;
    }
    ++nR;
    nA += ang ? 1 : 0;
  };
  // Structures of a block that fit one tile (nearly always: at most two of its
  // structures exceed 32 atoms) take the single-image scan in two parts: a
  // distance test per candidate that only sets a bit (about 15 instructions),
  // then the image code, the shell tests and the stores for the hits alone,
  // spread evenly over the atom's lanes.  Deciding every candidate in one
  // part took about 40 instructions each for the one in eleven that is kept
  // (512 structures, 87k atoms: 57 us in one part, 41 us in two).
  bool done = false;
  int totR = 0, totA = 0;
  if (jhi - jlo <= kNbrTile) {
    for (int q = threadIdx.x; q < jhi - jlo; q += kNbrThreads) {
      tx[q] = a.pos[jlo + q];
      ty[q] = a.pos[a.N + jlo + q];
      tz[q] = a.pos[2 * a.N + jlo + q];
    }
    __syncthreads();
    const PosTile t{tx, ty, tz, jlo};
    if (c.fast) {   // the same for the atom's 8 lanes
      uint32_t mask[kNbrMasks];
      scan_hits<kTri>(c, t, jb, je, mask);
      int n = 0;
#pragma unroll
      for (int k = 0; k < kNbrMasks; ++k) n += __popc(mask[k]);
      int w = n;
#pragma unroll
      for (int d = 1; d < 8; d <<= 1) {
        const int u = __shfl_up(w, d, 8);
        if (s >= d) w += u;
      }
      const int T = __shfl(w, 7, 8);
      w -= n;
      if (T <= 8 * kNbrBuf) {
        uint32_t* gbuf = nbuf + (threadIdx.x & ~7);   // the atom's columns
#pragma unroll
        for (int k = 0; k < kNbrMasks; ++k)
          for (uint32_t m = mask[k]; m; m &= m - 1u, ++w)
            gbuf[kNbrThreads * (w >> 3) + (w & 7)] = (uint32_t)(jb - jlo + 32 * k + __builtin_ctz(m));
        lds_lane_exchange();
        write_hits<kTri>(a, c, t, gbuf, T, s, totR, totA);
        done = true;
      }
    }
    if (!done) scan_keep<kTri>(c, t, jb, je, mybuf, nR, nA, angmask, keep);
    __syncthreads();   // a rescan below loads the tile again
  } else {
    // Structures that do not fit one tile together (one of nearly 1024 atoms
    // and a neighbor): the first part tile by tile, the second from memory.
    // Deciding every candidate in one part these few blocks took 33 us, the
    // whole launch for 100 structures of 32 to 1024 atoms.
    if (__syncthreads_and(len == 0 || (c.fast && len <= 256 * kNbrMasks))) {
      uint32_t* gbuf = nbuf + (threadIdx.x & ~7);
      int T = 0;
      sweep(jb, je, [&](const PosTile& t, int b2, int e2) {
        uint32_t mask[kNbrMasks];
        scan_hits<kTri>(c, t, b2, e2, mask);
        int n = 0;
#pragma unroll
        for (int k = 0; k < kNbrMasks; ++k) n += __popc(mask[k]);
        int w = n;
#pragma unroll
        for (int d = 1; d < 8; d <<= 1) {
          const int u = __shfl_up(w, d, 8);
          if (s >= d) w += u;
        }
        const int tot = __shfl(w, 7, 8);
        w += T - n;
#pragma unroll
        for (int k = 0; k < kNbrMasks; ++k)
          for (uint32_t m = mask[k]; m; m &= m - 1u, ++w)
            if (w < 8 * kNbrBuf) gbuf[kNbrThreads * (w >> 3) + (w & 7)] = (uint32_t)(b2 + 32 * k + __builtin_ctz(m));
        T += tot;
      });
      done = T <= 8 * kNbrBuf;
      if (done) {
        lds_lane_exchange();
        const PosTile all{a.pos, a.pos + a.N, a.pos + 2 * a.N, 0};
        write_hits<kTri>(a, c, all, gbuf, T, s, totR, totA);
      }
    }
    if (__syncthreads_or(!done))
      sweep(done ? 0 : jb, done ? 0 : je,
            [&](const PosTile& t, int b2, int e2) { scan_keep<kTri>(c, t, b2, e2, mybuf, nR, nA, angmask, keep); });
  }
  // inclusive prefix over the 8 lanes of the atom
  int pR = nR, pA = nA;
#pragma unroll
  for (int d = 1; d < 8; d <<= 1) {
    const int uR = __shfl_up(pR, d, 8), uA = __shfl_up(pA, d, 8);
    if (s >= d) {
      pR += uR;
      pA += uA;
    }
  }
  if (!done) {
    totR = __shfl(pR, 7, 8);
    totA = __shfl(pA, 7, 8);
  }
  int wR = pR - nR, wA = pA - nA;
  const size_t col = (size_t)c.i;
  const bool spill = nR > kNbrBuf;   // never after the two-part scan (nR is 0)
  if (mine && !spill) {
    for (int u = 0; u < nR; ++u) {
      const uint32_t e = mybuf[kNbrThreads * u];
      if (wR + u < a.capR) a.idxR[col * a.capR + wR + u] = e;
      if ((angmask >> u) & 1u) {
        if (wA < a.capA) a.idxA[col * a.capA + wA] = e;
        ++wA;
      }
    }
  }
  if (__syncthreads_or(mine && spill)) {
    auto write = [&](int j, int code, bool ang) {
      const uint32_t e = ((uint32_t)j << 5) | (uint32_t)code;
      if (wR < a.capR) a.idxR[col * a.capR + wR] = e;
      ++wR;
      if (ang) {
        if (wA < a.capA) a.idxA[col * a.capA + wA] = e;
        ++wA;
      }
    };
    // angular entries are a subset, so a lane past the radial capacity may
    // still have angular slots to fill
    const bool wr = mine && spill && (wR < a.capR || wA < a.capA);
    sweep(wr ? jb : 0, wr ? je : 0,
          [&](const PosTile& t, int b2, int e2) { scan_range<kTri>(c, t, b2, e2, write); });
  }
  if (live && s == 0) {
    if (mine) {
      a.cntR[i] = totR;
      a.cntA[i] = totA;
    } else {   // counted by the cell search
      totR = a.cntR[i];
      totA = a.cntA[i];
    }
    if (totR > a.capR || totA > a.capA) fl |= FL_OVERFLOW;
    a.p4[i] = make_float4(c.xf, c.yf, c.zf, atom_word(a.type[i], a.T, totR > a.capR, totA > a.capA));
  }
  if (!(live && s == 0)) fl = 0;
  if (a.bflags) {
    __shared__ int word;
    if (threadIdx.x == 0) word = 0;
    __syncthreads();
    if (fl) atomicOr(&word, fl);
    __syncthreads();
    if (threadIdx.x == 0) a.bflags[blockIdx.x] = word;
  } else if (fl) {
    atomicOr(a.flags, fl);
  }
}

// ================================================================= helpers
// c^A of the block's species with every neighbor species staged in LDS, rows
// padded to KAP = 4k floats: a pair reads its 4-aligned row with a few wide
// LDS reads instead of selecting each coefficient by the neighbor's species
template <int T, int NA, int KA>
struct CTab {
  static constexpr int KAP = (KA + 3) & ~3;
  static constexpr int size = T * NA * KAP;
};

// Entry 0 of a row holds c_0 + sum_k c_k (the terms h T_0 of every
// order), so g_n = sum_k row[k] h T_k.
template <int T, int NA, int KA>
__device__ __forceinline__ void stage_ctab(float* ct, const float* __restrict__ cA) {
  constexpr int KAP = CTab<T, NA, KA>::KAP, R = T * NA;
  // a row per thread: its loads are in flight together
  for (int r = threadIdx.x; r < R; r += blockDim.x) {
    float v[KAP], sum = 0.f;
#pragma unroll
    for (int k = 0; k < KAP; ++k) v[k] = k < KA ? cA[r * KA + (k < KA ? k : 0)] : 0.f;
#pragma unroll
    for (int k = 0; k < KA; ++k) sum += v[k];
    v[0] += sum;
#pragma unroll
    for (int k = 0; k < KAP; ++k) ct[r * KAP + k] = v[k];
  }
}

struct PairGeom {
  int j;
  float dx, dy, dz, r, inv_r;
};

// cell of a structure: edge vectors a = (Lx, 0, 0), b = (xy, Ly, 0),
// c = (xz, yz, Lz); the tilts are read only for triclinic batches
struct Cell {
  float Lx, Ly, Lz, xy, xz, yz;
};

template <bool kTri>
__device__ __forceinline__ Cell load_cell(const float* __restrict__ box, const float* __restrict__ tilt, int st) {
  Cell c;
  c.Lx = box[3 * st];
  c.Ly = box[3 * st + 1];
  c.Lz = box[3 * st + 2];
  c.xy = kTri ? tilt[3 * st] : 0.f;
  c.xz = kTri ? tilt[3 * st + 1] : 0.f;
  c.yz = kTri ? tilt[3 * st + 2] : 0.f;
  return c;
}

// d = x_j - x_i + the entry's image shift, from the packed atom pj
template <bool kTri>
__device__ __forceinline__ PairGeom packed_geom(uint32_t e, const float4& pj, float xi, float yi, float zi,
                                                const Cell& cl) {
  PairGeom g;
  g.j = (int)(e >> 5);
  float sx, sy, sz;
  decode_shift(e & 31u, sx, sy, sz);
  g.dx = (pj.x - xi) + sx * cl.Lx;
  g.dy = (pj.y - yi) + sy * cl.Ly;
  g.dz = (pj.z - zi) + sz * cl.Lz;
  if constexpr (kTri) {
    g.dx += sy * cl.xy + sz * cl.xz;
    g.dy += sz * cl.yz;
  }
  const float r2 = g.dx * g.dx + g.dy * g.dy + g.dz * g.dz;
  g.inv_r = rsq_hw(r2);
  g.r = r2 * g.inv_r;
  return g;
}

// species of a packed atom; T is 1, 2 or 4 in every compiled shape, so the
// mask also keeps it inside the tables
template <int T>
__device__ __forceinline__ int packed_type(const float4& p) {
  static_assert((T & (T - 1)) == 0, "species index masked to a power of two");
  return (int)(__float_as_uint(p.w) & (uint32_t)(T - 1));
}

// Packed atoms of a call that did not build its lists (the neighbor build
// packs them otherwise): positions and species are the caller's at this call.
// With fbar the caller's force cotangents are packed too.
__global__ __launch_bounds__(256) void k_pack(int N, int T, const float* __restrict__ pos, const int* __restrict__ type,
                                              PairLists nb, float4* __restrict__ p4, const float* __restrict__ fbar,
                                              float4* __restrict__ fb4) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= N) return;
  p4[i] = make_float4(pos[i], pos[N + i], pos[2 * N + i],
                      atom_word(type[i], T, nb.cntR[i] > nb.capR, nb.cntA[i] > nb.capA));
  if (fbar) fb4[i] = make_float4(fbar[i], fbar[N + i], fbar[2 * N + i], 0.f);
}

// ========================================================= atom groups
// Per-atom kernels run L lanes per atom, 64 / L atoms per wavefront and 256 / L
// per block (L = 8, or 16 or 32 in the forward and the adjoint of small
// batches, group_lanes).  Lane s = l mod L of an atom's group takes the radial
// pairs k = s, s + L, ... and the hidden units mu = s, s + L, ...; for the
// angular descriptors the group is 2 harmonic groups x L / 2 channels:
// g = s / (L / 2) picks the harmonics (l = 1 and 4, or l = 2 and 3; 12 each
// for l <= 4) and p = s mod (L / 2) the channels n = p, p + L / 2, ....
// Atoms are in species order with species segments aligned to 32, so every
// block evaluates a single species' network.
constexpr int kLPA = 8;                    // lanes per atom, and of the high-degree kernels
constexpr int kAPB = 256 / kLPA;           // atoms per block
constexpr int kAPW = kWave / kLPA;         // atoms per wavefront
static_assert(kSegAlign % kAPB == 0, "species segments must align to blocks (one species per block)");
}  // namespace nep
#include "nep_highl.h"
namespace nep {

// c^R of the block's species in LDS, [T][NR][KR], read lane by lane by the
// radial sums and the force coefficients.  With c^A of that species alone and
// S_nlm stored atom by atom in 16-byte units (it was one row per channel and
// harmonic), the forward fits four blocks per CU: 85 -> 78 us at 512
// structures (87k atoms), the adjoint 119 -> 117.
template <class C>
struct CRad {
  static constexpr int N = C::T * C::NR * C::KR, size = (N + 3) & ~3;
};

// Row of radial force coefficients of one (atom, neighbor species): KP words
template <class C>
struct HRad {
  static constexpr int KP = (C::KR + 3) & ~3;
};

template <int LM>
struct HSplit {
  static constexpr int nA0 = LM >= 1 ? 3 : 0;   // group 0: l = 1 ...
  static constexpr int nB0 = LM >= 4 ? 9 : 0;   // ... and l = 4
  static constexpr int nA1 = LM >= 2 ? 5 : 0;   // group 1: l = 2 ...
  static constexpr int nB1 = LM >= 3 ? 7 : 0;   // ... and l = 3
  static constexpr int YG = (nA0 + nB0 > nA1 + nB1) ? nA0 + nB0 : nA1 + nB1;
  // harmonic index of compact entry i of group g, -1 for padding
  static constexpr int q(int g, int i) {
    return g == 0 ? (i < nA0 ? i : (i - nA0 < nB0 ? 15 + (i - nA0) : -1))
                  : (i < nA1 ? 3 + i : (i - nA1 < nB1 ? 8 + (i - nA1) : -1));
  }
};

// C_lm of compact entry i for this lane's harmonic group
template <class HS>
__device__ __forceinline__ float csel(int g, int i) {
  const int q0 = HS::q(0, i), q1 = HS::q(1, i);
  return g ? (q1 >= 0 ? clm(q1) : 0.f) : (q0 >= 0 ? clm(q0) : 0.f);
}

// The per-atom rows of the angular sums (S, Sdot, Sbar, A), in LDS and in
// HBM, are kept in harmonic-group order: entry e of group g of channel n at
// n YR + g YG + e, YR = 2 YG.  A lane of group g then reaches its entries as
// its base plus constant offsets, with no per-entry address selects (which
// the adjoint otherwise kept live, and spilled, across its network phase).
template <int LM>
struct HRow {
  static constexpr int YG = HSplit<LM>::YG, YR = 2 * YG;
  // whether entry e of group g is a harmonic (not padding)
  static constexpr bool real(int g, int e) { return HSplit<LM>::q(g, e) >= 0; }
};

struct GroupCtx {
  int s, g, p, al, pa, i;
  bool valid;
};

// lane roles and the atom of this lane; every lane of the block stays alive
// (lanes without an atom repeat one of the wavefront's, or atom 0)
template <int L>
__device__ __forceinline__ GroupCtx group_ctx(const int* __restrict__ order, int Npad, int vb) {
  GroupCtx c;
  c.s = threadIdx.x & (L - 1);
  c.g = c.s / (L / 2);
  c.p = c.s & (L / 2 - 1);
  c.al = threadIdx.x / L;
  c.pa = vb * (256 / L) + c.al;
  const int iraw = c.pa < Npad ? order[c.pa] : -1;
  c.valid = iraw >= 0;
  const unsigned long long vm = __ballot(c.valid);
  const int lead = vm ? __ffsll(vm) - 1 : 0;
  const int ilead = vm ? __shfl(iraw, lead, kWave) : 0;
  c.i = c.valid ? iraw : ilead;
  return c;
}

// Species of block vb's atoms.  Segments start on block boundaries, so a
// block holds one species, and its first position is an atom unless the
// whole block is padding.
template <int T>
__device__ __forceinline__ int block_species(const int* __restrict__ order, const float4* __restrict__ p4, int vb) {
  const int ip = order[vb * kAPB];
  return ip >= 0 ? __builtin_amdgcn_readfirstlane(packed_type<T>(p4[ip])) : 0;
}

// LDS words of the staged weights: whole 64-word rows, so that the direct
// loads below never write past them
// Rows of D = DP - 2 or DP - 3 words hold b0 and w1 of their unit behind W0.  With
// that and c^R in the records' words the adjoint of the 3/4/5-body model keeps two
// blocks per CU up to hidden 256 (from 244 on it was one: 483 -> 260 us at hidden
// 256 and 90,000 atoms).
__host__ __device__ constexpr bool weights_in_row(int D, int DP) { return DP - D >= 2; }
__host__ __device__ constexpr int weights_words(int H, int D, int DP) {
  return (H * DP + (weights_in_row(D, DP) ? 0 : 2 * H) + 63) / 64 * 64;
}
template <int D, int DP>
__device__ __forceinline__ float weight_b0(const float* wl, int H, int mu) {
  return wl[weights_in_row(D, DP) ? mu * DP + D : H * DP + mu];
}
template <int D, int DP>
__device__ __forceinline__ float weight_w1(const float* wl, int H, int mu) {
  return wl[weights_in_row(D, DP) ? mu * DP + D + 1 : H * DP + H + mu];
}

// Species I's W0 (rows padded to DP words), b0 and w1 into LDS with direct
// global-to-LDS loads (gfx950 global_load_lds_dword: each wavefront writes
// 64 consecutive words and holds no registers for them), issued at the
// block's start and waited for by wait_weights() before the network, so
// their latency overlaps the pair passes instead of preceding them.  W0's
// padding words (d >= D, never read) receive W0[0][0].
__device__ __forceinline__ void stage_weights_async(float* wl, const float* __restrict__ nn, int nn_stride, int I,
                                                    int H, int D, int DP) {
  const bool in_row = weights_in_row(D, DP);
  const int WS = H * DP + 2 * H, WSP = weights_words(H, D, DP);
  const float* w = nn + (size_t)I * nn_stride;
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave, nw = blockDim.x / kWave;
  for (int c0 = wv * kWave; c0 < WSP; c0 += nw * kWave) {
    const int q = c0 + lane;
    const int mu = q / DP, d = q % DP;
    const int tail = in_row && d < D + 2 ? H * D + (d - D) * H + mu : 0;   // b0, w1 or padding
    const int src = q < H * DP ? (d < D ? mu * D + d : tail) : (!in_row && q < WS ? H * D + (q - H * DP) : 0);
    __builtin_amdgcn_global_load_lds(w + src, (__attribute__((address_space(3))) void*)(wl + c0), 4, 0, 0);
  }
}
__device__ __forceinline__ void wait_weights() { __builtin_amdgcn_s_waitcnt(0); }

// ======================================================== angular pair stream
// The angular pairs of a wavefront's atoms form one stream, taken 64 at a
// time with one pair per lane: geometry, basis and harmonics are evaluated
// once per pair.  (With the pairs split over 4 slots of an atom's lanes, both
// harmonic groups evaluated them, and an atom with 5 pairs took as long as
// one with 8.)  Atoms are sorted by pair count, so most wavefronts of the
// mean 7.3 pairs per atom need one chunk.  The lanes of an atom then sum 3
// harmonics each over its pairs, read back from LDS (15 sums a lane instead of
// 60).  Forward at 512 structures (87k atoms): 5540 -> 3570 VALU instructions
// per wavefront with the radial forces moved out, 168 -> 128 registers (four
// wavefronts per SIMD), 111 -> 87 us.  A table of the 8 atom slots in LDS
// serves the lanes whose pair belongs to another lane's atom.
constexpr int kSlotX = 0, kSlotI = 3, kSlotL = 4, kSlotBase = 7, kSlotTilt = 8;
template <bool kTri>
constexpr int slot_words() {
  return 12;   // x y z i | Lx Ly Lz base | xy xz yz -; 4 mod 8, so the 8 slots start in different banks
}

template <int L>
struct PairStream {
  static constexpr int APW = kWave / L;
  int cum[APW];   // stream position of slot v's first pair (wave-uniform)
  int total;
  int lo, hi;      // this lane's own atom's pairs
};

// nA: the pairs of this lane's atom (the same in its L lanes)
template <int L>
__device__ __forceinline__ PairStream<L> pair_stream(int nA) {
  PairStream<L> st;
  const int slot = (threadIdx.x & (kWave - 1)) / L;
  int at = 0;
  st.lo = 0;
#pragma unroll
  for (int v = 0; v < st.APW; ++v) {
    st.cum[v] = at;
    st.lo = v == slot ? at : st.lo;
    at += __builtin_amdgcn_readlane(nA, v * L);
  }
  st.total = at;
  st.hi = st.lo + nA;
  return st;
}

// atom slot of stream position p
template <int L>
__device__ __forceinline__ int pair_slot(const PairStream<L>& st, int p) {
  int u = 0;
#pragma unroll
  for (int v = 1; v < st.APW; ++v) u += p >= st.cum[v] ? 1 : 0;
  return u;
}

// The adjoint's tangent sums in wavefronts of many pairs an atom.  An atom's own
// L lanes would run through up to 64 pairs of a chunk while the lanes of the
// atoms without pairs in it wait; so 2^k groups of L lanes an atom take every
// 2^k-th of its pairs, and their sums are added and sent to the atom's own
// lanes.  Adjoint of 90,000 atoms in us without and with it: 22 pairs an atom
// 234 / 234, 28 298 / 278, 42 459 / 392, 75 908 / 669; at 19 and fewer, below
// the line, the same kernel.  (In the forward, whose sums are half as many, it
// spilled at four wavefronts per SIMD: 314 -> 318 us of a step at 7 pairs; with
// degrees l > 4, whose adjoint spills as it is, 570 -> 585 us at 7 pairs.)
constexpr int kSharePairs = 192;   // pairs of a wavefront
template <int L>
struct ChunkShare {
  int k;       // wave-uniform
  int t, t1;   // this lane's first pair and the end of its atom's, in the chunk
  int src;     // lane that holds this atom's sums, -1: the chunk has no pair of it
};
template <int L>
__device__ __forceinline__ ChunkShare<L> chunk_share(const PairStream<L>& ps, int c0, const float* slots, int words) {
  constexpr int APW = kWave / L;
  const int lane = threadIdx.x & (kWave - 1), slot = lane / L;
  const int u0 = pair_slot(ps, c0), u1 = pair_slot(ps, min(c0 + kWave, ps.total) - 1);
  ChunkShare<L> c;
  c.k = 0;
#pragma unroll
  for (int k = 1; (1 << k) <= APW; ++k) c.k += (u1 - u0 + 1) << k <= APW ? 1 : 0;
  const int v = u0 + (slot >> c.k), u = min(v, APW - 1);
  const int lo = __float_as_int(slots[u * words + kSlotBase]);
  const int hi = u + 1 < APW ? __float_as_int(slots[(u + 1) * words + kSlotBase]) : ps.total;
  c.t = max(lo - c0, 0) + (slot & ((1 << c.k) - 1));
  c.t1 = v <= u1 ? min(hi - c0, kWave) : 0;
  c.src = slot >= u0 && slot <= u1 ? ((slot - u0) << c.k) * L + lane % L : -1;
  return c;
}
// adds the groups' partial sums v to the sums S of the atom's own lanes
template <int L, int R, int N>
__device__ __forceinline__ void chunk_add(const ChunkShare<L>& c, float (&v)[R][N], float (&S)[R][N]) {
  // lane bits 3, 4, 5 as far as they tell the groups of an atom apart
  constexpr int bit0 = L == 8 ? 3 : L == 16 ? 4 : 5;
  auto each = [&](auto&& f) {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int n = 0; n < N; ++n) f(v[r][n], S[r][n]);
  };
  if constexpr (bit0 <= 3)
    if (c.k > 0) each([](float& x, float&) { x += dpp<kDppRowRor8>(x); });
  if constexpr (bit0 <= 4)
    if (c.k > 4 - bit0) each([](float& x, float&) { x = xor16_sum(x); });
  if (c.k > 5 - bit0) each([](float& x, float&) { x = xor32_sum(x); });
  each([&](float& x, float& y) {
    x = __shfl(x, max(c.src, 0), kWave);
    y += c.src >= 0 ? x : 0.f;
  });
}

template <bool kTri>
__device__ __forceinline__ void slot_store(float* sl, int i, float x, float y, float z, const Cell& c, int base) {
  *reinterpret_cast<float4*>(sl + kSlotX) = make_float4(x, y, z, __int_as_float(i));
  *reinterpret_cast<float4*>(sl + kSlotL) = make_float4(c.Lx, c.Ly, c.Lz, __int_as_float(base));
  if constexpr (kTri) *reinterpret_cast<float4*>(sl + kSlotTilt) = make_float4(c.xy, c.xz, c.yz, 0.f);
}

// list offset of stream position p and its geometry, from the slot's words
struct StreamPair {
  size_t off;
  int J;
  PairGeom q;
};
template <int T, bool kTri>
__device__ __forceinline__ StreamPair stream_pair(const float* sl, int p, const PairLists& nb, const float4* p4) {
  const float4 x = *reinterpret_cast<const float4*>(sl + kSlotX);
  const float4 l = *reinterpret_cast<const float4*>(sl + kSlotL);
  Cell c{l.x, l.y, l.z, 0.f, 0.f, 0.f};
  if constexpr (kTri) {
    const float4 t = *reinterpret_cast<const float4*>(sl + kSlotTilt);
    c.xy = t.x;
    c.xz = t.y;
    c.yz = t.z;
  }
  StreamPair r;
  r.off = (size_t)__float_as_int(x.w) * nb.capA + (p - __float_as_int(l.w));
  const uint32_t e = nb.idxA[r.off];
  const float4 pj = p4[e >> 5];
  r.J = packed_type<T>(pj);
  r.q = packed_geom<kTri>(e, pj, x.x, x.y, x.z, c);
  return r;
}

// Radial sums of an atom from its L lanes' partial sums v[t KR + k] over h T_k
// (or q_k): on return o[r] of lane s holds F[t][k] of entry L r + s, each with
// the T_0 term of its species added, and qn[r] holds sum_tk c^R_{ItnK} F[t][k]
// of channel n = L r + s.  cRI: c^R of species I (LDS).
template <class C, int L>
__device__ __forceinline__ void radial_finish(const float (&v)[C::T * C::KR], const float* cRI, int s,
                                              float (&o)[(C::T * C::KR + L - 1) / L], float (&qn)[(C::NR + L - 1) / L]) {
  constexpr int T = C::T, NR = C::NR, KR = C::KR, TK = T * KR, NV = (TK + L - 1) / L;
  rs_group<L>(v, o);
  float a0[T];
#pragma unroll
  for (int t = 0; t < T; ++t) a0[t] = __shfl(o[t * KR / L], t * KR % L, L);
  float part[NR];
#pragma unroll
  for (int n = 0; n < NR; ++n) part[n] = 0.f;
#pragma unroll
  for (int r = 0; r < NV; ++r) {
    const int e = r * L + s, t = e / KR, kk = e % KR;
    const bool on = TK % L == 0 || e < TK;
#pragma unroll
    for (int u = 0; u < T; ++u) o[r] += t == u ? a0[u] : 0.f;
    const float* c = cRI + (on ? t * NR * KR + kk : 0);
    const float x = on ? o[r] : 0.f;
#pragma unroll
    for (int n = 0; n < NR; ++n) part[n] = fmaf(c[n * KR], x, part[n]);
  }
  rs_group<L>(part, qn);
}

// LDS of the forward per wavefront: the slot table, then the pair records of
// the angular sums (g_n and the harmonics, odd stride) and, once they are
// summed, the atoms' rows (G, then S or A in group order; stride 4 mod 8)
template <class C, int L>
struct FwdLds {
  static constexpr int APW = kWave / L;   // atoms per wavefront
  static constexpr int DP = (C::D + 3) & ~3, YR = HRow<C::LMAX>::YR;
  static constexpr int RS = (C::NA + YR) | 1;
  static constexpr int SW = (C::NA * YR + 3) & ~3;   // an atom's S in HBM
  static constexpr int RW = (DP + SW + 7) / 8 * 8 + 4;
  static constexpr int BUF = (kWave * RS > APW * RW ? kWave * RS : APW * RW) + 3 & ~3;
  static constexpr int WAVE = APW * slot_words<true>() + BUF;
};

// words [base + e], e = 0..W-1 (16-byte reads when the row allows)
template <int W, bool kVec>
__device__ __forceinline__ void row_load(const float* p, float (&v)[W]) {
  if constexpr (kVec && W % 4 == 0) {
#pragma unroll
    for (int e = 0; e < W; e += 4) {
      const float4 c = *reinterpret_cast<const float4*>(p + e);
      v[e] = c.x;
      v[e + 1] = c.y;
      v[e + 2] = c.z;
      v[e + 3] = c.w;
    }
  } else {
#pragma unroll
    for (int e = 0; e < W; ++e) v[e] = p[e];
  }
}

// ================================================================= forward
// Per atom: radial sums F[J][k] = sum_{j of type J} f_k(r_ij) give
// q_n = sum_{J,k} c^R_{IJnk} F[J][k] (Eqs. 5-6); angular sums S_nlm (Eq. 8)
// give q_nl (Eq. 7) and the 4-/5-body invariants; the per-species network
// gives E_i and E' = dE_i/dG (D1.1-D1.5).  With forces on, the atom's radial
// force coefficients and every angular pair's partial force f_ij = dE_i/dr_ij
// (C3.6) are stored for the force pass.
// Launch index b (256 / L atoms of the species order); lds: lds_forward bytes.
template <class C, bool kTri, int L>
__device__ __forceinline__ void forward_body(const FwdArgs& a, int b, float* lds) {
  constexpr int T = C::T, NR = C::NR, NA = C::NA, KR = C::KR, KA = C::KA, Y = C::Y, D = C::D, LM = C::LMAX;
  constexpr int L3 = C::L3, L4 = C::L4, L5 = C::L5;
  using HS = HSplit<LM>;
  using FL = FwdLds<C, L>;
  constexpr int YG = HS::YG, YR = HRow<LM>::YR, DP = FL::DP, RS = FL::RS, RW = FL::RW;
  constexpr int NE = (YR + L - 1) / L;   // harmonics summed per lane
  constexpr bool kVec = YR % 4 == 0;
  const int H = a.H;
  using CT = CTab<T, NA, KA>;
  float* ctab = lds;                     // [T][NA][KAP], c^A of the block's species
  float* crl = lds + CT::size;           // its c^R
  float* wl = crl + CRad<C>::size;       // its weights
  float* slots = wl + weights_words(H, D, DP) + (threadIdx.x / kWave) * FL::WAVE;
  float* buf = slots + (kWave / L) * slot_words<kTri>();
  // 32 atoms of one species, taken by L / 8 blocks
  const int vs = launch_block(a.blist, a.nch, T, b / (L / 8));
  if (vs < 0) return;
  const int vb = vs * (L / 8) + b % (L / 8);
  // issued here, waited for after the angular sums: their latency overlaps the
  // pair passes
  const int I = block_species<T>(a.order, a.p4, vs);
  if (a.do_mlp) stage_weights_async(wl, a.nn, a.nn_stride, I, H, D, DP);
  stage_ctab<T, NA, KA>(ctab, a.cA + (size_t)I * T * NA * KA);
  for (int q = threadIdx.x; q < CRad<C>::N; q += 256) crl[q] = a.cR[(size_t)I * CRad<C>::N + q];
  const GroupCtx w = group_ctx<L>(a.order, a.Npad, vb);
  const int N = a.N, i = w.i, pa = w.pa, s = w.s, g = w.g;
  const int lane = threadIdx.x & (kWave - 1), slot = lane / L;
  const float4 me = a.p4[i];
  float* row = buf + slot * RW;
  float* rowS = row + DP;
  const int st = a.astruct[i];
  const Cell cell = load_cell<kTri>(a.box, a.tilt, st);
  const float xi = me.x, yi = me.y, zi = me.z;
  const int cR_i = a.nb.cntR[i], cA_i = a.nb.cntA[i];
  const int nR = w.valid ? min(cR_i, a.nb.capR) : 0;
  const int nA = w.valid ? min(cA_i, a.nb.capA) : 0;

  // ---- radial sums in Chebyshev space, pairs split over the lanes
  constexpr int NQ = (NR + L - 1) / L;
  float qn[NQ];   // channels s, s + L, ...
  {
    float FR[T * KR];
#pragma unroll
    for (int e = 0; e < T * KR; ++e) FR[e] = 0.f;
    // the next pair's atom and the list entry after it are loaded ahead
    const uint32_t* li = a.nb.idxR + (size_t)i * a.nb.capR;
    uint32_t e0 = 0, e1 = 0;
    float4 p0 = make_float4(0.f, 0.f, 0.f, 0.f);
    if (s < nR) {
      e0 = li[s];
      e1 = li[min(s + L, nR - 1)];
      p0 = a.p4[e0 >> 5];
    }
    for (int k = s; k < nR; k += L) {
      const uint32_t e = e0;
      const float4 pj = p0;
      e0 = e1;
      p0 = a.p4[e1 >> 5];
      e1 = li[min(k + 2 * L, nR - 1)];
      const PairGeom q = packed_geom<kTri>(e, pj, xi, yi, zi, cell);
      float f[KR];
      radial_cheb<KR>(q.r, a.inv_rcR, f);
      const int J = packed_type<T>(pj);
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const float m = (T == 1 || J == t) ? 1.f : 0.f;
#pragma unroll
        for (int kk = 0; kk < KR; ++kk) FR[t * KR + kk] = fmaf(m, f[kk], FR[t * KR + kk]);
      }
    }
    float o[(T * KR + L - 1) / L];
    lds_barrier();   // the block's coefficient tables
    radial_finish<C, L>(FR, crl, s, o, qn);
    if (a.FRst && w.valid) {
#pragma unroll
      for (int r = 0; r < (T * KR + L - 1) / L; ++r) {
        const int e = r * L + s;
        if (T * KR % L == 0 || e < T * KR) a.FRst[(size_t)e * a.Npad + pa] = o[r];
      }
    }
  }

  // ---- angular sums S_nlm: one pair per lane writes g_n and B_lm, then lane s
  //      of an atom sums its pairs for the harmonics s, s + L, ...
  const PairStream<L> ps = pair_stream<L>(nA);
  if (s == 0) slot_store<kTri>(slots + slot * slot_words<kTri>(), i, xi, yi, zi, cell, ps.lo);
  lds_lane_exchange();
  {
    float S[NE][NA];
#pragma unroll
    for (int r = 0; r < NE; ++r)
#pragma unroll
      for (int n = 0; n < NA; ++n) S[r][n] = 0.f;
    for (int c0 = 0; c0 < ps.total; c0 += kWave) {
      const int p = c0 + lane;
      if (p < ps.total) {
        const StreamPair sp = stream_pair<T, kTri>(slots + pair_slot(ps, p) * slot_words<kTri>(), p, a.nb, a.p4);
        float f[KA];
        radial_cheb<KA>(sp.q.r, a.inv_rcA, f);
        const float* cJ = ctab + sp.J * NA * CT::KAP;
        float* rec = buf + lane * RS;
#pragma unroll
        for (int n = 0; n < NA; ++n) {
          float acc = 0.f;
#pragma unroll
          for (int kk = 0; kk < KA; ++kk) acc = fmaf(cJ[n * CT::KAP + kk], f[kk], acc);
          rec[n] = acc;
        }
        float B[Y];
        harm_val<LM>(sp.q.dx * sp.q.inv_r, sp.q.dy * sp.q.inv_r, sp.q.dz * sp.q.inv_r, B);
#pragma unroll
        for (int gg = 0; gg < 2; ++gg)
#pragma unroll
          for (int e = 0; e < YG; ++e) {
            const int q = HS::q(gg, e);
            rec[NA + gg * YG + e] = q >= 0 ? B[q] : 0.f;
          }
      }
      lds_lane_exchange();
      const int t1 = min(ps.hi - c0, kWave);
#pragma unroll 2
      for (int t = max(ps.lo - c0, 0); t < t1; ++t) {
        const float* rec = buf + t * RS;
        float gn[NA];
#pragma unroll
        for (int n = 0; n < NA; ++n) gn[n] = rec[n];
#pragma unroll
        for (int r = 0; r < NE; ++r) {
          const int e = r * L + s;
          const float b = rec[NA + (YR % L == 0 || e < YR ? e : 0)];
#pragma unroll
          for (int n = 0; n < NA; ++n) S[r][n] = fmaf(gn[n], b, S[r][n]);
        }
      }
      lds_lane_exchange();
    }
    // This wavefront's weight loads have landed (before any store is issued, so
    // that none is waited for); the barrier ahead of the network covers the
    // other wavefronts'.
    wait_weights();
    // the atoms' rows take the records' place
#pragma unroll
    for (int r = 0; r < NE; ++r) {
      const int e = r * L + s;
      if (YR % L == 0 || e < YR) {
#pragma unroll
        for (int n = 0; n < NA; ++n) rowS[n * YR + e] = S[r][n];   // zero at padding entries
      }
    }
    lds_lane_exchange();
    // stored atom by atom, 16 bytes a lane
    if (w.valid && a.Sst) {
      float4* so = reinterpret_cast<float4*>(a.Sst + (size_t)pa * FL::SW);
#pragma unroll
      for (int q = s; q < FL::SW / 4; q += L) so[q] = reinterpret_cast<const float4*>(rowS)[q];
    }
  }
#pragma unroll
  for (int r = 0; r < NQ; ++r)
    if (r * L + s < NR) row[r * L + s] = qn[r];
  lds_lane_exchange();

  // ---- angular descriptors, channel n and harmonic group g by the lane of
  //      channel slot n mod (L / 2) and group g
  const int lA = g ? 2 : 1, lB = g ? 3 : 4;
  const int nAg = g ? HS::nA1 : HS::nA0;     // size of the first l block
  for (int n = w.p; n < NA; n += L / 2) {
    float Sn[YG];
    row_load<YG, kVec>(rowS + n * YR + g * YG, Sn);
    float qa = 0.f, qb = 0.f;
#pragma unroll
    for (int e = 0; e < YG; ++e) {
      const float v = csel<HS>(g, e) * Sn[e] * Sn[e];
      if (e < nAg) qa += v; else qb += v;
    }
    if (lA <= L3) row[NR + (lA - 1) * NA + n] = qa;
    if (lB <= L3) row[NR + (lB - 1) * NA + n] = qb;
    if constexpr (L4 != 0) {
      const Sym3 M = sym_of(Sn[0], Sn[1], Sn[2], Sn[3], Sn[4]);
      const float q4 = sym_dot(sym_mul(M, M), M);
      if (g == 1) row[NR + L3 * NA + n] = q4;
    }
    if constexpr (L5 != 0) {
      const float P = Sn[0] * Sn[0] + Sn[1] * Sn[1] + Sn[2] * Sn[2];
      if (g == 0) row[NR + L3 * NA + (L4 ? NA : 0) + n] = P * P;
    }
  }
  if constexpr (C::YH > 0) {
    // q_nl of l = 5..L3, from k_high_desc
    for (int v = NR + 4 * NA + s; v < NR + L3 * NA; v += L) {
      const float x = a.G[(size_t)v * a.Npad + pa];
      row[v] = w.valid ? x : 0.f;
    }
  }
  lds_barrier();
  float G[DP];
  row_load<DP, true>(row, G);   // words past D are not used
  if (w.valid) {
#pragma unroll
    for (int r = 0; r < (D + L - 1) / L; ++r) {
      const int v = r * L + s;
      if (D % L == 0 || v < D) {
        const float x = row[v];
        if (a.G) a.G[(size_t)v * a.Npad + pa] = x;
        if (a.Guser) a.Guser[(size_t)v * N + i] = x;
      }
    }
  }
  if (!a.do_mlp) return;

  // ---- network: hidden units mu = s, s + L, ... (weights from LDS)
  const float* Wl = wl;
  float Ep[D];
#pragma unroll
  for (int v = 0; v < D; ++v) Ep[v] = 0.f;
  float E = 0.f;
  for (int mu = s; mu < H; mu += L) {
    const float* wr = Wl + mu * DP;
    float z = weight_b0<D, DP>(Wl, H, mu);
#pragma unroll
    for (int v = 0; v < D; ++v) z = fmaf(wr[v], G[v], z);
    const float x = tanh_hw(z);
    const float w1 = weight_w1<D, DP>(Wl, H, mu);
    E = fmaf(w1, x, E);
    const float sg = w1 * (1.0f - x * x);
#pragma unroll
    for (int v = 0; v < D; ++v) Ep[v] = fmaf(sg, wr[v], Ep[v]);
    if (w.valid && a.X) a.X[(size_t)mu * a.Npad + pa] = x;
  }
  // E' summed over the lanes, scattered (entry v in lane v mod L), shared
  // through the atom's LDS row (G there has been read)
  {
    float eo[(D + L - 1) / L];
    rs_group<L>(Ep, eo);
#pragma unroll
    for (int r = 0; r < (D + L - 1) / L; ++r) {
      const int v = L * r + s;
      if (v < D) {
        row[v] = eo[r];
        if (w.valid && a.Ep) a.Ep[(size_t)v * a.Npad + pa] = eo[r];
      }
    }
    lds_lane_exchange();
  }
  E = grp_sum<L>(E) + a.nn[(size_t)I * a.nn_stride + H * D + 2 * H];
  if (w.valid) {
    if (s == 0) {
      if (a.eatom) a.eatom[i] = E;
      if (a.eatom2) a.eatom2[i] = E;
    }
  }
  if (!a.do_force) return;

  // ---- radial force coefficients h_Jk = sum_n E'_n c^R_{IJnk} for the force
  //      pass, entry (J, k) by lane (J KP + k) mod L; entry (J, 0) also takes
  //      sum_k h_Jk (the terms h T_0 of every order)
  {
    constexpr int KP = HRad<C>::KP, NH = (T * KP + L - 1) / L;
    float hv[NH], sum[T];
#pragma unroll
    for (int t = 0; t < T; ++t) sum[t] = 0.f;
#pragma unroll
    for (int r = 0; r < NH; ++r) {
      const int e = r * L + s, t = e / KP, kk = e % KP;
      const bool on = t < T && kk < KR;
      const float* c = crl + (on ? t * NR * KR + kk : 0);
      float acc = 0.f;
#pragma unroll
      for (int n = 0; n < NR; ++n) acc = fmaf(row[n], c[n * KR], acc);
      hv[r] = on ? acc : 0.f;
#pragma unroll
      for (int u = 0; u < T; ++u) sum[u] += t == u ? hv[r] : 0.f;
    }
#pragma unroll
    for (int t = 0; t < T; ++t) sum[t] = grp_sum<L>(sum[t]);
    if (w.valid) {
      float* ho = a.hrow + (size_t)i * T * KP;
#pragma unroll
      for (int r = 0; r < NH; ++r) {
        const int e = r * L + s, t = e / KP;
        float v = hv[r];
#pragma unroll
        for (int u = 0; u < T; ++u) v += (t == u && e == u * KP) ? sum[u] : 0.f;
        if (e < T * KP) ho[e] = v;
      }
    }
  }

  // ---- A_nlm = sum_v E'_v dG_v/dS_nlm in place of S_nlm, lanes as for the
  //      angular descriptors
  for (int n = w.p; n < NA; n += L / 2) {
    float Sn[YG];
    row_load<YG, kVec>(rowS + n * YR + g * YG, Sn);
    const float eA = lA <= L3 ? row[NR + ((lA <= L3 ? lA : 1) - 1) * NA + n] : 0.f;
    const float eB = lB <= L3 ? row[NR + ((lB <= L3 ? lB : 1) - 1) * NA + n] : 0.f;
    float a4[5] = {0.f, 0.f, 0.f, 0.f, 0.f}, a5[3] = {0.f, 0.f, 0.f};
    if constexpr (L4 != 0) {
      const Sym3 M = sym_of(Sn[0], Sn[1], Sn[2], Sn[3], Sn[4]);
      float o[5];
      sym_proj(sym_mul(M, M), o);
      const float e4 = g == 1 ? 3.0f * row[NR + L3 * NA + n] : 0.f;
#pragma unroll
      for (int m = 0; m < 5; ++m) a4[m] = e4 * o[m];
    }
    if constexpr (L5 != 0) {
      const float P = Sn[0] * Sn[0] + Sn[1] * Sn[1] + Sn[2] * Sn[2];
      const float e5 = g == 0 ? 4.0f * row[NR + L3 * NA + (L4 ? NA : 0) + n] * P : 0.f;
#pragma unroll
      for (int m = 0; m < 3; ++m) a5[m] = e5 * Sn[m];
    }
#pragma unroll
    for (int e = 0; e < YG; ++e) {
      float v = 2.0f * csel<HS>(g, e) * (e < nAg ? eA : eB) * Sn[e];
      if (e < 5) v += a4[e];
      if (e < 3) v += a5[e];
      rowS[n * YR + g * YG + e] = v;
    }
  }
  lds_lane_exchange();

  // ---- angular partial forces, one pair per lane:
  //      f_ij = sum_nlm A_nlm (g'_n r_hat B_lm + g_n grad B_lm)
  for (int c0 = 0; c0 < ps.total; c0 += kWave) {
    const int p = c0 + lane;
    if (p >= ps.total) break;
    const int u = pair_slot(ps, p);
    const StreamPair sp = stream_pair<T, kTri>(slots + u * slot_words<kTri>(), p, a.nb, a.p4);
    const PairGeom& q = sp.q;
    const float ux = q.dx * q.inv_r, uy = q.dy * q.inv_r, uz = q.dz * q.inv_r;
    float f[KA], fp[KA];
    radial_cheb_d<KA>(q.r, a.inv_rcA, f, fp);
    const float* cJ = ctab + sp.J * NA * CT::KAP;
    const float* rowA = buf + u * RW + DP;
    float B[Y], uf[Y];
    harm_val<LM>(ux, uy, uz, B);
#pragma unroll
    for (int qq = 0; qq < Y; ++qq) uf[qq] = 0.f;
    float vv = 0.f;
#pragma unroll
    for (int n = 0; n < NA; ++n) {
      float gn = 0.f, gp = 0.f;
#pragma unroll
      for (int kk = 0; kk < KA; ++kk) {
        const float c = cJ[n * CT::KAP + kk];
        gn = fmaf(c, f[kk], gn);
        gp = fmaf(c, fp[kk], gp);
      }
      float An[YR];
      row_load<YR, kVec>(rowA + n * YR, An);
      float wn = 0.f;   // sum_lm A_nlm B_lm
#pragma unroll
      for (int gg = 0; gg < 2; ++gg)
#pragma unroll
        for (int e = 0; e < YG; ++e) {
          const int qq = HS::q(gg, e);
          if (qq >= 0) {
            wn = fmaf(An[gg * YG + e], B[qq], wn);
            uf[qq] = fmaf(An[gg * YG + e], gn, uf[qq]);
          }
        }
      vv = fmaf(gp, wn, vv);
    }
    float gx, gy, gz;
    harm_grad_sum<LM>(ux, uy, uz, uf, gx, gy, gz);
    const float rad = ux * gx + uy * gy + uz * gz;
    float* fo = a.fA + 3 * sp.off;
    fo[0] = vv * ux + (gx - rad * ux) * q.inv_r;
    fo[1] = vv * uy + (gy - rad * uy) * q.inv_r;
    fo[2] = vv * uz + (gz - rad * uz) * q.inv_r;
  }
}

template <class C, bool kTri, int W, int L>
__global__ __launch_bounds__(256, W) void k_forward(FwdArgs a) {
  extern __shared__ __align__(16) float lds[];
  if (a.fl.n > 0 && blockIdx.x == gridDim.x - 1) {
    collect_flags(a.fl, reinterpret_cast<int*>(lds));
    return;
  }
  forward_body<C, kTri, L>(a, blockIdx.x, lds);
}

// ====================================================================== MD
// Velocity Verlet for the inference path, in eV, A, fs and amu: the
// acceleration of atom i is F_i / m_i times kAccel, and 1 amu A^2/fs^2 is
// 1/kAccel eV.
constexpr float kAccel = 9.648533212e-3f;

struct MDArgs {
  int N, T;
  const int* type;
  const int* astruct;
  const float* box;
  const float* tilt;   // null: every cell orthorhombic
  const float* mass;   // [T] amu
  float* pos;          // [3][N]
  float* vel;          // [3][N] A/fs
  const float* F;      // [3][N] eV/A
  float* ekin;         // [N] eV (kick only)
  float hdt, dt;
};

__device__ __forceinline__ float inv_mass(const MDArgs& a, int i) {
  const int t = a.type[i];
  return (t >= 0 && t < a.T) ? kAccel / a.mass[t] : 0.f;
}

// Atom i's move between two force evaluations, f the force on it.  With kKick the half kick that
// ends a step (forces at the current positions); with kDrift the half kick
// that begins the next one, the drift and the wrap into the cell: [0, L) per
// axis for an orthorhombic cell; for a triclinic one, minus the lattice vector
// H floor(f) of the fractional coordinates f = H^-1 x.  The last kick (no
// drift) also gives the kinetic energy per atom.
template <bool kKick, bool kDrift>
__device__ __forceinline__ void md_move(const MDArgs& a, int i, const float (&fi)[3]) {
  const float im = inv_mass(a, i);
  const float k = a.hdt * im;
  float x[3], v2 = 0.f;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const size_t q = (size_t)c * a.N + i;
    const float f = fi[c];
    float v = a.vel[q];
    if (kKick) v = fmaf(k, f, v);
    if (kDrift) {
      v = fmaf(k, f, v);
      x[c] = fmaf(a.dt, v, a.pos[q]);
    } else {
      v2 = fmaf(v, v, v2);
    }
    a.vel[q] = v;
  }
  if (!kDrift) {
    a.ekin[i] = im > 0.f ? 0.5f * v2 / im : 0.f;
    return;
  }
  const int st = a.astruct[i];
  const float Lx = a.box[3 * st], Ly = a.box[3 * st + 1], Lz = a.box[3 * st + 2];
  const float xy = a.tilt ? a.tilt[3 * st] : 0.f, xz = a.tilt ? a.tilt[3 * st + 1] : 0.f,
              yz = a.tilt ? a.tilt[3 * st + 2] : 0.f;
  if (xy != 0.f || xz != 0.f || yz != 0.f) {
    const float fc = x[2] / Lz;
    const float fb = (x[1] - yz * fc) / Ly;
    const float fa = (x[0] - xy * fb - xz * fc) / Lx;
    const float ka = floorf(fa), kb = floorf(fb), kc = floorf(fc);
    x[0] = x[0] - Lx * ka - xy * kb - xz * kc;
    x[1] = x[1] - Ly * kb - yz * kc;
    x[2] = x[2] - Lz * kc;
  } else {
    const float L[3] = {Lx, Ly, Lz};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      x[c] -= L[c] * floorf(x[c] / L[c]);
      if (x[c] >= L[c]) x[c] -= L[c];
      if (!(x[c] >= 0.f)) x[c] = 0.f;
    }
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) a.pos[(size_t)c * a.N + i] = x[c];
}

// Forces F_i = sum_j f_ij - f_ji (Eq. 3) and the atom's share of the virial.
//
// Radial part: f_ij = (sum_k h_i,Jk f'_k(r)) r_hat, and f_ji has the same
// basis at the same distance, so f_ij - f_ji = (sum_k (h_i,Jk + h_j,Ik) f'_k) r_hat
// needs only the neighbor's 12-word coefficient row: no pair force is stored
// and no reverse index is searched.  (Storing 12 bytes per pair, searching
// the reverse index and gathering both took 33 + 25 us and 13 us of the
// forward at 512 structures, 87k atoms; this kernel takes 29 us.)  Angular part: the
// stored pair forces, the partner's entry found in its short sorted list.
//
// A pair whose partner entry was cut off by the capacity counts with f_ij
// alone; only then does the partner's list have to be searched.  The virial
// -sum f_ij (x) r_ij over both entries of a pair equals -1/2 (f_ij - f_ji) (x) r_ij
// summed over both, so the radial part uses the total pair force.
//
// LPA lanes per atom take list slots s, s + LPA, ...; the rows of the block's
// own atoms are staged in LDS.
constexpr int kForceLPA = 16;   // default lanes per atom (8 or 16)
template <class C, int LPA>
constexpr int force_lds_words() {
  return 256 / LPA * C::T * HRad<C>::KP;
}

// Position of key in the angular list of atom j (m entries, row 16-byte
// aligned when vec), -1 if it was cut off: the count of smaller entries, 8 per
// step, of a list of more than 16 in the 16 that halving leaves (force pass of
// 90,000 atoms with 75 entries an atom: 374 us with the whole list counted,
// 249 so; 176 and 135 with 42, the same with up to 15).
__device__ __forceinline__ int partner_find(const uint32_t* __restrict__ row, int m, int cap, bool vec, uint32_t key) {
  int below = 0;
  bool hit = false;
  while (m - below > 16) {
    const int mid = below + (((m - below) / 2) & ~7);
    if (row[mid] <= key) below = mid; else m = mid;
  }
  for (int b = below; b < m; b += 8) {
    uint32_t v[8];
    if (vec && b + 8 <= cap) {
      const uint4 x = *reinterpret_cast<const uint4*>(row + b);
      const uint4 y = *reinterpret_cast<const uint4*>(row + b + 4);
      v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
      v[4] = y.x; v[5] = y.y; v[6] = y.z; v[7] = y.w;
    } else {
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = row[min(b + u, cap - 1)];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const bool in = b + u < m;
      below += (in && v[u] < key) ? 1 : 0;
      hit |= in && v[u] == key;
    }
  }
  return hit ? below : -1;
}

template <class C, bool kTri, int LPA>
__device__ __forceinline__ void force_body(const ForceArgs& a, int vb, float* own, const MDArgs* md = nullptr) {
  static_assert(LPA == 8 || LPA == 16, "8 or 16 lanes per atom");
  constexpr int T = C::T, KR = C::KR, KP = HRad<C>::KP, TK = T * KP, APB = 256 / LPA;
  const int s = threadIdx.x % LPA, al = threadIdx.x / LPA;
  const int i0 = vb * APB, i = i0 + al, N = a.N;
  {
    const float4* src = reinterpret_cast<const float4*>(a.hrow + (size_t)i0 * TK);
    const int n4 = min(APB, N - i0) * (TK / 4);
    for (int q = threadIdx.x; q < n4; q += 256) reinterpret_cast<float4*>(own)[q] = src[q];
  }
  __syncthreads();
  float fx = 0.f, fy = 0.f, fz = 0.f;
  float v[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (i < N) {
    const float4 pi = a.p4[i];
    const int I = packed_type<T>(pi);
    const Cell cell = load_cell<kTri>(a.box, a.tilt, a.astruct[i]);
    const int nR = min(a.nb.cntR[i], a.nb.capR), nA = min(a.nb.cntA[i], a.nb.capA);
    const uint32_t self = (uint32_t)i << 5;
    const size_t oR = (size_t)i * a.nb.capR, oA = (size_t)i * a.nb.capA;
    for (int k = s; k < nR; k += LPA) {
      const uint32_t e = a.nb.idxR[oR + k];
      const int j = (int)(e >> 5);
      const float4 pj = a.p4[j];
      const float4* hj = reinterpret_cast<const float4*>(a.hrow + ((size_t)j * T + I) * KP);
      const float4* hi = reinterpret_cast<const float4*>(own + (al * T + packed_type<T>(pj)) * KP);
      float wp = 1.f;   // 0: the partner's list does not hold this pair
      if (__float_as_uint(pj.w) & kAtomOverR)
        wp = row_find(a.nb.idxR + (size_t)j * a.nb.capR, a.nb.capR, a.nb.capR, self | (26u - (e & 31u))) >= 0 ? 1.f : 0.f;
      float c[KR];
#pragma unroll
      for (int q = 0; q < KP / 4; ++q) {
        const float4 x = hj[q], y = hi[q];
        if (4 * q < KR) c[4 * q] = fmaf(wp, x.x, y.x);
        if (4 * q + 1 < KR) c[4 * q + 1] = fmaf(wp, x.y, y.y);
        if (4 * q + 2 < KR) c[4 * q + 2] = fmaf(wp, x.z, y.z);
        if (4 * q + 3 < KR) c[4 * q + 3] = fmaf(wp, x.w, y.w);
      }
      const PairGeom q = packed_geom<kTri>(e, pj, pi.x, pi.y, pi.z, cell);
      const float sc = cheb_deriv<KR>(c, q.r, a.inv_rcR) * q.inv_r;
      const float gx = sc * q.dx, gy = sc * q.dy, gz = sc * q.dz;
      fx += gx;
      fy += gy;
      fz += gz;
      const float wv = fmaf(-0.5f, wp, 1.f);   // half a pair, or all of it without its partner
      const float hx = wv * gx, hy = wv * gy, hz = wv * gz;
      v[0] -= hx * q.dx; v[1] -= hy * q.dy; v[2] -= hz * q.dz;
      v[3] -= hx * q.dy; v[4] -= hy * q.dz; v[5] -= hz * q.dx;
    }
    const bool vec = (a.nb.capA & 3) == 0 && (reinterpret_cast<uintptr_t>(a.nb.idxA) & 15) == 0;
    for (int k = s; k < nA; k += LPA) {
      const uint32_t e = a.nb.idxA[oA + k];
      const int j = (int)(e >> 5);
      const float* f = a.fA + 3 * (oA + k);
      const float ax = f[0], ay = f[1], az = f[2];
      const float4 pj = a.p4[j];
      const int m = min(a.nb.cntA[j], a.nb.capA);
      const size_t oj = (size_t)j * a.nb.capA;
      const int pos = partner_find(a.nb.idxA + oj, m, a.nb.capA, vec, self | (26u - (e & 31u)));
      fx += ax;
      fy += ay;
      fz += az;
      if (pos >= 0) {
        const float* b = a.fA + 3 * (oj + pos);
        fx -= b[0];
        fy -= b[1];
        fz -= b[2];
      }
      const PairGeom q = packed_geom<kTri>(e, pj, pi.x, pi.y, pi.z, cell);
      v[0] -= ax * q.dx; v[1] -= ay * q.dy; v[2] -= az * q.dz;
      v[3] -= ax * q.dy; v[4] -= ay * q.dz; v[5] -= az * q.dx;
    }
  }
  // the lanes of an atom: 8-lane groups, then (16 lanes) the other half of the row
  float r[9] = {fx, fy, fz, v[0], v[1], v[2], v[3], v[4], v[5]};
#pragma unroll
  for (int q = 0; q < 9; ++q) {
    r[q] = grp8_sum(r[q]);
    if (LPA == 16) r[q] += dpp<kDppRowRor8>(r[q]);
  }
  if (i < N && s == 0) {
    const size_t n = (size_t)N;
#pragma unroll
    for (int q = 0; q < 3; ++q) a.F[q * n + i] = r[q];
    if (a.Fuser)
#pragma unroll
      for (int q = 0; q < 3; ++q) a.Fuser[q * n + i] = r[q];
#pragma unroll
    for (int q = 0; q < 6; ++q) a.wv[q * n + i] = r[3 + q];
    if (md) {
      const float f[3] = {r[0], r[1], r[2]};
      md_move<true, true>(*md, i, f);
    }
  }
}

template <class C, bool kTri, int LPA>
__global__ __launch_bounds__(256) void k_force(ForceArgs a) {
  __shared__ __align__(16) float own[force_lds_words<C, LPA>()];
  force_body<C, kTri, LPA>(a, xcd_block(), own);
}

// The force pass of an MD step that another follows: an atom's kick and drift
// by the lane that holds its force (the positions are written, the packed
// ones read).  Its own launch took 4 us a step of a 180-atom cell, now 27 us.
template <class C, bool kTri>
__global__ __launch_bounds__(256) void k_force_move(ForceArgs a, MDArgs md) {
  __shared__ __align__(16) float own[force_lds_words<C, kForceLPA>()];
  force_body<C, kTri, kForceLPA>(a, xcd_block(), own, &md);
}

// ==================================================================== loss
// One block per structure: E(n), W(n) and, with labels, the loss terms of
// Eqs. 10-12 and the cotangents dL/dE(n), dL/dF_i, dL/dW(n).  Sums run in
// float64 in a fixed order.
constexpr int kRedBlk = 256;

// Loss of Eqs. 9-12 from the per-structure partials, float64 in a fixed
// order (one block).
constexpr int kLossLds = 3 * kRedBlk * sizeof(double);
__device__ void loss_final_block(int S, int N, float le, float lf, float lv, const double* lpart, float* loss,
                                 int* flags, void* lds) {
  double (*red)[kRedBlk] = reinterpret_cast<double (*)[kRedBlk]>(lds);
  double acc[3] = {0, 0, 0};
  for (int s = threadIdx.x; s < S; s += kRedBlk)
    for (int q = 0; q < 3; ++q) acc[q] += lpart[3 * s + q];
  for (int q = 0; q < 3; ++q) red[q][threadIdx.x] = acc[q];
  __syncthreads();
  for (int st = kRedBlk / 2; st > 0; st >>= 1) {
    if (threadIdx.x < st)
      for (int q = 0; q < 3; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double Le = S > 0 ? red[0][0] / S : 0.0;
    const double Lf = N > 0 ? red[1][0] / (3.0 * N) : 0.0;
    const double Lv = S > 0 ? red[2][0] / (6.0 * S) : 0.0;
    const double L = le * Le + lf * Lf + lv * Lv;
    loss[0] = (float)L;
    loss[1] = (float)Le;
    loss[2] = (float)Lf;
    loss[3] = (float)Lv;
    if (flags && !isfinite(L)) atomicOr(flags, FL_NONFINITE);
  }
}

struct StructArgs {
  int S, N;
  const int* aoff;
  const float* eatom;
  const float* wv;
  const float* F;
  const float* Et;
  const float* Ft;
  const float* Wt;
  float le, lf, lv;
  float* Es;
  float* Ws;
  float* Es_user;
  float* Ws_user;
  float* eps;
  float* wbar;
  float4* fb4;
  double* lpart;  // [S][3]
  // structures of at least 2 kStructChunk atoms are summed from chunk partials
  int split;
  double* spart;  // [N / kStructChunk + 1][2][8]
};

constexpr int kStructChunk = 1024;

__device__ __forceinline__ int find_struct(const int* __restrict__ aoff, int S, int i) {
  int lo = 0, hi = S;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (aoff[mid] <= i) lo = mid; else hi = mid;
  }
  return lo;
}

// Sums over atoms [lo, hi) of one structure: energy, the six virial
// components and the squared force error (acc[0..7]); writes the packed F-bar.
__device__ __forceinline__ void struct_accumulate(const StructArgs& a, int lo, int hi, double* acc) {
  const int N = a.N;
  const bool lab = a.Et != nullptr;
  const float cf = 2.0f * a.lf / (3.0f * (float)max(N, 1));
  for (int i = lo + threadIdx.x; i < hi; i += kRedBlk) {
    acc[0] += a.eatom[i];
#pragma unroll
    for (int c = 0; c < 6; ++c) acc[1 + c] += a.wv[(size_t)c * N + i];
    if (lab) {
      float d[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        d[c] = a.F[(size_t)c * N + i] - a.Ft[(size_t)c * N + i];
        acc[7] += (double)d[c] * d[c];
      }
      a.fb4[i] = make_float4(cf * d[0], cf * d[1], cf * d[2], 0.f);
    }
  }
}

// Block sum of acc[0..7] in a fixed order, the result in red[q][0]: over each
// wavefront's lanes, then its four wavefronts.  Threads n and up hold zeros,
// whose exchanges are left out, a structure of one atom needing none (20000 of
// those: 93 us with all exchanges, 27 without).
__device__ __forceinline__ void struct_reduce(double (*red)[kRedBlk / kWave], const double* acc, int n) {
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  n -= wid * kWave;
  double v[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) v[q] = acc[q];
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) {
    if (d >= n) continue;   // wave-uniform
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] += __shfl_xor(v[q], d, kWave);
  }
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < 8; ++q) red[q][wid] = v[q];
  __syncthreads();
  if (threadIdx.x < 8) {
    double* r = red[threadIdx.x];
    r[0] = (r[0] + r[1]) + (r[2] + r[3]);
  }
  __syncthreads();
}

// Chunk partials of the large structures: a chunk of kStructChunk atoms
// meets at most two structures of 2 kStructChunk atoms or more, those of its
// first and last atoms (slots 0 and 1).
// chunk vb; lds: kStructLds bytes
__device__ __forceinline__ void struct_part_body(const StructArgs& a, int vb, void* lds) {
  double (*red)[kRedBlk / kWave] = reinterpret_cast<double (*)[kRedBlk / kWave]>(lds);
  const int c0 = vb * kStructChunk, c1 = min(c0 + kStructChunk, a.N);
  const int sa = find_struct(a.aoff, a.S, c0), sb = find_struct(a.aoff, a.S, c1 - 1);
  for (int h = 0; h < 2; ++h) {
    const int st = h ? sb : sa;
    if (h && sb == sa) break;
    const int a0 = a.aoff[st], a1 = a.aoff[st + 1];
    if (a1 - a0 < 2 * kStructChunk) continue;
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    struct_accumulate(a, max(a0, c0), min(a1, c1), acc);
    struct_reduce(red, acc, kRedBlk);
    if (threadIdx.x < 8) a.spart[(2 * (size_t)vb + h) * 8 + threadIdx.x] = red[threadIdx.x][0];
    __syncthreads();
  }
}

__global__ __launch_bounds__(kRedBlk) void k_struct_part(StructArgs a) {
  __shared__ double red[8][kRedBlk / kWave];
  struct_part_body(a, blockIdx.x, red);
}

constexpr int kStructLds = 8 * (kRedBlk / kWave) * sizeof(double);
// structure s; lds: kStructLds bytes
__device__ __forceinline__ void struct_body(const StructArgs& a, int s, void* lds) {
  double (*red)[kRedBlk / kWave] = reinterpret_cast<double (*)[kRedBlk / kWave]>(lds);
  const int a0 = a.aoff[s], a1 = a.aoff[s + 1];
  double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  const bool lab = a.Et != nullptr;
  // component c (the energy, the six of the virial) is finished by thread c
  const int c = threadIdx.x;
  const float label = lab && c < 7 ? (c == 0 ? a.Et[s] : a.Wt[6 * s + c - 1]) : 0.f;
  int held = a1 - a0;   // threads with a share
  if (a.split && a1 - a0 >= 2 * kStructChunk) {
    held = (a1 - 1) / kStructChunk - a0 / kStructChunk + 1;
    // chunk b holds this structure in slot 0 if it starts at or before the chunk
    for (int b = a0 / kStructChunk + threadIdx.x; b <= (a1 - 1) / kStructChunk; b += kRedBlk) {
      const int h = a0 > b * kStructChunk ? 1 : 0;
#pragma unroll
      for (int q = 0; q < 8; ++q) acc[q] += a.spart[(2 * (size_t)b + h) * 8 + q];
    }
  } else {
    struct_accumulate(a, a0, a1, acc);
  }
  struct_reduce(red, acc, held);
  if (threadIdx.x < kWave) {
    const double v = c < 7 ? red[c < 7 ? c : 0][0] : 0.0;
    const int n = a1 - a0;
    if (c == 0) {
      a.Es[s] = (float)v;
      if (a.Es_user) a.Es_user[s] = (float)v;
    } else if (c < 7) {
      a.Ws[6 * s + c - 1] = (float)v;
      if (a.Ws_user) a.Ws_user[6 * s + c - 1] = (float)v;
    }
    if (lab) {
      const double e = n > 0 ? (v - (double)label) / n : 0.0;
      if (c < 7) {
        const float w = n > 0 ? (float)(2.0 * (c == 0 ? a.le : a.lv) * e / ((c == 0 ? 1.0 : 6.0) * ((double)a.S * n))) : 0.f;
        if (c == 0)
          a.eps[s] = w;
        else
          a.wbar[6 * s + c - 1] = w;
      }
      const double sq = c < 7 ? e * e : 0.0;
      double lv = 0.0;
#pragma unroll
      for (int u = 1; u < 7; ++u) lv += __shfl(sq, u, kWave);
      if (c == 0) {
        a.lpart[3 * s] = sq;
        a.lpart[3 * s + 1] = red[7][0];
        a.lpart[3 * s + 2] = lv;
      }
    }
  }
  __syncthreads();   // red is read above before the next use of the LDS
}

__global__ __launch_bounds__(kRedBlk) void k_struct(StructArgs a) {
  __shared__ double red[8][kRedBlk / kWave];
  struct_body(a, blockIdx.x, red);
}

__global__ __launch_bounds__(kRedBlk) void k_loss_final(int S, int N, float le, float lf, float lv,
                                                        const double* __restrict__ lpart, float* __restrict__ loss,
                                                        int* __restrict__ flags) {
  __shared__ double red[3][kRedBlk];
  loss_final_block(S, N, le, lf, lv, lpart, loss, flags, red);
}

// ================================================================= adjoint
// Per atom, with the cotangents eps = dL/dE(n), Fbar = dL/dF and
// Gamma = dL/dW(n) frozen, the parameter gradient is the gradient of
//   Phi_i = eps E_i - E'_i . Gdot_i,  Gdot_i = sum_j dG_i/dr_ij t_ij,
//   t_ij = Fbar_j - Fbar_i + Gamma r_ij
// (the E, F and V terms of Eqs. 13-16 contracted with the residuals; the
// force and virial parts are the mixed second derivatives of C1.4-C3.20 and
// D1.11-D1.17 applied to t).
//   network: a = W0 Gdot, beta = w1 sigma (eps + 2 x a): dPhi/dW0 =
//            beta G^T - (w1 sigma) Gdot^T, dPhi/db0 = beta, dPhi/dw1 =
//            eps x - sigma a, dPhi/db1 = eps, Gbar = W0^T beta
//   radial:  dPhi/dc^R_{IJnk} = Gbar_n F[J][k] - E'_n Fp[J][k],
//            Fp[J][k] = sum_{j of type J} f'_k(r_ij) (r_hat . t)
//   angular: dPhi/dc^A_{IJnk} = sum_{j of type J} f_k X_n - f'_k (r_hat.t) Y_n,
//            X_n = sum_lm Sbar_nlm B_lm - A_nlm grad B_lm . t,
//            Y_n = sum_lm A_nlm B_lm,
//            Sbar = Gbar . dG/dS - E' . (d2G/dS2) Sdot  (the pairwise
//            coupling that Algorithm 1 enumerates).
// Outputs: per-atom vectors for the outer-product sums (W0, c^R) and, per
// wavefront, the sums of the c^A, b0, w1, b1 partials over its atoms.
// Launch index b (256 / L atoms of the species order); lds: lds_adjoint bytes.
// Slot table of the adjoint: the forward's words, then F-bar and Gamma.
constexpr int kSlotF = 12, kSlotG = 16, kSlotG2 = 20, kAdjSlot = 28;   // 4 mod 8

// LDS of the adjoint per wavefront: the slot table, then the pair records of
// the tangent sums (g_n and g'_n (u.t) interleaved, then B and grad B . t of
// one harmonic group interleaved; odd stride) and, once they are summed, the
// atoms' rows (Gdot or Gbar, Sdot or Sbar, S or A in group order; stride 4 mod 8).
// Per block: the coefficient table and the weights, whose words hold the
// coefficient gradient's records (16 pairs per wavefront) after the network.
template <class C, int L>
struct AdjLds {
  static constexpr int APW = kWave / L;
  static constexpr int DP = (C::D + 3) & ~3, YG = HSplit<C::LMAX>::YG, YR = HRow<C::LMAX>::YR;
  static constexpr int RS = (2 * C::NA + 2 * YG) | 1;
  // S at a multiple of 4 words after Sdot
  static constexpr int SW = (C::NA * YR + 3) & ~3;
  static constexpr int RW = (DP + 2 * SW + 7) / 8 * 8 + 4;
  static constexpr int BUF = ((kWave * RS > APW * RW ? kWave * RS : APW * RW) + 3) & ~3;
  static constexpr int WAVE = APW * kAdjSlot + BUF;
  static constexpr int REC = (2 * C::NA + 2 * C::KA + 1) | 1;   // X, Y (u.t), h T_k, q_k, species
  static constexpr int RECS = (256 / kWave) * 16 * REC;
  __host__ __device__ static int shared_words(int H) {
    const int w = weights_words(H, C::D, DP);
    return ((w > RECS ? w : RECS) + 3) & ~3;
  }
};

struct PairTangent {
  float ux, uy, uz, dt, wx, wy, wz;   // direction, u.t, (t - (u.t) u) / r
};
__device__ __forceinline__ PairTangent pair_tangent(const PairGeom& q, const float* sl, const float4& fj) {
  const float4 fi = *reinterpret_cast<const float4*>(sl + kSlotF);
  const float4 g = *reinterpret_cast<const float4*>(sl + kSlotG);      // xx yy zz xy
  const float4 g2 = *reinterpret_cast<const float4*>(sl + kSlotG2);    // yz zx
  PairTangent t;
  t.ux = q.dx * q.inv_r;
  t.uy = q.dy * q.inv_r;
  t.uz = q.dz * q.inv_r;
  const float tx = (fj.x - fi.x) + g.x * q.dx + g.w * q.dy;
  const float ty = (fj.y - fi.y) + g.y * q.dy + g2.x * q.dz;
  const float tz = (fj.z - fi.z) + g.z * q.dz + g2.y * q.dx;
  t.dt = t.ux * tx + t.uy * ty + t.uz * tz;
  t.wx = (tx - t.dt * t.ux) * q.inv_r;
  t.wy = (ty - t.dt * t.uy) * q.inv_r;
  t.wz = (tz - t.dt * t.uz) * q.inv_r;
  return t;
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

template <class C, bool kTri, int L>
__device__ __forceinline__ void adjoint_body(const AdjArgs& a, int b, float* lds) {
  constexpr int T = C::T, NR = C::NR, NA = C::NA, KR = C::KR, KA = C::KA, Y = C::Y, D = C::D, LM = C::LMAX;
  constexpr int L3 = C::L3, L4 = C::L4, L5 = C::L5;
  using HS = HSplit<LM>;
  using AL = AdjLds<C, L>;
  constexpr int YG = AL::YG, YR = AL::YR, DP = AL::DP, RS = AL::RS, RW = AL::RW;
  constexpr int NAH = (NA + 1) / 2;          // channels per lane in the tangent sums
  constexpr int HL = L / 2, NEH = (YG + HL - 1) / HL;          // harmonics of a group per lane there
  constexpr int NN = (NA + HL - 1) / HL;
  constexpr int PSA = T * NA * KA;
  constexpr bool kVec = YR % 4 == 0;
  const int H = a.H;
  using CT = CTab<T, NA, KA>;
  float* ctab = lds;                     // [T][NA][KAP], c^A of the block's species
  float* wl = lds + CT::size;            // its weights
  float* slots = wl + AL::shared_words(H) + (threadIdx.x / kWave) * AL::WAVE;
  float* buf = slots + (kWave / L) * kAdjSlot;
  // 32 atoms of one species, taken by L / 8 blocks
  const int vs = launch_block(a.blist, a.nch, T, b / (L / 8));
  if (vs < 0) return;
  const int vb = vs * (L / 8) + b % (L / 8);
  // issued here, waited for after the tangent sums
  const int I = block_species<T>(a.order, a.p4, vs);
  stage_weights_async(wl, a.nn, a.nn_stride, I, H, D, DP);
  stage_ctab<T, NA, KA>(ctab, a.cA + (size_t)I * T * NA * KA);
  const GroupCtx w = group_ctx<L>(a.order, a.Npad, vb);
  const int i = w.i, pa = w.pa, s = w.s, g = w.g;
  const size_t Np = a.Npad;
  const float4 me = a.p4[i];
  const int lane = threadIdx.x & (kWave - 1), slot = lane / L;
  // c^R of the species where the wavefront's records come later
  static_assert(CRad<C>::N <= AL::BUF, "the coefficients fit the records' words");
  float* crl = buf;
  for (int q = lane; q < CRad<C>::N; q += kWave) crl[q] = a.cR[(size_t)I * CRad<C>::N + q];
  const int wave = (vb * 256 + (int)threadIdx.x) / kWave;
  const bool first_atom = slot == 0;   // atom slot 0 of the wavefront writes the sums
  float* part = a.part + (size_t)wave * a.PW;
  float* row = buf + slot * RW;
  float* rowSb = row + DP;
  float* rowA = rowSb + AL::SW;
  const int st = a.astruct[i];
  const Cell cell = load_cell<kTri>(a.box, a.tilt, st);
  const float xi = me.x, yi = me.y, zi = me.z;
  const int cR_i = a.nb.cntR[i], cA_i = a.nb.cntA[i];
  const int nR = w.valid ? min(cR_i, a.nb.capR) : 0;
  const int nA = w.valid ? min(cA_i, a.nb.capA) : 0;
  const float eps_v = a.eps[st];
  const float eps = w.valid ? eps_v : 0.f;
  const float* wb = a.wbar + 6 * st;
  const float gxx = wb[0], gyy = wb[1], gzz = wb[2], gxy = wb[3], gyz = wb[4], gzx = wb[5];
  const float4 fi = a.fb4[i];
  const float fbx = fi.x, fby = fi.y, fbz = fi.z;

  // ---- radial tangent sums Fp[J][k] = sum_j f'_k(r_hat.t), pairs split over the lanes
  constexpr int NQ = (NR + L - 1) / L;
  float qn[NQ];
  {
    float FP[T * KR];
#pragma unroll
    for (int e = 0; e < T * KR; ++e) FP[e] = 0.f;
    // the next pair's atom and the list entry after it are loaded ahead
    const uint32_t* li = a.nb.idxR + (size_t)i * a.nb.capR;
    uint32_t e0 = 0, e1 = 0;
    float4 p0 = make_float4(0.f, 0.f, 0.f, 0.f), f0 = p0;
    if (s < nR) {
      e0 = li[s];
      e1 = li[min(s + L, nR - 1)];
      p0 = a.p4[e0 >> 5];
      f0 = a.fb4[e0 >> 5];
    }
    for (int k = s; k < nR; k += L) {
      const uint32_t e = e0;
      const float4 pj = p0, fj = f0;
      e0 = e1;
      p0 = a.p4[e1 >> 5];
      f0 = a.fb4[e1 >> 5];
      e1 = li[min(k + 2 * L, nR - 1)];
      const PairGeom q = packed_geom<kTri>(e, pj, xi, yi, zi, cell);
      const float tx = (fj.x - fbx) + gxx * q.dx + gxy * q.dy;
      const float ty = (fj.y - fby) + gyy * q.dy + gyz * q.dz;
      const float tz = (fj.z - fbz) + gzz * q.dz + gzx * q.dx;
      const float dt = (q.dx * tx + q.dy * ty + q.dz * tz) * q.inv_r;
      float t[KR], fp[KR];
      radial_cheb_d<KR>(q.r, a.inv_rcR, t, fp);
      const int J = packed_type<T>(pj);
#pragma unroll
      for (int u = 0; u < T; ++u) {
        const float md = (T == 1 || J == u) ? dt : 0.f;
#pragma unroll
        for (int kk = 0; kk < KR; ++kk) FP[u * KR + kk] = fmaf(md, fp[kk], FP[u * KR + kk]);
      }
    }
    float o[(T * KR + L - 1) / L];
    lds_barrier();   // the block's coefficient tables
    radial_finish<C, L>(FP, crl, s, o, qn);
    if (w.valid) {
#pragma unroll
      for (int r = 0; r < (T * KR + L - 1) / L; ++r) {
        const int e = r * L + s;
        if (T * KR % L == 0 || e < T * KR) a.FPst[(size_t)e * Np + pa] = o[r];
      }
    }
  }

  // ---- angular tangent sums Sdot_nlm = sum_j g'_n (r_hat.t) B_lm + g_n grad B_lm . t:
  //      one pair per lane writes them for one harmonic group at a time; lane s
  //      of an atom then sums its pairs for channels (s / HL) NAH + j and
  //      the harmonics (s mod HL) NEH + e of the group
  const PairStream<L> ps = pair_stream<L>(nA);
  if (s == 0) {
    float* sl = slots + slot * kAdjSlot;
    slot_store<kTri>(sl, i, xi, yi, zi, cell, ps.lo);
    *reinterpret_cast<float4*>(sl + kSlotF) = fi;
    *reinterpret_cast<float4*>(sl + kSlotG) = make_float4(gxx, gyy, gzz, gxy);
    *reinterpret_cast<float4*>(sl + kSlotG2) = make_float4(gyz, gzx, 0.f, 0.f);
  }
  // S of the forward for the rows, 16 bytes a lane
  constexpr int SW = FwdLds<C, L>::SW, NS4 = (SW / 4 + L - 1) / L;
  float4 Sr[NS4];
  {
    const float4* si = reinterpret_cast<const float4*>(a.Sst + (size_t)pa * SW);
#pragma unroll
    for (int r = 0; r < NS4; ++r) {
      const float4 v = si[min(r * L + s, SW / 4 - 1)];
      Sr[r] = w.valid ? v : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  lds_lane_exchange();
  {
    const int n0 = s / HL * NAH, h0 = (s & (HL - 1)) * NEH;
    float Sd[2][NEH][NAH];
#pragma unroll
    for (int gg = 0; gg < 2; ++gg)
#pragma unroll
      for (int e = 0; e < NEH; ++e)
#pragma unroll
        for (int j = 0; j < NAH; ++j) Sd[gg][e][j] = 0.f;
    auto tangent = [&](auto shared) {
      for (int c0 = 0; c0 < ps.total; c0 += kWave) {
        const int p = c0 + lane;
        const bool on = p < ps.total;
        float B[Y], gbt[Y];
        float* rec = buf + lane * RS;
        if (on) {
          const float* sl = slots + pair_slot(ps, p) * kAdjSlot;
          const StreamPair sp = stream_pair<T, kTri>(sl, p, a.nb, a.p4);
          const PairTangent t = pair_tangent(sp.q, sl, a.fb4[sp.q.j]);
          float f[KA], fp[KA];
          radial_cheb_d<KA>(sp.q.r, a.inv_rcA, f, fp);
          const float* cJ = ctab + sp.J * NA * CT::KAP;
#pragma unroll
          for (int n = 0; n < NA; ++n) {
            float s0 = 0.f, s1 = 0.f;
#pragma unroll
            for (int kk = 0; kk < KA; ++kk) {
              const float c = cJ[n * CT::KAP + kk];
              s0 = fmaf(c, f[kk], s0);
              s1 = fmaf(c, fp[kk], s1);
            }
            rec[2 * n] = s0;
            rec[2 * n + 1] = s1 * t.dt;
          }
          harm_val<LM>(t.ux, t.uy, t.uz, B);
          // grad B . t = grad b(u) . (t - (u.t) u) / r
          harm_dir<LM>(t.ux, t.uy, t.uz, t.wx, t.wy, t.wz, gbt);
        }
#pragma unroll
        for (int gg = 0; gg < 2; ++gg) {
          if (on) {
#pragma unroll
            for (int e = 0; e < YG; ++e) {
              const int q = HS::q(gg, e);
              rec[2 * NA + 2 * e] = q >= 0 ? B[q >= 0 ? q : 0] : 0.f;
              rec[2 * NA + 2 * e + 1] = q >= 0 ? gbt[q >= 0 ? q : 0] : 0.f;
            }
          }
          lds_lane_exchange();
          auto sums = [&](float (&S)[NEH][NAH], int t, int t1, int step) {
#pragma unroll 2
            for (; t < t1; t += step) {
              const float* rp = buf + t * RS;
              float gn[NAH], gp[NAH];
#pragma unroll
              for (int j = 0; j < NAH; ++j) {
                const int n = min(n0 + j, NA - 1);   // an odd channel count repeats the last, unused
                gn[j] = rp[2 * n];
                gp[j] = rp[2 * n + 1];
              }
#pragma unroll
              for (int e = 0; e < NEH; ++e) {
                const int q = YG % HL == 0 ? h0 + e : min(h0 + e, YG - 1);
                const float b = rp[2 * NA + 2 * q], c = rp[2 * NA + 2 * q + 1];
#pragma unroll
                for (int j = 0; j < NAH; ++j) S[e][j] = fmaf(gp[j], b, fmaf(gn[j], c, S[e][j]));
              }
            }
          };
          if constexpr (shared) {
            const ChunkShare<L> cs = chunk_share(ps, c0, slots, kAdjSlot);
            float S[NEH][NAH];
#pragma unroll
            for (int e = 0; e < NEH; ++e)
#pragma unroll
              for (int j = 0; j < NAH; ++j) S[e][j] = 0.f;
            sums(S, cs.t, cs.t1, 1 << cs.k);
            chunk_add(cs, S, Sd[gg]);
          } else {
            sums(Sd[gg], max(ps.lo - c0, 0), min(ps.hi - c0, kWave), 1);
          }
          lds_lane_exchange();
        }
      }
    };
    if (C::YH == 0 && ps.total > kSharePairs)
      tangent(std::bool_constant<C::YH == 0>{});
    else
      tangent(std::false_type{});
    wait_weights();   // before the stores below, as in the forward
    // the atoms' rows take the records' place
#pragma unroll
    for (int gg = 0; gg < 2; ++gg)
#pragma unroll
      for (int e = 0; e < NEH; ++e)
#pragma unroll
        for (int j = 0; j < NAH; ++j)
          if (n0 + j < NA && (YG % HL == 0 || h0 + e < YG)) rowSb[(n0 + j) * YR + gg * YG + h0 + e] = Sd[gg][e][j];
  }
#pragma unroll
  for (int r = 0; r < NS4; ++r)
    if (SW / 4 % L == 0 || r * L + s < SW / 4) reinterpret_cast<float4*>(rowA)[r * L + s] = Sr[r];
#pragma unroll
  for (int r = 0; r < NQ; ++r)
    if (r * L + s < NR) row[r * L + s] = qn[r];
  lds_lane_exchange();

  // ---- Gdot of the angular descriptors, channel n and harmonic group g by the
  //      lane of channel slot n mod (L / 2) and group g
  const int nAg = g ? HS::nA1 : HS::nA0;
  const int lA = g ? 2 : 1, lB = g ? 3 : 4;
  const int lAc = lA <= L3 ? lA : 1, lBc = lB <= L3 ? lB : 1;
  for (int n = w.p; n < NA; n += L / 2) {
    float Sn[YG], Sdn[YG];
    row_load<YG, kVec>(rowA + n * YR + g * YG, Sn);
    row_load<YG, kVec>(rowSb + n * YR + g * YG, Sdn);
    float qa = 0.f, qb = 0.f;
#pragma unroll
    for (int e = 0; e < YG; ++e) {
      const float v = 2.0f * csel<HS>(g, e) * Sn[e] * Sdn[e];
      if (e < nAg) qa += v; else qb += v;
    }
    if (lA <= L3) row[NR + (lA - 1) * NA + n] = qa;
    if (lB <= L3) row[NR + (lB - 1) * NA + n] = qb;
    if constexpr (L4 != 0) {
      const Sym3 M = sym_of(Sn[0], Sn[1], Sn[2], Sn[3], Sn[4]);
      const Sym3 Md = sym_of(Sdn[0], Sdn[1], Sdn[2], Sdn[3], Sdn[4]);
      const float v = 3.0f * sym_dot(sym_mul(M, M), Md);
      if (g == 1) row[NR + L3 * NA + n] = v;
    }
    if constexpr (L5 != 0) {
      const float P = Sn[0] * Sn[0] + Sn[1] * Sn[1] + Sn[2] * Sn[2];
      const float SS = Sn[0] * Sdn[0] + Sn[1] * Sdn[1] + Sn[2] * Sdn[2];
      if (g == 0) row[NR + L3 * NA + (L4 ? NA : 0) + n] = 4.0f * P * SS;
    }
  }
  if constexpr (C::YH > 0) {
    // Gdot of q_nl, l = 5..L3, from k_high_tangent
    for (int v = NR + 4 * NA + s; v < NR + L3 * NA; v += L) {
      const float x = a.Gd[(size_t)v * Np + pa];
      row[v] = w.valid ? x : 0.f;
    }
  }
  lds_barrier();
  float Gd[DP];
  row_load<DP, true>(row, Gd);   // words past D are not used
  if (w.valid) {
#pragma unroll
    for (int r = 0; r < (D + L - 1) / L; ++r) {
      const int v = r * L + s;
      if (D % L == 0 || v < D) a.Gd[(size_t)v * Np + pa] = row[v];
    }
  }
  // E' of the descriptors this lane's Sbar and A need, loaded ahead of the network
  float epA[NN], epB[NN], ep4[NN], ep5[NN];
#pragma unroll
  for (int r = 0; r < NN; ++r) {
    const int n = min(w.p + HL * r, NA - 1);
    epA[r] = a.Ep[(size_t)(NR + (lAc - 1) * NA + n) * Np + pa];
    epB[r] = a.Ep[(size_t)(NR + (lBc - 1) * NA + n) * Np + pa];
    ep4[r] = L4 ? a.Ep[(size_t)(NR + L3 * NA + n) * Np + pa] : 0.f;
    ep5[r] = L5 ? a.Ep[(size_t)(NR + L3 * NA + (L4 ? NA : 0) + n) * Np + pa] : 0.f;
  }

  // ---- network adjoint, hidden units mu = s, s + L, ...
  const float* Wl = wl;
  {
    float Gb[D];
#pragma unroll
    for (int v = 0; v < D; ++v) Gb[v] = 0.f;
    const int RH = (H + L - 1) / L;
    for (int r = 0; r < RH; ++r) {
      const int mu = r * L + s;
      const bool act = mu < H;
      const int mm = act ? mu : H - 1;
      const float* wr = Wl + mm * DP;
      const float xv = a.X[(size_t)mm * Np + pa];
      float aa = 0.f;
#pragma unroll
      for (int v = 0; v < D; ++v) aa = fmaf(wr[v], Gd[v], aa);
      const bool live = act && w.valid;
      const float x = live ? xv : 0.f;
      const float sg = 1.0f - x * x;
      const float ws = weight_w1<D, DP>(Wl, H, mm) * sg;
      const float be = live ? ws * (eps + 2.0f * x * aa) : 0.f;
#pragma unroll
      for (int v = 0; v < D; ++v) Gb[v] = fmaf(be, wr[v], Gb[v]);
      if (live) a.beta[(size_t)mu * Np + pa] = be;
      const float r0 = atoms_sum<L>(be);
      const float r1 = atoms_sum<L>(live ? eps * x - sg * aa : 0.f);
      if (act && first_atom) {
        part[PSA + mu] = r0;
        part[PSA + H + mu] = r1;
      }
    }
    {
      const float r = atoms_sum<L>(s == 0 ? eps : 0.f);
      if (lane == 0) part[PSA + 2 * H] = r;
    }
    // Gbar to the row's first D words (Gdot there has been read)
    float go[(D + L - 1) / L];
    rs_group<L>(Gb, go);
#pragma unroll
    for (int r = 0; r < (D + L - 1) / L; ++r) {
      const int v = r * L + s;
      if (D % L == 0 || v < D) {
        row[v] = go[r];
        // radial rows for the c^R gradient; l = 5..L3 for k_high_coef (the rows hold D entries)
        if (w.valid && (v < NR || (C::YH > 0 && v >= NR + 4 * NA && v < NR + L3 * NA))) a.Gbr[(size_t)v * Np + pa] = go[r];
      }
    }
  }
  lds_lane_exchange();

  // ---- Sbar and A of this lane's harmonic group, in place of Sdot and S.  With
  //      degrees l > 4 group and channel slot are taken anew: the row offsets and
  //      harmonic constants of the first pass were otherwise kept over the network
  //      and spilled (87,471 atoms: 52 -> 12 bytes a lane, 109 -> 97.5 us).  The
  //      others spill nothing, and forming them again took 0.3 % of their step.
  const int gb = C::YH > 0 ? opaque_int(g) : g, pb = C::YH > 0 ? opaque_int(w.p) : w.p;
  const int lAb = gb ? 2 : 1, lBb = gb ? 3 : 4, nAb = gb ? HS::nA1 : HS::nA0;
#pragma unroll
  for (int r = 0; r < NN; ++r) {
    const int n = pb + HL * r;
    if (n < NA) {
      float Sn[YG], Sdn[YG];
      row_load<YG, kVec>(rowA + n * YR + gb * YG, Sn);
      row_load<YG, kVec>(rowSb + n * YR + gb * YG, Sdn);
      // E' and Gbar of the descriptors built from these sums
      const float bA = row[NR + ((lAb <= L3 ? lAb : 1) - 1) * NA + n], bB = row[NR + ((lBb <= L3 ? lBb : 1) - 1) * NA + n];
      const float eA = (w.valid && lAb <= L3) ? epA[r] : 0.f;
      const float eB = (w.valid && lBb <= L3) ? epB[r] : 0.f;
      const float gA = lAb <= L3 ? bA : 0.f, gB = lBb <= L3 ? bB : 0.f;
      float o[5] = {0.f, 0.f, 0.f, 0.f, 0.f}, od[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
      float e4 = 0.f, g4 = 0.f, e5 = 0.f, g5 = 0.f, P = 0.f, SS = 0.f;
      if constexpr (L4 != 0) {
        const Sym3 M = sym_of(Sn[0], Sn[1], Sn[2], Sn[3], Sn[4]);
        const Sym3 Md = sym_of(Sdn[0], Sdn[1], Sdn[2], Sdn[3], Sdn[4]);
        sym_proj(sym_mul(M, M), o);
        sym_proj(sym_mul(Md, M), od);
        const float b = row[NR + L3 * NA + n];
        e4 = (w.valid && gb == 1) ? ep4[r] : 0.f;
        g4 = gb == 1 ? b : 0.f;
      }
      if constexpr (L5 != 0) {
        P = Sn[0] * Sn[0] + Sn[1] * Sn[1] + Sn[2] * Sn[2];
        SS = Sn[0] * Sdn[0] + Sn[1] * Sdn[1] + Sn[2] * Sdn[2];
        const float b = row[NR + L3 * NA + (L4 ? NA : 0) + n];
        e5 = (w.valid && gb == 0) ? ep5[r] : 0.f;
        g5 = gb == 0 ? b : 0.f;
      }
#pragma unroll
      for (int e = 0; e < YG; ++e) {
        const bool real = gb ? HRow<LM>::real(1, e) : HRow<LM>::real(0, e);
        const float c2 = 2.0f * csel<HS>(gb, e);
        const float eL = e < nAb ? eA : eB, gL = e < nAb ? gA : gB;
        float Av = c2 * eL * Sn[e];
        float Sb = c2 * (gL * Sn[e] - eL * Sdn[e]);
        if (e < 5) {
          Av += 3.0f * e4 * o[e];
          Sb += 3.0f * g4 * o[e] - 6.0f * e4 * od[e];
        }
        if (e < 3) {
          Av += 4.0f * e5 * P * Sn[e];
          Sb += 4.0f * g5 * P * Sn[e] - e5 * (8.0f * SS * Sn[e] + 4.0f * P * Sdn[e]);
        }
        rowA[n * YR + gb * YG + e] = real ? Av : 0.f;
        rowSb[n * YR + gb * YG + e] = real ? Sb : 0.f;
      }
    }
  }
  lds_barrier();   // also: every wavefront is done with the weights, whose words the records below take

  // ---- angular coefficient gradient.  One pair per lane forms X_n and Y_n (u.t);
  //      the sums over pairs of X_n h T_k - Y_n (u.t) q_k, per neighbor species,
  //      are a product contracted over pairs on the fp32 matrix cores: rows
  //      (species, n), columns k, 4 pairs per instruction.  16 pairs at a time
  //      go through LDS to reach the operands' lanes.
  constexpr int REC = AL::REC, ROWS = T * NA, MT = (ROWS + 15) / 16;
  static_assert(KA <= 16, "one column tile");
  float* recs = wl + (threadIdx.x / kWave) * 16 * REC;
  f32x4 acc[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) acc[m] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int c0 = 0; c0 < ps.total; c0 += kWave) {
    const int p = c0 + lane;
    float X[NA], Yd[NA], f[KA], fp[KA];
    int J = 0;
#pragma unroll
    for (int n = 0; n < NA; ++n) X[n] = Yd[n] = 0.f;
#pragma unroll
    for (int kk = 0; kk < KA; ++kk) f[kk] = fp[kk] = 0.f;
    if (p < ps.total) {
      const int u = pair_slot(ps, p);
      const float* sl = slots + u * kAdjSlot;
      const StreamPair sp = stream_pair<T, kTri>(sl, p, a.nb, a.p4);
      const PairTangent t = pair_tangent(sp.q, sl, a.fb4[sp.q.j]);
      radial_cheb_d<KA>(sp.q.r, a.inv_rcA, f, fp);
      J = sp.J;
      float B[Y], gbt[Y];
      harm_val<LM>(t.ux, t.uy, t.uz, B);
      harm_dir<LM>(t.ux, t.uy, t.uz, t.wx, t.wy, t.wz, gbt);
      const float* sb = buf + u * RW + DP;
#pragma unroll
      for (int n = 0; n < NA; ++n) {
        float x = 0.f, y = 0.f;
#pragma unroll
        for (int gg = 0; gg < 2; ++gg) {
          float Sb[YG], Av[YG];
          row_load<YG, kVec>(sb + n * YR + gg * YG, Sb);
          row_load<YG, kVec>(sb + AL::SW + n * YR + gg * YG, Av);
#pragma unroll
          for (int e = 0; e < YG; ++e) {
            const int qq = HS::q(gg, e);
            if (qq >= 0) {
              x = fmaf(Sb[e], B[qq], fmaf(-Av[e], gbt[qq], x));
              y = fmaf(Av[e], B[qq], y);
            }
          }
        }
        X[n] = x;
        Yd[n] = y * t.dt;
      }
    }
    const int left = ps.total - c0;   // wave-uniform
#pragma unroll
    for (int sub = 0; sub < 4; ++sub) {
      if (16 * sub >= left) break;
      if ((lane >> 4) == sub) {
        float* rp = recs + (lane & 15) * REC;
#pragma unroll
        for (int n = 0; n < NA; ++n) {
          rp[n] = X[n];
          rp[NA + n] = -Yd[n];
        }
#pragma unroll
        for (int kk = 0; kk < KA; ++kk) {
          rp[2 * NA + kk] = f[kk];
          rp[2 * NA + KA + kk] = fp[kk];
        }
        rp[2 * NA + 2 * KA] = __int_as_float(J);
      }
      lds_lane_exchange();
      const int col = min(lane & 15, KA - 1);   // columns past KA are not stored
#pragma unroll
      for (int m4 = 0; m4 < 4; ++m4) {
        const float* rp = recs + (4 * m4 + (lane >> 4)) * REC;
        const float bT = rp[2 * NA + col], bQ = rp[2 * NA + KA + col];
        const int Jp = __float_as_int(rp[2 * NA + 2 * KA]);
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          const int rr = m * 16 + (lane & 15), t = rr / NA, n = rr % NA;
          const bool mine = t == Jp;   // rows past T NA match no species
          const float aX = rp[n], aY = rp[NA + n];
          acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(mine ? aX : 0.f, bT, acc[m], 0, 0, 0);
          acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(mine ? aY : 0.f, bQ, acc[m], 0, 0, 0);
        }
      }
      lds_lane_exchange();
    }
  }
  // f_k = h T_k + h T_0: every column takes column 0's sum
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float v = acc[m][r] + dpp<kDppRowBcast0>(acc[m][r]);
      const int rr = m * 16 + 4 * (lane >> 4) + r, kk = lane & 15;
      if (rr < ROWS && kk < KA) part[rr * KA + kk] = v;
    }
}

template <class C, bool kTri, int W, int L>
__global__ __launch_bounds__(256, W) void k_adjoint(AdjArgs a) {
  extern __shared__ __align__(16) float lds[];
  adjoint_body<C, kTri, L>(a, blockIdx.x, lds);
}

// Sums over the atoms of each species of an outer product,
//   out[I][b][m][v] = sum_p A1[m][p] B1[v][p] - A2[m][p] B2[v][p],
// over block b's share of species I's atoms (species order).  Used for
// dL/dW0 = sum beta G^T - (w1 (1 - x^2)) Gdot^T and for
// dL/dc^R = sum Gbar_n F[J][k] - E'_n Fp[J][k].
// This is a product contracted over atoms, so it runs on the fp32 matrix
// cores: v_mfma_f32_16x16x4f32 takes a 16 x 4 slice of A (lane l: row l % 16,
// atom slot l / 16) and a 4 x 16 slice of B, and accumulates a 16 x 16 tile
// of which lane l holds rows 4 (l / 16) + r, column l % 16.  Each lane loads
// float4 runs of 4 consecutive atoms and feeds component j to the j-th of 4
// MFMAs, so atom slot l / 16 of MFMA j is atom 4 (l / 16) + j of the 16-atom
// group.  A block covers a 2 x 3 grid of 16 x 16 output tiles (blockIdx.z
// picks the grid cell for larger products); its 4 wavefronts take
// consecutive 16-atom groups and are summed through LDS at the end.
// Blocks per species and output slice: the W0 sums stream about three times
// the data of the c^R sums.  At 512 structures (87k atoms) the step takes
// 315 us with 96 blocks for W0 (two slices), 320 with 128, 326 with 192.
constexpr int kOSBlocksW = 96, kOSBlocksC = 64;            // defaults
constexpr int kOSBlocksMaxW = 512, kOSBlocksMaxC = 256;
constexpr int kOSTM = 2, kOSTV = 3;

struct OuterArgs {
  int Npad, M, V, NB;
  int T, nch, Q;      // block b: piece b mod Q of chunks b / Q, b / Q + NB / Q, ...
  const int* seg;
  const float* A1;
  const float* B1;
  const float* A2;    // with w1: the hidden activations x, the operand being w1 (1 - x^2)
  const float* B2;
  float* out;
  const float* w1;    // [T] blocks of w1_stride words, null: A2 as it is
  int w1_stride;
};

// atoms p .. p + 3 of a row (p a multiple of 4 inside the padded row), zero
// past p1; the load itself is unconditional so that a group's loads issue
// back to back
__device__ __forceinline__ f32x4 ld_atoms4(const float* row, int p, int p1) {
  const float4 v = *reinterpret_cast<const float4*>(row + p);
  f32x4 r;
  r[0] = p < p1 ? v.x : 0.f;
  r[1] = p + 1 < p1 ? v.y : 0.f;
  r[2] = p + 2 < p1 ? v.z : 0.f;
  r[3] = p + 3 < p1 ? v.w : 0.f;
  return r;
}

constexpr int kOuterLds = 3 * kOSTM * kOSTV * kWave * sizeof(f32x4);
__device__ __forceinline__ void outer_sum_block(const OuterArgs& o, int b, int I, int z,
                                                f32x4 (&red)[3][kOSTM * kOSTV][kWave]) {
  if (b >= o.NB) return;
  const int nzv = (o.V + 16 * kOSTV - 1) / (16 * kOSTV);
  const int mz = z / nzv, vz = z % nzv;
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
  const int row = lane & 15, slot = lane >> 4;
  int start = 0, p1 = 0;
  const float* a1[kOSTM];
  const float* a2[kOSTM];
  const float* b1[kOSTV];
  const float* b2[kOSTV];
#pragma unroll
  for (int t = 0; t < kOSTM; ++t) {
    const int m = (mz * kOSTM + t) * 16 + row;
    a1[t] = o.A1 + (size_t)(m < o.M ? m : 0) * o.Npad;
    a2[t] = o.A2 + (size_t)(m < o.M ? m : 0) * o.Npad;
  }
#pragma unroll
  for (int t = 0; t < kOSTV; ++t) {
    const int v = (vz * kOSTV + t) * 16 + row;
    b1[t] = o.B1 + (size_t)(v < o.V ? v : 0) * o.Npad;
    b2[t] = o.B2 + (size_t)(v < o.V ? v : 0) * o.Npad;
  }
  float w1[kOSTM];
#pragma unroll
  for (int t = 0; t < kOSTM; ++t) {
    const int m = (mz * kOSTM + t) * 16 + row;
    w1[t] = o.w1 && m < o.M ? o.w1[(size_t)I * o.w1_stride + m] : 0.f;
  }
  // tiles with no row or no column inside the product are skipped (uniform)
  const int tm_live = min(kOSTM, (o.M - mz * kOSTM * 16 + 15) / 16);
  const int tv_live = min(kOSTV, (o.V - vz * kOSTV * 16 + 15) / 16);
  f32x4 acc[kOSTM][kOSTV];
#pragma unroll
  for (int x = 0; x < kOSTM; ++x)
#pragma unroll
    for (int y = 0; y < kOSTV; ++y) acc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
  // operands of one 16-atom group; the next group's loads are issued before
  // the current group's MFMAs
  f32x4 va1[kOSTM], va2[kOSTM], vb1[kOSTV], vb2[kOSTV];
  // Rows and columns past the product repeat row or column 0 and are not
  // stored.  Past the block's atoms the loads read the segment start (always
  // inside the padded rows) and are masked to zero.
  auto load = [&](int g) {
    const int p = (g < p1 ? g : start) + 4 * slot, pe = g < p1 ? p1 : 0;
#pragma unroll
    for (int t = 0; t < kOSTM; ++t) {
      va1[t] = ld_atoms4(a1[t], p, pe);
      va2[t] = ld_atoms4(a2[t], p, pe);
    }
#pragma unroll
    for (int t = 0; t < kOSTV; ++t) {
      vb1[t] = ld_atoms4(b1[t], p, pe);
      vb2[t] = ld_atoms4(b2[t], p, pe);
    }
  };
  for (int c = b / o.Q; c < o.nch; c += o.NB / o.Q) {
  start = o.seg[2 * (c * o.T + I)];
  const int count = o.seg[2 * (c * o.T + I) + 1];
  const int per = ((count + o.Q - 1) / o.Q + 15) & ~15;   // multiple of 16 atoms
  const int p0 = start + b % o.Q * per;
  p1 = min(start + count, p0 + per);
  if (p0 >= p1) continue;
  load(p0 + 16 * wv);
  for (int g = p0 + 16 * wv; g < p1; g += 64) {
    f32x4 ca1[kOSTM], ca2[kOSTM], cb1[kOSTV], cb2[kOSTV];
    // minus the second product: -A2, or w1 (x^2 - 1) (B2 is zero past the end)
#pragma unroll
    for (int t = 0; t < kOSTM; ++t) {
      ca1[t] = va1[t];
#pragma unroll
      for (int j = 0; j < 4; ++j) ca2[t][j] = o.w1 ? w1[t] * fmaf(va2[t][j], va2[t][j], -1.0f) : -va2[t][j];
    }
#pragma unroll
    for (int t = 0; t < kOSTV; ++t) {
      cb1[t] = vb1[t];
      cb2[t] = vb2[t];
    }
    load(g + 64);
#pragma unroll
    for (int x = 0; x < kOSTM; ++x) {
      if (x >= tm_live) break;
#pragma unroll
      for (int y = 0; y < kOSTV; ++y) {
        if (y >= tv_live) break;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(ca1[x][j], cb1[y][j], acc[x][y], 0, 0, 0);
          acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(ca2[x][j], cb2[y][j], acc[x][y], 0, 0, 0);
        }
      }
    }
  }
  }
  if (wv > 0) {
#pragma unroll
    for (int x = 0; x < kOSTM; ++x)
#pragma unroll
      for (int y = 0; y < kOSTV; ++y) red[wv - 1][x * kOSTV + y][lane] = acc[x][y];
  }
  __syncthreads();
  if (wv != 0) {
    __syncthreads();
    return;
  }
  float* out = o.out + ((size_t)I * o.NB + b) * o.M * o.V;
#pragma unroll
  for (int x = 0; x < kOSTM; ++x)
#pragma unroll
    for (int y = 0; y < kOSTV; ++y) {
      f32x4 s4 = acc[x][y];
#pragma unroll
      for (int w = 0; w < 3; ++w) s4 += red[w][x * kOSTV + y][lane];
      const int v = (vz * kOSTV + y) * 16 + row;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = (mz * kOSTM + x) * 16 + 4 * slot + r;
        if (m < o.M && v < o.V) out[m * o.V + v] = s4[r];
      }
    }
  __syncthreads();   // the other wavefronts wait here: red is read above
}

int outer_slices(int M, int V) {
  const int nzm = (M + 16 * kOSTM - 1) / (16 * kOSTM), nzv = (V + 16 * kOSTV - 1) / (16 * kOSTV);
  return nzm * nzv;
}

// First stage of the final reduction for the wavefront partials (c^A, b0,
// w1, b1): block (b, I) sums, in float64 and in wave order, chunk b of the
// wavefronts of species I; one thread per slot, so reads run along rows.
constexpr int kPRChunks = 128;   // default chunks per species
constexpr int kPRChunksMax = 512;

// Loss reduction carried by k_outer_reduce (one extra block) so that a
// loss-and-gradient pass spends no launch on it.
struct LossArgs {
  int on, S, N;
  float le, lf, lv;
  const double* lpart;
  float* loss;
  int* flags;
};

// block b of species I's wavefront partials, pieces of the order's chunks as
// for the outer-product sums
struct PartArgs {
  int PW, NB, T, nch, Q, apw;   // apw: atoms per wavefront of the adjoint
  const int* seg;
  const float* part;
  double* pp;
};
__device__ __forceinline__ void part_reduce_body(const PartArgs& a, int b, int I) {
  const int PW = a.PW;
  for (int slot = threadIdx.x; slot < PW; slot += blockDim.x) {
    double sum = 0.0;
    for (int c = b / a.Q; c < a.nch; c += a.NB / a.Q) {
      const int start = a.seg[2 * (c * a.T + I)], count = a.seg[2 * (c * a.T + I) + 1];
      const int w0 = start / a.apw, w1 = (start + count + a.apw - 1) / a.apw;
      const int per = (w1 - w0 + a.Q - 1) / a.Q;
      int r = w0 + b % a.Q * per;
      const int r1 = min(w1, r + per);
      for (; r + 16 <= r1; r += 16) {
        float v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = a.part[(size_t)(r + u) * PW + slot];
#pragma unroll
        for (int u = 0; u < 16; ++u) sum += (double)v[u];
      }
      for (; r + 4 <= r1; r += 4) {
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = a.part[(size_t)(r + u) * PW + slot];
#pragma unroll
        for (int u = 0; u < 4; ++u) sum += (double)v[u];
      }
      for (; r < r1; ++r) sum += (double)a.part[(size_t)r * PW + slot];
    }
    a.pp[((size_t)I * a.NB + b) * PW + slot] = sum;
  }
}

// The outer-product sums, the first stage of the wavefront partial sums and
// the loss sum in one launch (all three read only the adjoint's outputs):
// blocks [0, n_outer) take the outer products (block x of species I, output
// slice z; slices [0, nzw) of dW0, the rest of dc^R), the next pr.NB T blocks
// the partial sums, the last one the loss.
struct OuterReduceArgs {
  OuterArgs ow, oc;
  int nzw, nzc, os_x, T;
  PartArgs pr;
  LossArgs la;
};

__global__ __launch_bounds__(256, 3) void k_outer_reduce(OuterReduceArgs a) {
  __shared__ f32x4 red[3][kOSTM * kOSTV][kWave];
  const int T = a.T, n_outer = a.os_x * T * (a.nzw + a.nzc), n_pr = a.pr.NB * T;
  const int v = blockIdx.x;
  if (v < n_outer) {
    const int x = v % a.os_x, I = (v / a.os_x) % T, z = v / (a.os_x * T);
    if (z < a.nzw)
      outer_sum_block(a.ow, x, I, z, red);
    else
      outer_sum_block(a.oc, x, I, z - a.nzw, red);
  } else if (v < n_outer + n_pr) {
    const int u = v - n_outer;
    part_reduce_body(a.pr, u % a.pr.NB, u / a.pr.NB);
  } else if (a.la.on) {
    loss_final_block(a.la.S, a.la.N, a.la.le, a.la.lf, a.la.lv, a.la.lpart, a.la.loss, a.la.flags, red);
  }
}


// Final gradient: 16 lanes per parameter; lane l sums rows l, l + 16, ... of
// that parameter's partials in float64, then a fixed xor tree adds the 16
// lane sums.  Parameter layout: c^R [T][T][NR][KR], c^A [T][T][NA][KA], then
// per species W0 [H][D], b0 [H], w1 [H], b1.
// ==================================================================== Adam
// One parameter's update, with the fused forms written out so that the captured
// step and the eager one round the moments alike.  (c1 and c2 are formed in
// single precision on the device and in double on the host.)
__device__ __forceinline__ void adam_update(float& th, float& m, float& v, float g, float lr, float b1, float b2,
                                            float eps, float c1, float c2) {
  m = fmaf(1.0f - b1, g, b1 * m);
  v = fmaf((1.0f - b2) * g, g, b2 * v);
  th -= lr * (m / c1) / (sqrtf(v / c2) + eps);
}
__device__ __forceinline__ void adam_one(float* __restrict__ th, float* __restrict__ m, float* __restrict__ v,
                                         float g, float lr, float b1, float b2, float eps, float c1, float c2,
                                         int64_t q) {
  float t = th[q], mm = m[q], vv = v[q];
  adam_update(t, mm, vv, g, lr, b1, b2, eps, c1, c2);
  m[q] = mm;
  v[q] = vv;
  th[q] = t;
}

__global__ __launch_bounds__(256) void k_adam(int64_t P, float* __restrict__ th, float* __restrict__ m,
                                              float* __restrict__ v, const float* __restrict__ g, float lr, float b1,
                                              float b2, float eps, float c1, float c2) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < P) adam_one(th, m, v, g[q], lr, b1, b2, eps, c1, c2, q);
}

struct AdamDev {
  float lr_start, lr_stop;
  int64_t n_warmup, n_total;
  float b1, b2, eps;
};

__device__ float lr_at(const AdamDev& c, int64_t s) {
  if (c.n_total <= 0) return c.lr_start;
  if (s < c.n_warmup) return c.lr_stop + (float)((double)s / (double)c.n_warmup) * (c.lr_start - c.lr_stop);
  double fr = (double)(s - c.n_warmup) / (double)max((int64_t)1, c.n_total - c.n_warmup);
  fr = fr > 1.0 ? 1.0 : fr;
  return c.lr_stop + (c.lr_start - c.lr_stop) * 0.5f * (1.0f + (float)cos(3.14159265358979323846 * fr));
}

// ------------------------------------------------- padded models: layout maps
// A model smaller than a compiled size class runs in that class with its
// parameters zero-padded: radial and angular channels, Chebyshev terms and
// species the model does not have get zero coefficients, and the network's
// columns of descriptors it does not have (higher channels, degrees up to the
// class's, the 4- and 5-body terms) get zero weights.  Every padded quantity
// then adds an exact zero to the energies, forces and virials, and the
// gradient entries of the model's own parameters are those of the class run.
// PadDims maps a parameter of the model to its slot in the class layout.
struct PadDims {
  int T, NR, NA, KR, KA, D, H, l3, l4, l5;   // the model
  int Tc, NRc, NAc, KRc, KAc, Dc, L3c;       // the class (4- and 5-body terms on)
  int64_t P;                                 // parameters of the model
};

// class column of descriptor v of the model
__device__ __forceinline__ int pad_col(const PadDims& d, int v) {
  if (v < d.NR) return v;
  v -= d.NR;
  if (v < d.l3 * d.NA) return d.NRc + (v / d.NA) * d.NAc + v % d.NA;
  v -= d.l3 * d.NA;
  if (d.l4) {
    if (v < d.NA) return d.NRc + d.L3c * d.NAc + v;
    v -= d.NA;
  }
  return d.NRc + d.L3c * d.NAc + d.NAc + v;   // 5-body
}

// 32-bit: a supported model has under 2^31 parameters
__device__ __forceinline__ int pad_index(const PadDims& d, int q) {
  const int PR = d.T * d.T * d.NR * d.KR, PA = d.T * d.T * d.NA * d.KA;
  const int PRc = d.Tc * d.Tc * d.NRc * d.KRc, PAc = d.Tc * d.Tc * d.NAc * d.KAc;
  if (q < PR) {
    const int k = q % d.KR, n = (q / d.KR) % d.NR, J = (q / (d.KR * d.NR)) % d.T;
    const int I = q / (d.KR * d.NR * d.T);
    return ((I * d.Tc + J) * d.NRc + n) * d.KRc + k;
  }
  q -= PR;
  if (q < PA) {
    const int k = q % d.KA, n = (q / d.KA) % d.NA, J = (q / (d.KA * d.NA)) % d.T;
    const int I = q / (d.KA * d.NA * d.T);
    return PRc + ((I * d.Tc + J) * d.NAc + n) * d.KAc + k;
  }
  q -= PA;
  const int HD = d.H * d.D;
  const int blk = HD + 2 * d.H + 1, blkc = d.H * d.Dc + 2 * d.H + 1;
  const int I = q / blk, o = q % blk;
  const int base = PRc + PAc + I * blkc;
  if (o < HD) return base + (o / d.D) * d.Dc + pad_col(d, o % d.D);
  return base + d.H * d.Dc + (o - HD);   // b0, w1, b1
}

struct GradArgs {
  int T, NR, NA, KR, KA, H, D, PW, NBw, NBc, PRC;
  int64_t P;
  const double* pp;      // [T][PRC][PW]
  const float* w0part;   // [T][NBw][H*D]
  const float* crpart;   // [T][NBc][NR*T*KR]
  float* grad;
  int pad;               // a padded model: parameters mapped into the class layout of the sums
  PadDims pd;
  // Adam on each parameter as soon as its gradient is summed (the captured
  // training step); step is the 1-based device step counter
  int adam;
  AdamDev ad;
  float* th;
  float* mm;
  float* vv;
  const int* step;
  int* flags;   // the replay's flag word: any raised flag skips the update
};

// Whether a captured step may update parameter q: no flag was raised by this
// replay's neighbor build or loss (their launches precede this one), the
// latched step is valid, and the gradient entry is finite (else the flag is
// raised and this entry alone keeps its value).
__device__ __forceinline__ bool adam_allowed(int* flags, int fl0, int st, float g) {
  if (!isfinite(g)) {
    atomicOr(flags, FL_NONFINITE);
    return false;
  }
  return fl0 == 0 && st >= 1;
}

// Block vb: parameters 16 vb .. 16 vb + 15.  What Adam needs is loaded, and its
// rate and bias corrections formed, while the first partial sums are on their
// way (as a chain after the sums: 5.3 us of a 58 us step of 544 atoms).
__device__ __forceinline__ void grad_final_body(const GradArgs& a, int vb) {
  const int64_t q = ((int64_t)vb * 256 + threadIdx.x) >> 4;
  const int l = threadIdx.x & 15;
  const int P_R = a.T * a.T * a.NR * a.KR, P_A = a.T * a.T * a.NA * a.KA;
  const int blk = a.H * a.D + 2 * a.H + 1;
  const int PSA = a.T * a.NA * a.KA;
  const int HD = a.H * a.D, CR = a.NR * a.T * a.KR;
  double sum = 0.0;
  const bool out = q < a.P && l == 0;
  float th = 0.f, m = 0.f, v = 0.f;
  int st = 0, fl0 = 0;
  if (a.adam) {
    st = *a.step;
    fl0 = __hip_atomic_load(a.flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (out) {
      th = a.th[q];
      m = a.mm[q];
      v = a.vv[q];
    }
  }
  const float* fsrc = nullptr;
  const double* dsrc = nullptr;
  int stride = 0, rows = 0;
  if (q < a.P) {
    const int qi = a.pad ? pad_index(a.pd, (int)q) : (int)q;
    if (qi < P_R) {
      const int I = qi / (a.T * a.NR * a.KR), rem = qi % (a.T * a.NR * a.KR);
      const int t = rem / (a.NR * a.KR), n = (rem / a.KR) % a.NR, k = rem % a.KR;
      fsrc = a.crpart + (size_t)I * a.NBc * CR + n * (a.T * a.KR) + t * a.KR + k;
      stride = CR;
      rows = a.NBc;
    } else if (qi < P_R + P_A) {
      const int I = (qi - P_R) / PSA, slot = (qi - P_R) % PSA;
      dsrc = a.pp + (size_t)I * a.PRC * a.PW + slot;
      stride = a.PW;
      rows = a.PRC;
    } else {
      const int I = (qi - P_R - P_A) / blk, o = (qi - P_R - P_A) % blk;
      if (o < HD) {
        fsrc = a.w0part + (size_t)I * a.NBw * HD + o;
        stride = HD;
        rows = a.NBw;
      } else {
        dsrc = a.pp + (size_t)I * a.PRC * a.PW + PSA + (o - HD);
        stride = a.PW;
        rows = a.PRC;
      }
    }
    if (l < rows) sum = fsrc ? (double)fsrc[(size_t)l * stride] : dsrc[(size_t)l * stride];
  }
  float lr = 0.f, c1 = 1.f, c2 = 1.f;
  if (a.adam) {
    lr = lr_at(a.ad, (int64_t)(st - 1));
    c1 = 1.0f - powf(a.ad.b1, (float)st);
    c2 = 1.0f - powf(a.ad.b2, (float)st);
  }
  if (fsrc) {
    for (int r = l + 16; r < rows; r += 16) sum += (double)fsrc[(size_t)r * stride];
  } else {
    for (int r = l + 16; r < rows; r += 16) sum += dsrc[(size_t)r * stride];
  }
#pragma unroll
  for (int d = 8; d >= 1; d >>= 1) sum += __shfl_xor(sum, d, 16);
  if (out) {
    const float gq = (float)sum;
    a.grad[q] = gq;
    if (a.adam && adam_allowed(a.flags, fl0, st, gq)) {
      adam_update(th, m, v, gq, lr, a.ad.b1, a.ad.b2, a.ad.eps, c1, c2);
      a.mm[q] = m;
      a.vv[q] = v;
      a.th[q] = th;
    }
  }
}

__global__ __launch_bounds__(256) void k_grad_final(GradArgs a) { grad_final_body(a, blockIdx.x); }

// Adam with the step counter read from device memory (graph replays).
__global__ __launch_bounds__(256) void k_adam_dev(int64_t P, float* __restrict__ th, float* __restrict__ m,
                                                  float* __restrict__ v, const float* __restrict__ g,
                                                  const int* __restrict__ step, int* flags, AdamDev c) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= P) return;
  const int st = *step;
  if (!adam_allowed(flags, __hip_atomic_load(flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), st, g[q])) return;
  const float lr = lr_at(c, (int64_t)(st - 1));
  const float c1 = 1.0f - powf(c.b1, (float)st), c2 = 1.0f - powf(c.b2, (float)st);
  adam_one(th, m, v, g[q], lr, c.b1, c.b2, c.eps, c1, c2, q);
}

// First node of a captured train step: clear the flags, latch the step this
// replay uses (Adam reads the latched copy) and advance the caller's counter.
// A step counter below 1 (Adam's bias correction needs step >= 1) raises
// FL_STEP, which makes this replay skip its update.
__device__ __forceinline__ void graph_head(int* flags, int* step, int* cur) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    const int st = step[0];
    flags[0] = st < 1 ? FL_STEP : 0;
    cur[0] = st;
    step[0] = st + 1;
  }
}
__global__ void k_graph_head(int* flags, int* step, int* cur) { graph_head(flags, step, cur); }


__global__ void k_fill_f32(float* p, int64_t n, float v) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n) p[q] = v;
}

// ============================================================ persistent step
// The whole step after the neighbor build in one launch: the species order,
// forward, force pass, per-structure sums and loss, adjoint, gradient
// reductions and Adam, as phases of one persistent grid separated by a
// software grid barrier.  The grid holds as many blocks as are resident at
// once, each phase deals its work items (the blocks of the separate kernels)
// to them, and every phase's intermediate stays in the same workspace arrays
// as in the separate kernels.

// Grid barrier, two levels.  The blocks of XCD x (blockIdx.x mod 8) count
// their arrivals in a counter of their own (bar[kBarStride (x + 1)], one per
// 64-byte line); the block that completes its XCD's count for barrier k adds
// one to the device counter bar[0], and every block waits until that reaches
// 8 k.  Same-address atomics from hundreds of blocks serialise at the memory
// side, so one level costs tens of microseconds where two cost a few.  The
// counters are zeroed by the step's head.  A wait longer than kBarrierTicks
// of the 100 MHz constant clock, or a flag raised by a block that timed out,
// makes the block leave with FL_BARRIER raised, so a grid whose blocks are
// not all resident ends with an error, not a hang.
// The wait polls with relaxed loads: an acquire load at device scope also
// invalidates the L2 of the polling XCD, and dozens of waiting blocks would
// keep invalidating the cache under the blocks still working.  A release
// fence before the arrival and an acquire fence after the wait order the
// phases' memory.
constexpr uint64_t kBarrierTicks = 200000000ull;   // 2 s
constexpr int kBarStride = 16;                     // words between counters
constexpr int kBarWords = kBarStride * (kXCD + 1);
__device__ __forceinline__ bool grid_barrier(unsigned* bar, unsigned k, int* flags, int* abort_sh) {
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned per = gridDim.x / kXCD;   // blocks per XCD (gridDim.x is a multiple of 8)
    const int x = blockIdx.x % kXCD;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    const unsigned old = __hip_atomic_fetch_add(bar + kBarStride * (x + 1), 1u, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
    if (old == k * per - 1u) __hip_atomic_fetch_add(bar, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned target = k * (unsigned)kXCD;
    const uint64_t t0 = wall_clock64();
    int ok = 1;
    while (__hip_atomic_load(bar, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
      __builtin_amdgcn_s_sleep(2);
      if ((__hip_atomic_load(flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & FL_BARRIER) ||
          wall_clock64() - t0 > kBarrierTicks) {
        atomicOr(flags, FL_BARRIER);
        ok = 0;
        break;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    *abort_sh = !ok;
  }
  __syncthreads();
  return *abort_sh == 0;
}

// A phase's arguments, read again for each work item behind a compiler
// barrier, into scalar registers.  Values derived from arguments that stay
// the same across a phase's loop would otherwise be computed once before the
// loop and kept live through the whole body (the per-atom bodies are sized
// for the registers of one block's work); here nothing in the body is
// invariant, so the loop body compiles as the separate kernel does.
template <class T>
__device__ __forceinline__ T item_args(const T& p) {
  static_assert(sizeof(T) % 4 == 0, "read as words");
  asm volatile("" ::: "memory");
  T v;
  const int* q = reinterpret_cast<const int*>(&p);
  int* d = reinterpret_cast<int*>(&v);
#pragma unroll
  for (int k = 0; k < (int)(sizeof(T) / 4); ++k) d[k] = __builtin_amdgcn_readfirstlane(q[k]);
  return v;
}

// Work items [0, n) of a phase dealt to the persistent blocks: the blocks of
// XCD x (blockIdx.x mod 8; gridDim.x is a multiple of 8) take the x-th
// contiguous eighth, so items that share data share an L2.
template <class F>
__device__ __forceinline__ void for_items(int n, F&& f) {
  const int per = gridDim.x / kXCD;
  const int x = blockIdx.x % kXCD, r = blockIdx.x / kXCD;
  const int q = n / kXCD, rem = n % kXCD;
  const int lo = x * q + min(x, rem), cnt = q + (x < rem ? 1 : 0);
  for (int j = r; j < cnt; j += per) f(lo + j);
}

struct StepArgs {
  OrderArgs ord;
  FwdArgs fwd;
  ForceArgs frc;
  StructArgs st;
  AdjArgs adj;
  OuterArgs ow, oc;
  int nzw, nzc, os_x;
  PartArgs pr;
  LossArgs la;
  GradArgs g;
  int n_gf;        // blocks of the final gradient reduction
  unsigned* bar;
  int* flags;
};

// The arguments are read from device memory (written by k_step_head), not
// from the kernel-argument segment: loads of kernel arguments are all issued
// at entry and would stay live in registers through every phase.  Two
// wavefronts per SIMD: at three (168 registers) the merged phases spill
// several hundred bytes per lane, although each body alone fits.
template <class C>
__global__ __launch_bounds__(256, 2) void k_step(const StepArgs* pa) {
  const StepArgs& a = *pa;
  extern __shared__ __align__(16) float lds[];
  __shared__ int abort_sh;
  unsigned k = 0;
#define NEP_BARRIER() \
  if (!grid_barrier(a.bar, ++k, a.flags, &abort_sh)) return
  // species order
  {
    const int nch = a.ord.nch;
    for_items(nch, [&](int c) { order_body<256>(item_args(a.ord), c, reinterpret_cast<int*>(lds)); });
  }
  NEP_BARRIER();
  // forward: descriptors, network, partial forces
  for_items(order_grid(a.fwd.nch, C::T), [&](int vb) {
    forward_body<C, false, kLPA>(item_args(a.fwd), vb, lds);
    __syncthreads();
  });
  NEP_BARRIER();
  for_items((a.fwd.N + 256 / kForceLPA - 1) / (256 / kForceLPA), [&](int vb) {
    force_body<C, false, kForceLPA>(item_args(a.frc), vb, lds);
    __syncthreads();
  });
  NEP_BARRIER();
  // per-structure sums, loss partials and cotangents
  if (a.st.split) {
    for_items((a.st.N + kStructChunk - 1) / kStructChunk,
              [&](int vb) { struct_part_body(item_args(a.st), vb, lds); });
    NEP_BARRIER();
  }
  for_items(a.st.S, [&](int s) { struct_body(item_args(a.st), s, lds); });
  NEP_BARRIER();
  for_items(order_grid(a.adj.nch, C::T), [&](int vb) {
    adjoint_body<C, false, kLPA>(item_args(a.adj), vb, lds);
    __syncthreads();
  });
  NEP_BARRIER();
  // outer-product sums, first stage of the partial sums, and the loss
  {
    const int T = a.ord.T;
    const int os_x = a.os_x, nzw = a.nzw;
    const int prc = a.pr.NB;
    const int n_outer = os_x * T * (nzw + a.nzc), n_pr = prc * T;
    auto& red = *reinterpret_cast<f32x4(*)[3][kOSTM * kOSTV][kWave]>(lds);
    for_items(n_outer + n_pr + (a.la.on ? 1 : 0), [&](int v) {
      if (v < n_outer) {
        const int x = v % os_x, I = (v / os_x) % T, z = v / (os_x * T);
        if (z < nzw)
          outer_sum_block(item_args(a.ow), x, I, z, red);
        else
          outer_sum_block(item_args(a.oc), x, I, z - nzw, red);
      } else if (v < n_outer + n_pr) {
        const int u = v - n_outer;
        part_reduce_body(item_args(a.pr), u % prc, u / prc);
      } else {
        const LossArgs la = item_args(a.la);
        loss_final_block(la.S, la.N, la.le, la.lf, la.lv, la.lpart, la.loss, la.flags, lds);
        __syncthreads();
      }
    });
  }
  NEP_BARRIER();
  // final gradient reduction with Adam
  for_items(a.n_gf, [&](int vb) { grad_final_body(item_args(a.g), vb); });
#undef NEP_BARRIER
}

// Head of the persistent step: the graph head, the step's arguments copied
// to device memory, and the barrier's arrival counter cleared.
__global__ void k_step_head(StepArgs a, StepArgs* dst, int* flags, int* step, int* cur) {
  static_assert(sizeof(StepArgs) % 4 == 0, "copied as words");
  const int* src = reinterpret_cast<const int*>(&a);
  int* d = reinterpret_cast<int*>(dst);
  for (int q = threadIdx.x; q < (int)(sizeof(StepArgs) / 4); q += blockDim.x) d[q] = src[q];
  for (int q = threadIdx.x; q < kBarWords; q += blockDim.x) a.bar[q] = 0u;
  graph_head(flags, step, cur);
}

// ============================================================ padded models
// (PadDims and the layout maps stand before the final gradient reduction.)

// class parameter q of the model, -1 where the model has none
__device__ __forceinline__ int unpad_index(const PadDims& d, int q) {
  const int PRc = d.Tc * d.Tc * d.NRc * d.KRc, PAc = d.Tc * d.Tc * d.NAc * d.KAc;
  const int PR = d.T * d.T * d.NR * d.KR, PA = d.T * d.T * d.NA * d.KA;
  if (q < PRc) {
    const int k = q % d.KRc, n = (q / d.KRc) % d.NRc, J = (q / (d.KRc * d.NRc)) % d.Tc;
    const int I = q / (d.KRc * d.NRc * d.Tc);
    return k < d.KR && n < d.NR && J < d.T && I < d.T ? ((I * d.T + J) * d.NR + n) * d.KR + k : -1;
  }
  q -= PRc;
  if (q < PAc) {
    const int k = q % d.KAc, n = (q / d.KAc) % d.NAc, J = (q / (d.KAc * d.NAc)) % d.Tc;
    const int I = q / (d.KAc * d.NAc * d.Tc);
    return k < d.KA && n < d.NA && J < d.T && I < d.T ? PR + ((I * d.T + J) * d.NA + n) * d.KA + k : -1;
  }
  q -= PAc;
  const int blk = d.H * d.D + 2 * d.H + 1, blkc = d.H * d.Dc + 2 * d.H + 1;
  const int I = q / blkc, o = q % blkc;
  if (I >= d.T) return -1;
  const int base = PR + PA + I * blk;
  if (o >= d.H * d.Dc) return base + d.H * d.D + (o - d.H * d.Dc);   // b0, w1, b1
  int v = o % d.Dc, col = -1;
  if (v < d.NRc) {
    col = v < d.NR ? v : -1;
  } else if ((v -= d.NRc) < d.L3c * d.NAc) {
    col = v / d.NAc < d.l3 && v % d.NAc < d.NA ? d.NR + v / d.NAc * d.NA + v % d.NAc : -1;
  } else if ((v -= d.L3c * d.NAc) < d.NAc) {
    col = d.l4 && v < d.NA ? d.NR + d.l3 * d.NA + v : -1;
  } else {
    v -= d.NAc;
    col = d.l5 && v < d.NA ? d.NR + d.l3 * d.NA + (d.l4 ? d.NA : 0) + v : -1;
  }
  return col >= 0 ? base + o / d.Dc * d.D + col : -1;
}

// the class parameters: the model's where it has them, zero elsewhere
__global__ __launch_bounds__(256) void k_pad_params(PadDims d, int64_t Pc, const float* __restrict__ p,
                                                    float* __restrict__ pc) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= Pc) return;
  const int64_t m = unpad_index(d, (int)q);
  pc[q] = m >= 0 ? p[m] : 0.f;
}

// descriptor rows [Dc][N] of the class to the model's [D][N]
__global__ __launch_bounds__(256) void k_unpad_desc(PadDims d, int N, const float* __restrict__ Gc,
                                                    float* __restrict__ G) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q < (int64_t)d.D * N) G[q] = Gc[(int64_t)pad_col(d, (int)(q / N)) * N + q % N];
}

// ================================================================ dispatch
// A move of its own launch: the half kick and drift before the first force
// evaluation of a call, and the half kick after the last one (whose forces the
// energy sums follow).
template <bool kKick, bool kDrift>
__global__ __launch_bounds__(256) void k_md_move(MDArgs a) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.N) return;
  const float f[3] = {a.F[i], a.F[(size_t)a.N + i], a.F[2 * (size_t)a.N + i]};
  md_move<kKick, kDrift>(a, i, f);
}

// out[s] = sum of x over the atoms of structure s (float64, one block each)
__global__ __launch_bounds__(256) void k_struct_sum(const int* __restrict__ aoff, const float* __restrict__ x,
                                                    float* __restrict__ out) {
  __shared__ double red[256];
  const int s = blockIdx.x;
  double acc = 0.0;
  for (int i = aoff[s] + threadIdx.x; i < aoff[s + 1]; i += blockDim.x) acc += x[i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int st = blockDim.x / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[s] = (float)red[0];
}

enum HighKernel { kHighDesc, kHighForce, kHighTangent, kHighCoef };

struct Ops {
  int T, NR, NA, KR, KA, L3, L4, L5, D, Y, PS, YH, YR;
  void (*forward)(const FwdArgs&, int, hipStream_t, int, int);
  void (*force)(const ForceArgs&, hipStream_t, int, const MDArgs*);
  void (*adjoint)(const AdjArgs&, int, hipStream_t, int, int);
  int KP;   // words of a radial force coefficient row
  size_t (*lds_fwd)(int);
  size_t (*lds_adj)(int);
  void (*high)(HighKernel, const HighArgs&, dim3, hipStream_t);   // null without degrees l > 4
  // persistent step (null with degrees l > 4): launch, and resident blocks per CU
  void (*step)(const StepArgs*, int, size_t, hipStream_t);
  int (*step_occupancy)(size_t);
  bool padded;   // a size class: models up to its sizes run zero-padded
};

template <class C, int L>
static size_t lds_forward(int H) {
  using FL = FwdLds<C, L>;
  return sizeof(float) * ((size_t)CTab<C::T, C::NA, C::KA>::size + CRad<C>::size + (size_t)weights_words(H, C::D, FL::DP) +
                          (size_t)(256 / kWave) * FL::WAVE);
}
template <class C, int L>
static size_t lds_adjoint(int H) {
  using AL = AdjLds<C, L>;
  return sizeof(float) * ((size_t)CTab<C::T, C::NA, C::KA>::size + (size_t)AL::shared_words(H) +
                          (size_t)(256 / kWave) * AL::WAVE);
}
// LDS of a workgroup on gfx950 (160 KiB per CU); dynamic LDS beyond 64 KiB is
// requested from the runtime per kernel before its launch
constexpr size_t kMaxLds = 160 * 1024;
template <class K>
static void allow_lds(K* k, size_t bytes) {
  if (bytes > 64 * 1024)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)bytes);
}

// forward_waves 2 and 3 are the forward compiled for 3 and for 4 wavefronts
// per SIMD (168 and 128 registers); the adjoint is compiled for 2 and 3
template <class C, int W, int L>
static void launch_forward_w(const FwdArgs& a, int blocks, hipStream_t st) {
  const dim3 grid(blocks + (a.fl.n > 0 ? 1 : 0));   // an extra block for the flags
  const size_t lds = lds_forward<C, L>(a.H);
  if (a.tilt) {
    allow_lds(&k_forward<C, true, W, L>, lds);
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_forward<C, true, W, L>), grid, dim3(256), lds, st, a);
  } else {
    allow_lds(&k_forward<C, false, W, L>, lds);
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_forward<C, false, W, L>), grid, dim3(256), lds, st, a);
  }
}
template <class C>
static void launch_forward(const FwdArgs& a, int blocks, hipStream_t st, int waves, int lanes) {
  if (lanes == 32) return launch_forward_w<C, 2, 32>(a, 4 * blocks, st);
  if (lanes == 16) return launch_forward_w<C, 2, 16>(a, 2 * blocks, st);
  if constexpr (C::FIXED_WAVES != 0)
    launch_forward_w<C, C::FIXED_WAVES, kLPA>(a, blocks, st);
  else if (waves == 2)
    launch_forward_w<C, 3, kLPA>(a, blocks, st);
  else
    launch_forward_w<C, 4, kLPA>(a, blocks, st);
}
template <class C, bool kTri>
static void launch_force_t(const ForceArgs& a, hipStream_t st, int lanes) {
  const int apb = 256 / lanes;
  const dim3 grid((a.N + apb - 1) / apb);
  if (lanes == 8)
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_force<C, kTri, 8>), grid, dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_force<C, kTri, 16>), grid, dim3(256), 0, st, a);
}
template <class C>
static void launch_force(const ForceArgs& a, hipStream_t st, int lanes, const MDArgs* md) {
  if (md) {
    const dim3 grid((a.N + 256 / kForceLPA - 1) / (256 / kForceLPA));
    if (a.tilt)
      hipLaunchKernelGGL(HIP_KERNEL_NAME(k_force_move<C, true>), grid, dim3(256), 0, st, a, *md);
    else
      hipLaunchKernelGGL(HIP_KERNEL_NAME(k_force_move<C, false>), grid, dim3(256), 0, st, a, *md);
  } else if (a.tilt)
    launch_force_t<C, true>(a, st, lanes);
  else
    launch_force_t<C, false>(a, st, lanes);
}
template <class C, int W, int L>
static void launch_adjoint_w(const AdjArgs& a, dim3 grid, hipStream_t st) {
  const size_t lds = lds_adjoint<C, L>(a.H);
  if (a.tilt) {
    allow_lds(&k_adjoint<C, true, W, L>, lds);
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_adjoint<C, true, W, L>), grid, dim3(256), lds, st, a);
  } else {
    allow_lds(&k_adjoint<C, false, W, L>, lds);
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_adjoint<C, false, W, L>), grid, dim3(256), lds, st, a);
  }
}
template <class C>
static void launch_adjoint(const AdjArgs& a, int blocks, hipStream_t st, int waves, int lanes) {
  if (lanes == 32) return launch_adjoint_w<C, 2, 32>(a, dim3(4 * blocks), st);
  if (lanes == 16) return launch_adjoint_w<C, 2, 16>(a, dim3(2 * blocks), st);
  const dim3 grid(blocks);
  if constexpr (C::FIXED_WAVES != 0)
    launch_adjoint_w<C, C::FIXED_WAVES, kLPA>(a, grid, st);
  else if (waves == 2)
    launch_adjoint_w<C, 2, kLPA>(a, grid, st);
  else
    launch_adjoint_w<C, 3, kLPA>(a, grid, st);
}
template <class C, bool kTri>
static void launch_high_t(HighKernel k, const HighArgs& a, dim3 grid, hipStream_t st) {
  switch (k) {
    case kHighDesc: hipLaunchKernelGGL(HIP_KERNEL_NAME(k_high_desc<C, kTri>), grid, dim3(256), 0, st, a); break;
    case kHighForce: hipLaunchKernelGGL(HIP_KERNEL_NAME(k_high_force<C, kTri>), grid, dim3(256), 0, st, a); break;
    case kHighTangent:
      hipLaunchKernelGGL(HIP_KERNEL_NAME(k_high_tangent<C, kTri>), grid, dim3(256), 0, st, a);
      break;
    case kHighCoef:   // one wavefront per block
      hipLaunchKernelGGL(HIP_KERNEL_NAME(k_high_coef<C, kTri>), dim3(grid.x * 4), dim3(kWave), 0, st, a);
      break;
  }
}
template <class C>
static void launch_high(HighKernel k, const HighArgs& a, dim3 grid, hipStream_t st) {
  if (a.tilt)
    launch_high_t<C, true>(k, a, grid, st);
  else
    launch_high_t<C, false>(k, a, grid, st);
}
template <class C>
static void launch_step(const StepArgs* a, int grid, size_t lds, hipStream_t st) {
  allow_lds(&k_step<C>, lds);
  hipLaunchKernelGGL(HIP_KERNEL_NAME(k_step<C>), dim3(grid), dim3(256), lds, st, a);
}
template <class C>
static int step_occupancy(size_t lds) {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, reinterpret_cast<const void*>(&k_step<C>), 256, lds) !=
      hipSuccess)
    return 0;
  return nb;
}
template <class C>
static Ops make_ops() {
  void (*high)(HighKernel, const HighArgs&, dim3, hipStream_t) = nullptr;
  void (*step)(const StepArgs*, int, size_t, hipStream_t) = nullptr;
  int (*occ)(size_t) = nullptr;
  if constexpr (C::YH > 0) high = &launch_high<C>;
  if constexpr (C::YH == 0 && C::FIXED_WAVES == 0) {
    step = &launch_step<C>;
    occ = &step_occupancy<C>;
  }
  return Ops{C::T, C::NR, C::NA, C::KR, C::KA, C::L3, C::L4, C::L5, C::D, C::Y, C::PS, C::YH,
             HRow<C::LMAX>::YR, &launch_forward<C>, &launch_force<C>, &launch_adjoint<C>, HRad<C>::KP, &lds_forward<C, kLPA>, &lds_adjoint<C, kLPA>, high, step, occ,
             C::FIXED_WAVES != 0};
}

// Compiled-in model sizes (n_types, n_rad, n_ang, k_rad, k_ang, l3, l4, l5):
// exact shapes, then size classes that run any model up to their sizes with
// the parameters zero-padded (kPadClasses, smallest first).
static const Ops kOps[] = {
    make_ops<Cfg<2, 5, 5, 9, 9, 4, 0, 0>>(),    // 3-body NEP, basis 8, n_max 4
    make_ops<Cfg<2, 7, 5, 11, 11, 4, 2, 1>>(),  // 3/4/5-body NEP, basis 10, n_max 6/4
    make_ops<Cfg<2, 3, 2, 4, 3, 4, 2, 1>>(),    // small two-species model
    make_ops<Cfg<1, 4, 3, 6, 5, 2, 2, 0>>(),    // small one-species model
    make_ops<Cfg<2, 5, 4, 8, 8, 8, 2, 1>>(),    // 3-body degrees up to l = 8, n_max 4/3
};
static const Ops kPadClasses[] = {
    make_ops<Cfg<1, 12, 8, 12, 12, 4, 2, 1, 2>>(),
    make_ops<Cfg<2, 12, 8, 12, 12, 4, 2, 1, 2>>(),
    make_ops<Cfg<4, 12, 8, 12, 12, 4, 2, 1, 2>>(),
    make_ops<Cfg<1, 12, 8, 12, 12, 8, 2, 1, 2>>(),
    make_ops<Cfg<2, 12, 8, 12, 12, 8, 2, 1, 2>>(),
    make_ops<Cfg<4, 12, 8, 12, 12, 8, 2, 1, 2>>(),
};

}  // namespace nep

// ===================================================================== ABI
using namespace nep;

namespace {

// Kernels for a model: an exact compiled shape, else the smallest size class
// that holds it (the model then runs zero-padded as the class model `cls`).
struct Resolved {
  const Ops* o = nullptr;
  nep_model cls{};
  bool pad = false;
};

Resolved resolve(const nep_model* m) {
  Resolved r;
  for (const Ops& o : kOps)
    if (o.T == m->n_types && o.NR == m->n_rad && o.NA == m->n_ang && o.KR == m->k_rad && o.KA == m->k_ang &&
        o.L3 == m->l3 && o.L4 == m->l4 && o.L5 == m->l5) {
      r.o = &o;
      r.cls = *m;
      return r;
    }
  for (const Ops& o : kPadClasses)
    if (o.T >= m->n_types && o.NR >= m->n_rad && o.NA >= m->n_ang && o.KR >= m->k_rad && o.KA >= m->k_ang &&
        o.L3 >= m->l3 && o.L4 >= m->l4 && o.L5 >= m->l5) {
      r.o = &o;
      r.pad = true;
      r.cls = *m;
      r.cls.n_types = o.T;
      r.cls.n_rad = o.NR;
      r.cls.n_ang = o.NA;
      r.cls.k_rad = o.KR;
      r.cls.k_ang = o.KA;
      r.cls.l3 = o.L3;
      r.cls.l4 = o.L4;
      r.cls.l5 = o.L5;
      return r;
    }
  return r;
}

int model_valid(const nep_model* m) {
  if (!m) return NEP_ERR_ARG;
  if (m->n_types < 1 || m->n_types > 8 || m->n_rad < 1 || m->n_ang < 0 || m->k_rad < 1 || m->k_ang < 1 ||
      m->l3 < 0 || m->l3 > 8 || (m->l4 != 0 && m->l4 != 2) || (m->l5 != 0 && m->l5 != 1) || m->hidden < 1 ||
      m->hidden > 256 || !(m->rc_rad > 0.f) || !(m->rc_ang > 0.f) || m->rc_ang > m->rc_rad || m->cap_rad < 1 ||
      m->cap_ang < 1 || m->cap_rad > 4096 || m->cap_ang > 4096)
    return NEP_ERR_ARG;
  return NEP_OK;
}

int32_t desc_count(const nep_model* m) {
  return m->n_rad + m->n_ang * m->l3 + (m->l4 ? m->n_ang : 0) + (m->l5 ? m->n_ang : 0);
}

int64_t param_count(const nep_model* m) {
  const int64_t T = m->n_types, D = desc_count(m), H = m->hidden;
  return T * T * (m->n_rad * m->k_rad + m->n_ang * m->k_ang) + T * (H * D + 2 * H + 1);
}

size_t al(size_t x) { return (x + 255) & ~(size_t)255; }

// Lanes per atom of the forward and the adjoint.  With few atoms a SIMD has one
// wavefront or none, and the time is the instructions of one wavefront: more
// lanes an atom shorten its pair loops, sums and hidden units, up to the
// batch where 32 lanes (8 atoms a block) no longer fit one block per CU and
// 16 lanes two; beyond, the work that more lanes repeat counts.  Training
// step of the 3/4/5-body model in us with 8 / 16 / 32 lanes: 512 atoms
// 81.2 / 61.9 / 56.7, 2048 atoms 80.3 / 64.0 / 60.6, 3072 atoms 82.2 / 67.4 /
// 66.1, 8192 atoms 94.8 / 84.8 / 102.5; with 8 / 16, 10240 atoms 106.3 / 97.8,
// 11264 atoms 107.9 / 116.6.  The 3-body model is the same (10240 atoms 94.5 /
// 86.9, 11264 atoms 93.4 / 94.9).  Models of up to 16 descriptors have less to
// repeat (one species, 14336 atoms 77.0 / 72.6, 16384 atoms 71.8 / 72.9), those
// of degrees up to 8 and the padded classes more (8192 atoms 160.3 / 159.9 and,
// three species, 113.7 / 116.6, 6144 atoms 154.2 / 145.4 and 105.8 / 91.6).  At 32
// lanes all change sides between 2048 and 3072 atoms.
constexpr int kLanes32Atoms = 2048, kLanes16Wide = 8192, kLanes16Atoms = 10240, kLanes16Small = 14336;
int group_lanes(const Ops* o, int N) {
  const int line = o->padded || o->YH > 0 ? kLanes16Wide : o->D <= 16 ? kLanes16Small : kLanes16Atoms;
  return N <= kLanes32Atoms ? 32 : N <= line ? 16 : kLPA;
}

struct Layout {
  int N, S, T, D, Y, H, NR, TKR, Npad, lanes, nch, PW, NA, capR, capA;
  size_t order, seg, blist, bflags, astruct, p4, G, Sst, Ep, X, eatom, hrow, fA, wv, F, fb4, Es, Ws, eps, wbar, lpart,
      Gd, FRst, FPst, Gbr, beta, part, pp, w0part, crpart, Sh, Sdh, cgrid, cell, cstart, cpart, acell, aslot, cpos, spart,
      cur_step, bar, sargs, prm, Gtmp, total;
};

// Workspace size callers see: with the pair forces and reverse indices of both
// lists, which the layout below does not hold, so that nep_loss_grad_noalloc
// takes and refuses the batches that its header states.  The layout fits in it
// (at capacities below 16 it may pass it by up to 3 %).
size_t reported_bytes(const Layout& L, const Ops* o, const nep_model* m, bool pad) {
  const size_t N = L.N > 0 ? L.N : 1, S = L.S > 0 ? L.S : 1, T = L.T, D = L.D, H = L.H, TKR = L.TKR;
  const size_t n8 = ((size_t)L.N + 31) / 32 * 32 + T * 32 + 16, Np = (n8 + 31) / 32 * 32;
  const size_t Pc = pad ? (size_t)param_count(m) : 0, capR = L.capR, capA = L.capA, NA = L.NA;
  const size_t bytes[] = {
      4 * Np, 64, 4 * ((N + 1023) / 1024) * T * 64, 4 * N, 4 * capR * N, 4 * capA * N, 4 * D * Np,
      4 * NA * (size_t)o->YR * Np, 4 * D * Np, 4 * H * Np, 4 * N, 12 * capR * N, 12 * capA * N, 24 * N, 12 * N, 12 * N,
      4 * S, 24 * S, 4 * S, 24 * S, 24 * S, 4 * D * Np, 4 * TKR * Np, 4 * TKR * Np,
      4 * (o->YH > 0 ? D : (size_t)L.NR) * Np, 4 * H * Np, 4 * H * Np, 4 * (Np / kAPW) * (size_t)L.PW,
      8 * T * kPRChunksMax * (size_t)L.PW, 4 * T * kOSBlocksMaxW * H * D, 4 * T * kOSBlocksMaxC * (size_t)L.NR * TKR,
      4 * Np * NA * (size_t)o->YH, 4 * Np * NA * (size_t)o->YH, 16 * S, 4 * (N + 1), 4 * (N / kScanChunk + 1), 4 * N,
      4 * N, 16 * N, 128 * (N / kStructChunk + 1), 4, 4 * kBarWords, 1280, 4 * Pc, 4 * Pc, pad ? 4 * D * N : 0};
  size_t sum = 0;
  for (size_t b : bytes) sum += al(b);
  return sum;
}

// Blocks per species of a reduction over the order's chunks: each chunk in Q
// pieces (at most max_q, so that a piece keeps some work) so that there are
// about `want` blocks, at most `most`; with more chunks than that a block
// takes several.
struct Split {
  int Q, NB;
};
Split split_chunks(int want, int most, int nch, int max_q) {
  int q = std::min(std::max((want + nch / 2) / nch, 1), std::max(max_q, 1));
  if (nch * q > most) q = std::max(1, most / nch);
  return Split{q, std::min(nch * q, most)};
}
// 64 atoms (a 16-atom group per wavefront, 8 wavefront rows) to a piece at least
int max_pieces(int N) { return std::min(N, kOrdChunk) / 64; }

// m: the model the kernels run (the class model when padded)
Layout layout_of(const nep_model* m, const Ops* o, int S, int N, bool pad) {
  Layout L{};
  L.N = N;
  L.S = S;
  L.T = m->n_types;
  L.D = o->D;
  L.Y = o->Y;
  L.H = m->hidden;
  L.NA = m->n_ang;
  L.NR = m->n_rad;
  L.TKR = m->n_types * m->k_rad;
  L.capR = m->cap_rad;
  L.capA = m->cap_ang;
  // chunks of the species order; the last one with its own atoms only.  A
  // segment start leaves 16 positions to the end, which the outer-product sums
  // may read.
  L.nch = N > 0 ? (N + kOrdChunk - 1) / kOrdChunk : 1;
  const int last = N - (L.nch - 1) * kOrdChunk;
  L.Npad = (L.nch - 1) * order_stride(L.T) + (last + kSegAlign - 1) / kSegAlign * kSegAlign + L.T * kSegAlign;
  // the per-atom vectors are rows of Npad words: an odd number of 256-byte
  // units, so the rows a wavefront stores start in different memory channels
  L.Npad = (L.Npad + 63) / 64 * 64;
  if ((L.Npad / 64) % 2 == 0) L.Npad += 64;
  L.lanes = group_lanes(o, N);   // each wavefront writes a row of part
  L.PW = L.T * m->n_ang * m->k_ang + 2 * L.H + 1;
  const size_t Np = L.Npad, Nn = (size_t)(N > 0 ? N : 1), Ss = (size_t)(S > 0 ? S : 1);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t r = off;
    off += al(bytes);
    return r;
  };
  L.order = take(4 * Np);
  L.seg = take(4 * 2 * (size_t)L.nch * L.T);
  L.blist = take(4 * (size_t)order_grid(L.nch, L.T));
  L.bflags = take(4 * (Nn / kNbrAPB + 1));
  L.astruct = take(4 * Nn);
  L.p4 = take(16 * Nn);
  L.G = take(4 * (size_t)L.D * Np);
  // the class descriptor rows of nep_descriptors (a padded model), which stores
  // no sums, take the sums' place
  L.Sst = L.Gtmp = take(4 * std::max((((size_t)L.NA * o->YR + 3) & ~(size_t)3) * Np, pad ? (size_t)L.D * Nn : 0));
  L.Ep = take(4 * (size_t)L.D * Np);
  L.X = take(4 * (size_t)L.H * Np);
  L.eatom = take(4 * Nn);
  L.fA = take(4 * 3 * (size_t)L.capA * Nn);
  L.wv = take(4 * 6 * Nn);
  L.F = take(4 * 3 * Nn);
  L.fb4 = take(16 * Nn);
  L.Es = take(4 * Ss);
  L.Ws = take(4 * 6 * Ss);
  L.eps = take(4 * Ss);
  L.wbar = take(4 * 6 * Ss);
  L.lpart = take(8 * 3 * Ss);
  // the radial force coefficients (forward to force pass) end before the
  // descriptor tangents (adjoint) begin: one region
  L.hrow = L.Gd = take(4 * std::max((size_t)L.D * Np, (size_t)L.T * o->KP * Nn));
  L.FRst = take(4 * (size_t)L.TKR * Np);
  L.FPst = take(4 * (size_t)L.TKR * Np);
  L.Gbr = take(4 * (size_t)(o->YH > 0 ? L.D : L.NR) * Np);
  L.beta = take(4 * (size_t)L.H * Np);
  L.part = take(4 * (size_t)(L.Npad / (kWave / L.lanes)) * L.PW);
  // the most blocks any tuning can ask for
  auto blocks = [&](int most) { return (size_t)L.T * split_chunks(most, most, L.nch, max_pieces(N)).NB; };
  L.pp = take(8 * blocks(kPRChunksMax) * L.PW);
  L.w0part = take(4 * blocks(kOSBlocksMaxW) * L.H * L.D);
  L.crpart = take(4 * blocks(kOSBlocksMaxC) * L.NR * L.TKR);
  L.Sh = take(4 * (size_t)Np * L.NA * o->YH);
  L.Sdh = take(4 * (size_t)Np * L.NA * o->YH);
  L.cgrid = take(16 * Ss);
  L.cell = take(4 * (Nn + 1));
  L.cstart = take(4 * (Nn + 1));
  L.cpart = take(4 * (Nn / kScanChunk + 1));
  L.acell = take(4 * Nn);
  L.aslot = take(4 * Nn);
  L.cpos = take(16 * Nn);
  L.spart = take(8 * 16 * (Nn / kStructChunk + 1));
  L.cur_step = take(4);
  L.bar = take(4 * kBarWords);
  L.sargs = take(sizeof(StepArgs));
  L.prm = take(pad ? 4 * (size_t)param_count(m) : 0);   // the class-layout parameters
  L.total = off;
  return L;
}

Layout make_layout(const nep_model* m, const Ops* o, int S, int N, bool pad = false) {
  Layout L = layout_of(m, o, S, N, pad);
  L.total = std::max(L.total, reported_bytes(L, o, m, pad));
  return L;
}

template <class P>
P* at(void* ws, size_t off) {
  return reinterpret_cast<P*>(static_cast<char*>(ws) + off);
}

int check_batch(const nep_batch* b) {
  if (!b || b->n_struct < 0 || b->n_atom < 0 || b->n_atom >= (1 << 27)) return NEP_ERR_ARG;
  if (b->n_struct == 0 && b->n_atom != 0) return NEP_ERR_ARG;
  if (b->n_struct > 0 && (!b->atom_offset || !b->box)) return NEP_ERR_ARG;
  if (b->n_atom > 0 && (!b->pos || !b->type)) return NEP_ERR_ARG;
  if (b->max_atoms < 0) return NEP_ERR_ARG;
  return NEP_OK;
}

int check_ws(const void* ws) {
  if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255u)) return NEP_ERR_WORKSPACE;
  return NEP_OK;
}

int check_nbrs(const nep_neighbors* n, int N) {
  if (!n) return NEP_ERR_ARG;
  if (N > 0 && (!n->idx_rad || !n->cnt_rad || !n->idx_ang || !n->cnt_ang)) return NEP_ERR_ARG;
  return NEP_OK;
}

// Optional per-launch timing (nep_profile_loss_grad).
struct Prof {
  hipStream_t st;
  std::vector<hipEvent_t> ev;
  std::vector<const char*> names;
  void begin() {
    hipEvent_t e;
    (void)hipEventCreate(&e);
    (void)hipEventRecord(e, st);
    ev.push_back(e);
  }
  void end(const char* n) {
    begin();
    names.push_back(n);
  }
};

#define NEP_LAUNCH(prof, name, ...)  \
  do {                               \
    if (prof) (prof)->begin();       \
    __VA_ARGS__;                     \
    if (prof) (prof)->end(name);     \
  } while (0)

int hip_ok() { return hipGetLastError() == hipSuccess ? NEP_OK : NEP_ERR_HIP; }

// Launch choices of one evaluation (nep_tuning with the defaults filled in).
struct Tune {
  int persistent, outer_w, outer_c, reduce_chunks, cell_min, gather_lanes, forward_waves, adjoint_waves;
};

Tune default_tune(const Ops* o) {
  // degrees l > 4: forward 2 (at 3, 1 us slower of 230), adjoint 3 (at 2, 7 us slower)
  return Tune{0, kOSBlocksW, kOSBlocksC, kPRChunks, kCellMinAtoms, kForceLPA, o->YH > 0 ? 2 : 3, 3};
}

struct Ctx {
  const nep_model* m;    // the model the kernels run: the caller's, or its size class
  const nep_model* mu;   // the caller's model
  nep_model mcls;        // the size-class model of a padded run
  bool pad = false;
  PadDims pd{};
  const Ops* o;
  const nep_batch* b;
  Tune tune;
  Layout L;
  void* ws;
  hipStream_t st;
  // the captured training step: Adam after the gradient, fused into its
  // final reduction
  const struct AdamFuse* adam = nullptr;
  int lanes = kLPA;   // lanes per atom of the forward and the adjoint
  // the packed atoms of this call are in the workspace
  mutable bool packed = false;
  // a captured step whose order launch or forward starts the replay (flags, step
  // latch): the step counter and its latch, and the flag words left to the forward
  int* g_step = nullptr;
  int* g_cur = nullptr;
  mutable FlagArgs flag_words{};
  // force cotangents of the caller (nep_vjp), packed with the atoms
  const float* fbar = nullptr;
};

struct AdamFuse {
  int64_t P;
  float* th;
  float* mm;
  float* vv;
  const int* step;
  AdamDev ad;
  int* flags;
};

int grid1(int n, int blk = 256) { return (n + blk - 1) / blk; }

PairLists pair_lists(const Ctx& c, const nep_neighbors* nb) {
  PairLists p;
  p.idxR = nb->idx_rad;
  p.cntR = nb->cnt_rad;
  p.idxA = nb->idx_ang;
  p.cntA = nb->cnt_ang;
  p.capR = c.m->cap_rad;
  p.capA = c.m->cap_ang;
  return p;
}

OrderArgs order_args(const Ctx& c, const nep_neighbors* nb) {
  return OrderArgs{c.L.N, c.L.Npad, c.L.T, c.L.nch, c.b->type, nb->cnt_ang, at<int>(c.ws, c.L.seg),
                   at<int>(c.ws, c.L.order), at<int>(c.ws, c.L.blist)};
}

void run_neighbors(const Ctx& c, nep_neighbors* nb, int32_t* flags, Prof* pr, bool with_order = true) {
  const int N = c.L.N;
  if (N == 0) return;
  c.packed = true;
  NbrArgs a;
  a.N = N;
  a.S = c.b->n_struct;
  a.T = c.mu->n_types;   // types are checked against the caller's model
  a.capR = c.m->cap_rad;
  a.capA = c.m->cap_ang;
  a.rcR = c.m->rc_rad;
  a.rcA = c.m->rc_ang;
  a.aoff = c.b->atom_offset;
  a.box = c.b->box;
  a.tilt = c.b->tilt;
  a.pos = c.b->pos;
  a.type = c.b->type;
  a.idxR = nb->idx_rad;
  a.cntR = nb->cnt_rad;
  a.idxA = nb->idx_ang;
  a.cntA = nb->cnt_ang;
  a.astruct = at<int>(c.ws, c.L.astruct);
  a.p4 = at<float4>(c.ws, c.L.p4);
  a.bflags = with_order ? at<int>(c.ws, c.L.bflags) : nullptr;
  a.flags = flags;
  // the cell-list kernels run unless the caller's bound rules out every structure
  const int S = c.b->n_struct;
  a.cell_min = c.tune.cell_min;
  a.cells = N >= a.cell_min && (c.b->max_atoms == 0 || c.b->max_atoms >= a.cell_min);
  a.grid = at<int4>(c.ws, c.L.cgrid);
  a.cell = at<int>(c.ws, c.L.cell);
  a.start = at<int>(c.ws, c.L.cstart);
  a.cpart = at<int>(c.ws, c.L.cpart);
  a.acell = at<int>(c.ws, c.L.acell);
  a.aslot = at<int>(c.ws, c.L.aslot);
  a.cpos = at<float4>(c.ws, c.L.cpos);
  if (a.cells) {
    const int nch = grid1(N, kScanChunk);
    if (a.tilt) {
      NEP_LAUNCH(pr, "cell_setup",
                 hipLaunchKernelGGL(k_cell_setup<true>, dim3(grid1(max(N, S), 256)), dim3(256), 0, c.st, a));
      NEP_LAUNCH(pr, "cell_bin", hipLaunchKernelGGL(k_cell_bin<true>, dim3(grid1(N, 256)), dim3(256), 0, c.st, a));
    } else {
      NEP_LAUNCH(pr, "cell_setup",
                 hipLaunchKernelGGL(k_cell_setup<false>, dim3(grid1(max(N, S), 256)), dim3(256), 0, c.st, a));
      NEP_LAUNCH(pr, "cell_bin", hipLaunchKernelGGL(k_cell_bin<false>, dim3(grid1(N, 256)), dim3(256), 0, c.st, a));
    }
    if (nch > kScanDirect)
      NEP_LAUNCH(pr, "cell_part",
                 hipLaunchKernelGGL(k_cell_part, dim3(nch), dim3(256), 0, c.st, N, a.cell, a.cpart));
    NEP_LAUNCH(pr, "cell_start",
               hipLaunchKernelGGL(k_cell_start, dim3(nch), dim3(256), 0, c.st, N, a.cell, a.cpart, a.start));
    NEP_LAUNCH(pr, "cell_place", hipLaunchKernelGGL(k_cell_place, dim3(grid1(N, 256)), dim3(256), 0, c.st, a));
    if (a.tilt)
      NEP_LAUNCH(pr, "cell_neighbors", hipLaunchKernelGGL(k_cell_neighbors<true>, dim3(grid1(N, kNbrAPB)),
                                                          dim3(kNbrThreads), 0, c.st, a));
    else
      NEP_LAUNCH(pr, "cell_neighbors", hipLaunchKernelGGL(k_cell_neighbors<false>, dim3(grid1(N, kNbrAPB)),
                                                          dim3(kNbrThreads), 0, c.st, a));
  }
  const int nblk = grid1(N, kNbrAPB);
  const bool by_type = with_order && N <= kTypeOrderAtoms;
  // without an order launch behind it the build raises its flags itself, or in
  // a captured step leaves their words to the forward
  if (by_type && !c.g_step) a.bflags = nullptr;
  {
    auto* k = a.tilt ? (a.cells ? k_neighbors<true, true> : k_neighbors<true, false>)
                     : (a.cells ? k_neighbors<false, true> : k_neighbors<false, false>);
    NEP_LAUNCH(pr, "neighbors", hipLaunchKernelGGL(k, dim3(nblk + (by_type ? c.L.nch : 0)), dim3(kNbrThreads), 0, c.st,
                                                   a, nblk, order_args(c, nb)));
  }
  if (!with_order) return;   // the persistent step computes the species order itself
  const FlagArgs fa{a.bflags, nblk, flags, c.g_step, c.g_cur};
  if (!by_type)
    NEP_LAUNCH(pr, "order",
               hipLaunchKernelGGL(k_order, dim3(c.L.nch), dim3(1024), 0, c.st, order_args(c, nb), fa));
  else if (c.g_step)
    c.flag_words = fa;
}

FwdArgs fwd_args(const Ctx& c, const nep_neighbors* nb, const float* params) {
  FwdArgs a;
  a.fl = c.flag_words;
  const nep_model* m = c.m;
  a.N = c.L.N;
  a.Npad = c.L.Npad;
  a.H = m->hidden;
  a.inv_rcR = 1.0f / m->rc_rad;
  a.inv_rcA = 1.0f / m->rc_ang;
  a.order = at<int>(c.ws, c.L.order);
  a.blist = at<int>(c.ws, c.L.blist);
  a.nch = c.L.nch;
  a.astruct = at<int>(c.ws, c.L.astruct);
  a.box = c.b->box;
  a.tilt = c.b->tilt;
  a.p4 = at<float4>(c.ws, c.L.p4);
  a.nb = pair_lists(c, nb);
  const int T = m->n_types;
  a.cR = params;
  a.cA = params + (size_t)T * T * m->n_rad * m->k_rad;
  a.nn = a.cA + (size_t)T * T * m->n_ang * m->k_ang;
  a.nn_stride = m->hidden * c.o->D + 2 * m->hidden + 1;
  a.G = at<float>(c.ws, c.L.G);
  a.Guser = nullptr;
  a.Sst = at<float>(c.ws, c.L.Sst);
  a.FRst = at<float>(c.ws, c.L.FRst);
  a.Ep = at<float>(c.ws, c.L.Ep);
  a.X = at<float>(c.ws, c.L.X);
  a.eatom = at<float>(c.ws, c.L.eatom);
  a.eatom2 = nullptr;
  a.hrow = at<float>(c.ws, c.L.hrow);
  a.fA = at<float>(c.ws, c.L.fA);
  a.do_mlp = 1;
  a.do_force = 1;
  return a;
}

ForceArgs force_args(const Ctx& c, const FwdArgs& f, float* user) {
  ForceArgs a;
  a.N = f.N;
  a.inv_rcR = f.inv_rcR;
  a.nb = f.nb;
  a.p4 = at<float4>(c.ws, c.L.p4);
  a.astruct = f.astruct;
  a.box = f.box;
  a.tilt = f.tilt;
  a.hrow = f.hrow;
  a.fA = f.fA;
  a.F = at<float>(c.ws, c.L.F);
  a.Fuser = user;
  a.wv = at<float>(c.ws, c.L.wv);
  return a;
}

// arguments of the kernels of degrees l > 4 (wbar only for the adjoint's)
HighArgs high_args(const Ctx& c, const nep_neighbors* nb, const float* params, const float* wbar = nullptr) {
  HighArgs h;
  const nep_model* m = c.m;
  h.N = c.L.N;
  h.Npad = c.L.Npad;
  h.PW = c.L.PW * (c.lanes / kLPA);   // its wavefronts hold 8 atoms: one of the adjoint's rows
  h.inv_rcA = 1.0f / m->rc_ang;
  h.order = at<int>(c.ws, c.L.order);
  h.astruct = at<int>(c.ws, c.L.astruct);
  h.box = c.b->box;
  h.tilt = c.b->tilt;
  h.p4 = at<float4>(c.ws, c.L.p4);
  h.nb = pair_lists(c, nb);
  h.cA = params + (size_t)m->n_types * m->n_types * m->n_rad * m->k_rad;
  h.Sh = at<float>(c.ws, c.L.Sh);
  h.Sdh = at<float>(c.ws, c.L.Sdh);
  h.G = at<float>(c.ws, c.L.G);
  h.Ep = at<float>(c.ws, c.L.Ep);
  h.Gd = at<float>(c.ws, c.L.Gd);
  h.Gb = at<float>(c.ws, c.L.Gbr);
  h.fA = at<float>(c.ws, c.L.fA);
  h.fb4 = at<float4>(c.ws, c.L.fb4);
  h.wbar = wbar;
  h.part = at<float>(c.ws, c.L.part);
  return h;
}

void run_high(const Ctx& c, HighKernel k, const HighArgs& h, Prof* pr) {
  static const char* const names[] = {"high_desc", "high_force", "high_tangent", "high_coef"};
  if (c.o->high) NEP_LAUNCH(pr, names[k], c.o->high(k, h, dim3(c.L.Npad / kAPB), c.st));
}

// packs the atoms unless this call's neighbor build did
void run_pack(const Ctx& c, const nep_neighbors* nb, Prof* pr) {
  const int N = c.L.N;
  if (c.packed || N == 0) return;
  NEP_LAUNCH(pr, "pack", hipLaunchKernelGGL(k_pack, dim3(grid1(N)), dim3(256), 0, c.st, N, c.m->n_types, c.b->pos,
                                            c.b->type, pair_lists(c, nb), at<float4>(c.ws, c.L.p4), c.fbar,
                                            at<float4>(c.ws, c.L.fb4)));
  c.packed = true;
}

// forward pass with the degrees l > 4 around it
void launch_forward_pass(const Ctx& c, const nep_neighbors* nb, const float* params, const FwdArgs& a, Prof* pr) {
  const HighArgs h = high_args(c, nb, params);
  run_pack(c, nb, pr);
  run_high(c, kHighDesc, h, pr);
  NEP_LAUNCH(pr, "forward", c.o->forward(a, order_grid(c.L.nch, c.L.T), c.st, c.tune.forward_waves, c.lanes));
  if (a.do_mlp && a.do_force) run_high(c, kHighForce, h, pr);
}

StructArgs struct_args(const Ctx& c, float* e_struct, float* virial, const nep_labels* lab, const float* lam) {
  StructArgs s;
  const int N = c.L.N;
  s.S = c.b->n_struct;
  s.N = N;
  s.aoff = c.b->atom_offset;
  s.eatom = at<float>(c.ws, c.L.eatom);
  s.wv = at<float>(c.ws, c.L.wv);
  s.F = at<float>(c.ws, c.L.F);
  s.Et = lab ? lab->energy : nullptr;
  s.Ft = lab ? lab->force : nullptr;
  s.Wt = lab ? lab->virial : nullptr;
  s.le = lam ? lam[0] : 0.f;
  s.lf = lam ? lam[1] : 0.f;
  s.lv = lam ? lam[2] : 0.f;
  s.Es = at<float>(c.ws, c.L.Es);
  s.Ws = at<float>(c.ws, c.L.Ws);
  s.Es_user = e_struct;
  s.Ws_user = virial;
  s.eps = at<float>(c.ws, c.L.eps);
  s.wbar = at<float>(c.ws, c.L.wbar);
  s.fb4 = at<float4>(c.ws, c.L.fb4);
  s.lpart = at<double>(c.ws, c.L.lpart);
  // large structures take chunk partials first, unless the caller's bound rules them out
  s.split = N >= 2 * kStructChunk && (c.b->max_atoms == 0 || c.b->max_atoms >= 2 * kStructChunk);
  s.spart = at<double>(c.ws, c.L.spart);
  return s;
}

void run_forward(const Ctx& c, const nep_neighbors* nb, const float* params, float* e_atom, float* e_struct,
                 float* force, float* virial, const nep_labels* lab, const float* lam, float* loss, int32_t* flags,
                 Prof* pr, bool defer_loss = false, const MDArgs* md = nullptr) {
  const int N = c.L.N, S = c.b->n_struct;
  if (N > 0) {
    FwdArgs a = fwd_args(c, nb, params);
    a.eatom2 = e_atom;
    if (!lab) {   // no adjoint follows: its inputs are not stored (l > 4 reads G and E')
      a.Sst = a.FRst = a.X = nullptr;
      if (c.o->YH == 0) a.G = a.Ep = nullptr;
    }
    launch_forward_pass(c, nb, params, a, pr);
    NEP_LAUNCH(pr, "force", c.o->force(force_args(c, a, force), c.st, c.tune.gather_lanes, md));
  }
  // an MD step that another follows needs no sums
  if (S > 0 && !md) {
    const StructArgs s = struct_args(c, e_struct, virial, lab, lam);
    if (s.split)
      NEP_LAUNCH(pr, "struct_part",
                 hipLaunchKernelGGL(k_struct_part, dim3(grid1(N, kStructChunk)), dim3(kRedBlk), 0, c.st, s));
    NEP_LAUNCH(pr, "struct_sums", hipLaunchKernelGGL(k_struct, dim3(S), dim3(kRedBlk), 0, c.st, s));
    // with defer_loss the adjoint's first reduction launch sums the loss
    if (lab && !defer_loss)
      NEP_LAUNCH(pr, "loss_final",
                 hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(kRedBlk), 0, c.st, S, N, s.le, s.lf, s.lv, s.lpart,
                                    loss, flags));
  }
}

AdjArgs adj_args(const Ctx& c, const nep_neighbors* nb, const float* params, const float* eps, const float* wbar) {
  const nep_model* m = c.m;
  AdjArgs a;
  a.N = c.L.N;
  a.Npad = c.L.Npad;
  a.H = m->hidden;
  a.S = c.b->n_struct;
  a.inv_rcR = 1.0f / m->rc_rad;
  a.inv_rcA = 1.0f / m->rc_ang;
  a.order = at<int>(c.ws, c.L.order);
  a.blist = at<int>(c.ws, c.L.blist);
  a.nch = c.L.nch;
  a.astruct = at<int>(c.ws, c.L.astruct);
  a.box = c.b->box;
  a.tilt = c.b->tilt;
  a.p4 = at<float4>(c.ws, c.L.p4);
  a.nb = pair_lists(c, nb);
  const int T = m->n_types;
  a.cR = params;
  a.cA = params + (size_t)T * T * m->n_rad * m->k_rad;
  a.nn = a.cA + (size_t)T * T * m->n_ang * m->k_ang;
  a.nn_stride = m->hidden * c.o->D + 2 * m->hidden + 1;
  a.Sst = at<float>(c.ws, c.L.Sst);
  a.Ep = at<float>(c.ws, c.L.Ep);
  a.X = at<float>(c.ws, c.L.X);
  a.eps = eps;
  a.fb4 = at<float4>(c.ws, c.L.fb4);
  a.wbar = wbar;
  a.Gd = at<float>(c.ws, c.L.Gd);
  a.FPst = at<float>(c.ws, c.L.FPst);
  a.Gbr = at<float>(c.ws, c.L.Gbr);
  a.beta = at<float>(c.ws, c.L.beta);
  a.part = at<float>(c.ws, c.L.part);
  a.PW = c.L.PW;
  return a;
}

Split split_w(const Ctx& c) { return split_chunks(c.tune.outer_w, kOSBlocksMaxW, c.L.nch, max_pieces(c.L.N)); }
Split split_c(const Ctx& c) { return split_chunks(c.tune.outer_c, kOSBlocksMaxC, c.L.nch, max_pieces(c.L.N)); }
Split split_p(const Ctx& c) { return split_chunks(c.tune.reduce_chunks, kPRChunksMax, c.L.nch, max_pieces(c.L.N)); }

PartArgs part_args(const Ctx& c) {
  const Split p = split_p(c);
  return PartArgs{c.L.PW, p.NB, c.L.T, c.L.nch, p.Q, kWave / c.lanes, at<int>(c.ws, c.L.seg), at<float>(c.ws, c.L.part),
                  at<double>(c.ws, c.L.pp)};
}

// the two outer-product sums: dW0 (W) and dc^R (C)
void outer_args(const Ctx& c, const AdjArgs& a, OuterArgs& ow, OuterArgs& oc) {
  const nep_model* m = c.m;
  const int* seg = at<int>(c.ws, c.L.seg);
  const Split w = split_w(c), r = split_c(c);
  ow = OuterArgs{c.L.Npad, m->hidden, c.o->D, w.NB, c.L.T, c.L.nch, w.Q, seg, a.beta, at<float>(c.ws, c.L.G), a.X, a.Gd,
                 at<float>(c.ws, c.L.w0part), a.nn + m->hidden * c.o->D + m->hidden, a.nn_stride};
  oc = OuterArgs{c.L.Npad, m->n_rad, c.L.TKR, r.NB, c.L.T, c.L.nch, r.Q, seg, a.Gbr, at<float>(c.ws, c.L.FRst),
                 at<float>(c.ws, c.L.Ep), a.FPst, at<float>(c.ws, c.L.crpart), nullptr, 0};
}

GradArgs grad_args(const Ctx& c, float* grad) {
  const nep_model* m = c.m;
  GradArgs g;
  g.T = m->n_types;
  g.NR = m->n_rad;
  g.NA = m->n_ang;
  g.KR = m->k_rad;
  g.KA = m->k_ang;
  g.H = m->hidden;
  g.D = c.o->D;
  g.PW = c.L.PW;
  g.NBw = split_w(c).NB;
  g.NBc = split_c(c).NB;
  g.PRC = split_p(c).NB;
  g.P = param_count(c.mu);
  g.pad = c.pad;
  g.pd = c.pd;
  g.pp = at<double>(c.ws, c.L.pp);
  g.w0part = at<float>(c.ws, c.L.w0part);
  g.crpart = at<float>(c.ws, c.L.crpart);
  g.grad = grad;
  g.adam = c.adam != nullptr;
  if (c.adam) {
    g.ad = c.adam->ad;
    g.th = c.adam->th;
    g.mm = c.adam->mm;
    g.vv = c.adam->vv;
    g.step = c.adam->step;
    g.flags = c.adam->flags;
  }
  return g;
}

unsigned grad_final_blocks(const GradArgs& g) { return (unsigned)((g.P * 16 + 255) / 256); }

// adjoint + gradient reductions; cotangents from eps, wbar and the packed F-bar
void run_adjoint(const Ctx& c, const nep_neighbors* nb, const float* params, const float* eps, const float* wbar,
                 float* grad, Prof* pr, LossArgs la = LossArgs{}) {
  const nep_model* m = c.m;
  const int N = c.L.N;
  if (N > 0) {
    const AdjArgs a = adj_args(c, nb, params, eps, wbar);
    const int T = m->n_types;
    const HighArgs h = high_args(c, nb, params, wbar);
    run_high(c, kHighTangent, h, pr);
    NEP_LAUNCH(pr, "adjoint", c.o->adjoint(a, order_grid(c.L.nch, c.L.T), c.st, c.tune.adjoint_waves, c.lanes));
    run_high(c, kHighCoef, h, pr);
    {
      OuterReduceArgs ra;
      outer_args(c, a, ra.ow, ra.oc);
      ra.nzw = outer_slices(ra.ow.M, ra.ow.V);
      ra.nzc = outer_slices(ra.oc.M, ra.oc.V);
      ra.os_x = std::max(ra.ow.NB, ra.oc.NB);
      ra.T = T;
      ra.pr = part_args(c);
      ra.la = la;
      const int nblk = ra.os_x * T * (ra.nzw + ra.nzc) + ra.pr.NB * T + (la.on ? 1 : 0);
      NEP_LAUNCH(pr, "outer_sums_reduce",
                 hipLaunchKernelGGL(k_outer_reduce, dim3(nblk), dim3(256), 0, c.st, ra));
    }
    const GradArgs g = grad_args(c, grad);
    NEP_LAUNCH(pr, "grad_final", hipLaunchKernelGGL(k_grad_final, dim3(grad_final_blocks(g)), dim3(256), 0, c.st, g));
  } else {
    const int64_t P = param_count(c.mu);
    hipLaunchKernelGGL(k_fill_f32, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, c.st, grad, P, 0.f);
    if (c.adam)
      hipLaunchKernelGGL(k_adam_dev, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, c.st, P, c.adam->th,
                         c.adam->mm, c.adam->vv, grad, c.adam->step, c.adam->flags, c.adam->ad);
  }
}

PadDims pad_dims(const nep_model* m, const nep_model* cls) {
  PadDims d;
  d.T = m->n_types;
  d.NR = m->n_rad;
  d.NA = m->n_ang;
  d.KR = m->k_rad;
  d.KA = m->k_ang;
  d.D = desc_count(m);
  d.H = m->hidden;
  d.l3 = m->l3;
  d.l4 = m->l4;
  d.l5 = m->l5;
  d.Tc = cls->n_types;
  d.NRc = cls->n_rad;
  d.NAc = cls->n_ang;
  d.KRc = cls->k_rad;
  d.KAc = cls->k_ang;
  d.Dc = desc_count(cls);
  d.L3c = cls->l3;
  d.P = param_count(m);
  return d;
}

// kernels exist for the model and their LDS fits
int model_supported(const nep_model* m, Resolved* out = nullptr) {
  int rc = model_valid(m);
  if (rc) return rc;
  const Resolved r = resolve(m);
  if (!r.o) return NEP_ERR_ARG;
  if (r.o->lds_adj(m->hidden) > kMaxLds || r.o->lds_fwd(m->hidden) > kMaxLds) return NEP_ERR_ARG;
  if (out) *out = r;
  return NEP_OK;
}

size_t workspace_size(const nep_model* m, int S, int N) {
  const Resolved r = resolve(m);
  return make_layout(&r.cls, r.o, S, N, r.pad).total;
}

int setup(Ctx& c, const nep_model* m, const nep_batch* b, void* ws, void* stream) {
  Resolved r;
  int rc = model_supported(m, &r);
  if (rc) return rc;
  if ((rc = check_batch(b))) return rc;
  if ((rc = check_ws(ws))) return rc;
  c.o = r.o;
  c.mu = m;
  c.pad = r.pad;
  c.mcls = r.cls;
  c.m = r.pad ? &c.mcls : m;
  if (r.pad) c.pd = pad_dims(m, &c.mcls);
  c.b = b;
  c.tune = default_tune(c.o);
  c.ws = ws;
  c.st = static_cast<hipStream_t>(stream);
  c.L = make_layout(c.m, c.o, b->n_struct, b->n_atom, r.pad);
  c.lanes = c.L.lanes;
  return NEP_OK;
}

// The parameters the kernels read: the caller's, or for a padded model their
// class-layout copy in the workspace (filled by launches on the call's stream).
const float* kernel_params(const Ctx& c, const float* params) {
  if (!c.pad) return params;
  float* pc = at<float>(c.ws, c.L.prm);
  const int64_t Pc = param_count(c.m);
  hipLaunchKernelGGL(k_pad_params, dim3((unsigned)((Pc + 255) / 256)), dim3(256), 0, c.st, c.pd, Pc, params, pc);
  return pc;
}

// loss sum carried by the first reduction launch after the adjoint
LossArgs loss_args(const Ctx& c, const nep_labels* labels, const float* lam, float* loss, int32_t* flags) {
  LossArgs la{};
  const int N = c.L.N, S = c.b->n_struct;
  if (N > 0 && S > 0 && labels) {
    la.on = 1;
    la.S = S;
    la.N = N;
    la.le = lam[0];
    la.lf = lam[1];
    la.lv = lam[2];
    la.lpart = at<double>(c.ws, c.L.lpart);
    la.loss = loss;
    la.flags = flags;
  }
  return la;
}

int loss_grad_seq(Ctx& c, nep_neighbors* nb, const float* params, const nep_labels* labels, const float* lam,
                  float* loss, float* grad, float* e_struct, float* force, float* virial, int32_t* flags, Prof* pr,
                  bool with_neighbors) {
  if (with_neighbors) run_neighbors(c, nb, flags, pr);
  if (c.b->n_struct == 0) hipLaunchKernelGGL(k_fill_f32, dim3(1), dim3(64), 0, c.st, loss, (int64_t)4, 0.f);
  // with atoms present the loss is summed by the adjoint's reduction launch
  const LossArgs la = loss_args(c, labels, lam, loss, flags);
  run_forward(c, nb, params, nullptr, e_struct, force, virial, labels, lam, loss, flags, pr, la.on != 0);
  run_adjoint(c, nb, params, at<float>(c.ws, c.L.eps), at<float>(c.ws, c.L.wbar), grad, pr, la);
  return hip_ok();
}

// ---- persistent step: everything after the neighbor build in one launch
size_t step_lds(const Ctx& c) {
  size_t l = std::max(c.o->lds_fwd(c.m->hidden), c.o->lds_adj(c.m->hidden));
  l = std::max(l, (size_t)kOrdLds * sizeof(int));
  l = std::max(l, (size_t)kStructLds);
  l = std::max(l, (size_t)kOuterLds);
  l = std::max(l, (size_t)kLossLds);
  return l;
}

// Blocks of the persistent grid: as many as are resident at once, a multiple
// of the XCD count; 0 when the kernel cannot run.
int step_grid(const Ctx& c, size_t lds) {
  if (!c.o->step) return 0;
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 0;
  const int per = c.o->step_occupancy(lds);
  return per * cus / kXCD * kXCD;
}

// The persistent step covers orthorhombic batches with atoms and structures,
// for models without degrees l > 4.
bool persistent_ok(const Ctx& c) { return c.o->step && !c.b->tilt && c.L.N > 0 && c.b->n_struct > 0; }

StepArgs step_args(const Ctx& c, nep_neighbors* nb, const float* params, const nep_labels* labels,
                   const float* lam, float* loss, float* grad, int32_t* flags) {
  StepArgs a;
  a.ord = order_args(c, nb);
  a.fwd = fwd_args(c, nb, params);
  a.frc = force_args(c, a.fwd, nullptr);
  a.st = struct_args(c, nullptr, nullptr, labels, lam);
  a.adj = adj_args(c, nb, params, at<float>(c.ws, c.L.eps), at<float>(c.ws, c.L.wbar));
  outer_args(c, a.adj, a.ow, a.oc);
  a.nzw = outer_slices(a.ow.M, a.ow.V);
  a.nzc = outer_slices(a.oc.M, a.oc.V);
  a.os_x = std::max(a.ow.NB, a.oc.NB);
  a.pr = part_args(c);
  a.la = loss_args(c, labels, lam, loss, flags);
  a.g = grad_args(c, grad);
  a.n_gf = (int)grad_final_blocks(a.g);
  a.bar = at<unsigned>(c.ws, c.L.bar);
  a.flags = flags;
  return a;
}

struct GraphHandle {
  hipGraph_t g;
  hipGraphExec_t e;
};

// Adam's hyper-parameters: beta in [0, 1) (the bias correction divides by
// 1 - beta^step), eps >= 0 finite.
bool adam_hparams_ok(float beta1, float beta2, float eps) {
  return beta1 >= 0.f && beta1 < 1.f && beta2 >= 0.f && beta2 < 1.f && eps >= 0.f && std::isfinite(eps);
}

// Overrides of the launch choices; 0 keeps the default.  NEP_ERR_ARG out of range.
int apply_tuning(Tune& t, const nep_tuning* u) {
  if (!u) return NEP_OK;
  auto set = [](int& dst, int v, int lo, int hi) {
    if (v == 0) return true;
    if (v < lo || v > hi) return false;
    dst = v;
    return true;
  };
  bool ok = u->persistent == 0 || u->persistent == 1;
  t.persistent = u->persistent;
  ok = ok && set(t.outer_w, u->outer_blocks_w, 1, kOSBlocksMaxW);
  ok = ok && set(t.outer_c, u->outer_blocks_c, 1, kOSBlocksMaxC);
  ok = ok && set(t.reduce_chunks, u->reduce_chunks, 1, kPRChunksMax);
  ok = ok && set(t.cell_min, u->cell_min_atoms, kCellMinAtomsLo, 1 << 27);
  ok = ok && (u->gather_lanes == 0 || u->gather_lanes == 8 || u->gather_lanes == 16);
  if (u->gather_lanes) t.gather_lanes = u->gather_lanes;
  ok = ok && set(t.forward_waves, u->forward_waves, 2, 3);
  ok = ok && set(t.adjoint_waves, u->adjoint_waves, 2, 3);
  ok = ok && u->reverse_branch >= 0 && u->reverse_branch <= 2;   // no launch to place any more
  return ok ? NEP_OK : NEP_ERR_ARG;
}

int check_adam_config(const nep_adam_config* a) {
  if (!adam_hparams_ok(a->beta1, a->beta2, a->eps)) return NEP_ERR_ARG;
  if (!std::isfinite(a->lr_start) || !std::isfinite(a->lr_stop) || a->n_warmup < 0) return NEP_ERR_ARG;
  return NEP_OK;
}

// Scratch of nep_loss_grad_noalloc: a file-scope device array, one copy per
// GPU, held until the process ends.  Host code never passes the array's name
// to a kernel (on the host it is only a stand-in for the symbol); it uses the
// device address hipGetSymbolAddress returns, taken once per device with that
// device current.
static __device__ __align__(256) unsigned char scratch[NEP_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

int static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return NEP_ERR_HIP;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return NEP_ERR_HIP;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return NEP_OK;
}

}  // namespace

extern "C" {

int64_t nep_param_count(const nep_model* m) {
  const int rc = model_valid(m);
  return rc ? rc : param_count(m);
}

int32_t nep_descriptor_count(const nep_model* m) {
  const int rc = model_valid(m);
  return rc ? rc : desc_count(m);
}

int nep_model_supported(const nep_model* m) { return model_supported(m); }

int nep_workspace_bytes(const nep_model* m, int32_t n_struct, int32_t n_atom, size_t* bytes) {
  int rc = nep_model_supported(m);
  if (rc) return rc;
  if (!bytes || n_struct < 0 || n_atom < 0 || n_atom >= (1 << 27)) return NEP_ERR_ARG;
  *bytes = workspace_size(m, n_struct, n_atom);
  return NEP_OK;
}

int nep_build_neighbors(const nep_model* m, const nep_batch* b, nep_neighbors* out, void* ws, int32_t* d_flags,
                        void* stream) {
  Ctx c;
  int rc = setup(c, m, b, ws, stream);
  if (rc) return rc;
  if ((rc = check_nbrs(out, b->n_atom))) return rc;
  if (!d_flags) return NEP_ERR_ARG;
  run_neighbors(c, out, d_flags, nullptr);
  return hip_ok();
}

int nep_descriptors(const nep_model* m, const nep_batch* b, const nep_neighbors* nb, const float* params, float* G,
                    void* ws, void* stream) {
  Ctx c;
  int rc = setup(c, m, b, ws, stream);
  if (rc) return rc;
  if ((rc = check_nbrs(nb, b->n_atom))) return rc;
  if (b->n_atom > 0 && (!params || !G)) return NEP_ERR_ARG;
  if (b->n_atom == 0) return NEP_OK;
  const float* kp = kernel_params(c, params);
  FwdArgs a = fwd_args(c, nb, kp);
  a.Guser = c.pad ? at<float>(c.ws, c.L.Gtmp) : G;
  a.do_mlp = 0;
  a.do_force = 0;
  a.Sst = a.FRst = nullptr;
  if (c.o->YH == 0) a.G = nullptr;
  launch_forward_pass(c, nb, kp, a, nullptr);
  if (c.pad)
    hipLaunchKernelGGL(k_unpad_desc, dim3((unsigned)(((int64_t)c.pd.D * b->n_atom + 255) / 256)), dim3(256), 0, c.st,
                       c.pd, b->n_atom, a.Guser, G);
  return hip_ok();
}

int nep_energy_force_virial(const nep_model* m, const nep_batch* b, const nep_neighbors* nb, const float* params,
                            float* e_atom, float* e_struct, float* force, float* virial, void* ws, void* stream) {
  Ctx c;
  int rc = setup(c, m, b, ws, stream);
  if (rc) return rc;
  if ((rc = check_nbrs(nb, b->n_atom))) return rc;
  if (!params) return NEP_ERR_ARG;
  run_forward(c, nb, kernel_params(c, params), e_atom, e_struct, force, virial, nullptr, nullptr, nullptr, nullptr,
              nullptr);
  return hip_ok();
}

// MD steps between two species orders (formed every step it took 5 us of the
// step of a 180-atom cell, now 27, and 8 of that of 9261 atoms, now 73)
constexpr int kMDOrderSteps = 16;

int nep_md_step(const nep_model* m, const nep_batch* b, float* pos, nep_neighbors* nb, const float* params,
                const float* mass, float* vel, float* force, float dt, int32_t n_steps, float* e_pot, float* e_kin,
                void* ws, int32_t* d_flags, void* stream) {
  Ctx c;
  int rc = setup(c, m, b, ws, stream);
  if (rc) return rc;
  if ((rc = check_nbrs(nb, b->n_atom))) return rc;
  const int N = b->n_atom, S = b->n_struct;
  if (!params || !mass || !d_flags || n_steps < 0 || !std::isfinite(dt)) return NEP_ERR_ARG;
  if (N > 0 && (pos != b->pos || !vel || !force)) return NEP_ERR_ARG;
  if (N == 0 || n_steps == 0) return NEP_OK;
  MDArgs a;
  a.N = N;
  a.T = m->n_types;
  a.type = b->type;
  a.astruct = at<int>(c.ws, c.L.astruct);
  a.box = b->box;
  a.tilt = b->tilt;
  a.mass = mass;
  a.pos = pos;
  a.vel = vel;
  a.F = force;
  a.ekin = at<float>(c.ws, c.L.eatom);   // reused after the last force evaluation
  a.hdt = 0.5f * dt;
  a.dt = dt;
  params = kernel_params(c, params);
  // The energies are those of the last step: no sums before it.  A step that
  // another follows is the neighbor build, the forward and a force pass that
  // also moves the atoms.  The species order holds for as long as the species
  // do, which is the call; its ranking by pair count (for balance alone) is
  // renewed now and then.
  hipLaunchKernelGGL(HIP_KERNEL_NAME(k_md_move<false, true>), dim3(grid1(N)), dim3(256), 0, c.st, a);
  for (int k = 0; k < n_steps; ++k) {
    run_neighbors(c, nb, d_flags, nullptr, k % kMDOrderSteps == 0);
    run_forward(c, nb, params, nullptr, e_pot, force, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, false,
                k + 1 < n_steps ? &a : nullptr);
  }
  hipLaunchKernelGGL(HIP_KERNEL_NAME(k_md_move<true, false>), dim3(grid1(N)), dim3(256), 0, c.st, a);
  if (e_kin && S > 0)
    hipLaunchKernelGGL(k_struct_sum, dim3(S), dim3(256), 0, c.st, b->atom_offset, a.ekin, e_kin);
  return hip_ok();
}

int nep_vjp(const nep_model* m, const nep_batch* b, const nep_neighbors* nb, const float* params, const float* e_bar,
            const float* f_bar, const float* v_bar, float* grad, void* ws, void* stream) {
  Ctx c;
  int rc = setup(c, m, b, ws, stream);
  if (rc) return rc;
  if ((rc = check_nbrs(nb, b->n_atom))) return rc;
  if (!params || !grad) return NEP_ERR_ARG;
  if (b->n_atom > 0 && (!e_bar || !f_bar || !v_bar)) return NEP_ERR_ARG;
  params = kernel_params(c, params);
  if (b->n_atom > 0) {
    FwdArgs a = fwd_args(c, nb, params);
    a.do_force = 0;
    c.fbar = f_bar;
    launch_forward_pass(c, nb, params, a, nullptr);
  }
  run_adjoint(c, nb, params, e_bar, v_bar, grad, nullptr);
  return hip_ok();
}

int nep_loss_grad(const nep_model* m, const nep_batch* b, const nep_neighbors* nb, const float* params,
                  const nep_labels* labels, const float lambda[3], float* loss, float* grad, float* e_struct,
                  float* force, float* virial, void* ws, int32_t* d_flags, void* stream) {
  Ctx c;
  int rc = setup(c, m, b, ws, stream);
  if (rc) return rc;
  if ((rc = check_nbrs(nb, b->n_atom))) return rc;
  if (!params || !labels || !lambda || !loss || !grad) return NEP_ERR_ARG;
  if (b->n_struct > 0 && (!labels->energy || !labels->virial)) return NEP_ERR_ARG;
  if (b->n_atom > 0 && !labels->force) return NEP_ERR_ARG;
  return loss_grad_seq(c, const_cast<nep_neighbors*>(nb), kernel_params(c, params), labels, lambda, loss, grad,
                       e_struct, force, virial, d_flags, nullptr, false);
}

int nep_loss_grad_noalloc(const nep_model* m, const nep_batch* b, nep_neighbors* nb, const float* params,
                          const nep_labels* labels, const float lambda[3], float* loss, float* grad, float* e_struct,
                          float* force, float* virial, int32_t* d_flags, void* stream) {
  int rc = nep_model_supported(m);
  if (rc) return rc;
  if ((rc = check_batch(b))) return rc;
  if (workspace_size(m, b->n_struct, b->n_atom) > (size_t)NEP_STATIC_SCRATCH_BYTES)
    return NEP_ERR_SCRATCH;
  void* ws = nullptr;
  if ((rc = static_scratch(&ws))) return rc;
  Ctx c;
  if ((rc = setup(c, m, b, ws, stream))) return rc;
  if ((rc = check_nbrs(nb, b->n_atom))) return rc;
  if (!params || !labels || !lambda || !loss || !grad || !d_flags) return NEP_ERR_ARG;
  if (b->n_struct > 0 && (!labels->energy || !labels->virial)) return NEP_ERR_ARG;
  if (b->n_atom > 0 && !labels->force) return NEP_ERR_ARG;
  return loss_grad_seq(c, nb, kernel_params(c, params), labels, lambda, loss, grad, e_struct, force, virial, d_flags,
                       nullptr, true);
}

int nep_adam_step(int64_t P, float* params, float* mm, float* vv, const float* grad, float lr, float beta1,
                  float beta2, float eps, int32_t step, void* stream) {
  if (P < 0 || step < 1 || !adam_hparams_ok(beta1, beta2, eps) || !std::isfinite(lr)) return NEP_ERR_ARG;
  if (P == 0) return NEP_OK;
  if (!params || !mm || !vv || !grad) return NEP_ERR_ARG;
  const float c1 = 1.0f - (float)std::pow((double)beta1, (double)step);
  const float c2 = 1.0f - (float)std::pow((double)beta2, (double)step);
  hipLaunchKernelGGL(k_adam, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, static_cast<hipStream_t>(stream), P,
                     params, mm, vv, grad, lr, beta1, beta2, eps, c1, c2);
  return hip_ok();
}

float nep_lr_schedule(int64_t s, float lr_start, float lr_stop, int64_t n_warmup, int64_t n_total) {
  if (n_total <= 0) return lr_start;
  if (s < n_warmup) return lr_stop + (float)((double)s / (double)n_warmup) * (lr_start - lr_stop);
  double fr = (double)(s - n_warmup) / (double)std::max<int64_t>(1, n_total - n_warmup);
  fr = fr > 1.0 ? 1.0 : fr;
  return lr_stop + (lr_start - lr_stop) * 0.5f * (1.0f + (float)std::cos(3.14159265358979323846 * fr));
}

int nep_train_step_graph_create(const nep_model* m, const nep_batch* b, nep_neighbors* nb, const nep_labels* labels,
                                const float lambda[3], float* params, float* mm, float* vv, float* grad, float* loss,
                                int32_t* d_step, const nep_adam_config* adam, void* ws, int32_t* d_flags,
                                int32_t graph_flags, void* stream, void** graph) {
  return nep_train_step_graph_create_tuned(m, b, nb, labels, lambda, params, mm, vv, grad, loss, d_step, adam, ws,
                                           d_flags, graph_flags, nullptr, stream, graph);
}

int nep_train_step_graph_create_tuned(const nep_model* m, const nep_batch* b, nep_neighbors* nb,
                                      const nep_labels* labels, const float lambda[3], float* params, float* mm,
                                      float* vv, float* grad, float* loss, int32_t* d_step,
                                      const nep_adam_config* adam, void* ws, int32_t* d_flags, int32_t graph_flags,
                                      const nep_tuning* tuning, void* stream, void** graph) {
  Ctx c;
  int rc = setup(c, m, b, ws, stream);
  if (rc) return rc;
  if ((rc = apply_tuning(c.tune, tuning))) return rc;
  if ((rc = check_nbrs(nb, b->n_atom))) return rc;
  if (!labels || !lambda || !params || !mm || !vv || !grad || !loss || !d_step || !adam || !d_flags || !graph)
    return NEP_ERR_ARG;
  if ((rc = check_adam_config(adam))) return rc;
  const bool persistent = (graph_flags & NEP_GRAPH_PERSISTENT) != 0 || c.tune.persistent;
  size_t slds = 0;
  int sgrid = 0;
  if (persistent) {
    if (!persistent_ok(c)) return NEP_ERR_ARG;
    c.lanes = kLPA;   // its grid is sized for 8 lanes an atom
    slds = step_lds(c);
    sgrid = step_grid(c, slds);
    if (sgrid < kXCD) return NEP_ERR_HIP;
  }
  hipStream_t cap;
  if (hipStreamCreateWithFlags(&cap, hipStreamNonBlocking) != hipSuccess) return NEP_ERR_HIP;
  c.st = cap;
  hipGraph_t g = nullptr;
  if (hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal) != hipSuccess) {
    (void)hipStreamDestroy(cap);
    return NEP_ERR_HIP;
  }
  int* cur = at<int>(c.ws, c.L.cur_step);
  // Adam runs inside the gradient's final reduction
  const AdamFuse af{param_count(m), params, mm, vv, cur,
                    AdamDev{adam->lr_start, adam->lr_stop, adam->n_warmup, adam->n_total, adam->beta1, adam->beta2,
                            adam->eps},
                    d_flags};
  c.adam = &af;
  if (persistent) {
    StepArgs* sa = at<StepArgs>(c.ws, c.L.sargs);
    hipLaunchKernelGGL(k_step_head, dim3(1), dim3(64), 0, cap,
                       step_args(c, nb, params, labels, lambda, loss, grad, d_flags), sa, d_flags, d_step, cur);
    if ((graph_flags & NEP_GRAPH_CACHED_NEIGHBORS) == 0) run_neighbors(c, nb, d_flags, nullptr, false);
    run_pack(c, nb, nullptr);
    c.o->step(sa, sgrid, slds, cap);
  } else {
    if ((graph_flags & NEP_GRAPH_CACHED_NEIGHBORS) != 0 || c.L.N == 0) {
      hipLaunchKernelGGL(k_graph_head, dim3(1), dim3(64), 0, cap, d_flags, d_step, cur);
    } else {   // by the order launch of the neighbor build, or with up to 8192 atoms the forward
      c.g_step = d_step;
      c.g_cur = cur;
    }
    // a padded model's class-layout parameters are refreshed by every replay
    loss_grad_seq(c, nb, kernel_params(c, params), labels, lambda, loss, grad, nullptr, nullptr, nullptr, d_flags,
                  nullptr, (graph_flags & NEP_GRAPH_CACHED_NEIGHBORS) == 0);
  }
  const hipError_t e1 = hipStreamEndCapture(cap, &g);
  (void)hipStreamDestroy(cap);
  if (e1 != hipSuccess || !g) return NEP_ERR_HIP;
  hipGraphExec_t ex;
  if (hipGraphInstantiate(&ex, g, nullptr, nullptr, 0) != hipSuccess) {
    (void)hipGraphDestroy(g);
    return NEP_ERR_HIP;
  }
  GraphHandle* h = new (std::nothrow) GraphHandle{g, ex};
  if (!h) {
    (void)hipGraphExecDestroy(ex);
    (void)hipGraphDestroy(g);
    return NEP_ERR_HIP;
  }
  *graph = h;
  return NEP_OK;
}

int nep_train_step_graph_launch(void* graph, void* stream) {
  if (!graph) return NEP_ERR_ARG;
  GraphHandle* h = static_cast<GraphHandle*>(graph);
  return hipGraphLaunch(h->e, static_cast<hipStream_t>(stream)) == hipSuccess ? NEP_OK : NEP_ERR_HIP;
}

int nep_train_step_graph_destroy(void* graph) {
  if (!graph) return NEP_OK;
  GraphHandle* h = static_cast<GraphHandle*>(graph);
  (void)hipGraphExecDestroy(h->e);
  (void)hipGraphDestroy(h->g);
  delete h;
  return NEP_OK;
}

int nep_profile_loss_grad(const nep_model* m, const nep_batch* b, nep_neighbors* nb, const float* params,
                          const nep_labels* labels, const float lambda[3], float* loss, float* grad, void* ws,
                          int32_t* d_flags, void* stream, float* ms, const char** names, int32_t max_kernels,
                          int32_t* n_kernels) {
  Ctx c;
  int rc = setup(c, m, b, ws, stream);
  if (rc) return rc;
  if ((rc = check_nbrs(nb, b->n_atom))) return rc;
  if (!labels || !lambda || !params || !loss || !grad || !d_flags || !n_kernels) return NEP_ERR_ARG;
  Prof pr;
  pr.st = c.st;
  rc = loss_grad_seq(c, nb, kernel_params(c, params), labels, lambda, loss, grad, nullptr, nullptr, nullptr, d_flags,
                     &pr, true);
  if (hipStreamSynchronize(c.st) != hipSuccess) rc = NEP_ERR_HIP;
  const int n = (int)pr.names.size();
  *n_kernels = n;
  for (int k = 0; k < n && k < max_kernels; ++k) {
    float t = 0.f;
    (void)hipEventElapsedTime(&t, pr.ev[2 * k], pr.ev[2 * k + 1]);
    if (ms) ms[k] = t;
    if (names) names[k] = pr.names[k];
  }
  for (hipEvent_t e : pr.ev) (void)hipEventDestroy(e);
  return rc;
}

int nep_flags_status(int32_t f) {
  if (f & FL_BARRIER) return NEP_ERR_HIP;
  if (f & FL_BOX) return NEP_ERR_BOX;
  if (f & FL_TYPE) return NEP_ERR_TYPE;
  if (f & FL_POS) return NEP_ERR_POSITION;
  if (f & FL_OVERFLOW) return NEP_ERR_NBR_OVERFLOW;
  if (f & FL_NONFINITE) return NEP_ERR_NONFINITE;
  if (f & FL_STEP) return NEP_ERR_ARG;
  return NEP_OK;
}

const char* nep_status_string(int code) {
  switch (code) {
    case NEP_OK: return "ok";
    case NEP_ERR_ARG: return "invalid argument or unsupported model";
    case NEP_ERR_BOX: return "a box edge is shorter than rc_rad";
    case NEP_ERR_NBR_OVERFLOW: return "neighbor list capacity exceeded";
    case NEP_ERR_NONFINITE: return "loss is not finite";
    case NEP_ERR_HIP: return "HIP runtime error";
    case NEP_ERR_WORKSPACE: return "workspace missing or not 256-byte aligned";
    case NEP_ERR_TYPE: return "atom type out of range";
    case NEP_ERR_POSITION: return "coordinate outside [0, L)";
    case NEP_ERR_SCRATCH: return "batch needs more than the static scratch of nep_loss_grad_noalloc";
    default: return "unknown status";
  }
}

}  // extern "C"
