// Device kernels of libsrmd for gfx950 (MI355X).
//
// One time step (paper sections 5-7) runs in one of two forms with the same
// per-particle arithmetic in the same order, so both give the same trajectory bit
// for bit at the same launch shape.
//
// Launch chains, captured in HIP graphs; the decision to rebuild the neighbour list
// lives on the device (the paper's device-side flag of section 6), so no step needs
// the host:
//   list rebuild, only when the flag is set (every kernel exits at once otherwise):
//     small systems: the spatial sort already ran at the end of the previous step, so
//                    only the list build runs here, or inside k_step;
//     large systems: k_bin (cells, arrival slots, tile counts), k_scan (cell
//                    offsets, one workgroup per tile), k_scatter, k_gather
//                    (deterministic rank by particle id, gather of every
//                    per-particle array: the reorder of section 7), then the list
//                    kernel.  A chain holds these once per 1 to 32 steps; a step
//                    that finds a rebuild due exits, and so do those after it, up
//                    to the next of these places;
//     list kernels: k_list_wave (a wave per particle), k_list_cell (a wave per piece
//                    of a cell), k_list_stage (16-bit lists into LDS copies of the
//                    neighbourhoods of 256 particles, with k_stage_expand for their
//                    readers outside the step), k_list_thread (a thread per
//                    particle), k_list_row, k_list_allpairs (all pairs in index
//                    order, no sort: the O(N^2) builder of section 6);
//   k_step    pair forces with t_p lanes per particle (sections 3 and 5) fused with
//             the leapfrog / Nose-Hoover update; float64 partial sums per block; its
//             last workgroup (or k_finish, one workgroup, as a launch of its own)
//             ends the step: fixed-order float64 reduction of the partials,
//             thermostat update, thermodynamic record, the displacement test that
//             sets the rebuild flag (section 6), and for small systems the whole
//             spatial sort in LDS when a rebuild is due.
//
// Persistent (k_multi): every step of a call in one cooperative launch of 500
// steps, a system split over several workgroups separated by grid barriers, or many
// systems (a batch of replicas) over the workgroups; the same phases as above run
// inside it.
#include <algorithm>

#include "srmd_internal.h"

namespace srmd {

// ---------------------------------------------------------------- helpers

// Blocks are dispatched round-robin over the 8 XCDs (block b runs on XCD b % 8).
// Remap so that each XCD works on one contiguous range of (spatially sorted)
// particles and its L2 holds that region's positions.
__device__ __forceinline__ int xcd_remap(int b, int G) {
  const int q = G >> 3, r = G & 7, x = b & 7, k = b >> 3;
  return x * q + min(x, r) + k;
}

// float32 minimum image of one coordinate difference: the specified sequence
// m = rint(d * invL) (ties to even), d = fma(-m, L, d).
__device__ __forceinline__ float min_image(float d, float L, float invL) {
  const float m = __builtin_rintf(d * invL);
  return __builtin_fmaf(-m, L, d);
}

// float32 squared distance from a to b; d = b - a after the minimum image.
__device__ __forceinline__ float dist2(const float4 a, const float4 b, const SysConst &c, float &dx, float &dy,
                                       float &dz) {
  dx = min_image(b.x - a.x, c.L[0], c.invL[0]);
  dy = min_image(b.y - a.y, c.L[1], c.invL[1]);
  dz = min_image(b.z - a.z, c.L[2], c.invL[2]);
  return __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
}

__device__ __forceinline__ int ptype(const float4 r) { return __float_as_int(r.w); }

// Cell coordinate along one axis, clamped to [0, nc - 1] in float32 before the
// conversion: x + L/2 can round to L, and a non-finite coordinate (a blown-up run,
// reported through the error word) lands in cell 0 (fmaxf returns the non-NaN
// operand), so no input can produce a cell index outside the grid.
__device__ __forceinline__ int cell_coord(float x, float halfL, float scale, int nc) {
  const float f = fminf(fmaxf(floorf((x + halfL) * scale), 0.0f), (float)(nc - 1));
  return (int)f;
}

// Native 4-vectors, for whole-element copies that stay in registers.
typedef float raw_f4 __attribute__((ext_vector_type(4)));
typedef int raw_i4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void cell_coords(const float4 r, const SysConst &c, int &cx, int &cy, int &cz) {
  cx = cell_coord(r.x, c.halfL[0], c.cscale[0], c.nc[0]);
  cy = cell_coord(r.y, c.halfL[1], c.cscale[1], c.nc[1]);
  cz = cell_coord(r.z, c.halfL[2], c.cscale[2], c.nc[2]);
}

// Address of entry k of particle i in the tp-interleaved column-major list:
// groups of tp consecutive entries of one particle are stored contiguously, and
// consecutive particles' groups follow each other, so the tp lanes of a wave that
// serve consecutive particles read one contiguous span per iteration.  tp = 1 is
// the paper's column-major layout (section 5).
__device__ __forceinline__ long long nbl_addr(int i, int k, const SysConst &c) {
  return ((long long)(k >> c.tp_shift) * c.nvp + i) * c.tp + (k & (c.tp - 1));
}

// Linear index of cell (x, y, z): the order of the spatial sort.  Small systems:
// row-major, x fastest.  Large systems: the grid is cut into columns of about 5 x 5
// cells along z; the columns follow each other in a serpentine over (x, y), each is
// traversed along z (up and down in turn) layer by layer, and a layer row by row.
// Consecutive particles then form slabs of a column, so that the neighbourhood of a
// few hundred of them is small enough for LDS (256 particles of the LJ liquid: about
// 1800 particles; a stretch of x-rows of the row-major order: 4300).  A row of cells
// along x inside one tile stays consecutive.
struct Tile {
  int t, x0, w;  // tile index, first cell and width along an axis
};

__device__ __forceinline__ Tile tile_of(const SysConst &c, int axis, int x) {
  Tile r{0, 0, c.nc[axis]};
  if (c.tiles[axis] > 1) {
    const int q = c.tile_q[axis], rem = c.tile_rem[axis], wide = rem * (q + 1);
    r.t = x < wide ? (x * c.tile_mq1[axis]) >> 16 : rem + (((x - wide) * c.tile_mq[axis]) >> 16);
    r.x0 = r.t * q + min(r.t, rem);
    r.w = q + (r.t < rem ? 1 : 0);
  }
  return r;
}

// Position of a column in the serpentine.
__device__ __forceinline__ int column_seq(const SysConst &c, int tx, int ty) {
  return ty * c.tiles[0] + ((ty & 1) ? c.tiles[0] - 1 - tx : tx);
}

__device__ __forceinline__ int cell_id(const SysConst &c, int x, int y, int z) {
  const int nx = c.nc[0], ny = c.nc[1], nz = c.nc[2];
  if (c.tiles[0] == 1 && c.tiles[1] == 1) return (z * ny + y) * nx + x;
  const Tile X = tile_of(c, 0, x), Y = tile_of(c, 1, y);
  const int before = (Y.t & 1) ? nx - X.x0 - X.w : X.x0;  // cells along x of the columns before it in its row of tiles
  const int zz = (column_seq(c, X.t, Y.t) & 1) ? nz - 1 - z : z;
  return nz * (nx * Y.x0 + Y.w * before) + (zz * Y.w + (y - Y.x0)) * X.w + (x - X.x0);
}

// The x extent of one stencil row: up to two runs of consecutive cells
// [a0, a1] and [b0, b1] (the second one only when the +-2 window wraps round the box
// or reaches into the next tile of the cell order; tiles are at least 5 wide, so not
// both), in the order dx = -2 .. +2; every cell when the axis has fewer than 5.
__device__ __forceinline__ void row_runs(const SysConst &c, int cx, int &a0, int &a1, int &b0, int &b1) {
  const int nx = c.nc[0];
  b0 = 0;
  b1 = -1;
  if (c.full_axis & 1) {
    a0 = 0;
    a1 = nx - 1;
    return;
  }
  const int lo = cx - 2, hi = cx + 2;
  if (lo < 0) {
    a0 = lo + nx;
    a1 = nx - 1;
    b0 = 0;
    b1 = hi;
  } else if (hi >= nx) {
    a0 = lo;
    a1 = nx - 1;
    b0 = 0;
    b1 = hi - nx;
  } else {
    a0 = lo;
    a1 = hi;
    if (c.tiles[0] > 1) {
      const Tile T = tile_of(c, 0, hi);
      if (T.x0 > lo) {
        a1 = T.x0 - 1;
        b0 = T.x0;
        b1 = hi;
      }
    }
  }
}

// Pair table staged in LDS, one 32-byte row per type pair so that a pair's
// constants arrive in two 16-byte LDS reads.
struct alignas(16) PairRow {
  float rc2, sig2, eps24, eps4;  // rc^2, sigma^2, 24 eps, 4 eps
  float ushift, fc, rc, pad;     // U(rc), F(rc), rc
};

// Constants of the shifted-force Coulomb term of a type pair (kernel method 3).
struct alignas(16) CoulRow {
  float qq, rcc2, inv_rcc2, two_inv_rcc;  // q_a q_b, r_cc^2, 1 / r_cc^2, 2 / r_cc
};

// Constants of the two-power potential of a type pair (kernel method 4): B, n B,
// and the half exponents m/2, n/2 (A and m A are in the PairRow's eps4 and eps24).
struct alignas(16) MieRow {
  float b, nb;
  int hm, hn;
};

// Constants of a further potential of a type pair (kernel method 5).
struct alignas(16) GenRow {
  float g0, g1, g2, g3;
};

struct SharedPairs {
  PairRow row[kMaxPairs];
  CoulRow crow[kMaxPairs];
  MieRow mrow[kMaxPairs];
  GenRow grow[kMaxPairs];
};

__device__ __forceinline__ void stage_pairs(SharedPairs &sp, const SysConst &c) {
  const int t = threadIdx.x;
  if (t < kMaxPairs) {
    PairRow r;
    r.rc2 = c.pt.rc2[t];
    r.sig2 = c.pt.sig2[t];
    r.eps24 = c.pt.eps24[t];
    r.eps4 = c.pt.eps4[t];
    r.ushift = c.pt.ushift[t];
    r.fc = c.pt.fc[t];
    r.rc = c.pt.rc[t];
    r.pad = 0.f;
    sp.row[t] = r;
    CoulRow q;
    q.qq = c.pt.qq[t];
    q.rcc2 = c.pt.rcc2;
    q.inv_rcc2 = c.pt.inv_rcc2;
    q.two_inv_rcc = c.pt.two_inv_rcc;
    sp.crow[t] = q;
    MieRow g;
    g.b = c.pt.mie_b[t];
    g.nb = c.pt.mie_nb[t];
    g.hm = c.pt.mie_hm[t];
    g.hn = c.pt.mie_hn[t];
    sp.mrow[t] = g;
    sp.grow[t] = GenRow{c.pt.gen[t][0], c.pt.gen[t][1], c.pt.gen[t][2], c.pt.gen[t][3]};
  }
}

// Position of particle i widened once for the float64 coordinate differences.
struct Wide {
  double x, y, z;
};

__device__ __forceinline__ Wide widen(const float4 p) { return Wide{(double)p.x, (double)p.y, (double)p.z}; }

// One pair contribution (12-6 Lennard-Jones, paper section 2 cutoff methods).
// The in/out decision uses the specified float32 squared distance (the same bits
// as the list build and the CPU reference).  The value uses the coordinate
// differences recomputed in float64 with the same image shift and rounded once to
// float32: across the periodic boundary x_j - x_i is close to L, and rounding it
// in float32 first would cost about ulp(L/2) of absolute accuracy.
// Accumulates the force on i (-fr * d, with fr = F(r)/r and d = r_j - r_i), the
// pair energy u and fr * r^2 (= r . F) for the virial.
// x^h for 0 <= h < 32 by binary exponentiation (five squarings, fixed order).
__device__ __forceinline__ float pow_int(float x, int h) {
  float r = 1.0f;
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    if (h & (1 << k)) r *= x;
    x *= x;
  }
  return r;
}

// Energy u and force over distance fr = F(r)/r (F = -dU/dr, positive repulsive) of
// the further pair potentials of paper section 2 (the paper names them only; these
// are the textbook forms), in float32 from the pair's constants g (kind uniform over
// the system):
//  2 Yukawa        U = eps (sig/r) exp(-kappa (r - sig)) = g0 exp(-g1 r) / r
//                  (g0 = eps sig exp(kappa sig), g1 = kappa)
//  3 Buckingham    U = A exp(-r/rho) - C / r^6               (g0 = A, g1 = 1/rho, g2 = C)
//  4 Gaussian core U = eps exp(-(r/sig)^2)                    (g0 = eps, g1 = 1/sig^2)
//  5 Dzugutov      U = eps [5.82 (x^-16 - 1.28) exp(1.1 / (x - 1.87)) (x < 1.87)
//                         + 1.28 exp(0.27 / (x - 1.94)) (x < 1.94)],  x = r/sig
//                                                            (g0 = eps, g1 = 1/sig)
//  6 Girifalco     U = -alpha [1/(s(s-1)^3) + 1/(s(s+1)^3) - 2/s^4]
//                      + beta [1/(s(s-1)^9) + 1/(s(s+1)^9) - 2/s^10],  s = r/d
//                                                            (g0 = alpha, g1 = beta, g2 = 1/d)
__device__ __forceinline__ void pair_further(int kind, const GenRow &g, float r, float inv_r, float &u, float &fr) {
  const float inv_r2 = inv_r * inv_r;
  if (kind == 2) {
    u = g.g0 * expf(-g.g1 * r) * inv_r;
    fr = u * __builtin_fmaf(g.g1, r, 1.0f) * inv_r2;
  } else if (kind == 3) {
    const float e = g.g0 * expf(-g.g1 * r);
    const float d6 = g.g2 * inv_r2 * inv_r2 * inv_r2;
    u = e - d6;
    fr = (e * g.g1 * inv_r - 6.0f * d6 * inv_r2);
  } else if (kind == 4) {
    const float e = g.g0 * expf(-r * r * g.g1);
    u = e;
    fr = 2.0f * g.g1 * e;
  } else if (kind == 5) {
    const float x = r * g.g1;
    float uu = 0.0f, du = 0.0f;
    if (x < 1.87f) {
      const float q = 1.0f / (x - 1.87f);
      const float e = expf(1.1f * q);
      const float ix2 = 1.0f / (x * x);
      const float xm = pow_int(ix2, 8);
      uu = 5.82f * (xm - 1.28f) * e;
      du = 5.82f * e * (-16.0f * xm / x - (xm - 1.28f) * 1.1f * q * q);
    }
    if (x < 1.94f) {
      const float q = 1.0f / (x - 1.94f);
      const float e = 1.28f * expf(0.27f * q);
      uu += e;
      du -= e * 0.27f * q * q;
    }
    u = g.g0 * uu;
    fr = -g.g0 * du * g.g1 * inv_r;
  } else {
    const float s = r * g.g2, is = 1.0f / s;
    const float ia = 1.0f / (s - 1.0f), ib = 1.0f / (s + 1.0f);
    const float ia3 = ia * ia * ia, ib3 = ib * ib * ib, ia9 = ia3 * ia3 * ia3, ib9 = ib3 * ib3 * ib3;
    const float is4 = is * is * is * is, is10 = is4 * is4 * is * is;
    const float att = is * (ia3 + ib3) - 2.0f * is4;
    const float rep = is * (ia9 + ib9) - 2.0f * is10;
    const float datt = -is * is * (ia3 + ib3) - 3.0f * is * (ia3 * ia + ib3 * ib) + 8.0f * is4 * is;
    const float drep = -is * is * (ia9 + ib9) - 9.0f * is * (ia9 * ia + ib9 * ib) + 20.0f * is10 * is;
    u = -g.g0 * att + g.g1 * rep;
    fr = (g.g0 * datt - g.g1 * drep) * g.g2 * inv_r;
  }
}

template <int METHOD>
__device__ __forceinline__ void pair_acc(const float4 pi, const Wide &wi, const float4 pj, int ti, int ntypes,
                                         const SharedPairs &sp, const SysConst &c, float &fx, float &fy, float &fz,
                                         float &u, float &w) {
  const float ex = pj.x - pi.x, ey = pj.y - pi.y, ez = pj.z - pi.z;
  const float mx = __builtin_rintf(ex * c.invL[0]), my = __builtin_rintf(ey * c.invL[1]),
              mz = __builtin_rintf(ez * c.invL[2]);
  float dx = __builtin_fmaf(-mx, c.L[0], ex), dy = __builtin_fmaf(-my, c.L[1], ey), dz = __builtin_fmaf(-mz, c.L[2], ez);
  const float r2s = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
  const int pidx = ti * ntypes + ptype(pj);
  const PairRow &pr = sp.row[pidx];
  if (METHOD == 4) {
    // two-power potential A s^m - B s^n, s = sigma/r, with the cutoff method carried
    // by U(rc) (zero when truncated) and F(rc) (nonzero for shifted force only)
    if (r2s < pr.rc2) {
      dx = (float)(((double)pj.x - wi.x) - (double)mx * c.Ld[0]);
      dy = (float)(((double)pj.y - wi.y) - (double)my * c.Ld[1]);
      dz = (float)(((double)pj.z - wi.z) - (double)mz * c.Ld[2]);
      const float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
      const float inv_r2 = __builtin_amdgcn_rcpf(r2);
      const MieRow &mr = sp.mrow[pidx];
      const float s2 = pr.sig2 * inv_r2;
      const float sm = pow_int(s2, mr.hm), sn = pow_int(s2, mr.hn);
      float fr = (pr.eps24 * sm - mr.nb * sn) * inv_r2;
      float e = pr.eps4 * sm - mr.b * sn - pr.ushift;
      const float inv_r = __builtin_amdgcn_rsqf(r2);
      const float r = r2 * inv_r;
      fr = __builtin_fmaf(-pr.fc, inv_r, fr);
      e = __builtin_fmaf(r - pr.rc, pr.fc, e);
      fx = __builtin_fmaf(-fr, dx, fx);
      fy = __builtin_fmaf(-fr, dy, fy);
      fz = __builtin_fmaf(-fr, dz, fz);
      u += e;
      w = __builtin_fmaf(fr, r2, w);
    }
    return;
  }
  if (METHOD == 5) {
    // a further potential of paper section 2, cutoff method by U(rc) and F(rc)
    if (r2s < pr.rc2) {
      dx = (float)(((double)pj.x - wi.x) - (double)mx * c.Ld[0]);
      dy = (float)(((double)pj.y - wi.y) - (double)my * c.Ld[1]);
      dz = (float)(((double)pj.z - wi.z) - (double)mz * c.Ld[2]);
      const float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
      const float inv_r = __builtin_amdgcn_rsqf(r2);
      const float r = r2 * inv_r;
      float e, fr;
      pair_further(c.pot_kind, sp.grow[pidx], r, inv_r, e, fr);
      fr = __builtin_fmaf(-pr.fc, inv_r, fr);
      e = __builtin_fmaf(r - pr.rc, pr.fc, e - pr.ushift);
      fx = __builtin_fmaf(-fr, dx, fx);
      fy = __builtin_fmaf(-fr, dy, fy);
      fz = __builtin_fmaf(-fr, dz, fz);
      u += e;
      w = __builtin_fmaf(fr, r2, w);
    }
    return;
  }
}

// One pair contribution of 12-6 Lennard-Jones (paper section 2 cutoff methods;
// METHOD 0-2) or of shifted-force Lennard-Jones plus shifted-force Coulomb (METHOD 3,
// paper section 9: q_a q_b (1/r - 1/r_cc + (r - r_cc)/r_cc^2), force
// q_a q_b (1/r^2 - 1/r_cc^2), each term with its own float32 in/out decision).
// Straight-line code: a pair out of range (or ok = false, an idle slot) contributes
// zeros by selects instead of a branch, so the pairs of a batch are independent
// instruction streams that the compiler interleaves.  IMG = false: the caller knows
// that no pair in range crosses the periodic boundary; then every image integer is 0,
// the float32 differences are the correctly rounded ones and both the decision and the
// value use them (the same bits as the general form).  ONE: a single particle type,
// whose constants are uniform over the wave (scalar registers) instead of LDS rows.
template <int METHOD, bool IMG, bool ONE>
__device__ __forceinline__ void lj_pair(const float4 pi, const Wide &wi, const float4 pj, bool ok, int row0,
                                        const SharedPairs &sp, const SysConst &c, float &fx, float &fy, float &fz,
                                        float &u, float &w) {
  float dx = pj.x - pi.x, dy = pj.y - pi.y, dz = pj.z - pi.z;
  float mx = 0.f, my = 0.f, mz = 0.f;
  if (IMG) {
    mx = __builtin_rintf(dx * c.invL[0]);
    my = __builtin_rintf(dy * c.invL[1]);
    mz = __builtin_rintf(dz * c.invL[2]);
    dx = __builtin_fmaf(-mx, c.L[0], dx);
    dy = __builtin_fmaf(-my, c.L[1], dy);
    dz = __builtin_fmaf(-mz, c.L[2], dz);
  }
  const float r2s = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
  const int pidx = ONE ? 0 : row0 + ptype(pj);
  const float rc2 = ONE ? c.pt.rc2[0] : sp.row[pidx].rc2, sig2 = ONE ? c.pt.sig2[0] : sp.row[pidx].sig2;
  const float eps24 = ONE ? c.pt.eps24[0] : sp.row[pidx].eps24, eps4 = ONE ? c.pt.eps4[0] : sp.row[pidx].eps4;
  const float ushift = ONE ? c.pt.ushift[0] : sp.row[pidx].ushift;
  const bool in_lj = ok & (r2s < rc2);
  float r2 = r2s;
  if (IMG) {
    // (the product of an image integer and the float32 side is exact in float64)
    dx = (float)__builtin_fma(-(double)mx, c.Ld[0], (double)pj.x - wi.x);
    dy = (float)__builtin_fma(-(double)my, c.Ld[1], (double)pj.y - wi.y);
    dz = (float)__builtin_fma(-(double)mz, c.Ld[2], (double)pj.z - wi.z);
    r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
  }
  const float inv_r2 = __builtin_amdgcn_rcpf(r2);
  const float s2 = sig2 * inv_r2;
  const float s6 = s2 * s2 * s2;
  const float s12 = s6 * s6;
  float fr = eps24 * __builtin_fmaf(2.0f, s12, -s6) * inv_r2;
  float e = __builtin_fmaf(eps4, s12 - s6, -ushift);
  if (METHOD >= 2) {  // shifted force: F(r) - F(rc); U(r) - U(rc) + (r - rc) F(rc)
    const float fc = ONE ? c.pt.fc[0] : sp.row[pidx].fc, rc = ONE ? c.pt.rc[0] : sp.row[pidx].rc;
    const float inv_r = __builtin_amdgcn_rsqf(r2);
    const float r = r2 * inv_r;
    fr = __builtin_fmaf(-fc, inv_r, fr);
    e = __builtin_fmaf(r - rc, fc, e);
    if (METHOD == 3) {
      const CoulRow &cr = sp.crow[pidx];
      const bool in_c = ok & (r2s < cr.rcc2);
      fr = in_lj ? fr : 0.f;
      e = in_lj ? e : 0.f;
      const float frc = __builtin_fmaf(cr.qq * inv_r, inv_r2 - cr.inv_rcc2, fr);
      const float ec = __builtin_fmaf(cr.qq, __builtin_fmaf(r, cr.inv_rcc2, inv_r) - cr.two_inv_rcc, e);
      fr = in_c ? frc : fr;
      e = in_c ? ec : e;
    }
  }
  if (METHOD != 3) {
    fr = in_lj ? fr : 0.f;
    e = in_lj ? e : 0.f;
  }
  fx = __builtin_fmaf(-fr, dx, fx);
  fy = __builtin_fmaf(-fr, dy, fy);
  fz = __builtin_fmaf(-fr, dz, fz);
  u += e;
  w = __builtin_fmaf(fr, r2, w);
}

// The selects of lj_pair leave a pair out of range a product with 0, which a non-finite
// coordinate (of the neighbour, or the particle's own in an idle slot) turns into NaN; such
// a pair contributes nothing (no distance to it is below a cutoff).  So a lane whose sums are
// not finite takes its entries again one by one and leaves those out: the same sums unless a
// pair in range is itself not finite.  count(): the lane's entries; entry(m): its entry m.
template <int METHOD, class Count, class Entry>
__device__ __forceinline__ void finite_sums(const float4 pi, Count count, Entry entry, const SharedPairs &sp,
                                            const SysConst &c, float &fx, float &fy, float &fz, float &u, float &w) {
  if (fabsf((fx + fy) + (fz + w)) < __builtin_inff()) return;
  const int row0 = ptype(pi) * c.ntypes;
  const Wide wi = widen(pi);
  fx = fy = fz = u = w = 0.f;
  const int mine = count();
#pragma unroll 1
  for (int m = 0; m < mine; ++m) {
    const float4 q = entry(m);
    float dx, dy, dz;
    if (dist2(pi, q, c, dx, dy, dz) < __builtin_inff())
      lj_pair<METHOD, true, false>(pi, wi, q, true, row0, sp, c, fx, fy, fz, u, w);
  }
}

// Pairs evaluated together: a group is skipped (uniformly) once every lane's list has
// ended.  1, 2 and 4 measured within 1 % of each other; with whole batches of 8 a wave
// of lists of 10 entries did 16 pairs of work.
constexpr int kPairGroup = 2;

// The list of one lane (entries k = t, t + TP, ... of particle i; mine of them, at most
// wmax in this wave), B entries at a time: the positions of a batch are issued
// together, then the next batch's indices, which arrive while the batch is evaluated.
// The entries of one slot of all lanes of a wave are consecutive words of the list, so
// a slot's address is uniform (row + m * stride) plus the lane.
template <int TP, int METHOD, int B, bool IMG, bool ONE, class IdxPtr>
__device__ __forceinline__ void force_loop(int i, const float4 pi, const float4 *__restrict__ pos, IdxPtr row,
                                           long long stride, int mine, int wmax, int (&j)[B], const SharedPairs &sp,
                                           const SysConst &c, float &fx, float &fy, float &fz, float &u, float &w) {
  const int lane = threadIdx.x & 63;
  const int ti = ptype(pi);
  const int row0 = ti * c.ntypes;
  const Wide wi = widen(pi);
  for (int m0 = 0; m0 < wmax; m0 += B) {
    bool ok[B];
    float4 q[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
      ok[b] = m0 + b < mine;
      q[b] = pos[ok[b] ? j[b] : i];
    }
    if (m0 + B < wmax) {
#pragma unroll
      for (int b = 0; b < B; ++b) j[b] = __builtin_nontemporal_load(row + (long long)min(m0 + B + b, wmax - 1) * stride + lane);
    }
#pragma unroll
    for (int g = 0; g < B; g += kPairGroup) {
      if (m0 + g < wmax) {  // uniform
#pragma unroll
        for (int b = g; b < g + kPairGroup; ++b) {
          if constexpr (METHOD <= 3) {
            lj_pair<METHOD, IMG, ONE>(pi, wi, q[b], ok[b], row0, sp, c, fx, fy, fz, u, w);
          } else {
            if (ok[b]) pair_acc<METHOD>(pi, wi, q[b], ti, c.ntypes, sp, c, fx, fy, fz, u, w);
          }
        }
      }
    }
  }
}

// List entries of one lane taken together: about the entries a lane has at liquid
// densities (90 per particle / TP), so that few slots of the last batch idle.
template <int TP>
struct Batch {
  static constexpr int value = TP <= 2 ? 16 : TP == 4 ? 8 : TP == 8 ? 16 : TP == 16 ? 8 : TP == 32 ? 4 : 2;
};

// The launch-chain kernels take at most 8 entries per batch and prefetch the next
// batch's indices, so two batches' loads are in flight within 128 registers (the
// persistent kernel, at 2 waves per SIMD, keeps the full batches).
template <int TP>
struct StepBatch {
  static constexpr int value = Batch<TP>::value > 8 ? 8 : Batch<TP>::value;
};

// The value of lane (this lane) ^ O, O a power of two below 64, by VALU lane
// exchanges: quad permutations for 1 and 2, two bank-masked row shifts for 4, a
// row rotation for 8, and the row and half-wave swaps of gfx950 for 16 and 32.
template <int O>
__device__ __forceinline__ unsigned xor_lane(unsigned v) {
  if constexpr (O == 1) {
    return (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false);  // quad_perm [1, 0, 3, 2]
  } else if constexpr (O == 2) {
    return (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, false);  // quad_perm [2, 3, 0, 1]
  } else if constexpr (O == 4) {
    // lanes 0-3 and 8-11 of a row read lane + 4 (row_shl:4), lanes 4-7 and 12-15 lane - 4 (row_shr:4)
    const int t = __builtin_amdgcn_update_dpp(0, (int)v, 0x104, 0xF, 0x5, false);
    return (unsigned)__builtin_amdgcn_update_dpp(t, (int)v, 0x114, 0xF, 0xA, false);
  } else if constexpr (O == 8) {
    return (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, false);  // row_ror:8
  } else if constexpr (O == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);  // odd rows <-> even rows
    return ((threadIdx.x >> 4) & 1) ? r[0] : r[1];
  } else {
    static_assert(O == 32, "xor_lane: O must be 1, 2, 4, 8, 16 or 32");
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);  // upper half <-> lower half
    return ((threadIdx.x >> 5) & 1) ? r[0] : r[1];
  }
}

template <int O>
__device__ __forceinline__ float xor_lane(float v) {
  return __uint_as_float(xor_lane<O>(__float_as_uint(v)));
}

// Sum over the TP lanes of a particle: the butterfly lane ^ TP/2, ..., lane ^ 1 (the
// whole wave must be active).
template <int TP, int O = TP / 2>
__device__ __forceinline__ float lane_sum(float v) {
  if constexpr (O == 0) {
    return v;
  } else {
    return lane_sum<TP, O / 2>(v + xor_lane<O>(v));
  }
}

// Wave-wide reductions by DPP lane swizzles (VALU operand exchanges, no LDS round
// trip as in a shuffle).  Within each 16-lane row: the quad exchanges lane ^ 1 and
// lane ^ 2, the half-row mirror (lane i with 7 - i of its 8) and the row mirror
// (i with 15 - i), each pairing two disjoint halves, so that every lane of a row
// ends with the row's total, bitwise the same in all 16 (each step combines the
// same two values in either order).  Then lane 15 of rows 0 and 2 is combined into
// rows 1 and 3, and lane 31 into rows 2 and 3, so lane 63 holds
// (row 3 + row 2) + (row 1 + row 0), which is read back to every lane.  Lanes of the
// rows a broadcast does not reach combine with the identity.  The whole wave must
// be active.
constexpr int kDppXor1 = 0xB1;        // quad_perm [1, 0, 3, 2]
constexpr int kDppXor2 = 0x4E;        // quad_perm [2, 3, 0, 1]
constexpr int kDppMirror = 0x140;     // row_mirror
constexpr int kDppHalfMirror = 0x141; // row_half_mirror
constexpr int kDppBcast15 = 0x142;    // row_bcast:15
constexpr int kDppBcast31 = 0x143;    // row_bcast:31

template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned dpp32(unsigned old, unsigned v) {
  return (unsigned)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, ROWS, 0xF, false);
}

template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned long long dpp64(unsigned long long old, unsigned long long v) {
  const unsigned lo = dpp32<CTRL, ROWS>((unsigned)old, (unsigned)v);
  const unsigned hi = dpp32<CTRL, ROWS>((unsigned)(old >> 32), (unsigned)(v >> 32));
  return ((unsigned long long)hi << 32) | lo;
}

template <class Op>
__device__ __forceinline__ unsigned long long wave_reduce64(unsigned long long v, unsigned long long id, Op op) {
  v = op(v, dpp64<kDppXor1, 0xF>(id, v));
  v = op(v, dpp64<kDppXor2, 0xF>(id, v));
  v = op(v, dpp64<kDppHalfMirror, 0xF>(id, v));
  v = op(v, dpp64<kDppMirror, 0xF>(id, v));
  v = op(v, dpp64<kDppBcast15, 0xA>(id, v));
  v = op(v, dpp64<kDppBcast31, 0xC>(id, v));
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, 63);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), 63);
  return ((unsigned long long)hi << 32) | lo;
}

__device__ __forceinline__ double bits_f64(unsigned long long b) { return __longlong_as_double((long long)b); }
__device__ __forceinline__ unsigned long long f64_bits(double d) { return (unsigned long long)__double_as_longlong(d); }

__device__ __forceinline__ double wave_sum(double v) {
  return bits_f64(wave_reduce64(f64_bits(v), f64_bits(0.0), [](unsigned long long a, unsigned long long b) {
    return f64_bits(bits_f64(a) + bits_f64(b));
  }));
}

__device__ __forceinline__ double wave_max(double v) {
  return bits_f64(wave_reduce64(f64_bits(v), f64_bits(-__builtin_inf()), [](unsigned long long a, unsigned long long b) {
    return f64_bits(fmax(bits_f64(a), bits_f64(b)));
  }));
}

__device__ __forceinline__ unsigned long long wave_min_u64(unsigned long long v) {
  return wave_reduce64(v, ~0ull, [](unsigned long long a, unsigned long long b) { return b < a ? b : a; });
}

__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long v) {
  return wave_reduce64(v, 0ull, [](unsigned long long a, unsigned long long b) { return b > a ? b : a; });
}

__device__ __forceinline__ int wave_or(int v) {
  return (int)wave_reduce64((unsigned)v, 0ull, [](unsigned long long a, unsigned long long b) { return a | b; });
}

// Largest of the lanes' non-negative integers, uniform (a scalar register).
__device__ __forceinline__ int wave_max_i32(int v) {
  auto up = [](int a, int b) { return a > b ? a : b; };
  v = up(v, (int)dpp32<kDppXor1, 0xF>(0u, (unsigned)v));
  v = up(v, (int)dpp32<kDppXor2, 0xF>(0u, (unsigned)v));
  v = up(v, (int)dpp32<kDppHalfMirror, 0xF>(0u, (unsigned)v));
  v = up(v, (int)dpp32<kDppMirror, 0xF>(0u, (unsigned)v));
  v = up(v, (int)dpp32<kDppBcast15, 0xA>(0u, (unsigned)v));
  v = up(v, (int)dpp32<kDppBcast31, 0xC>(0u, (unsigned)v));
  return __builtin_amdgcn_readlane(v, 63);
}

// Force on particle i from lane t of its TP lanes (entries k = t, t+TP, ...), by whole
// waves: lanes with active = false (i past the end) idle with i clamped to a valid
// particle.  The lane's entries are taken B at a time (the paper prefetches one entry
// ahead, section 5; on MI355X the latency of a dependent load chain dominates, so many
// loads go in flight).  The first batch is issued before the list length arrives
// (clamped to the capacity n_max / TP of a lane), so the length and the first indices
// share a round trip.  A wave whose particles are all farther than the cutoff from
// every face takes the loop without image arithmetic, and a system of one type the
// loop with scalar constants (25 and 20 instructions of about 60 per pair).  SLIM: the
// general loop only (the rare unstaged units of the staged kernels, the persistent kernel).
template <int TP, int METHOD, int B, bool SLIM, class IdxPtr>
__device__ __forceinline__ void force_lane(int i, int t, bool active, const float4 pi, const float4 *__restrict__ pos,
                                           IdxPtr nbl, IdxPtr nnb, const SharedPairs &sp, const SysConst &c,
                                           float &fx, float &fy, float &fz, float &u, float &w) {
  const long long stride = (long long)c.nvp * TP;
  // particle of the wave's first lane, a multiple of 64 / TP (also in a wave that idles
  // with its lanes clamped), so that the wave's words stay inside the list's nvp columns
  const int lane = threadIdx.x & 63;
  const int i0 = __builtin_amdgcn_readfirstlane(i - lane / TP) & ~(64 / TP - 1);
  const IdxPtr row = nbl + (long long)i0 * TP;
  const int cap = c.n_max / TP;  // entries of one lane the list can hold
  int j[B];
#pragma unroll
  for (int b = 0; b < B; ++b) j[b] = __builtin_nontemporal_load(row + (long long)min(b, cap - 1) * stride + lane);
  const int nn = active ? nnb[i] : 0;
  const int mine = nn > t ? (nn - t + TP - 1) / TP : 0;  // entries of this lane
  int wmax = 0;  // entries of the wave's longest lane
  if constexpr (TP >= 16) {  // few particles per wave: their lengths by scalar reads
#pragma unroll
    for (int k = 0; k < 64; k += TP) wmax = max(wmax, __builtin_amdgcn_readlane(nn, k));
    wmax = (wmax + TP - 1) / TP;
  } else {
    wmax = wave_max_i32(mine);
  }
  // from 16 lanes per particle the wave at a face sets the pace of the step: one form
  const bool near = TP >= 16 || fabsf(pi.x) >= c.inner[0] || fabsf(pi.y) >= c.inner[1] || fabsf(pi.z) >= c.inner[2];
  if constexpr (METHOD <= 3 && !SLIM) {
    if (c.ntypes == 1 && METHOD != 3) {
      if (TP >= 16 || __any(near))
        force_loop<TP, METHOD, B, true, true>(i, pi, pos, row, stride, mine, wmax, j, sp, c, fx, fy, fz, u, w);
      else
        force_loop<TP, METHOD, B, false, true>(i, pi, pos, row, stride, mine, wmax, j, sp, c, fx, fy, fz, u, w);
    } else {
      if (TP >= 16 || __any(near))
        force_loop<TP, METHOD, B, true, false>(i, pi, pos, row, stride, mine, wmax, j, sp, c, fx, fy, fz, u, w);
      else
        force_loop<TP, METHOD, B, false, false>(i, pi, pos, row, stride, mine, wmax, j, sp, c, fx, fy, fz, u, w);
    }
  } else {
    force_loop<TP, METHOD, B, true, false>(i, pi, pos, row, stride, mine, wmax, j, sp, c, fx, fy, fz, u, w);
  }
  if constexpr (METHOD <= 3)
    finite_sums<METHOD>(
        pi, [&] { return mine; }, [&](int m) { return pos[*(row + (long long)m * stride + lane)]; }, sp, c, fx, fy, fz,
        u, w);
}

// Least of the lanes' values (at most 1e30), uniform.
__device__ __forceinline__ float wave_min_f32(float v) {
  auto dn = [](float a, unsigned b) { return fminf(a, __uint_as_float(b)); };
  const unsigned id = __float_as_uint(1e30f);
  v = dn(v, dpp32<kDppXor1, 0xF>(id, __float_as_uint(v)));
  v = dn(v, dpp32<kDppXor2, 0xF>(id, __float_as_uint(v)));
  v = dn(v, dpp32<kDppHalfMirror, 0xF>(id, __float_as_uint(v)));
  v = dn(v, dpp32<kDppMirror, 0xF>(id, __float_as_uint(v)));
  v = dn(v, dpp32<kDppBcast15, 0xA>(id, __float_as_uint(v)));
  v = dn(v, dpp32<kDppBcast31, 0xC>(id, __float_as_uint(v)));
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// ---- staged lists in the force loop (large systems)

// The copies of a workgroup's units' regions into LDS (unit after unit, place 0 of each
// a far-away particle that no distance test passes).  Returns the first place of the
// calling wave's unit, or -1 when its lists are plain ones (a region that was too large
// for the list build); the others all fit, as stage_lds holds stage_cap places and one
// more for every unit.  Every thread of the block must call it; a barrier must follow.
template <int TP>
__device__ __forceinline__ int stage_fill(const SysConst &c, const SysPtrs &p, const float4 *__restrict__ pos, int lb,
                                          float4 *s_region) {
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int ppb = nthr / TP, units = ppb / kStageSlots, u0 = lb * units;
  const int mine = __builtin_amdgcn_readfirstlane(tid) / (TP * kStageSlots);
  int at = 0, place = -1;
  for (int u = 0; u < units; ++u) {
    if ((u0 + u) * kStageSlots >= c.n) break;
    const int n = p.stage_n[u0 + u];
    if (n == 0) continue;
    if (u == mine) place = at;
    const unsigned *src = p.stage_src + (size_t)(u0 + u) * c.stage_cap;
    float4 *dst = s_region + at + 1;
    if (tid == 0) s_region[at] = make_float4(1e18f, 1e18f, 1e18f, 0.f);
    for (int k0 = tid; k0 < n; k0 += 4 * nthr) {
      unsigned j[4];
      float4 v[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) j[b] = src[min(k0 + b * nthr, n - 1)];
#pragma unroll
      for (int b = 0; b < 4; ++b) v[b] = pos[j[b]];
#pragma unroll
      for (int b = 0; b < 4; ++b)
        if (k0 + b * nthr < n) dst[k0 + b * nthr] = v[b];
    }
    at += n + 1;
  }
  return place;
}

// force_loop over a staged list: two entries per word, neighbour positions from the LDS
// copy.  The lists are padded with place 0 up to the unit's longest, so that a loop
// without image arithmetic needs no test for the end of a lane's list.
template <int TP, int METHOD, bool IMG, bool ONE>
__device__ __forceinline__ void stage_loop(const float4 pi, const float4 *region, const unsigned *row, long long stride,
                                           int col, int mine, int words, unsigned (&j)[4], const SharedPairs &sp,
                                           const SysConst &c, float &fx, float &fy, float &fz, float &u, float &w) {
  const int ti = ptype(pi);
  const int row0 = ti * c.ntypes;
  const Wide wi = widen(pi);
  for (int w0 = 0; w0 < words; w0 += 4) {
    float4 q[8];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      q[2 * b] = region[j[b] & 0xffffu];
      q[2 * b + 1] = region[j[b] >> 16];
    }
    if (w0 + 4 < words) {
#pragma unroll
      for (int b = 0; b < 4; ++b) j[b] = __builtin_nontemporal_load(row + (long long)min(w0 + 4 + b, words - 1) * stride + col);
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      if (w0 + b < words) {  // uniform
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const bool ok = (!IMG && METHOD <= 3) || 2 * (w0 + b) + h < mine;
          if constexpr (METHOD <= 3) {
            lj_pair<METHOD, IMG, ONE>(pi, wi, q[2 * b + h], ok, row0, sp, c, fx, fy, fz, u, w);
          } else {
            if (ok) pair_acc<METHOD>(pi, wi, q[2 * b + h], ti, c.ntypes, sp, c, fx, fy, fz, u, w);
          }
        }
      }
    }
  }
}

// force_lane over a staged list: the same pairs in the same order.  The gathers from L2
// bound force_lane (the texture-address path takes a cycle per lane: 63 % busy, and the
// 32-bit indices are 70 % of the bytes); from LDS a neighbour costs a quarter of that
// and an index half the bytes.  k_step at one lane per particle, 1 024 000 particles: 178
// -> 162 us by the column order alone, 125 us with the copies (five blocks per compute
// unit; with a third more LDS per block, four, 131 us), bound by VALU issue (78 % busy);
// 256 000: 50.5 -> 44.5 us; at four lanes per particle, 64 000: 20.8 -> 20.4 us.
template <int TP, int METHOD>
__device__ __forceinline__ void force_lane_staged(int i, int t, bool active, const float4 pi, const float4 *region,
                                                  const SysPtrs &p, const SharedPairs &sp, const SysConst &c, float &fx,
                                                  float &fy, float &fz, float &u, float &w) {
  const long long stride = (long long)c.nvp * TP;
  const int lane = threadIdx.x & 63;
  const int i0 = __builtin_amdgcn_readfirstlane(i - lane / TP) & ~(64 / TP - 1);
  const unsigned *row = p.list16 + (long long)i0 * TP;
  const int col = active ? lane : 0;   // lanes past the last particle read a list that was written
  const int cap = c.n_max / (2 * TP);  // words of one lane the list can hold
  unsigned j[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) j[b] = __builtin_nontemporal_load(row + (long long)min(b, cap - 1) * stride + col);
  const int nn = active ? p.nnb[i] : 0;
  const int mine = nn > t ? (nn - t + TP - 1) / TP : 0;
  const int words = (wave_max_i32(mine) + 1) / 2;
  // words past the wave's longest list are not padded: no place outside the region
#pragma unroll
  for (int b = 0; b < 4; ++b) j[b] = b < words ? j[b] : 0u;
  const bool near = fabsf(pi.x) >= c.inner[0] || fabsf(pi.y) >= c.inner[1] || fabsf(pi.z) >= c.inner[2];
  if constexpr (METHOD <= 3) {
    if (c.ntypes == 1 && METHOD != 3) {
      if (__any(near))
        stage_loop<TP, METHOD, true, true>(pi, region, row, stride, col, mine, words, j, sp, c, fx, fy, fz, u, w);
      else
        stage_loop<TP, METHOD, false, true>(pi, region, row, stride, col, mine, words, j, sp, c, fx, fy, fz, u, w);
    } else {
      if (__any(near))
        stage_loop<TP, METHOD, true, false>(pi, region, row, stride, col, mine, words, j, sp, c, fx, fy, fz, u, w);
      else
        stage_loop<TP, METHOD, false, false>(pi, region, row, stride, col, mine, words, j, sp, c, fx, fy, fz, u, w);
    }
  } else {
    stage_loop<TP, METHOD, true, false>(pi, region, row, stride, col, mine, words, j, sp, c, fx, fy, fz, u, w);
  }
  if constexpr (METHOD <= 3) {
    // the list's length and column anew: kept over the loop above they would be spilled (two
    // registers of each thread, 8 MB a step at 1 024 000 particles)
    auto anew = [](int v) {
      __asm__("" : "+v"(v));
      return v;
    };
    finite_sums<METHOD>(
        pi,
        [&] {
          const int nk = active ? p.nnb[anew(i)] : 0;
          return nk > t ? (nk - t + TP - 1) / TP : 0;
        },
        [&](int m) {
          const unsigned two = row[(long long)(m >> 1) * stride + (active ? anew((int)threadIdx.x) & 63 : 0)];
          return region[m & 1 ? two >> 16 : two & 0xffffu];
        },
        sp, c, fx, fy, fz, u, w);
  }
}

// Inclusive prefix sum over the lanes of a wave, exact for integers: within each row
// the shifted copies by 1, 2 and 3 lanes, then the partial sums shifted by 4 (into
// the upper three banks of 4 lanes) and by 8 (into the upper two), then the row
// totals by the broadcasts of lanes 15 and 31.  The whole wave must be active.
__device__ __forceinline__ unsigned wave_incl_scan(unsigned v) {
  unsigned t = v + (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);  // row_shr:1
  t += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);             // row_shr:2
  t += (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x113, 0xF, 0xF, false);             // row_shr:3
  t += (unsigned)__builtin_amdgcn_update_dpp(0, (int)t, 0x114, 0xF, 0xE, false);             // row_shr:4
  t += (unsigned)__builtin_amdgcn_update_dpp(0, (int)t, 0x118, 0xF, 0xC, false);             // row_shr:8
  t += (unsigned)__builtin_amdgcn_update_dpp(0, (int)t, kDppBcast15, 0xA, 0xF, false);
  t += (unsigned)__builtin_amdgcn_update_dpp(0, (int)t, kDppBcast31, 0xC, 0xF, false);
  return t;
}

// Reduction of one BlockPartial over groups of `group` threads (a multiple of 64):
// lanes by butterfly, then the group's waves in index order; the result is valid
// in the first thread of each group.  Every thread of the block must call it.
// With group = blockDim.x this is the block-wide reduction; the batched kernel
// uses groups to reproduce the blocks of the single-system kernels exactly.
// used: the group's waves that can hold data (the rest hold zero partials, whose fold
// changes nothing: no partial is -0.0, since every sum starts from +0.0)
__device__ void group_reduce(BlockPartial &v, BlockPartial *s_waves, int group, int used = 64) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, wpg = min(group >> 6, used);
  v.pe = wave_sum(v.pe);
  v.w = wave_sum(v.w);
  v.ke_half = wave_sum(v.ke_half);
  v.ke_int = wave_sum(v.ke_int);
  v.disp2 = wave_max(v.disp2);
  v.t0 = wave_min_u64(v.t0);
  v.t1 = wave_max_u64(v.t1);
  v.nonfinite = wave_or(v.nonfinite);
  if (lane == 0) s_waves[wv] = v;
  __syncthreads();
  if ((threadIdx.x % group) == 0) {
    const int w0 = wv;  // first wave of this group
    BlockPartial a = s_waves[w0];
    for (int k = 1; k < wpg; ++k) {
      const BlockPartial &q = s_waves[w0 + k];
      a.pe += q.pe;
      a.w += q.w;
      a.ke_half += q.ke_half;
      a.ke_int += q.ke_int;
      a.disp2 = fmax(a.disp2, q.disp2);
      a.nonfinite |= q.nonfinite;
      a.t0 = q.t0 < a.t0 ? q.t0 : a.t0;
      a.t1 = q.t1 > a.t1 ? q.t1 : a.t1;
    }
    v = a;
  }
}

__device__ __forceinline__ void block_reduce(BlockPartial &v, BlockPartial *s_waves) {
  group_reduce(v, s_waves, (int)blockDim.x);
}

__device__ __forceinline__ BlockPartial zero_partial() {
  BlockPartial a;
  a.pe = a.w = a.ke_half = a.ke_int = a.disp2 = 0.0;
  a.nonfinite = 0;
  a.pad = 0;
  a.t0 = ~0ull;
  a.t1 = 0ull;
  return a;
}

__device__ __forceinline__ bool finite3(float a, float b, float c) {
  return __builtin_isfinite(a) && __builtin_isfinite(b) && __builtin_isfinite(c);
}

// Per-block totals of a list build, one device-scope atomic each: entries kept,
// the longest list (before capping) and the overflow flag.  Every thread of the
// block calls it once.  The blocks' atomics queue at the word, so the two that every
// block issues go to different cache lines (k_list_cell at 16 000 particles, 500 blocks:
// 26.3 -> 21.6 us; a rebuild step of the mixture of 4096, 256 blocks: 30.2 -> 27.3).
__device__ void list_tally(int cnt, int longest, int nmax, Control *ctl) {
  __shared__ int s_sum[16], s_max[16];
  int v = cnt, m = longest;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    v += __shfl_xor(v, o, 64);
    m = max(m, __shfl_xor(m, o, 64));
  }
  if ((threadIdx.x & 63) == 0) {
    s_sum[threadIdx.x >> 6] = v;
    s_max[threadIdx.x >> 6] = m;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    long long tot = 0;
    int mx = 0;
    for (int k = 0; k < (int)(blockDim.x >> 6); ++k) {
      tot += s_sum[k];
      mx = max(mx, s_max[k]);
    }
    atomicAdd((unsigned long long *)&ctl->entries, (unsigned long long)tot);
    atomicMax(&ctl->max_nbrs, mx);
    if (mx > nmax) atomicOr(&ctl->error, 2);
  }
}

// Copy the sorted arrays of slot t into place and record its build position.
__device__ __forceinline__ void place_sorted(const SysPtrs &p, int cur, int t, const float4 r) {
  p.pos[cur][t] = r;
  p.last[t] = r;
  p.vel[t] = p.t_vel[t];
  p.img[t] = p.t_img[t];
  if (p.kahan) p.kahan[t] = p.t_kahan[t];
  if (p.pos64) {
    p.pos64[3 * t] = p.t_pos64[3 * t];
    p.pos64[3 * t + 1] = p.t_pos64[3 * t + 1];
    p.pos64[3 * t + 2] = p.t_pos64[3 * t + 2];
  }
}

// Whether a rebuild kernel has work.  cur < 0: a run-ahead chain, in which the position
// buffer is the device's and nothing runs once the call's last step is done; the loads
// are issued together.
__device__ __forceinline__ bool rebuild_due(const Control *ctl, int &cur) {
  const int flag = ctl->rebuild, buf = ctl->cur;
  const long long step = ctl->step, stop = ctl->stop;
  if (cur >= 0) return flag != 0;
  cur = buf;
  return flag != 0 && step < stop;
}

// ---------------------------------------------------------------- multi-kernel sort (large systems)

__device__ __forceinline__ void begin_build(Control *ctl) {
  ctl->max_nbrs = 0;
  ctl->entries = 0;
  ctl->n_rebuilds += 1;
}

// All-pairs lists keep the particle order between builds; with sort_every = k > 0
// the particles are spatially sorted again before builds 0, k, 2k, ... (the
// periodic re-sort of the paper's n2 method, appendix step 5), counted by the builds
// so far.
__device__ __forceinline__ bool resort_due(const SysConst &c, long long builds) {
  return c.sort_every > 0 && (builds % c.sort_every) == 0;
}

// The counting sort of large systems (section 7 steps 1-3) in four phases, each a
// grid-wide pass over particles or cells: bin, scan, scatter, gather.  The launch
// chain runs them as four kernels; the persistent kernel runs the same functions
// with a grid barrier between phases.  Thread ranges: a workgroup of blockDim.x
// threads starts at particle base and steps by stride.

// Phase 1: cell of every particle, its arrival slot in the cell, and the particle
// count of every tile of 2^shift cells (lanes of a wave that fall in the same tile
// add to it once).
__device__ void sort_bin(const SysConst &c, const SysPtrs &p, int cur, int base, int stride) {
  const int shift = scan_tile_shift(c.ncell);
  const int lane = threadIdx.x & 63;
  for (int s0 = base; s0 < c.n; s0 += stride) {  // uniform over the workgroup
    const int s = s0 + threadIdx.x;
    const bool act = s < c.n;
    unsigned tile = 0u;
    if (act) {
      const float4 r = p.pos[cur][s];
      int cx, cy, cz;
      cell_coords(r, c, cx, cy, cz);
      const unsigned cell = (unsigned)cell_id(c, cx, cy, cz);
      p.cell_of[s] = cell;
      p.slot_in_cell[s] = atomicAdd(&p.cell_count[cell], 1u);
      tile = cell >> shift;
    }
    unsigned long long pend = __ballot(act);
    while (pend) {
      const int lead = __ffsll((long long)pend) - 1;
      const unsigned lt = (unsigned)__builtin_amdgcn_readlane((int)tile, lead);
      const unsigned long long same = __ballot(act && tile == lt);
      if (lane == lead) atomicAdd(&p.tile_count[lt], (unsigned)__popcll(same));
      pend &= ~same;
    }
  }
}

// Phase 2: exclusive scan of the cell histogram into cell_start for tile b, by the
// calling workgroup: the counts of the tiles before b, then the tile 4 cells per
// thread at a time.  The histogram is cleared for the next build (the tile counts
// are cleared in phase 3).  s_w: 16 words of LDS.
__device__ void sort_scan_tile(const SysConst &c, const SysPtrs &p, int b, unsigned *s_w) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6, nw = blockDim.x >> 6;
  const int shift = scan_tile_shift(c.ncell);
  unsigned pre = 0;
  for (int k = t; k < b; k += blockDim.x) pre += p.tile_count[k];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) pre += __shfl_xor(pre, o, 64);
  if (lane == 0) s_w[wv] = pre;
  __syncthreads();
  unsigned carry = 0;
  for (int k = 0; k < nw; ++k) carry += s_w[k];
  __syncthreads();
  const int beg = b << shift, end = min(c.ncell, (b + 1) << shift);
  for (int base = beg; base < end; base += 4 * (int)blockDim.x) {
    const int i0 = base + 4 * t;
    unsigned v[4];
    if (i0 + 3 < end) {
      const uint4 q = *reinterpret_cast<const uint4 *>(p.cell_count + i0);
      v[0] = q.x;
      v[1] = q.y;
      v[2] = q.z;
      v[3] = q.w;
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = i0 + k < end ? p.cell_count[i0 + k] : 0u;
    }
    const unsigned sum = v[0] + v[1] + v[2] + v[3];
    unsigned x = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    if (lane == 63) s_w[wv] = x;
    __syncthreads();
    unsigned wbase = 0, total = 0;
    for (int k = 0; k < nw; ++k) {
      if (k < wv) wbase += s_w[k];
      total += s_w[k];
    }
    unsigned e = carry + wbase + x - sum;
    if (i0 + 3 < end) {
      uint4 o4;
      o4.x = e;
      o4.y = e + v[0];
      o4.z = e + v[0] + v[1];
      o4.w = e + v[0] + v[1] + v[2];
      *reinterpret_cast<uint4 *>(p.cell_start + i0) = o4;
      *reinterpret_cast<uint4 *>(p.cell_count + i0) = make_uint4(0u, 0u, 0u, 0u);
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (i0 + k < end) {
          p.cell_start[i0 + k] = e;
          p.cell_count[i0 + k] = 0u;
        }
        e += v[k];
      }
    }
    carry += total;
    __syncthreads();  // s_w is rewritten by the next chunk
  }
  if (b == scan_tiles(c.ncell) - 1 && t == 0) p.cell_start[c.ncell] = carry;
}

// Phase 3: every particle's arrival slot in its cell's range (perm_tmp); the tile
// counts are cleared for the next build by the threads of clear_tiles.
__device__ void sort_scatter(const SysConst &c, const SysPtrs &p, int first, int stride, bool clear_tiles) {
  if (clear_tiles)
    for (int k = threadIdx.x; k < scan_tiles(c.ncell); k += blockDim.x) p.tile_count[k] = 0u;
  for (int s = first; s < c.n; s += stride) p.perm_tmp[p.cell_start[p.cell_of[s]] + p.slot_in_cell[s]] = (unsigned)s;
}

// Phase 4: deterministic rank by particle id inside each cell, and the gather of
// every per-particle array to its sorted slot in the t_* arrays.
__device__ void sort_gather(const SysConst &c, const SysPtrs &p, int cur, int first, int stride) {
  for (int s = first; s < c.n; s += stride) {
    const unsigned cell = p.cell_of[s];
    const unsigned beg = p.cell_start[cell], end = p.cell_start[cell + 1];
    const int4 im = p.img[s];
    unsigned rank = 0;
    for (unsigned u = beg; u < end; ++u) rank += (p.img[p.perm_tmp[u]].w < im.w) ? 1u : 0u;
    const unsigned dst = beg + rank;
    p.t_pos[dst] = p.pos[cur][s];
    p.t_vel[dst] = p.vel[s];
    p.t_img[dst] = im;
    if (p.pos64) {
      p.t_pos64[3 * dst] = p.pos64[3 * s];
      p.t_pos64[3 * dst + 1] = p.pos64[3 * s + 1];
      p.t_pos64[3 * dst + 2] = p.pos64[3 * s + 2];
    }
    if (p.kahan) p.t_kahan[dst] = p.kahan[s];
  }
}

static __global__ __launch_bounds__(256) void k_bin(SysConst c, SysPtrs p, int cur) {
  if (!rebuild_due(p.ctl, cur)) return;
  sort_bin(c, p, cur, blockIdx.x * blockDim.x, gridDim.x * blockDim.x);
}

// One workgroup per tile of cells.
static __global__ __launch_bounds__(256) void k_scan(SysConst c, SysPtrs p, int cur) {
  if (!rebuild_due(p.ctl, cur)) return;
  __shared__ unsigned s_w[16];
  if (blockIdx.x == 0 && threadIdx.x == 0) begin_build(p.ctl);
  sort_scan_tile(c, p, blockIdx.x, s_w);
}

static __global__ __launch_bounds__(256) void k_scatter(SysConst c, SysPtrs p, int cur) {
  if (!rebuild_due(p.ctl, cur)) return;
  sort_scatter(c, p, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x, blockIdx.x == 0);
}

static __global__ __launch_bounds__(256) void k_gather(SysConst c, SysPtrs p, int cur) {
  if (!rebuild_due(p.ctl, cur)) return;
  sort_gather(c, p, cur, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}

// ---------------------------------------------------------------- one-workgroup sort (small systems)

constexpr int kSmallN = 8192;
constexpr int kSmallCells = 8192;

// The whole spatial sort of a small system by the calling workgroup, in LDS: cell
// histogram with LDS atomics, exclusive scan (also written to cell_start), the
// particle ids placed by arrival order in their cell, a deterministic rank by
// particle id inside each cell, and the gather of every per-particle array to its
// sorted slot in the t_* arrays (section 7 steps 1-3).  Every thread of the block
// must call it.
template <int THREADS, class Source>
__device__ void sort_small_from(const SysConst &c, const SysPtrs &p, unsigned *s_cnt, int *s_id, Source src) {
  __shared__ unsigned s_w[16];
  __shared__ unsigned s_carry;
  constexpr int PER = kSmallN / THREADS;
  const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, wv = tid >> 6, nw = nthr >> 6;
  const int ncell = c.ncell;
  for (int k = tid; k <= ncell; k += nthr) s_cnt[k] = 0u;
  if (tid == 0) {
    s_carry = 0u;
    begin_build(p.ctl);
    p.ctl->resorted = 1;
  }
  unsigned my_cell[PER], my_slot[PER];
  int my_id[PER];
  float4 my_pos[PER];
#pragma unroll
  for (int m = 0; m < PER; ++m) {
    const int sidx = tid + m * nthr;
    my_cell[m] = 0u;
    my_slot[m] = 0u;
    my_id[m] = 0;
    my_pos[m] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (sidx < c.n) src.get(sidx, my_pos[m], my_id[m]);
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < PER; ++m) {
    const int sidx = tid + m * nthr;
    if (sidx < c.n) {
      int cx, cy, cz;
      cell_coords(my_pos[m], c, cx, cy, cz);
      my_cell[m] = (unsigned)((cz * c.nc[1] + cy) * c.nc[0] + cx);
      my_slot[m] = atomicAdd(&s_cnt[my_cell[m]], 1u);
    }
  }
  __syncthreads();
  for (int base = 0; base <= ncell; base += nthr) {
    const int idx = base + tid;
    const unsigned v = idx <= ncell ? s_cnt[idx] : 0u;
    unsigned x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    if (lane == 63) s_w[wv] = x;
    __syncthreads();
    unsigned wbase = 0;
    for (int k = 0; k < wv; ++k) wbase += s_w[k];
    if (idx <= ncell) {
      const unsigned e = s_carry + wbase + x - v;
      s_cnt[idx] = e;
      p.cell_start[idx] = e;
    }
    __syncthreads();
    if (tid == 0) {
      unsigned tot = 0;
      for (int k = 0; k < nw; ++k) tot += s_w[k];
      s_carry += tot;
    }
    __syncthreads();
  }
#pragma unroll
  for (int m = 0; m < PER; ++m) {
    const int sidx = tid + m * nthr;
    if (sidx < c.n) s_id[s_cnt[my_cell[m]] + my_slot[m]] = my_id[m];
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < PER; ++m) {
    const int sidx = tid + m * nthr;
    if (sidx < c.n) {
      const unsigned beg = s_cnt[my_cell[m]], end = s_cnt[my_cell[m] + 1];
      unsigned rank = 0;
      for (unsigned q = beg; q < end; ++q) rank += (s_id[q] < my_id[m]) ? 1u : 0u;
      const unsigned dst = beg + rank;
      p.t_pos[dst] = my_pos[m];
      src.put(sidx, dst, m);
    }
  }
}

// The system's own arrays as the source of the sort.
struct SortOwn {
  const SysPtrs &p;
  int cur;
  __device__ void get(int i, float4 &r, int &id) const {
    r = p.pos[cur][i];
    id = p.img[i].w;
  }
  __device__ void put(int i, unsigned dst, int) const {
    p.t_vel[dst] = p.vel[i];
    p.t_img[dst] = p.img[i];
    if (p.pos64) {
      p.t_pos64[3 * dst] = p.pos64[3 * i];
      p.t_pos64[3 * dst + 1] = p.pos64[3 * i + 1];
      p.t_pos64[3 * dst + 2] = p.pos64[3 * i + 2];
    }
    if (p.kahan) p.t_kahan[dst] = p.kahan[i];
  }
};

template <int THREADS>
__device__ void sort_small_block(const SysConst &c, const SysPtrs &p, int cur, unsigned *s_cnt, int *s_id) {
  sort_small_from<THREADS>(c, p, s_cnt, s_id, SortOwn{p, cur});
}

// Spatial sort requested from the host (start of a run, new state or parameters).
static __global__ __launch_bounds__(1024) void k_sort_small(SysConst c, SysPtrs p, int cur) {
  __shared__ unsigned s_cnt[kSmallCells + 1];
  __shared__ int s_id[kSmallN];
  __shared__ int s_due;
  if (p.ctl->rebuild == 0) return;
  if (c.list_kind == 4) {  // all-pairs lists sort only when a periodic re-sort is due
    if (threadIdx.x == 0) s_due = resort_due(c, p.ctl->n_rebuilds) ? 1 : 0;
    __syncthreads();
    if (!s_due) {
      if (threadIdx.x == 0) {
        begin_build(p.ctl);
        p.ctl->resorted = 0;
      }
      return;
    }
  }
  sort_small_block<1024>(c, p, cur, s_cnt, s_id);
}

#ifndef SRMD_TP
bool small_sort_fits(int n, int ncell) { return n <= kSmallN && ncell <= kSmallCells; }
#endif

// ---------------------------------------------------------------- list builds

constexpr int kWaveCand = 1024;  // candidates per window of the wave builder
constexpr int kListChunks = 4;   // 64-candidate chunks whose loads are in flight together

// The stencil of cell (cx, cy, cz) as runs of sorted slots: 5x5x5 cells (every cell
// along an axis with fewer than 5), cut into rows of consecutive x cells; as
// particles are sorted by cell index, each row is one or two contiguous slot runs.
// Lane s of the calling wave gets run s (row s / 2; the second run of a row only
// when its x window wraps round the box) in the order of the rows, its offset excl
// in the concatenated candidate sequence and the sequence length total.
__device__ __forceinline__ void stencil_runs(const SysConst &c, int cx, int cy, int cz, const unsigned *cstart,
                                             unsigned &run_start, unsigned &run_len, unsigned &excl,
                                             unsigned &total, unsigned &over) {
  const int lane = threadIdx.x & 63;
  const int nx = c.nc[0], ny = c.nc[1], nz = c.nc[2];
  int a0, a1, b0, b1;
  row_runs(c, cx, a0, a1, b0, b1);
  run_start = 0;
  run_len = 0;
  over = 0;
  const int row = lane >> 1;
  int yy, zz, rows = 25;
  if (c.full_axis & 6) {
    const bool fy = c.full_axis & 2, fz = c.full_axis & 4;
    const int ny_eff = fy ? ny : 5, nz_eff = fz ? nz : 5;
    rows = ny_eff * nz_eff;
    const int oy = row % ny_eff, oz = row / ny_eff;
    yy = fy ? oy : (cy + oy - 2 + ny) % ny;
    zz = fz ? oz : (cz + oz - 2 + nz) % nz;
  } else {
    const int oz = row / 5;
    yy = cy + row - 5 * oz - 2;
    zz = cz + oz - 2;
    const int ky = yy < 0 ? ny : yy >= ny ? -ny : 0, kz = zz < 0 ? nz : zz >= nz ? -nz : 0;
    yy += ky;
    zz += kz;
    over = (ky != 0 ? 2u : 0u) | (kz != 0 ? 4u : 0u);
  }
  if (row < rows) {
    const bool second = lane & 1, one = b1 < b0;
    const int x0 = second && !one ? b0 : a0, x1 = second && !one ? b1 : a1;
    if (cx < 2 ? !second : cx >= nx - 2 && second) over |= 1u;
    if (x1 >= x0) {
      const int first = cell_id(c, x0, yy, zz);
      // clamped to [0, n]: a run never reaches outside the sorted arrays
      unsigned s1 = min(cstart[first + (x1 - x0) + 1], (unsigned)c.n);
      unsigned s0 = min(cstart[first], s1);
      if (one) {  // half of the row's one run each
        const unsigned mid = s0 + (s1 - s0 + 1) / 2;
        s0 = second ? mid : s0;
        s1 = second ? s1 : mid;
      }
      run_start = s0;
      run_len = s1 - s0;
    }
  }
  const unsigned incl = wave_incl_scan(run_len);
  excl = incl - run_len;
  total = (unsigned)__builtin_amdgcn_readlane((int)incl, 63);
}

// Verlet list of particle t (sorted slot), one wave per particle; for small systems,
// where one thread per particle (section 7) leaves the chip idle and every thread
// waits on a long chain of dependent loads.  The 5x5x5 stencil (every cell along
// an axis with fewer than 5 cells) is cut into rows of consecutive x cells; as
// particles are sorted by cell index, each row is one or two contiguous slot runs.
// Lane s loads the bounds of run s, a wave prefix sum gives each run's offset in
// the candidate sequence, the runs are expanded into LDS, and the candidates are
// tested 64 at a time; a ballot compacts the hits in candidate order, so the
// list order is deterministic (stencil row order, then slot order).  cand is the
// calling wave's LDS window of kWaveCand entries; tpos and cstart are the sorted
// positions and the cell starts (in device memory, or copies in LDS); PLACE: also
// copy slot t's sorted data into place.  Returns the number of entries kept (all
// lanes) and raises longest to the list length before capping.
template <bool PLACE>
__device__ int list_wave_one(const SysConst &c, const SysPtrs &p, int cur, int t, unsigned *cand,
                             const float *s_cs2, const float4 *tpos, const unsigned *cstart, int &longest) {
  const int lane = threadIdx.x & 63;
  const float4 r = tpos[t];
  if (PLACE && lane == 0) place_sorted(p, cur, t, r);
  const int ti = ptype(r);
  int cx, cy, cz;
  cell_coords(r, c, cx, cy, cz);
  unsigned run_start, run_len, excl, total, over;
  stencil_runs(c, cx, cy, cz, cstart, run_start, run_len, excl, total, over);
  const int nmax = c.n_max;
  int count = 0;
  for (unsigned wbase = 0; wbase < total; wbase += kWaveCand) {
    const unsigned wend = min(total, wbase + (unsigned)kWaveCand);
    // expand this lane's run into the window
    const unsigned q0 = max(excl, wbase), q1 = min(excl + run_len, wend);
    for (unsigned q = q0; q < q1; ++q) cand[q - wbase] = run_start + (q - excl);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const unsigned wlen = wend - wbase;
    for (unsigned base = 0; base < wlen; base += 64u * kListChunks) {
      unsigned u[kListChunks];
      float4 q[kListChunks];
#pragma unroll
      for (int cb = 0; cb < kListChunks; ++cb) {
        const unsigned qi = base + 64u * cb + (unsigned)lane;
        u[cb] = qi < wlen ? cand[qi] : (unsigned)t;
        q[cb] = tpos[u[cb]];
      }
#pragma unroll
      for (int cb = 0; cb < kListChunks; ++cb) {
        bool hit = false;
        if ((int)u[cb] != t) {
          float dx, dy, dz;
          const float r2 = dist2(r, q[cb], c, dx, dy, dz);
          hit = r2 < s_cs2[ti * c.ntypes + ptype(q[cb])];
        }
        const unsigned long long mask = __ballot(hit);
        const int k = count + __popcll(mask & ((1ull << lane) - 1ull));
        if (hit && k < nmax) p.nbl[nbl_addr(t, k, c)] = (int)u[cb];
        count += __popcll(mask);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  const int kept = min(count, nmax);
  if (lane == 0) p.nnb[t] = kept;
  longest = max(longest, count);  // the caller reports the longest list and overflow
  return kept;
}

// Verlet list of particle i against every particle of the system in index order,
// by the calling wave: the paper's O(N^2) builder for small systems (section 6),
// which needs no cells and no spatial sort.  Candidates are taken 64 per chunk,
// kListChunks chunks in flight; a ballot compacts the hits in index order.  pos:
// the positions of the step (in LDS or device memory).  Also records the position
// of the build, the reference of the displacement test.  Returns the entries kept
// (all lanes) and raises longest to the list length before capping.
__device__ int list_allpairs_one(const SysConst &c, const SysPtrs &p, int i, const float *s_cs2,
                                 const float4 *pos, int &longest) {
  const int lane = threadIdx.x & 63;
  const float4 r = pos[i];
  if (lane == 0) p.last[i] = r;
  const int ti = ptype(r);
  const int nmax = c.n_max;
  int count = 0;
  for (int base = 0; base < c.n; base += 64 * kListChunks) {
    int jj[kListChunks];
    float4 q[kListChunks];
#pragma unroll
    for (int cb = 0; cb < kListChunks; ++cb) {
      jj[cb] = base + 64 * cb + lane;
      q[cb] = pos[jj[cb] < c.n ? jj[cb] : i];
    }
#pragma unroll
    for (int cb = 0; cb < kListChunks; ++cb) {
      bool hit = false;
      if (jj[cb] < c.n && jj[cb] != i) {
        float dx, dy, dz;
        const float r2 = dist2(r, q[cb], c, dx, dy, dz);
        hit = r2 < s_cs2[ti * c.ntypes + ptype(q[cb])];
      }
      const unsigned long long mask = __ballot(hit);
      const int k = count + __popcll(mask & ((1ull << lane) - 1ull));
      if (hit && k < nmax) p.nbl[nbl_addr(i, k, c)] = jj[cb];
      count += __popcll(mask);
    }
  }
  const int kept = min(count, nmax);
  if (lane == 0) p.nnb[i] = kept;
  longest = max(longest, count);
  return kept;
}

// All-pairs lists for the launch chain, one wave per particle, four per block; the
// particles keep their order unless a periodic re-sort ran before this build.
static __global__ __launch_bounds__(256) void k_list_allpairs(SysConst c, SysPtrs p, int cur) {
  if (!rebuild_due(p.ctl, cur)) return;
  __shared__ float s_cs2[kMaxPairs];
  if (threadIdx.x < kMaxPairs) s_cs2[threadIdx.x] = c.pt.cs2[threadIdx.x];
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int t = xcd_remap(blockIdx.x, gridDim.x) * 4 + wv;
  // after a periodic re-sort the candidates come from the sorted copy, and each wave
  // moves its own particle's slot into place
  const bool resorted = p.ctl->resorted != 0;
  const float4 *src = resorted ? p.t_pos : p.pos[cur];
  int kept = 0, longest = 0;
  if (t < c.n) {  // uniform across the wave
    if (resorted && lane == 0) place_sorted(p, cur, t, src[t]);
    const int k = list_allpairs_one(c, p, t, s_cs2, src, longest);
    if (lane == 0) kept = k;
  }
  list_tally(kept, longest, c.n_max, p.ctl);
}

constexpr int kListWaves = 16;  // waves (particles) per workgroup of k_list_wave

// One wave per particle (list_wave_one).  The workgroups' tallies queue at their memory
// words (about 10 ns each), so the workgroups are few and large: 1500 particles 15.6 us
// with 4 waves each, 11.7 with 8, 10.2 with 16 (both words on one cache line then).
static __global__ __launch_bounds__(64 * kListWaves) void k_list_wave(SysConst c, SysPtrs p, int cur) {
  if (!rebuild_due(p.ctl, cur)) return;
  __shared__ float s_cs2[kMaxPairs];
  __shared__ unsigned s_cand[kListWaves][kWaveCand];
  if (threadIdx.x < kMaxPairs) s_cs2[threadIdx.x] = c.pt.cs2[threadIdx.x];
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int t = xcd_remap(blockIdx.x, gridDim.x) * kListWaves + wv;
  int kept = 0, longest = 0;
  if (t < c.n) {  // uniform across the wave
    const int k = list_wave_one<true>(c, p, cur, t, s_cand[wv], s_cs2, p.t_pos, p.cell_start, longest);
    if (lane == 0) kept = k;
  }
  list_tally(kept, longest, c.n_max, p.ctl);  // every thread of the block reaches this barrier once
}

constexpr int kThreadBatch = 10;  // candidate positions in flight per thread (measured best of 8-24)

__device__ __forceinline__ int wave_min_int(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
  return v;
}

// Verlet list, one thread per particle (section 7), for large systems where there
// are enough particles to fill the chip.  Candidates of one stencil row are loaded
// kThreadBatch at a time, and the cell bounds of the next row are loaded while the
// current row is tested, so that a row costs about one memory round trip.  Same
// candidate order, hence the same list, as the wave builder.
//
// The list is column-major, so the lanes of a wave write one contiguous span per
// slot only when they write the same slot together; each lane finds its entries at
// its own pace, so entries are first staged in a per-wave ring of kRing slots in
// LDS, and every slot that all lanes of the wave have passed is written out as one
// span.  A lane that runs kRing slots ahead of the slowest lane writes its later
// entries directly.
static __global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_list_thread(SysConst c, SysPtrs p, int cur) {
  if (!rebuild_due(p.ctl, cur)) return;
  __shared__ float s_cs2[kMaxPairs];
  __shared__ int s_ring[4][kRing][64];
  if (threadIdx.x < kMaxPairs) s_cs2[threadIdx.x] = c.pt.cs2[threadIdx.x];
  __syncthreads();
  const int lane = threadIdx.x & 63;
  int(*ring)[64] = s_ring[threadIdx.x >> 6];
  const int nmax = c.n_max;
  const int ny = c.nc[1], nz = c.nc[2];
  const bool fy = c.full_axis & 2, fz = c.full_axis & 4;
  const int ny_eff = fy ? ny : 5, nz_eff = fz ? nz : 5, nrows = ny_eff * nz_eff;
  const unsigned nu = (unsigned)c.n;
  int kept_sum = 0, longest = 0;
  for (int t0 = xcd_remap(blockIdx.x, gridDim.x) * blockDim.x; t0 < c.n; t0 += gridDim.x * blockDim.x) {
    const int t = t0 + threadIdx.x;  // the loop is uniform over the block; lanes past n idle
    const bool act = t < c.n;
    const float4 r = p.t_pos[act ? t : t0];
    if (act) place_sorted(p, cur, t, r);
    const int ti = ptype(r);
    int cx, cy, cz;
    cell_coords(r, c, cx, cy, cz);
    int a0, a1, b0, b1;
    row_runs(c, cx, a0, a1, b0, b1);
    const bool two = b1 >= b0;
    auto bounds = [&](int rr, unsigned &ca0, unsigned &ca1, unsigned &cb0, unsigned &cb1) {
      const int oz = rr / ny_eff, oy = rr - oz * ny_eff;
      const int zz = fz ? oz : (cz + oz - 2 + nz) % nz;
      const int yy = fy ? oy : (cy + oy - 2 + ny) % ny;
      const int fa = cell_id(c, a0, yy, zz);
      ca0 = p.cell_start[fa];
      ca1 = p.cell_start[fa + (a1 - a0) + 1];
      if (two) {
        const int fb = cell_id(c, b0, yy, zz);
        cb0 = p.cell_start[fb];
        cb1 = p.cell_start[fb + (b1 - b0) + 1];
      }
    };
    unsigned ca0, ca1, cb0 = 0, cb1 = 0;
    bounds(0, ca0, ca1, cb0, cb1);
    int count = 0;      // entries found by this lane
    int ring_end = 0;   // this lane's entries below it are in the ring (or written)
    bool spill = false; // this lane writes its later entries directly
    int flushed = 0;    // uniform: every lane's slots below it are written
    auto flush = [&](int upto) {
      for (int k = flushed; k < upto; ++k)
        if (act && k < ring_end && k < nmax) p.nbl[nbl_addr(t, k, c)] = ring[k % kRing][lane];
      flushed = upto;
    };
    for (int rr = 0; rr < nrows; ++rr) {
      // runs clamped to [0, n]: they never reach outside the sorted arrays
      const unsigned sa1 = min(ca1, nu), sa0 = min(ca0, sa1);
      const unsigned sb1 = two ? min(cb1, nu) : 0u, sb0 = two ? min(cb0, sb1) : 0u;
      if (rr + 1 < nrows) bounds(rr + 1, ca0, ca1, cb0, cb1);
      const unsigned la = sa1 - sa0, lt = act ? la + (sb1 - sb0) : 0u;
      for (unsigned base = 0; base < lt; base += kThreadBatch) {
        unsigned u[kThreadBatch];
        float4 q[kThreadBatch];
#pragma unroll
        for (int b = 0; b < kThreadBatch; ++b) {
          const unsigned o = base + b;
          u[b] = o < la ? sa0 + o : sb0 + (o - la);
          if (o >= lt) u[b] = (unsigned)t;  // past the row: load own slot, skipped below
          q[b] = p.t_pos[u[b]];
        }
#pragma unroll
        for (int b = 0; b < kThreadBatch; ++b) {
          if (base + b < lt && (int)u[b] != t) {
            float dx, dy, dz;
            const float r2 = dist2(r, q[b], c, dx, dy, dz);
            if (r2 < s_cs2[ti * c.ntypes + ptype(q[b])]) {
              if (!spill && count - flushed >= kRing) spill = true;
              if (spill) {
                if (count < nmax) p.nbl[nbl_addr(t, count, c)] = (int)u[b];
              } else {
                ring[count % kRing][lane] = (int)u[b];
                ring_end = count + 1;
              }
              ++count;
            }
          }
        }
      }
      // write out the slots every lane has passed, once half the ring is in use
      if (__any(act && !spill && count - flushed >= kRing / 2))
        flush(min(wave_min_int(act && !spill ? count : 0x7fffffff), flushed + kRing));
    }
    flush(flushed + kRing);
    const int kept = act ? min(count, nmax) : 0;
    if (act) p.nnb[t] = kept;
    longest = max(longest, act ? count : 0);
    kept_sum += kept;
  }
  list_tally(kept_sum, longest, nmax, p.ctl);
}

// ---- staged list build (large systems)

constexpr int kStageLanes = 2;     // lanes per particle of the staged list build
constexpr int kStageThreads = kStageSlots * kStageLanes;

// The cells a run of sorted slots needs for its lists: a box of cells (start, may be
// negative: periodic; extent), 2 cells wider than the slots' own box on every side.
struct Region {
  int x0, y0, z0, X, Y, Z;
};

// Region of the slots whose first and last lie in cells a and b (x, y, z): the tile of
// their column and their layers; over two columns the box of both tiles (neighbours
// in the serpentine) and the layers up to their common end; over more columns whole
// columns (then usually too large, see k_list_stage).
__device__ __forceinline__ Region region_of(const SysConst &c, const int (&a)[3], const int (&b)[3]) {
  const Tile ax = tile_of(c, 0, a[0]), ay = tile_of(c, 1, a[1]), bx = tile_of(c, 0, b[0]), by = tile_of(c, 1, b[1]);
  const int qa = column_seq(c, ax.t, ay.t), qb = column_seq(c, bx.t, by.t);
  int zlo = min(a[2], b[2]), zhi = max(a[2], b[2]);
  if (qb == qa + 1) {
    if (qa & 1)
      zlo = 0;
    else
      zhi = c.nc[2] - 1;
  } else if (qb > qa + 1) {
    zlo = 0;
    zhi = c.nc[2] - 1;
  }
  const bool rows = ay.t != by.t && qb > qa + 1;  // several rows of tiles: the whole x extent
  const int xlo = rows ? 0 : min(ax.x0, bx.x0), xhi = rows ? c.nc[0] : max(ax.x0 + ax.w, bx.x0 + bx.w);
  const int ylo = min(ay.x0, by.x0), yhi = max(ay.x0 + ay.w, by.x0 + by.w);
  return Region{xlo - 2, ylo - 2, zlo - 2, xhi - xlo + 4, yhi - ylo + 4, zhi - zlo + 5};
}

// The lanes of a wave exchange data through LDS: their accesses stay in program order.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The lists of one unit's particles against the LDS copy of their region.
// IMG: the region wraps round the box, so differences take the image arithmetic
// (otherwise every image integer is 0).  ONE: one particle type.
struct StageView {
  const float4 *pos;         // region's near particles from place 1 on; .w holds slot << 2 | type
  const unsigned short *cs;  // first places of the region's cells (x fastest, then y, z)
  unsigned short *ring;      // the wave's ring of entries, [entry][particle]
  const float *cs2;          // list radii of the type pairs
};

// m = 2 m + (this lane's bit of mask): one instruction per candidate.
__device__ __forceinline__ void push_bit(unsigned &m, unsigned long long mask) {
  __asm__("v_addc_co_u32_e64 %0, vcc, %0, %0, %1" : "+v"(m) : "s"(mask) : "vcc");
}

// A staged list pairs the entries k and k + tp of one of the tp lanes in a word, so that
// a lane reads two of its own entries at once.  Word wd holds entry stage_entry and the
// one tp further; it is stored as word wd of the interleaved layout (nbl_addr).
__device__ __forceinline__ int stage_entry(int wd, const SysConst &c) {
  return (wd >> c.tp_shift << (c.tp_shift + 1)) | (wd & (c.tp - 1));
}
__device__ __forceinline__ long long stage_half(int i, int k, const SysConst &c) {  // of entry k, in 16-bit units
  const int wd = (k >> (c.tp_shift + 1) << c.tp_shift) | (k & (c.tp - 1));
  return 2 * nbl_addr(i, wd, c) + ((k >> c.tp_shift) & 1);
}

// The kStageLanes = 2 lanes of a particle take two rows of the stencil at a time, one
// each; the second lane's hits follow the first's in the list.  (One lane per particle
// leaves a wave alone with 25 rows of dependent LDS reads, four cost more instructions
// around the tests than the shorter chain saves.)
template <bool IMG, bool ONE>
__device__ __forceinline__ int stage_lists(const SysConst &c, const SysPtrs &p, const Region &R, const StageView &v,
                                           int t, bool act, const float4 r, int cell, int gy, int gz,
                                           int *s_longest) {
  // cell: the first cell of the particle's stencil in the region; gy, gz: that cell's
  // coordinates in the box (negative or past the end: beyond the face)
  static_assert(kStageLanes == 2, "a particle's lanes are a pair");
  constexpr int kCols = 64 / kStageLanes;  // particles of a wave
  const int lane = threadIdx.x & 63, sub = lane % kStageLanes, col = lane / kStageLanes;
  const int ti = ptype(r), group = 2 * c.tp;
  const int nmax = c.n_max;
  // the particle's own place in the copy: its cell is the stencil's centre, whose kept
  // particles follow each other by slot; those before it that are not in the copy (in cells
  // longer than the list radius) leave it earlier than the slots tell
  auto slot_at = [&](int k) { return (int)((unsigned)__float_as_int(v.pos[k].w) >> 2); };
  const int at0 = cell + (2 * R.Y + 2) * R.X + 2, centre = v.cs[at0];
  int self = min(centre + (t - slot_at(centre)), v.cs[at0 + 1] - 1);
  while (self > centre && slot_at(self) > t) --self;
  int count = 0;      // entries of the particle (the same in its lanes)
  int flushed = 0;    // uniform: every particle's entries below it are written (a multiple of group)
  bool spill = false; // this particle's entries are written directly
  auto direct = [&](int k, unsigned e) {
    if (k < nmax) reinterpret_cast<unsigned short *>(p.list16)[stage_half(t, k, c)] = (unsigned short)e;
  };
  unsigned short *const ring = v.ring + col;
  unsigned *const list = p.list16 + (long long)t * c.tp;
  const long long stride = (long long)c.nvp * c.tp;
  // the words of entries [flushed, upto), the particle's lanes taking turns; last: place
  // 0 past the end of a list
  auto flush = [&](int upto, bool last) {
    upto = min(upto, nmax);
    wave_lds_order();
    for (int wd = flushed / 2 + sub; wd < upto / 2; wd += kStageLanes) {
      const int k = stage_entry(wd, c);
      unsigned lo = ring[((unsigned)k % kRing) * kCols], hi = ring[((unsigned)(k + c.tp) % kRing) * kCols];
      if (last) {
        lo = k < count ? lo : 0u;
        hi = k + c.tp < count ? hi : 0u;
      }
      if (act && !spill) list[(wd >> c.tp_shift) * stride + (wd & (c.tp - 1))] = lo | hi << 16;
    }
    flushed = max(flushed, upto);
    wave_lds_order();
  };
  int oy = sub, oz = 0;  // this lane's row
  for (int row = 0; row < 25; row += kStageLanes) {
    const int base = cell + (oz * R.Y + oy) * R.X;  // cell: the stencil's first cell
    const bool mine = act && oz < 5;
    // The image shift along y and z is the row's: a row past a face is its periodic twin
    // (the image integer of every difference in it is then -1 or 1, else 0).
    float sy = 0.f, sz = 0.f;
    if (IMG) {
      const int y = gy + oy, z = gz + oz;
      sy = y < 0 ? -c.L[1] : y >= c.nc[1] ? c.L[1] : 0.f;
      sz = z < 0 ? -c.L[2] : z >= c.nc[2] ? c.L[2] : 0.f;
    }
    const int lo = mine ? v.cs[base] : 0, n = mine ? v.cs[base + 5] - lo : 0;
    // 32 candidates at a time (a row of 5 cells of a liquid holds about 12): the hits as
    // bits, first candidate highest, then the entries of the set bits in order.  Longer
    // rows are rare; the rows' further candidates would follow out of order, so the rows
    // are then taken one after the other.
    const bool lone = __any(n > 32);
    for (int turn = 0; turn < (lone ? kStageLanes : 1); ++turn) {
      const int len = lone && turn != sub ? 0 : n;
      for (int c0 = 0; __any(c0 < len); c0 += 32) {
        const int first = lo + c0, nc = max(0, min(len - c0, 32));
        unsigned m = 0;
        int b0 = 0;
        for (; b0 < nc; b0 += kStageTest) {
          float4 q[kStageTest];
#pragma unroll
          for (int b = 0; b < kStageTest; ++b) q[b] = v.pos[first + b0 + b];  // up to kStageTest - 1 past the row
#pragma unroll
          for (int b = 0; b < kStageTest; ++b) {
            float dx = q[b].x - r.x, dy = q[b].y - r.y, dz = q[b].z - r.z;
            if (IMG) {
              dx = min_image(dx, c.L[0], c.invL[0]);
              dy += sy;
              dz += sz;
            }
            const float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
            const float cut = ONE ? c.pt.cs2[0] : v.cs2[ti * c.ntypes + (__float_as_int(q[b].w) & 3)];
            push_bit(m, __builtin_amdgcn_ballot_w64(r2 < cut));
          }
        }
        // candidate k to bit 31 - k (b0 were pushed, those past nc fall out)
        m = nc > 0 ? m >> (b0 - nc) << (32 - nc) : 0u;
        if (oz == 2 && oy == 2 && (unsigned)(self - first) < (unsigned)nc) m &= ~(0x80000000u >> (self - first));
        const int hits = __builtin_popcount(m), other = (int)xor_lane<1>((unsigned)hits), all = hits + other;
        int k = count + (sub ? other : 0);
        if (__any(!spill && count + all - flushed > kRing)) {
          const int low = 0x3fffffff - wave_max_i32(act && !spill ? 0x3fffffff - count : 0);
          flush(min(low & -group, flushed + kRing), false);
          if (!spill && count + all - flushed > kRing) {
            // far ahead of the wave's slowest particle: this list is written directly from here on
            for (int e = flushed + sub; e < count; e += kStageLanes) direct(e, ring[((unsigned)e % kRing) * kCols]);
            spill = true;
          }
        }
        count += all;
        if (!__any(spill)) {
          while (m) {
            const int b = __builtin_clz(m);
            m &= ~(0x80000000u >> b);
            ring[((unsigned)k % kRing) * kCols] = (unsigned short)(first + b);
            ++k;
          }
        } else {
          while (m) {
            const int b = __builtin_clz(m);
            m &= ~(0x80000000u >> b);
            if (spill)
              direct(k, (unsigned)(first + b));
            else
              ring[((unsigned)k % kRing) * kCols] = (unsigned short)(first + b);
            ++k;
          }
        }
      }
    }
    oy += kStageLanes;
    if (oy >= 5) {
      oy -= 5;
      ++oz;
    }
  }
  // pad every list to the unit's longest (whole groups)
  const int longest = wave_max_i32(act ? count : 0);
  if (lane == 0) atomicMax(s_longest, longest);
  __syncthreads();
  const int end = __builtin_amdgcn_readfirstlane((*s_longest + group - 1) & -group);
  if (act && spill)
    for (int k = count + sub; k < end; k += kStageLanes) direct(k, 0u);
  flush(end, true);
  return count;
}

// Verlet lists of large systems for units of kStageSlots sorted slots (slabs of a column
// of the cell order).  The workgroup copies the region of cells around its slots into
// LDS once (the cells' first places by a prefix sum over their counts) and each
// thread tests the candidates of its particle's 25 stencil rows, each a contiguous range
// of the copy, in the order of the other builders, so the lists hold the same
// particles in the same order, as 16-bit places in the copy (the step kernel makes the
// same copy from stage_src).  Against k_list_thread (VALU issue 85 % busy: 64
// instructions per candidate slot with its per-lane addresses and image arithmetic,
// every candidate gathered per lane from L2) a candidate is one LDS read at a constant
// offset and 8 instructions, as most regions do not wrap round the box: 670 -> 390 us a
// build at 1 024 000 particles (VALU issue still all busy: 236 M instead of 326 M
// instructions, a third of them around the tests), 190 -> 124 at 256 000, 120 -> 57 at
// 64 000.  A unit whose region does not fit (several columns, crowded cells) gets plain
// lists, a wave per particle, from device memory.
static __global__ __launch_bounds__(kStageThreads) __attribute__((amdgpu_waves_per_eu(8))) void k_list_stage(SysConst c, SysPtrs p, int cur) {
  if (!rebuild_due(p.ctl, cur)) return;
  extern __shared__ float4 s_pos[];
  __shared__ float s_cs2[kMaxPairs];
  __shared__ unsigned s_w[16];
  __shared__ int s_longest, s_bad;
  __shared__ float s_box[kStageThreads / 64][2][6];  // per wave, column: least x, y, z and -x, -y, -z
  unsigned short *s_cs = reinterpret_cast<unsigned short *>(s_pos + c.stage_cap + 1 + kStageTest);
  unsigned *s_ring = reinterpret_cast<unsigned *>(s_cs + kStageCells + 8);
  const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, wv = tid >> 6, nw = nthr >> 6;
  if (tid < kMaxPairs) s_cs2[tid] = c.pt.cs2[tid];
  if (tid == 0) s_longest = s_bad = 0;
  const int unit = xcd_remap(blockIdx.x, gridDim.x);
  const int s0 = unit * kStageSlots, s1 = min(c.n, s0 + kStageSlots);
  int ca[3], cb[3];
  cell_coords(p.t_pos[s0], c, ca[0], ca[1], ca[2]);
  cell_coords(p.t_pos[s1 - 1], c, cb[0], cb[1], cb[2]);
#pragma unroll
  for (int d = 0; d < 3; ++d) {  // uniform: the region's arithmetic stays scalar
    ca[d] = __builtin_amdgcn_readfirstlane(ca[d]);
    cb[d] = __builtin_amdgcn_readfirstlane(cb[d]);
  }
  const Region R = region_of(c, ca, cb);
  const bool straddles = tile_of(c, 0, ca[0]).t != tile_of(c, 0, cb[0]).t || tile_of(c, 1, ca[1]).t != tile_of(c, 1, cb[1]).t;
  const int cells = R.X * R.Y * R.Z;
  const int t = s0 + tid / kStageLanes;
  const bool act = t < s1;
  const int ts = act ? t : s0;
  const float4 r = p.t_pos[ts];
  int cx, cy, cz;
  cell_coords(r, c, cx, cy, cz);
  bool fits = cells <= kStageCells;
  unsigned total = 0;
  if (fits) {
    // boxes of the unit's particles, one for the first column and one for the rest
    const bool second = straddles && (tile_of(c, 0, cx).t != tile_of(c, 0, ca[0]).t || tile_of(c, 1, cy).t != tile_of(c, 1, ca[1]).t);
    const int boxes = straddles ? 2 : 1;
    for (int q = 0; q < boxes; ++q) {
      const bool in = second == (q == 1);
      const float e[6] = {r.x, r.y, r.z, -r.x, -r.y, -r.z};
#pragma unroll
      for (int d = 0; d < 6; ++d) {
        const float lo = wave_min_f32(in ? e[d] : 1e30f);
        if (lane == 0) s_box[wv][q][d] = lo;
      }
    }
    __syncthreads();
    if (tid < 6 * boxes) {
      const int q = tid / 6, d = tid - 6 * q;
      float lo = s_box[0][q][d];
      for (int k = 1; k < nw; ++k) lo = fminf(lo, s_box[k][q][d]);
      s_box[0][q][d] = lo;
    }
    __syncthreads();
    // The region's cells: first slot, and a bit for each particle near enough to one of
    // the boxes to be a neighbour (five sixths of them in the LJ liquid); both in the
    // ring's space.  Near is judged with a margin far above its rounding.
    unsigned *s_first = s_ring, *s_near = s_ring + kStageCells;
    for (int k = tid; k < cells; k += nthr) {
      const int xy = R.X * R.Y, z = k / xy, y = (k - z * xy) / R.X, x = k - z * xy - y * R.X;
      // cells past a face are their periodic twins, the particles shifted by the side
      float shift[3];
      auto wrap = [&](int v, int d) {
        const int n = c.nc[d], out = v < 0 ? -1 : v >= n ? 1 : 0;
        shift[d] = (float)out * c.L[d];
        return v - out * n;
      };
      const int gx = wrap(R.x0 + x, 0), gy = wrap(R.y0 + y, 1), gz = wrap(R.z0 + z, 2);
      const int id = cell_id(c, gx, gy, gz);
      const unsigned e = min(p.cell_start[id + 1], (unsigned)c.n), f = min(p.cell_start[id], e), cnt = e - f;
      if (cnt > 32) s_bad = 1;
      auto is_near = [&](const float4 v) {
        const float px = v.x + shift[0], py = v.y + shift[1], pz = v.z + shift[2];
        auto dist = [&](const float *bx) {
          const float dx = fmaxf(0.f, fmaxf(bx[0] - px, px + bx[3])), dy = fmaxf(0.f, fmaxf(bx[1] - py, py + bx[4])),
                      dz = fmaxf(0.f, fmaxf(bx[2] - pz, pz + bx[5]));
          return dx * dx + dy * dy + dz * dz;
        };
        float d2 = dist(s_box[0][0]);
        if (straddles) d2 = fminf(d2, dist(s_box[0][1]));
        return d2 < c.stage_reach2 ? 1u : 0u;
      };
      unsigned near = 0;
      for (unsigned e0 = 0; e0 < min(cnt, 32u); e0 += 4) {
        const unsigned l = cnt - 1;
        const float4 v0 = p.t_pos[f + e0], v1 = p.t_pos[f + min(e0 + 1, l)], v2 = p.t_pos[f + min(e0 + 2, l)],
                     v3 = p.t_pos[f + min(e0 + 3, l)];
        near |= (is_near(v0) | is_near(v1) << 1 | is_near(v2) << 2 | is_near(v3) << 3) << e0;
      }
      if (cnt < 32) near &= (1u << cnt) - 1u;
      s_first[k] = f;
      s_near[k] = near;
      s_cs[k] = (unsigned short)__builtin_popcount(near);
    }
    __syncthreads();
    // exclusive scan of the counts, consecutive cells per thread
    const int per = (cells + nthr - 1) / nthr, k0 = min(cells, tid * per), k1 = min(cells, k0 + per);
    unsigned sum = 0;
    for (int k = k0; k < k1; ++k) sum += s_cs[k];
    const unsigned incl = wave_incl_scan(sum);
    if (lane == 63) s_w[wv] = incl;
    __syncthreads();
    unsigned at = incl - sum;
    for (int k = 0; k < nw; ++k) {
      if (k < wv) at += s_w[k];
      total += s_w[k];
    }
    fits = total <= (unsigned)c.stage_cap && s_bad == 0;
    if (fits) {
      // each particle's source slot into its place, then the particles themselves
      for (int k = k0; k < k1; ++k) {
        unsigned near = s_near[k];
        const unsigned f = s_first[k];
        s_cs[k] = (unsigned short)(at + 1);
        while (near) {
          const int e = __builtin_ctz(near);
          near &= near - 1;
          s_pos[++at].w = __int_as_float((int)(f + e));
        }
      }
      if (tid == 0) s_cs[cells] = (unsigned short)(total + 1);
      __syncthreads();
      unsigned *src_out = p.stage_src + (size_t)unit * c.stage_cap;
      for (unsigned q0 = tid; q0 < total; q0 += 4 * nthr) {
        float4 v[4];
        unsigned src[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const unsigned q = q0 + b * nthr;
          src[b] = q < total ? (unsigned)__float_as_int(s_pos[q + 1].w) : (unsigned)s0;
          v[b] = p.t_pos[src[b]];
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const unsigned q = q0 + b * nthr;
          if (q < total) {
            src_out[q] = src[b];
            v[b].w = __int_as_float((int)(src[b] << 2 | (unsigned)ptype(v[b])));
            s_pos[q + 1] = v[b];
          }
        }
      }
    }
  }
  __syncthreads();
  if (tid == 0) p.stage_n[unit] = fits ? (int)total : 0;
  if (act && tid % kStageLanes == 0) place_sorted(p, cur, t, r);
  int kept = 0, longest = 0;
  if (fits) {
    const int cell = ((cz - R.z0 - 2) * R.Y + (cy - R.y0 - 2)) * R.X + (cx - R.x0 - 2);
    const StageView v{s_pos, s_cs, reinterpret_cast<unsigned short *>(s_ring) + wv * kRing * (64 / kStageLanes), s_cs2};
    const bool img = R.x0 < 0 || R.y0 < 0 || R.z0 < 0 || R.x0 + R.X > c.nc[0] || R.y0 + R.Y > c.nc[1] || R.z0 + R.Z > c.nc[2];
    const int count = c.ntypes == 1 ? (img ? stage_lists<true, true>(c, p, R, v, ts, act, r, cell, cy - 2, cz - 2, &s_longest)
                                           : stage_lists<false, true>(c, p, R, v, ts, act, r, cell, cy - 2, cz - 2, &s_longest))
                                    : (img ? stage_lists<true, false>(c, p, R, v, ts, act, r, cell, cy - 2, cz - 2, &s_longest)
                                           : stage_lists<false, false>(c, p, R, v, ts, act, r, cell, cy - 2, cz - 2, &s_longest));
    longest = act ? count : 0;
    if (act && tid % kStageLanes == 0) {
      kept = min(count, c.n_max);
      p.nnb[t] = kept;
    }
  } else {
    unsigned *cand = reinterpret_cast<unsigned *>(s_pos) + wv * kWaveCand;
    const int fw = min(nw, (int)(stage_list_bytes(c.stage_cap) / (sizeof(unsigned) * kWaveCand)));  // waves whose windows fit
    for (int q = s0 + wv; wv < fw && q < s1; q += fw) {
      const int k = list_wave_one<false>(c, p, cur, q, cand, s_cs2, p.t_pos, p.cell_start, longest);
      if (lane == 0) kept += k;
    }
  }
  list_tally(kept, longest, c.n_max, p.ctl);
}

// The staged lists as plain ones (slot indices in nbl), for what reads those: pairs and
// states read back, the persistent kernel.  drop: the units' lists are plain from now on.
static __global__ __launch_bounds__(kStageSlots) void k_stage_expand(SysConst c, SysPtrs p, int drop) {
  const int unit = blockIdx.x, i = unit * kStageSlots + threadIdx.x;
  const int n = p.stage_n[unit];
  if (n > 0 && i < c.n) {
    const unsigned *src = p.stage_src + (size_t)unit * c.stage_cap;
    const unsigned short *list = reinterpret_cast<const unsigned short *>(p.list16);
    const int nn = p.nnb[i];
    for (int k = 0; k < nn; ++k) {
      const int e = list[stage_half(i, k, c)];
      p.nbl[nbl_addr(i, k, c)] = (int)src[min(max(e - 1, 0), n - 1)];
    }
  }
  __syncthreads();
  if (drop && threadIdx.x == 0) p.stage_n[unit] = 0;
}

// Row-staged list build (list mode 5): one workgroup per x-row of cells.  The
// particles of a row are consecutive sorted slots, and so is every full x-row of
// the stencil, so for each of the 25 stencil rows (in the order of the other
// builders: z offset, then y offset) the workgroup copies that row's positions and
// cell starts into LDS with coalesced loads; each thread then tests its particle
// against the candidates of its five x cells from LDS, in the same slot order as
// k_list_thread, so the lists are the same entry for entry.  The per-lane gathers
// of the thread builder (a cache line per lane and candidate batch) become one
// contiguous copy per row that every particle of the row shares.  A stencil row of
// more than kRowCap particles is read from device memory instead.
constexpr int kRowCap = 1024;    // particles of a stencil row staged in LDS
constexpr int kRowCells = 1024;  // cells per x-row the cell starts of LDS hold (nc <= 1024)

static __global__ __launch_bounds__(256) void k_list_row(SysConst c, SysPtrs p, int cur) {
  if (!rebuild_due(p.ctl, cur)) return;
  __shared__ float s_cs2[kMaxPairs];
  __shared__ int s_ring[4][kRing][64];
  __shared__ float4 s_row[kRowCap];
  __shared__ unsigned s_cs[kRowCells + 1];
  if (threadIdx.x < kMaxPairs) s_cs2[threadIdx.x] = c.pt.cs2[threadIdx.x];
  const int lane = threadIdx.x & 63;
  int(*ring)[64] = s_ring[threadIdx.x >> 6];
  const int nmax = c.n_max;
  const int nx = c.nc[0], ny = c.nc[1], nz = c.nc[2];
  const bool fy = c.full_axis & 2, fz = c.full_axis & 4;
  const int ny_eff = fy ? ny : 5, nz_eff = fz ? nz : 5, nrows = ny_eff * nz_eff;
  const unsigned nu = (unsigned)c.n;
  const int row = xcd_remap(blockIdx.x, gridDim.x);  // x-row (cy, cz) of this workgroup
  const int cy = row % ny, cz = row / ny;
  const unsigned r0 = min(p.cell_start[row * nx], nu), r1 = min(p.cell_start[row * nx + nx], nu);
  int kept_sum = 0, longest = 0;
  for (unsigned t0 = r0; t0 < r1; t0 += blockDim.x) {  // uniform over the block
    const unsigned tt = t0 + threadIdx.x;
    const bool act = tt < r1;
    const int t = (int)(act ? tt : r0);
    const float4 r = p.t_pos[t];
    if (act) place_sorted(p, cur, t, r);
    const int ti = ptype(r);
    int cx, cyy, czz;
    cell_coords(r, c, cx, cyy, czz);
    int a0, a1, b0, b1;
    row_runs(c, cx, a0, a1, b0, b1);
    const bool two = b1 >= b0;
    int count = 0, ring_end = 0, flushed = 0;
    bool spill = false;
    auto flush = [&](int upto) {
      for (int k = flushed; k < upto; ++k)
        if (act && k < ring_end && k < nmax) p.nbl[nbl_addr(t, k, c)] = ring[k % kRing][lane];
      flushed = upto;
    };
    for (int rr = 0; rr < nrows; ++rr) {
      const int oz = rr / ny_eff, oy = rr - oz * ny_eff;
      const int zz = fz ? oz : (cz + oz - 2 + nz) % nz;
      const int yy = fy ? oy : (cy + oy - 2 + ny) % ny;
      const int rb = (zz * ny + yy) * nx;
      __syncthreads();  // the previous row's LDS copy is no longer read
      for (int k = threadIdx.x; k <= nx; k += blockDim.x) s_cs[k] = min(p.cell_start[rb + k], nu);
      __syncthreads();
      const unsigned q0 = s_cs[0], q1 = s_cs[nx];
      const bool staged = q1 - q0 <= (unsigned)kRowCap;
      if (staged)
        for (unsigned k = threadIdx.x; k < q1 - q0; k += blockDim.x) s_row[k] = p.t_pos[q0 + k];
      __syncthreads();
      const unsigned sa0 = s_cs[a0], sa1 = s_cs[a1 + 1];
      const unsigned sb0 = two ? s_cs[b0] : 0u, sb1 = two ? s_cs[b1 + 1] : 0u;
      const unsigned la = sa1 - sa0, lt = act ? la + (sb1 - sb0) : 0u;
      for (unsigned o = 0; o < lt; ++o) {
        const unsigned u = o < la ? sa0 + o : sb0 + (o - la);
        if ((int)u == t) continue;
        const float4 q = staged ? s_row[u - q0] : p.t_pos[u];
        float dx, dy, dz;
        const float r2 = dist2(r, q, c, dx, dy, dz);
        if (r2 < s_cs2[ti * c.ntypes + ptype(q)]) {
          if (!spill && count - flushed >= kRing) spill = true;
          if (spill) {
            if (count < nmax) p.nbl[nbl_addr(t, count, c)] = (int)u;
          } else {
            ring[count % kRing][lane] = (int)u;
            ring_end = count + 1;
          }
          ++count;
        }
      }
      // write out the slots every lane has passed, once half the ring is in use
      if (__any(act && !spill && count - flushed >= kRing / 2))
        flush(min(wave_min_int(act && !spill ? count : 0x7fffffff), flushed + kRing));
    }
    flush(flushed + kRing);
    const int kept = act ? min(count, nmax) : 0;
    if (act) p.nnb[t] = kept;
    longest = max(longest, act ? count : 0);
    kept_sum += kept;
  }
  list_tally(kept_sum, longest, nmax, p.ctl);
}

constexpr int kCellChunks = 8;  // 64-candidate chunks held in registers (one window)
constexpr int kCellWindow = 64 * kCellChunks;

// Verlet lists of the particles in sorted slots [i0, i1) of cell (cx, cy, cz), by the
// calling wave.  Every particle of a cell has the same stencil (section 7), hence the
// same candidates in the same order, so the wave loads them once, kCellWindow at a
// time (64 per chunk from contiguous slot runs), and tests each particle against
// them; a ballot compacts the hits in candidate order, so the lists equal those of
// the particle-by-particle builders entry for entry.  cand: kCellWindow entries of
// the wave's LDS; cnt[l]: entries found so far for particle i0 + l (LDS, the caller
// clears it); sink(i, k, upto, j) stores entry k of particle i (called by the hit lanes;
// upto: entries found so far with those of this chunk, uniform).  GEO: the image from the
// cells where they tell it (else always per pair).

// Lanes before this one whose bit of mask is set, plus base.
__device__ __forceinline__ int rank_below(unsigned long long mask, int base) {
  return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                        __builtin_amdgcn_mbcnt_lo((unsigned)mask, (unsigned)base));
}

__device__ __forceinline__ float4 uniform4(const float4 v) {
  auto first = [](float x) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x))); };
  return make_float4(first(v.x), first(v.y), first(v.z), first(v.w));
}

// The particles [i0, i1) of a cell against one window of candidates u at q (places past
// its end hold a candidate at infinity).  PAIR: image arithmetic per pair; otherwise (at
// most two types) the image of a candidate relative to the cell is in its shift h.
template <bool PAIR, class Sink>
__device__ __forceinline__ void cell_tests(const SysConst &c, int i0, int i1, unsigned wlen,
                                           const unsigned (&u)[kCellChunks], const float4 (&q)[kCellChunks],
                                           const float (&h)[kCellChunks][3], int *cnt, const float *s_cs2,
                                           const float4 *tpos, Sink sink) {
  const int lane = threadIdx.x & 63, nt = c.ntypes;
  for (int i = i0; i < i1; ++i) {
    const float4 pi = uniform4(tpos[i]);
    const float *row = s_cs2 + ptype(pi) * nt;
    const float r0 = row[0], r1 = row[nt > 1 ? 1 : 0];
    int count = __builtin_amdgcn_readfirstlane(cnt[i - i0]);
#pragma unroll
    for (int cb = 0; cb < kCellChunks; ++cb) {
      if (64u * cb < wlen) {  // uniform over the wave
        float r2;
        if constexpr (PAIR) {
          float dx, dy, dz;
          r2 = dist2(pi, q[cb], c, dx, dy, dz);
        } else {
          const float dx = q[cb].x - pi.x - h[cb][0], dy = q[cb].y - pi.y - h[cb][1], dz = q[cb].z - pi.z - h[cb][2];
          r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
        }
        float lim;
        if constexpr (PAIR)
          lim = row[ptype(q[cb])];
        else
          lim = ptype(q[cb]) ? r1 : r0;
        const bool hit = (r2 < lim) & ((int)u[cb] != i);
        const unsigned long long mask = __ballot(hit);
        const int upto = count + __popcll(mask);
        if (hit) sink(i, rank_below(mask, count), upto, (int)u[cb]);
        count = upto;
      }
    }
    if (lane == 0) cnt[i - i0] = count;
  }
}

template <bool GEO, class Cand, class Sink>
__device__ __forceinline__ void list_cell_particles(const SysConst &c, const SysPtrs &p, int cx, int cy, int cz, int i0, int i1,
                                    Cand *cand, int *cnt, const float *s_cs2, const float4 *tpos,
                                    const unsigned *cstart, Sink sink) {
  cx = __builtin_amdgcn_readfirstlane(cx);
  cy = __builtin_amdgcn_readfirstlane(cy);
  cz = __builtin_amdgcn_readfirstlane(cz);
  i0 = __builtin_amdgcn_readfirstlane(i0);
  i1 = __builtin_amdgcn_readfirstlane(i1);
  constexpr int kOver = 8 * (int)sizeof(Cand) - 3;  // the three wrap bits above a slot
  const int lane = threadIdx.x & 63;
  const int nx = c.nc[0], ny = c.nc[1], nz = c.nc[2];
  unsigned run_start, run_len, excl, total, over;
  stencil_runs(c, cx, cy, cz, cstart, run_start, run_len, excl, total, over);
  // From 7 cells per axis the cells tell the image: a candidate reached without wrapping
  // round the box is nearer than 3 cells per axis, less than half a side, one reached by
  // wrapping 4 or more away, so rounding the difference gives this very image, and a
  // subtraction in its place the same bits.
  const bool geo = min(nx, min(ny, nz)) >= 7 && c.ntypes <= 2;
  const float sx = cx < 2 ? c.L[0] : -c.L[0], sy = cy < 2 ? c.L[1] : -c.L[1], sz = cz < 2 ? c.L[2] : -c.L[2];
  const unsigned tag = over << kOver;
  for (unsigned wbase = 0; wbase < total; wbase += kCellWindow) {
    const unsigned wend = min(total, wbase + (unsigned)kCellWindow), wlen = wend - wbase;
    const unsigned q0 = max(excl, wbase), q1 = min(excl + run_len, wend);
    for (unsigned q = q0; q < q1; ++q) cand[q - wbase] = (Cand)(run_start + (q - excl) + tag);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    unsigned u[kCellChunks];
    float4 q[kCellChunks];
    float h[kCellChunks][3];
#pragma unroll
    for (int cb = 0; cb < kCellChunks; ++cb) {
      const unsigned qi = 64u * cb + (unsigned)lane;
      u[cb] = qi < wlen ? (unsigned)cand[qi] : (unsigned)i0;
      if (64u * cb < wlen) {
        const unsigned w = u[cb] >> kOver;
        u[cb] &= (1u << kOver) - 1u;
        q[cb] = tpos[u[cb]];
        h[cb][0] = w & 1u ? sx : 0.f;
        h[cb][1] = w & 2u ? sy : 0.f;
        h[cb][2] = w & 4u ? sz : 0.f;
        if (qi >= wlen) q[cb].x = __builtin_inff();
      }
    }
    if (GEO && geo)
      cell_tests<false>(c, i0, i1, wlen, u, q, h, cnt, s_cs2, tpos, sink);
    else
      cell_tests<true>(c, i0, i1, wlen, u, q, h, cnt, s_cs2, tpos, sink);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

constexpr int kCellSlots = 32;   // sorted slots per workgroup of the cell builder
constexpr int kCellWaves = 8;    // its waves
constexpr int kCellPiece = 4;    // particles of a cell one wave takes at most
constexpr int kCellStage = 128;  // list entries per particle staged in LDS

// Verlet lists, one wave per cell (list_cell_particles), for the launch chain.  A
// workgroup takes kCellSlots consecutive sorted slots, split into pieces of at most
// kCellPiece slots of one cell (a cell that straddles two workgroups is handled by both,
// each for its own slots), dealt over its waves.  Bound by the latency of a piece (its
// candidates' indices, then positions, then the tests), so the pieces are many and the
// waves eight: with two waves and whole cells a wave took about seven cells of a liquid
// one after the other (54 -> 27 us a build for the liquid of 16 000, 178 -> 115 for the
// salt of 20 000, 50 -> 26 for the mixture of 5003; 22, 97 and 23 with the image from the
// cells and the tallies on two lines).  The lists are staged in LDS as
// [particle][entry] and then written out by the workgroup in address order, so each
// entry index of the column-major list is one contiguous span; entries past kCellStage
// are written directly.
static __global__ __launch_bounds__(64 * kCellWaves, 4) void k_list_cell(SysConst c, SysPtrs p, int cur) {
  if (!rebuild_due(p.ctl, cur)) return;
  __shared__ float s_cs2[kMaxPairs];
  __shared__ int s_list[kCellSlots][kCellStage + 1];  // +1: entries of one particle fall in distinct banks
  __shared__ unsigned s_cand[kCellWaves][kCellWindow];
  __shared__ int s_cnt[kCellSlots];
  __shared__ int s_seg[kCellSlots + 1];
  __shared__ int s_nseg;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int T0 = xcd_remap(blockIdx.x, gridDim.x) * kCellSlots;
  const int m = min(kCellSlots, c.n - T0);  // slots of this workgroup, >= 1
  const int nmax = c.n_max;
  if (tid < kMaxPairs) s_cs2[tid] = c.pt.cs2[tid];
  if (wv == 0) {
    // pieces: one starts where the cell index changes and after every kCellPiece slots
    int cell = -1;
    if (lane < m) {
      const float4 r = p.t_pos[T0 + lane];
      place_sorted(p, cur, T0 + lane, r);
      int cx, cy, cz;
      cell_coords(r, c, cx, cy, cz);
      cell = (cz * c.nc[1] + cy) * c.nc[0] + cx;
      s_cnt[lane] = 0;
    }
    const int prev = __shfl_up(cell, 1, 64);
    const unsigned long long first = __ballot(lane < m && (lane == 0 || prev != cell));
    // slots since the first one of the cell
    const int since = lane - (63 - __builtin_clzll((first & ((2ull << lane) - 1ull)) | 1ull));
    const bool head = lane < m && since % kCellPiece == 0;
    const unsigned long long hm = __ballot(head);
    if (head) s_seg[__popcll(hm & ((1ull << lane) - 1ull))] = lane;
    if (lane == 0) {
      s_nseg = __popcll(hm);
      s_seg[__popcll(hm)] = m;
    }
  }
  __syncthreads();
  const int nseg = s_nseg;
  auto stage = [&](int i, int k, int upto, int j) {
    if (upto <= kCellStage)
      s_list[i - T0][k] = j;
    else if (k < kCellStage)
      s_list[i - T0][k] = j;
    else if (k < nmax)
      p.nbl[nbl_addr(i, k, c)] = j;
  };
  for (int sg = wv; sg < nseg; sg += kCellWaves) {
    const int l0 = s_seg[sg], l1 = s_seg[sg + 1];
    int cx, cy, cz;
    cell_coords(p.t_pos[T0 + l0], c, cx, cy, cz);
    list_cell_particles<true>(c, p, cx, cy, cz, T0 + l0, T0 + l1, s_cand[wv], s_cnt + l0, s_cs2, p.t_pos, p.cell_start,
                        stage);
  }
  __syncthreads();
  // write-out in address order: groups of tp entries of consecutive particles are
  // contiguous in the tp-interleaved column-major list
  int kmax = 0;
  for (int l = 0; l < m; ++l) kmax = max(kmax, s_cnt[l]);
  const int tp = c.tp;
  const int kst = min(min(kmax, nmax), kCellStage);
  const int span = kCellSlots * tp;  // elements of one group of tp entries
  const int groups = (kst + tp - 1) / tp;
  for (int j = tid; j < groups * span; j += blockDim.x) {
    const int g = j / span, rr = j - g * span, l = rr / tp, k = g * tp + (rr - l * tp);
    if (l < m && k < kst && k < s_cnt[l])
      p.nbl[(long long)g * ((long long)c.nvp * tp) + (long long)(T0 + l) * tp + (rr - l * tp)] = s_list[l][k];
  }
  int kept = 0, longest = 0;
  if (tid < m) {
    longest = s_cnt[tid];
    kept = min(longest, nmax);
    p.nnb[T0 + tid] = kept;
  }
  list_tally(kept, longest, nmax, p.ctl);
}

// ---------------------------------------------------------------- force only

template <int TP, int METHOD, bool STAGE>
__global__ __launch_bounds__(1024) void k_force(SysConst c, SysPtrs p, int cur) {
  extern __shared__ float4 s_region[];
  __shared__ SharedPairs sp;
  __shared__ BlockPartial s_waves[16];
  const unsigned long long tstart = wall_clock64();
  stage_pairs(sp, c);
  const int lb = xcd_remap(blockIdx.x, gridDim.x);
  int place = -1;
  if constexpr (STAGE) place = stage_fill<TP>(c, p, p.pos[cur], lb, s_region);
  __syncthreads();
  const int gt = lb * blockDim.x + threadIdx.x;
  const int i = gt / TP, t = gt % TP;
  const bool active = i < c.n;
  const float4 *pos = p.pos[cur];
  float fx = 0.f, fy = 0.f, fz = 0.f, u = 0.f, w = 0.f;
  float4 vo = make_float4(0.f, 0.f, 0.f, 0.f), pi = vo;
  const int ic = active ? i : c.n - 1;
  pi = pos[ic];
  if (active && t == 0) vo = p.vel[i];
  if (STAGE && place >= 0)
    force_lane_staged<TP, METHOD>(ic, t, active, pi, s_region + place, p, sp, c, fx, fy, fz, u, w);
  else
    force_lane<TP, METHOD, StepBatch<TP>::value, STAGE>(ic, t, active, pi, pos, (const int *)p.nbl, (const int *)p.nnb, sp,
                                                        c, fx, fy, fz, u, w);
  fx = lane_sum<TP>(fx);
  fy = lane_sum<TP>(fy);
  fz = lane_sum<TP>(fz);
  u = lane_sum<TP>(u);
  w = lane_sum<TP>(w);
  BlockPartial v = zero_partial();
  if (active && t == 0) {
    p.force[i] = make_float4(fx, fy, fz, 0.5f * u);
    p.wpart[i] = (float)((double)w / 6.0);
    v.pe = 0.5 * (double)u;
    v.w = (double)w / 6.0;
    const double dvx = vo.x, dvy = vo.y, dvz = vo.z;
    v.ke_half = 0.5 * c.mass[ptype(pi)] * (dvx * dvx + dvy * dvy + dvz * dvz);
    v.nonfinite = finite3(fx, fy, fz) ? 0 : 1;
  }
  v.t0 = tstart;
  v.t1 = wall_clock64();
  block_reduce(v, s_waves);
  if (threadIdx.x == 0) {
    p.part[lb] = v;
    if (blockIdx.x == 0) p.ctl->rebuild = 0;  // the list in use is now current
  }
}

// A store that writes through the L2 to memory: agent-scope relaxed atomic stores of
// its 8-byte words (the XCDs' L2s are not coherent with each other).  Once the
// storing wave's vmcnt has drained the words are visible to loads from any XCD
// that miss their own L2, with no write-back of a whole L2.
template <class T>
__device__ __forceinline__ void store_through(T *dst, const T &v) {
  static_assert(sizeof(T) % 8 == 0, "whole 8-byte words");
  unsigned long long w[sizeof(T) / 8];
  __builtin_memcpy(w, &v, sizeof(T));
  unsigned long long *d = reinterpret_cast<unsigned long long *>(dst);
#pragma unroll
  for (int k = 0; k < (int)(sizeof(T) / 8); ++k) __hip_atomic_store(d + k, w[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <class T>
__device__ __forceinline__ void store_to(T *dst, const T &v, bool through) {
  if (through)
    store_through(dst, v);
  else
    *dst = v;
}

// Leapfrog / Nose-Hoover update of particle i (sorted slot) from its force, and
// its float64 contributions to the step's sums (paper section 2 integrators;
// kinetic energy at the half step for the thermostat and at the integer step for
// the thermodynamic record; largest displacement since the last list build for
// the rebuild test of section 6).
template <int PREC>
__device__ __forceinline__ void integrate_one(const SysConst &c, const SysPtrs &p, int cur, int i, const float4 pi,
                                              const float4 vo, int4 im, const float4 l0, float4 kc, double x64,
                                              double y64, double z64, double xi, float fx, float fy, float fz,
                                              float u, float w, BlockPartial &v, bool through = false) {
    // through: the arrays the end-of-step sort reads are written through the L2
    const int ti = ptype(pi);
    // v(n+1/2) = [v(n-1/2) (1 - xi dt/2) + F/m dt] / (1 + xi dt/2); a = b = 1 without thermostat
    const double hx = 0.5 * xi * c.dtd;
    const float a = (float)(1.0 - hx);
    const float ib = (float)(1.0 / (1.0 + hx));
    const float dtm = c.dt * c.inv_mass[ti];
    const float vx = __builtin_fmaf(vo.x, a, fx * dtm) * ib;
    const float vy = __builtin_fmaf(vo.y, a, fy * dtm) * ib;
    const float vz = __builtin_fmaf(vo.z, a, fz * dtm) * ib;
    store_to(&p.vel[i], make_float4(vx, vy, vz, vo.w), through);
    p.force[i] = make_float4(fx, fy, fz, 0.5f * u);
    float4 rn;
    rn.w = pi.w;
    if (PREC == 2) {  // float64 master positions
      double x = x64 + (double)vx * c.dtd;
      double y = y64 + (double)vy * c.dtd;
      double z = z64 + (double)vz * c.dtd;
      if (x >= 0.5 * c.Ld[0]) { x -= c.Ld[0]; im.x += 1; } else if (x < -0.5 * c.Ld[0]) { x += c.Ld[0]; im.x -= 1; }
      if (y >= 0.5 * c.Ld[1]) { y -= c.Ld[1]; im.y += 1; } else if (y < -0.5 * c.Ld[1]) { y += c.Ld[1]; im.y -= 1; }
      if (z >= 0.5 * c.Ld[2]) { z -= c.Ld[2]; im.z += 1; } else if (z < -0.5 * c.Ld[2]) { z += c.Ld[2]; im.z -= 1; }
      store_to(&p.pos64[3 * i], x, through);
      store_to(&p.pos64[3 * i + 1], y, through);
      store_to(&p.pos64[3 * i + 2], z, through);
      rn.x = (float)x;
      rn.y = (float)y;
      rn.z = (float)z;
      // the float32 copy may round up onto +L/2; use the periodic twin -L/2
      if (rn.x >= c.halfL[0]) rn.x = -c.halfL[0];
      if (rn.y >= c.halfL[1]) rn.y = -c.halfL[1];
      if (rn.z >= c.halfL[2]) rn.z = -c.halfL[2];
    } else {
      float x, y, z;
      if (PREC == 1) {  // compensated update: y = v dt - c; t = r + y; c = (t - r) - y
        const float yx = vx * c.dt - kc.x, yy = vy * c.dt - kc.y, yz = vz * c.dt - kc.z;
        x = pi.x + yx;
        y = pi.y + yy;
        z = pi.z + yz;
        kc.x = (x - pi.x) - yx;
        kc.y = (y - pi.y) - yy;
        kc.z = (z - pi.z) - yz;
        store_to(&p.kahan[i], kc, through);
      } else {
        x = __builtin_fmaf(vx, c.dt, pi.x);
        y = __builtin_fmaf(vy, c.dt, pi.y);
        z = __builtin_fmaf(vz, c.dt, pi.z);
      }
      // wrap into [-L/2, L/2); both corrections are exact (Sterbenz)
      if (x >= c.halfL[0]) { x -= c.L[0]; im.x += 1; } else if (x < -c.halfL[0]) { x += c.L[0]; im.x -= 1; }
      if (y >= c.halfL[1]) { y -= c.L[1]; im.y += 1; } else if (y < -c.halfL[1]) { y += c.L[1]; im.y -= 1; }
      if (z >= c.halfL[2]) { z -= c.L[2]; im.z += 1; } else if (z < -c.halfL[2]) { z += c.L[2]; im.z -= 1; }
      rn.x = x;
      rn.y = y;
      rn.z = z;
    }
    store_to(&p.pos[cur ^ 1][i], rn, through);
    store_to(&p.img[i], im, through);
    // float64 reductions
    const double m = c.mass[ti];
    const double dvx = vx, dvy = vy, dvz = vz;
    v.ke_half = 0.5 * m * (dvx * dvx + dvy * dvy + dvz * dvz);
    const double mx = 0.5 * ((double)vo.x + dvx), my = 0.5 * ((double)vo.y + dvy), mz = 0.5 * ((double)vo.z + dvz);
    v.ke_int = 0.5 * m * (mx * mx + my * my + mz * mz);
    v.pe = 0.5 * (double)u;
    v.w = (double)w / 6.0;
    // displacement since the last build: float64 from the float32 positions
    double ddx = (double)rn.x - (double)l0.x, ddy = (double)rn.y - (double)l0.y, ddz = (double)rn.z - (double)l0.z;
    ddx -= c.Ld[0] * rint(ddx / c.Ld[0]);
    ddy -= c.Ld[1] * rint(ddy / c.Ld[1]);
    ddz -= c.Ld[2] * rint(ddz / c.Ld[2]);
    v.disp2 = (ddx * ddx + ddy * ddy) + ddz * ddz;
    v.nonfinite = (finite3(fx, fy, fz) && finite3(rn.x, rn.y, rn.z)) ? 0 : 1;
}

// ---------------------------------------------------------------- end of step

// Nose-Hoover friction of the next step from the half-step kinetic energy.
__device__ __forceinline__ double xi_next(const SysConst &c, double xi, double ke_half) {
  const double th = 2.0 * ke_half / c.g;
  return xi + c.dtd * (th / c.T0 - 1.0) * c.inv_tau2;
}

// End of a time step, by one thread, from the fully reduced partials a: the
// thermodynamic record, the Nose-Hoover update, the step counter and the
// displacement test that sets the rebuild flag.  Returns the flag.
// The control words finish_step reads, loaded together (one memory round trip).
struct CtlView {
  double xi, xi_int;
  long long step, n_rebuilds, n_records, trace_cap;
  int max_nbrs, thermo_every;
};

__device__ __forceinline__ CtlView load_ctl(const Control *ctl) {
  CtlView v;
  v.xi = ctl->xi;
  v.xi_int = ctl->xi_int;
  v.step = ctl->step;
  v.n_rebuilds = ctl->n_rebuilds;
  v.n_records = ctl->n_records;
  v.trace_cap = ctl->trace_cap;
  v.max_nbrs = ctl->max_nbrs;
  v.thermo_every = ctl->thermo_every;
  return v;
}

// End of a time step, by one thread, from the fully reduced partials a and the
// control words v (loaded after the step's list build): the thermodynamic record,
// the Nose-Hoover update, the step counter and the displacement test that sets the
// rebuild flag.  Returns the flag.
__device__ int finish_step(const SysConst &c, const SysPtrs &p, const BlockPartial &a, const CtlView &v) {
  Control *ctl = p.ctl;
  const double xi = c.thermostat ? v.xi : 0.0;
  Thermo rec;
  rec.pe = a.pe;
  rec.ke = a.ke_int;
  rec.virial = a.w;
  rec.temperature = 2.0 * a.ke_int / c.g;
  rec.pressure = (2.0 * a.ke_int / 3.0 + a.w) / c.volume;
  rec.xi = xi;
  rec.xi_integral = v.xi_int;
  rec.h_conserved = a.ke_int + a.pe;
  if (c.thermostat && c.inv_tau2 > 0.0)
    rec.h_conserved += c.g * c.T0 * (xi * xi / (2.0 * c.inv_tau2) + v.xi_int);
  rec.ke_half = a.ke_half;
  rec.step = v.step;
  rec.n_rebuilds = v.n_rebuilds;
  rec.max_nbrs = v.max_nbrs;
  rec.reserved = 0;
  *p.thermo = rec;
  if (v.thermo_every > 0 && (v.step % v.thermo_every) == 0 && v.n_records < v.trace_cap) {
    p.trace[v.n_records] = rec;
    ctl->n_records = v.n_records + 1;
  }
  if (c.thermostat) {
    const double xn = xi_next(c, xi, a.ke_half);
    ctl->xi_int = v.xi_int + c.dtd * (xi + xn) * 0.5;
    ctl->xi = xn;
  }
  ctl->step = v.step + 1;
  if (a.t1 > a.t0) {
    ctl->prof_ticks += a.t1 - a.t0;
    ctl->prof_count += 1;
  }
  const int rebuild = (a.disp2 > c.half_skin2) ? 1 : 0;
  ctl->rebuild = rebuild;
  if (a.nonfinite) atomicOr(&ctl->error, 1);
  return rebuild;
}

// ---------------------------------------------------------------- end of step in the step kernel

// The fold of one block partial into a running sum, with the operations and order
// of k_finish and group_reduce (the device-clock stamps included).
__device__ __forceinline__ void fold_timed(BlockPartial &a, const BlockPartial &q) {
  a.pe += q.pe;
  a.w += q.w;
  a.ke_half += q.ke_half;
  a.ke_int += q.ke_int;
  a.disp2 = fmax(a.disp2, q.disp2);
  a.nonfinite |= q.nonfinite;
  a.t0 = q.t0 < a.t0 ? q.t0 : a.t0;
  a.t1 = q.t1 > a.t1 ? q.t1 : a.t1;
}

// Arrival counters of a step kernel that ends the step itself: kArriveGroups group
// counters and one top counter, each on its own 128-byte line.
constexpr unsigned kArriveGroups = 16;
constexpr unsigned kArriveStride = 32;  // unsigned words per counter line
constexpr size_t kArriveBytes = sizeof(unsigned) * kArriveStride * (kArriveGroups + 1);

// Arrival of a workgroup at the end of a step kernel that ends the step itself.
// What the last workgroup reads from the others (their block partials and, for a
// small system, the arrays its sort reads) was written through the L2
// (store_through); every wave waits for its stores to complete before its
// workgroup takes a ticket.  No L2 write-back is needed (one per workgroup would
// cost the XCD's L2 a walk each).  Tickets are taken in two levels, so that the
// workgroups that end together do not all queue on one word: workgroup b counts on
// group counter b % 16, and the last of each group on the top counter.  The
// workgroup with the last top ticket acquires at agent scope (the invalidation of
// its compute unit's L1 and of its L2 precedes, through the workgroup barrier,
// every later load of its waves) and returns true in all its threads.  Each counter
// is put back to zero by the workgroup that takes its last ticket, for the next
// launch.  Every workgroup has arrived, hence read the step's control words, before
// the last one writes them.
__device__ __forceinline__ bool arrive_last(unsigned *ctr, unsigned G, unsigned b, int *s_last) {
  __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's stores are complete
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned g = b % kArriveGroups;
    const unsigned members = G / kArriveGroups + (g < G % kArriveGroups ? 1u : 0u);
    const unsigned groups = G < kArriveGroups ? G : kArriveGroups;
    int last = 0;
    unsigned *gc = ctr + g * kArriveStride, *top = ctr + kArriveGroups * kArriveStride;
    if (__hip_atomic_fetch_add(gc, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == members) {
      __hip_atomic_store(gc, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (__hip_atomic_fetch_add(top, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == groups) {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        __hip_atomic_store(top, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = 1;
      }
    }
    *s_last = last;
  }
  __syncthreads();
  return *s_last != 0;
}

// The reduction of k_finish<0> (1024 threads: thread t sums the block partials t,
// t + 1024, ... in order, a butterfly per wave, then thread 0 folds in order the
// waves that hold data) by a workgroup of any multiple of 64 threads, its wave v
// standing in for the waves v, v + W, ... of that workgroup.  Bitwise the result of
// k_finish; valid in thread 0.
__device__ BlockPartial finish_reduce(const BlockPartial *part, int G, BlockPartial *s_waves) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = (int)(blockDim.x >> 6);
  const int used = min(16, (G + 63) / 64);
  for (int vw = wv; vw < used; vw += nw) {
    BlockPartial a = zero_partial();
    for (int b = vw * 64 + lane; b < G; b += 1024) fold_timed(a, part[b]);
    a.pe = wave_sum(a.pe);
    a.w = wave_sum(a.w);
    a.ke_half = wave_sum(a.ke_half);
    a.ke_int = wave_sum(a.ke_int);
    a.disp2 = wave_max(a.disp2);
    a.t0 = wave_min_u64(a.t0);
    a.t1 = wave_max_u64(a.t1);
    a.nonfinite = wave_or(a.nonfinite);
    if (lane == 0) s_waves[vw] = a;
  }
  __syncthreads();
  BlockPartial a = zero_partial();
  if (threadIdx.x == 0) {
    a = s_waves[0];
    for (int k = 1; k < used; ++k) fold_timed(a, s_waves[k]);
  }
  return a;
}

// Cell index of a position (the major key of the spatial sort).
__device__ __forceinline__ int cell_index(const float4 r, const SysConst &c) {
  int cx, cy, cz;
  cell_coords(r, c, cx, cy, cz);
  return (cz * c.nc[1] + cy) * c.nc[0] + cx;
}

// The spatial sort of sort_small_block (order by cell, then particle id; the same
// cell starts and gathered arrays) by a workgroup of any size, its working arrays
// in LDS only: s_cnt (ncell + 1 words) and s_id (n words).  A histogram pass, the
// exclusive scan (also written to cell_start), a placement pass that moves each
// cell's cursor past its particles (so that afterwards s_cnt[k] ends cell k), and a
// rank-and-gather pass; cells are recomputed from the positions in every pass.
// Each thread takes B particles of a pass at a time, their loads issued together
// (B / 2 in the gather pass, which loads three arrays), so that a pass over a few
// thousand particles costs one memory round trip rather than one per particle; when
// all particles fit one such batch, the placement works from registers instead
// (below).  The scan's per-wave prefix sums are DPP lane shifts.
template <int B>
__device__ void sort_small_shared(const SysConst &c, const SysPtrs &p, int cur, unsigned *s_cnt, int *s_id) {
  constexpr int BG = B > 1 ? B / 2 : 1;
  __shared__ unsigned s_w[16];
  __shared__ unsigned s_carry;
  const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, wv = tid >> 6, nw = (nthr + 63) >> 6;
  const int ncell = c.ncell, n = c.n;
  const float4 *pos = p.pos[cur];
  for (int k = tid; k <= ncell; k += nthr) s_cnt[k] = 0u;
  if (tid == 0) {
    s_carry = 0u;
    begin_build(p.ctl);
    p.ctl->resorted = 1;
  }
  __syncthreads();
  // When each thread has at most B particles (one batch), their cells, ids and slots
  // within their cells (the histogram counter before their increment) stay in
  // registers, and the placement needs neither the positions again nor a second
  // atomic: particle k goes to start(cell) + slot.  key = cell << 13 | slot (cells
  // and slots below 8192, as N <= 8192).
  const bool one = B > 1 && n <= B * nthr;
  unsigned key[B];
  int idr[B];
  // (loads past n are clamped to the last particle and their results unused, so that
  // every load is issued unconditionally)
  for (int base = tid; base < n; base += B * nthr) {
    float4 r[B];
#pragma unroll
    for (int k = 0; k < B; ++k) {
      const int i = min(base + k * nthr, n - 1);
      r[k] = pos[i];
      if (one) idr[k] = p.img[i].w;
    }
#pragma unroll
    for (int k = 0; k < B; ++k)
      if (base + k * nthr < n) {
        const unsigned cell = (unsigned)cell_index(r[k], c);
        const unsigned slot = atomicAdd(&s_cnt[cell], 1u);
        if (one) key[k] = cell << 13 | slot;
      }
  }
  __syncthreads();
  for (int base = 0; base <= ncell; base += nthr) {
    const int idx = base + tid;
    const unsigned v = idx <= ncell ? s_cnt[idx] : 0u;
    const unsigned x = wave_incl_scan(v);
    if (lane == 63 || tid == nthr - 1) s_w[wv] = x;
    __syncthreads();
    unsigned wbase = 0;
    for (int k = 0; k < wv; ++k) wbase += s_w[k];
    if (idx <= ncell) {
      const unsigned e = s_carry + wbase + x - v;
      s_cnt[idx] = e;
      p.cell_start[idx] = e;
    }
    __syncthreads();
    if (tid == 0) {
      unsigned tot = 0;
      for (int k = 0; k < nw; ++k) tot += s_w[k];
      s_carry += tot;
    }
    __syncthreads();
  }
  if (one) {
    // s_cnt holds the cell starts (and s_cnt[ncell] = n)
#pragma unroll
    for (int k = 0; k < B; ++k)
      if (tid + k * nthr < n) s_id[s_cnt[key[k] >> 13] + (key[k] & 8191u)] = idr[k];
  } else {
    for (int base = tid; base < n; base += B * nthr) {
      float4 r[B];
      int id[B];
#pragma unroll
      for (int k = 0; k < B; ++k) {
        const int i = min(base + k * nthr, n - 1);
        r[k] = pos[i];
        id[k] = p.img[i].w;
      }
#pragma unroll
      for (int k = 0; k < B; ++k)
        if (base + k * nthr < n) s_id[atomicAdd(&s_cnt[cell_index(r[k], c)], 1u)] = id[k];
    }
  }
  __syncthreads();
  for (int base = tid; base < n; base += BG * nthr) {
    float4 r[BG];
    raw_f4 v[BG];
    raw_i4 im[BG];
#pragma unroll
    for (int k = 0; k < BG; ++k) {
      const int i = min(base + k * nthr, n - 1);
      r[k] = pos[i];
      im[k] = reinterpret_cast<const raw_i4 *>(p.img)[i];
      v[k] = reinterpret_cast<const raw_f4 *>(p.vel)[i];
    }
#pragma unroll
    for (int k = 0; k < BG; ++k) {
      const int i = base + k * nthr;
      if (i < n) {
        const int cell = cell_index(r[k], c);
        // cell bounds: starts (one batch) or the cursors moved to the cells' ends
        const unsigned beg = one ? s_cnt[cell] : cell > 0 ? s_cnt[cell - 1] : 0u;
        const unsigned end = one ? s_cnt[cell + 1] : s_cnt[cell];
        unsigned rank = 0;
        for (unsigned q = beg; q < end; ++q) rank += (s_id[q] < im[k].w) ? 1u : 0u;
        const unsigned dst = beg + rank;
        p.t_pos[dst] = r[k];
        reinterpret_cast<raw_f4 *>(p.t_vel)[dst] = v[k];
        reinterpret_cast<raw_i4 *>(p.t_img)[dst] = im[k];
        if (p.pos64) {
          p.t_pos64[3 * dst] = p.pos64[3 * i];
          p.t_pos64[3 * dst + 1] = p.pos64[3 * i + 1];
          p.t_pos64[3 * dst + 2] = p.pos64[3 * i + 2];
        }
        if (p.kahan) p.t_kahan[dst] = p.kahan[i];
      }
    }
  }
}

// Particles per thread whose loads the end-of-step sort issues together.
constexpr int kTailSortBatch = 8;

// LDS bytes of sort_small_shared for n particles in ncell cells.
__host__ __device__ constexpr size_t tail_sort_lds(int n, int ncell) { return 4 * ((size_t)ncell + 1 + (size_t)n); }

// The end of a step in the workgroup that arrived last (arrive_last): the
// reduction, record, thermostat update and rebuild decision of k_finish<0>, and on
// a small system's step that decides a rebuild the spatial sort of the new
// positions pos[next] (dynamic LDS of tail_sort_lds bytes).
__device__ void step_tail(const SysConst &c, const SysPtrs &p, int G, int next, BlockPartial *s_waves, int *s_flag,
                          unsigned *s_dyn) {
  CtlView cv{};
  if (threadIdx.x == 0) cv = load_ctl(p.ctl);  // beside the partials: one round trip
  const BlockPartial a = finish_reduce(p.part, G, s_waves);
  if (threadIdx.x == 0) {
    s_flag[0] = finish_step(c, p, a, cv);
    s_flag[1] = resort_due(c, cv.n_rebuilds) ? 1 : 0;
    p.ctl->cur = next;
  }
  __syncthreads();
  if (s_flag[0] && c.small_sort) {
    if (c.list_kind == 4 && !s_flag[1]) {  // all-pairs lists sort only when a re-sort is due
      if (threadIdx.x == 0) {
        begin_build(p.ctl);
        p.ctl->resorted = 0;
      }
    } else {
      sort_small_shared<kTailSortBatch>(c, p, next, s_dyn, reinterpret_cast<int *>(s_dyn + c.ncell + 1));
    }
  }
}

// ---------------------------------------------------------------- fused step

// Waves per SIMD the step kernel is compiled for: blocks of 1024 threads need four.  The
// staged form at one lane per particle takes five (with float32 positions): its LDS copy
// leaves room for five blocks of 256; but not with the further potentials (method 5), whose
// loop then spills 40 registers (100 steps at 256 000 particles with 5 and 4 waves: Yukawa
// 14.77 and 14.35 ms, Gaussian 9.13 and 8.95, Dzugutov 8.17 and 8.03).
template <int TP, int METHOD, int PREC, bool STAGE>
struct kStepWaves {
  static constexpr int value = STAGE && TP == 1 && METHOD < 5 && PREC == 0 ? 5 : 4;
};

template <int TP, int METHOD, int PREC, bool STAGE>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(kStepWaves<TP, METHOD, PREC, STAGE>::value))) void k_step(SysConst c, SysPtrs p, int cur, int tail) {
  extern __shared__ unsigned s_tail_lds[];  // list build and tail of small systems; STAGE: the region copies
  __shared__ SharedPairs sp;
  __shared__ BlockPartial s_waves[16];
  __shared__ int s_flag[2];
  __shared__ float s_cs2[kMaxPairs];
  const unsigned long long tstart = wall_clock64();
  // cur < 0: a step of a run-ahead chain; -1 follows a rebuild slot, -2 does not and
  // waits for the next one when the flag is set.  Every workgroup reads the words before
  // the last one, which ends the step, writes them.
  if (cur < 0) {
    const int flag = p.ctl->rebuild, buf = p.ctl->cur;
    const long long now = p.ctl->step, stop = p.ctl->stop;
    if (now >= stop || (cur == -2 && flag != 0)) return;
    cur = buf;
  }
  stage_pairs(sp, c);
  // tail 2: a small system's list is built here, at the start of a step whose
  // rebuild flag is set (no list kernel in the chain): each wave builds the lists of
  // the block's own particles one after the other (the wave builder or the all-pairs
  // builder: the same lists as their list kernels), placing their sorted data; the
  // step then reads positions from the sorted copy, which the other workgroups may
  // not have placed yet
  const int build = !STAGE && tail == 2 ? p.ctl->rebuild : 0;
  // the friction of the step, read before the list build: the build's tallies are
  // atomics on the same control line from every workgroup, and a load queued behind
  // them waits several microseconds
  const double xi = c.thermostat ? p.ctl->xi : 0.0;
  if (build && threadIdx.x < kMaxPairs) s_cs2[threadIdx.x] = c.pt.cs2[threadIdx.x];
  const int lb = xcd_remap(blockIdx.x, gridDim.x);
  float4 *const s_region = reinterpret_cast<float4 *>(s_tail_lds);
  int place = -1;
  if constexpr (STAGE) place = stage_fill<TP>(c, p, p.pos[cur], lb, s_region);
  __syncthreads();
  // the positions of the step: the sorted copy on a build step after a sort, else in place
  const float4 *pos = p.pos[cur];
  if (build) {
    const int wv = threadIdx.x >> 6, nw = (int)(blockDim.x >> 6), ppb = (int)blockDim.x / TP;
    const bool allp = c.list_kind == 4;  // all pairs: sorted only when a periodic re-sort was due
    const bool sorted = !allp || p.ctl->resorted != 0;
    if (sorted) pos = p.t_pos;
    int kept = 0, longest = 0;
    for (int q = wv; q < ppb; q += nw) {
      const int slot = lb * ppb + q;
      if (slot < c.n) {  // uniform across the wave
        int k;
        if (allp) {
          if (sorted && (threadIdx.x & 63) == 0) place_sorted(p, cur, slot, pos[slot]);
          k = list_allpairs_one(c, p, slot, s_cs2, pos, longest);
        } else {
          k = list_wave_one<true>(c, p, cur, slot, s_tail_lds + wv * kWaveCand, s_cs2, pos, p.cell_start, longest);
        }
        if ((threadIdx.x & 63) == 0) kept += k;
      }
    }
    list_tally(kept, longest, c.n_max, p.ctl);  // every thread of the block reaches this barrier once
    __syncthreads();  // the block's lists and placed data are visible to all its waves
  }
  const int gt = lb * blockDim.x + threadIdx.x;
  const int i = gt / TP, t = gt % TP;
  const bool active = i < c.n;
  float fx = 0.f, fy = 0.f, fz = 0.f, u = 0.f, w = 0.f;
  float4 pi = make_float4(0.f, 0.f, 0.f, 0.f);
  // integrator operands are loaded before the force loop so their latency overlaps it
  float4 vo = pi, l0 = pi, kc = pi;
  int4 im = make_int4(0, 0, 0, 0);
  double x64 = 0.0, y64 = 0.0, z64 = 0.0;
  const int ic = active ? i : c.n - 1;
  pi = pos[ic];
  if (active) {
    if (t == 0) {
      vo = p.vel[i];
      im = p.img[i];
      l0 = p.last[i];
      if (PREC == 1) kc = p.kahan[i];
      if (PREC == 2) {
        x64 = p.pos64[3 * i];
        y64 = p.pos64[3 * i + 1];
        z64 = p.pos64[3 * i + 2];
      }
    }
  }
  if (STAGE && place >= 0)
    force_lane_staged<TP, METHOD>(ic, t, active, pi, s_region + place, p, sp, c, fx, fy, fz, u, w);
  else
    force_lane<TP, METHOD, StepBatch<TP>::value, STAGE>(ic, t, active, pi, pos, (const int *)p.nbl, (const int *)p.nnb, sp,
                                                        c, fx, fy, fz, u, w);
  fx = lane_sum<TP>(fx);
  fy = lane_sum<TP>(fy);
  fz = lane_sum<TP>(fz);
  u = lane_sum<TP>(u);
  w = lane_sum<TP>(w);
  BlockPartial v = zero_partial();
  if (active && t == 0)
    integrate_one<PREC>(c, p, cur, i, pi, vo, im, l0, kc, x64, y64, z64, xi, fx, fy, fz, u, w, v,
                        tail && c.small_sort);
  v.t0 = tstart;
  v.t1 = wall_clock64();
  block_reduce(v, s_waves);
  if (threadIdx.x == 0) {
    store_to(&p.part[lb], v, tail != 0);
    // the list of this step has been consumed (with the tail, finish_step decides the flag)
    if (blockIdx.x == 0 && !tail) p.ctl->rebuild = 0;
  }
  // tail: the last workgroup to arrive ends the step (k_finish<0> not launched)
  if (tail && arrive_last(p.arrive, gridDim.x, blockIdx.x, &s_flag[0])) step_tail(c, p, gridDim.x, cur ^ 1, s_waves, s_flag, s_tail_lds);
}

// One workgroup after the step (MODE 0) or force-only (MODE 1) kernel: fixed-order
// float64 reduction of the G block partials (each thread sums its blocks in index
// order, then lanes by butterfly and waves in order), the Nose-Hoover update, the
// thermodynamic record, the displacement test that sets the rebuild flag, and for
// small systems the spatial sort for the next list build (positions pos[next]).
template <int MODE>
__global__ __launch_bounds__(1024) void k_finish(SysConst c, SysPtrs p, int G, int next) {
  __shared__ BlockPartial s_waves[16];
  __shared__ int s_rebuild, s_due;
  __shared__ unsigned s_cnt[MODE == 0 ? kSmallCells + 1 : 1];
  __shared__ int s_id[MODE == 0 ? kSmallN : 1];
  // the control words are final (the kernels before this one in the stream wrote
  // them), so they load beside the partials: one memory round trip instead of two
  CtlView cv{};
  if (MODE == 0 && threadIdx.x == 0) cv = load_ctl(p.ctl);
  BlockPartial a = zero_partial();
  for (int b = threadIdx.x; b < G; b += blockDim.x) {
    const BlockPartial q = p.part[b];
    a.pe += q.pe;
    a.w += q.w;
    a.ke_half += q.ke_half;
    a.ke_int += q.ke_int;
    a.disp2 = fmax(a.disp2, q.disp2);
    a.nonfinite |= q.nonfinite;
    a.t0 = q.t0 < a.t0 ? q.t0 : a.t0;
    a.t1 = q.t1 > a.t1 ? q.t1 : a.t1;
  }
  // threads at or past G hold zero partials: only the first (G + 63) / 64 waves are folded
  group_reduce(a, s_waves, (int)blockDim.x, (G + 63) / 64);
  if (threadIdx.x == 0) {
    Control *ctl = p.ctl;
    int rebuild = 0;
    if (MODE == 1) {
      Thermo *th = p.thermo;
      th->pe = a.pe;
      th->virial = a.w;
      th->ke = a.ke_half;  // kinetic energy of the stored (half-step) velocities
      th->ke_half = a.ke_half;
      th->temperature = 2.0 * a.ke_half / c.g;
      th->pressure = (2.0 * a.ke_half / 3.0 + a.w) / c.volume;
      th->xi = c.thermostat ? ctl->xi : 0.0;
      th->xi_integral = ctl->xi_int;
      th->h_conserved = a.ke_half + a.pe;
      th->max_nbrs = ctl->max_nbrs;
      th->n_rebuilds = ctl->n_rebuilds;
      th->step = ctl->step;
      if (a.nonfinite) ctl->error |= 1;
    } else {
      rebuild = finish_step(c, p, a, cv);
      s_due = resort_due(c, cv.n_rebuilds) ? 1 : 0;
    }
    s_rebuild = rebuild;
  }
  __syncthreads();
  if (MODE == 0 && s_rebuild && c.small_sort) {
    if (c.list_kind == 4 && !s_due) {
      if (threadIdx.x == 0) {
        begin_build(p.ctl);
        p.ctl->resorted = 0;
      }
    } else {
      sort_small_block<1024>(c, p, next, s_cnt, s_id);
    }
  }
}

// ---------------------------------------------------------------- persistent launches

// Butterfly of a BlockPartial over the 64 lanes of a wave (the first step of
// group_reduce), result valid in every lane.
__device__ __forceinline__ void wave_reduce(BlockPartial &v) {
  v.pe = wave_sum(v.pe);
  v.w = wave_sum(v.w);
  v.ke_half = wave_sum(v.ke_half);
  v.ke_int = wave_sum(v.ke_int);
  v.disp2 = wave_max(v.disp2);
  v.nonfinite = wave_or(v.nonfinite);
}

// a += q with the operations of the block and k_finish reductions.
__device__ __forceinline__ void fold(BlockPartial &a, const BlockPartial &q) {
  a.pe += q.pe;
  a.w += q.w;
  a.ke_half += q.ke_half;
  a.ke_int += q.ke_int;
  a.disp2 = fmax(a.disp2, q.disp2);
  a.nonfinite |= q.nonfinite;
}

// A pointer read from a descriptor in memory is generic to the compiler; loads
// through this global-address-space view compile to global (not flat) loads, which
// keep the list loads of the force loop pipelined.
#define SRMD_GLOBAL __attribute__((address_space(1)))

template <class T>
__device__ __forceinline__ const SRMD_GLOBAL T *global_view(const T *q) {
  return (const SRMD_GLOBAL T *)q;
}

__device__ __forceinline__ float4 gload(const float4 *q, int i) {
  const raw_f4 v = ((const SRMD_GLOBAL raw_f4 *)q)[i];
  return make_float4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ int4 gload(const int4 *q, int i) {
  const raw_i4 v = ((const SRMD_GLOBAL raw_i4 *)q)[i];
  return make_int4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ int gload(const int *q, int i) { return ((const SRMD_GLOBAL int *)q)[i]; }

// Threads of a persistent workgroup: 512 for one system, whose steps wait for the
// barrier between many small pieces, and 1024 for a batch at up to 8 threads per
// particle, where a workgroup has thousands of particles to itself and the positions in
// LDS allow one workgroup per compute unit: 256 replicas of the mixture (500 to 8000
// particles, tp = 1) step in 470 us with 16 waves against 620 with 8.  From 16 threads per
// particle a step is 16 times as many waves' work and the 512-thread kernel, which keeps
// more entries in flight, stays.
constexpr int kPersistThreads = 512;
constexpr int kBatchThreads = 1024;
constexpr int kBatchMaxTp = 8;
constexpr int kCoopMaxGroups = 256;  // workgroups of one system (arrival words per parity)
constexpr int kMaxJobs = 64;         // jobs of one workgroup
constexpr int kLdsUnits = 64;        // wave partials of one piece kept in LDS (else in memory)

// Grid-wide barrier k (k = 1, 2, ... in one launch) of the G workgroups that share
// one system, over that system's array of arrival words (one per workgroup and
// barrier parity, cleared by the host before the launch).  Piece w publishes
// (k << 1) | bit in its word: an arrival costs one store and no read-modify-write on
// a shared counter, and bit carries a flag whose OR over the pieces every piece
// receives (the rebuild decision).  The first wave polls the G words of parity k & 1
// until each holds barrier k; two parities suffice because no piece can reach
// barrier k + 2 before every piece has left barrier k.  The wait is bounded (about
// one second of the 100 MHz device clock): on time-out the workgroup sets error bit 2
// and the kernel ends instead of hanging.  Release / acquire fences at agent scope
// order every store before the barrier against every load after it, once per
// workgroup: the release after each wave has waited for its own stores to complete
// (the L2 write-back acts on the whole cache), with the arrival store waiting for the
// write-back to complete; the acquire by the polling wave, whose invalidate of the
// compute unit's L1 and of the L2 precedes, through the workgroup barrier, every
// later load of the other waves.  With G = 1 the barrier is the workgroup barrier.
__device__ __forceinline__ bool coop_barrier(unsigned *flags, unsigned G, unsigned w, unsigned k, int bit,
                                             Control *ctl, int *s_ok, int *s_any) {
  if (G == 1) {
    __syncthreads();
    if (threadIdx.x == 0) *s_any = bit;
    __syncthreads();
    return true;
  }
  __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's stores have reached the L2
  __syncthreads();
  unsigned *slot = flags + (k & 1u) * kCoopMaxGroups;
  if (threadIdx.x == 0) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    // the L2 write-back must complete before the arrival is visible; the compiler's own
    // wait after the write-back is dropped when no store of this wave is outstanding
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __hip_atomic_store(slot + w, (k << 1) | (unsigned)(bit != 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (threadIdx.x < 64) {
    const unsigned long long t0 = wall_clock64();
    int ok = 1;
    bool any = false;
    while (true) {
      bool done = true, mine = false;
      for (unsigned l = threadIdx.x; l < G; l += 64) {
        const unsigned f = __hip_atomic_load(slot + l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        done = done && (f >> 1) >= k;
        mine = mine || (f & 1u);
      }
      if (__all(done)) {
        any = __any(mine);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
      if (wall_clock64() - t0 > 100000000ull) {
        ok = 0;
        break;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (threadIdx.x == 0) {
      if (!ok) atomicOr(&ctl->error, 4);
      *s_ok = ok;
      *s_any = any ? 1 : 0;
    }
  }
  __syncthreads();
  return *s_ok != 0;
}

// Positions of all n particles into LDS, eight loads in flight per thread.
template <int NT>
__device__ __forceinline__ void fill_positions(float4 *dst, const float4 *src, int n) {
  for (int base = 0; base < n; base += 8 * NT) {
    float4 v[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) v[m] = gload(src, min(base + m * NT + (int)threadIdx.x, n - 1));
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const int k = base + m * NT + (int)threadIdx.x;
      if (k < n) dst[k] = v[m];
    }
  }
}

// Cell lists of a batch: slots of one round of a workgroup, list entries per particle
// staged in LDS (as 16-bit slots; rows of an odd number of words, so that the write-out
// reads distinct banks), and the LDS of the stage and the waves' candidate windows.
constexpr int kRoundSlots = 128;
constexpr int kRoundRow = kCellStage + 2;
constexpr int round_list_bytes(int threads) {
  return 2 * (kRoundSlots * kRoundRow + threads / 64 * kCellWindow);
}

// Verlet lists of a batched replica by cells, for the slots of this piece (w of g).  A
// round takes kRoundSlots consecutive sorted slots, cut into pieces of at most kCellPiece
// slots of one cell that are dealt over the waves (list_cell_particles), stages their
// entries in LDS and writes them out in address order.  Pieces are taken from a counter, so
// that waves with emptier cells take more of them.  Bound by the instructions of a piece
// (about 750 per wave); a build of 5300 particles of the mixture takes 0.95 ms on one
// compute unit, 1.35 with a wave per cell whose lanes wrote each entry to memory by
// themselves and read the constants through the descriptor.
// stage: round_list_bytes(NT) bytes.  Returns this thread's entries and longest list.
template <int TP, int NT>
__device__ __forceinline__ void list_rounds(const SysConst &cg, const SysPtrs &p, int w, int g, unsigned short *stage,
                            const float *s_cs2, const float4 *tpos, const unsigned *cstart, int &kept, int &longest) {
  constexpr int NW = NT / 64;
  __shared__ int s_cnt[2][kRoundSlots], s_seg[2][2][65], s_nseg[2][2], s_kmax[2], s_next[2];
  // the constants used below, in registers: through the replica's descriptor in memory
  // they would be read again after every store
  SysConst c;
  c.n = cg.n;
  c.ntypes = cg.ntypes;
  c.nvp = cg.nvp;
  c.n_max = cg.n_max;
  c.tp = TP;
  c.tp_shift = cg.tp_shift;
  c.full_axis = cg.full_axis;
  c.tiles[0] = c.tiles[1] = 1;  // small systems: row-major cells
  for (int k = 0; k < 3; ++k) {
    c.nc[k] = cg.nc[k];
    c.L[k] = cg.L[k];
    c.invL[k] = cg.invL[k];
    c.halfL[k] = cg.halfL[k];
    c.cscale[k] = cg.cscale[k];
  }
  int *const nbl = p.nbl, *const nnb = p.nnb;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int nmax = c.n_max;
  unsigned short *cand = stage + kRoundSlots * kRoundRow + wv * kCellWindow;
  // the pieces of the round at T0, by waves 0 and 1 (64 slots each): one starts where the
  // cell changes and after every kCellPiece slots
  auto cut = [&](int T0, int par) {
    if (wv < 2) {
      const int l = 64 * wv + lane, m = c.n - T0;
      int cell = -1;
      if (l < m) {
        int cx, cy, cz;
        cell_coords(tpos[T0 + l], c, cx, cy, cz);
        cell = (cz * c.nc[1] + cy) * c.nc[0] + cx;
      }
      s_cnt[par][l] = 0;
      const int prev = __shfl_up(cell, 1, 64);
      const unsigned long long first = __ballot(l < m && (lane == 0 || prev != cell));
      const int since = lane - (63 - __builtin_clzll((first & ((2ull << lane) - 1ull)) | 1ull));
      const bool head = l < m && since % kCellPiece == 0;
      const unsigned long long hm = __ballot(head);
      if (head) s_seg[par][wv][__popcll(hm & ((1ull << lane) - 1ull))] = l;
      if (lane == 0) {
        s_nseg[par][wv] = __popcll(hm);
        s_seg[par][wv][__popcll(hm)] = min(64 * (wv + 1), max(m, 64 * wv));
        s_kmax[par] = 0;
        s_next[par] = NW;
      }
    }
  };
  int T0 = w * kRoundSlots, par = 0;
  if (T0 < c.n) cut(T0, 0);
  __syncthreads();
  for (; T0 < c.n; T0 += g * kRoundSlots, par ^= 1) {
    const int n0 = s_nseg[par][0], nseg = n0 + s_nseg[par][1];
    auto sink = [&](int i, int k, int upto, int j) {
      unsigned short *row = stage + (i - T0) * kRoundRow;
      if (upto <= kCellStage)
        row[k] = (unsigned short)j;
      else if (k < kCellStage)
        row[k] = (unsigned short)j;
      else if (k < nmax)
        nbl[nbl_addr(i, k, c)] = j;
    };
    for (int sg = wv; sg < nseg;) {
      const int h = sg >= n0, q = sg - (h ? n0 : 0);
      const int l0 = s_seg[par][h][q], l1 = s_seg[par][h][q + 1];
      int cx, cy, cz;
      cell_coords(tpos[T0 + l0], c, cx, cy, cz);
      list_cell_particles<true>(c, p, cx, cy, cz, T0 + l0, T0 + l1, cand, s_cnt[par] + l0, s_cs2, tpos, cstart, sink);
      if (lane < l1 - l0) atomicMax(&s_kmax[par], s_cnt[par][l0 + lane]);
      if (lane == 0) sg = atomicAdd(&s_next[par], 1);
      sg = __builtin_amdgcn_readfirstlane(sg);
    }
    __syncthreads();
    if (T0 + g * kRoundSlots < c.n) cut(T0 + g * kRoundSlots, par ^ 1);
    const int m = min(kRoundSlots, c.n - T0);
    const int kst = min(min(s_kmax[par], nmax), kCellStage);
    const int groups = (kst + TP - 1) / TP;
    for (int j = tid; j < groups * kRoundSlots * TP; j += NT) {
      const int gr = j / (kRoundSlots * TP), rr = j % (kRoundSlots * TP), l = rr / TP, k = gr * TP + rr % TP;
      if (l < m && k < min(s_cnt[par][l], kst))
        nbl[(long long)gr * ((long long)c.nvp * TP) + (long long)T0 * TP + rr] = stage[l * kRoundRow + k];
    }
    if (tid < m) {
      const int cn = s_cnt[par][tid];
      longest = max(longest, cn);
      kept += min(cn, nmax);
      nnb[T0 + tid] = min(cn, nmax);
    }
    __syncthreads();
  }
}

// Small systems (N <= 8192, at most 8192 cells) advanced nsteps in one cooperative
// launch: one system over many workgroups (a single large enough system), many
// systems over the workgroups (a batch of replicas: the ensembles of small systems
// the paper's introduction points to), or both (a batch whose largest replicas are
// split over several workgroups and whose smallest share one).  Workgroup b runs the
// jobs jobs[job_off[b] .. job_off[b+1]) one after the other in every step.
//
// Piece w of g of a system owns the virtual blocks w, w + g, ... of that system's
// single-system step launch (G blocks of vb threads): its waves run the blocks' wave
// units (64 threads of that launch: the same particles, t_p lanes and list entries)
// with all positions of the step in LDS, and each block's wave partials are folded in
// index order into the block partial, as the step kernel does.  The partials buffer
// of a system holds two sets of G block partials (by step parity) and then one
// partial per wave unit.  After the barrier
// every piece reads the G block partials and repeats the fixed-order reduction of
// k_finish (so the thermostat needs no second barrier); piece 0 alone writes the
// record and the control block.  The rebuild decision travels with the barrier.  On
// a step that decides a rebuild, piece 0 sorts (as k_finish does), a barrier follows,
// the pieces build the lists of particles wave, wave + NW g, ... (or rounds of cells), and another barrier
// follows.  A system follows its single-system trajectory bit for bit at the same
// (tp, ppb), whatever the pieces and the other jobs of its workgroups.
//
// BIG: one larger system alone (more than 8192 particles or cells), positions read
// from device memory rather than LDS.  Its spatial sort is the four-phase counting
// sort of the launch chain, run by all pieces at the start of a step that rebuilds,
// with a grid barrier after each phase.
// Waves per SIMD the persistent kernel is compiled for: in a batch (kBatchThreads) the
// four of its workgroup; else three from 16 lanes per particle up (measured +12 % at
// KA 4096, 32 bytes of spills), the register count's own two below, where three would
// spill 150 bytes per lane.
template <int TP, int NT>
struct kMultiWaves {
  static constexpr int value = NT == kBatchThreads ? NT / 256 : TP >= 16 ? 3 : 1;
};

// List entries in flight per lane: four waves per SIMD hide the loads of four (4, 6 and 8
// measure the same on the replica batch; eight spill more).
template <int TP, int NT>
struct kMultiBatch {
  static constexpr int value = NT == kBatchThreads ? 4 : Batch<TP>::value;
};

// The persistent kernel of one small system runs its phases once per step, a few waves per
// SIMD: its size counts, also of code that a step does not reach.  From 8 threads per
// particle it takes the general pair loop alone, and its cell lists the image per pair alone
// (500 steps of the liquid at 2048, 4096 and 8000 particles: 14.6, 15.5 and 19.6 us a step;
// with the loops and tests for every case 15.3, 16.6 and 20.6; the mixture 14.2, 16.0 and
// 19.7 against 15.2, 17.2 and 21.0).  Fewer threads per particle have more pairs per lane and
// the large-system form more of them per wave, for which the loops without images pay.
template <int TP, bool BIG, int NT>
struct kMultiSlim {
  static constexpr bool value = NT == kPersistThreads && TP >= 8 && !BIG;
};

template <int TP, int METHOD, bool BIG, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(kMultiWaves<TP, NT>::value))) void k_multi(
    const ReplicaDesc *__restrict__ reps, const CoopJob *__restrict__ jobs, const int *__restrict__ job_off, int nsteps,
    int lds_bytes) {
  constexpr int NW = NT / 64;
  extern __shared__ float4 s_dyn[];
  __shared__ SharedPairs sp;
  __shared__ BlockPartial s_waves[16];
  __shared__ BlockPartial s_wp[kLdsUnits];
  __shared__ float s_cs2[kMaxPairs];
  __shared__ int s_ok, s_any, s_bit, s_due;
  __shared__ int s_rebuild[kMaxJobs], s_cur[kMaxJobs], s_resorted[kMaxJobs];
  __shared__ unsigned s_k[kMaxJobs];
  __shared__ double s_xi[kMaxJobs];
  __shared__ unsigned s_scan[16];
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
  const int j0 = job_off[blockIdx.x];
  const int nj = min(job_off[blockIdx.x + 1] - j0, kMaxJobs);
  // every piece reads its system's control block before piece 0 can write it
  for (int j = 0; j < nj; ++j) {
    const CoopJob J = jobs[j0 + j];
    const ReplicaDesc &R = reps[J.rep];
    if (tid == 0) {
      s_rebuild[j] = R.p.ctl->rebuild;
      s_resorted[j] = R.p.ctl->resorted;
      s_xi[j] = R.c.thermostat ? R.p.ctl->xi : 0.0;
      s_cur[j] = R.cur;
      s_k[j] = 1u;
    }
    if (!coop_barrier(R.p.bar_flags, J.g, J.w, 1u, 0, R.p.ctl, &s_ok, &s_any)) return;
  }
  bool prefilled = false;  // the positions of this step are already in LDS
  for (int step = 0; step < nsteps; ++step) {
    for (int j = 0; j < nj; ++j) {
      const CoopJob J = jobs[j0 + j];
      const ReplicaDesc &R = reps[J.rep];
      const SysConst &c = R.c;
      const SysPtrs &p = R.p;
      const int G = R.G, vb = R.vb, wpv = vb >> 6;
      const SRMD_GLOBAL int *nblg = global_view(p.nbl);
      const SRMD_GLOBAL int *nnbg = global_view(p.nnb);
      __syncthreads();  // the previous job's LDS use has ended
      int cur = s_cur[j];
      unsigned k = s_k[j];
      const int rebuild = s_rebuild[j];
      const double xi = s_xi[j];
      stage_pairs(sp, c);
      if (tid < kMaxPairs) s_cs2[tid] = c.pt.cs2[tid];
      if (tid == 0) s_bit = 0;
      __syncthreads();
      if (BIG && rebuild) {  // the counting sort of the launch chain, phase by phase
        const int base = J.w * NT, stride = J.g * NT;
        sort_bin(c, p, cur, base, stride);
        if (!coop_barrier(p.bar_flags, J.g, J.w, ++k, 0, p.ctl, &s_ok, &s_any)) return;
        if (J.w == 0 && tid == 0) begin_build(p.ctl);
        for (int b = J.w; b < scan_tiles(c.ncell); b += J.g) sort_scan_tile(c, p, b, s_scan);
        if (!coop_barrier(p.bar_flags, J.g, J.w, ++k, 0, p.ctl, &s_ok, &s_any)) return;
        sort_scatter(c, p, base + tid, stride, J.w == 0);
        if (!coop_barrier(p.bar_flags, J.g, J.w, ++k, 0, p.ctl, &s_ok, &s_any)) return;
        sort_gather(c, p, cur, base + tid, stride);
        if (!coop_barrier(p.bar_flags, J.g, J.w, ++k, 0, p.ctl, &s_ok, &s_any)) return;
      }
      if (!BIG && rebuild && c.list_kind == 4) {
        // all pairs from the positions of the step in LDS, no cells; after a periodic
        // re-sort from the sorted copy, with this piece's slots moved into place
        const bool resorted = s_resorted[j] != 0;
        fill_positions<NT>(s_dyn, resorted ? p.t_pos : p.pos[cur], c.n);
        if (resorted)
          for (int t = J.w * NT + tid; t < c.n; t += J.g * NT)
            place_sorted(p, cur, t, gload(p.t_pos, t));
        __syncthreads();
        int kept = 0, longest = 0;
        for (int t = J.w * NW + wv; t < c.n; t += J.g * NW) {
          const int kt = list_allpairs_one(c, p, t, s_cs2, s_dyn, longest);
          if (lane == 0) kept += kt;
        }
        list_tally(kept, longest, c.n_max, p.ctl);
        if (!coop_barrier(p.bar_flags, J.g, J.w, ++k, 0, p.ctl, &s_ok, &s_any)) return;
        prefilled = true;  // s_dyn holds this step's positions
      } else if (rebuild) {  // the spatial sort has been done (host request, end of step, or above)
        // the sorted positions and the cell starts go to LDS when they fit beside the
        // candidate windows, so the list build reads no device memory but its own list
        const int cs_words = (c.ncell + 1 + 3) & ~3;
        // by cells when each wave gets several; with about one cell per wave the most
        // crowded cell would set the pace, so then one wave per particle
        const bool by_cell = 4 * J.g * NW <= c.ncell;
        constexpr bool kRounds = !BIG && NT == kBatchThreads;
        const int list_lds = kRounds && by_cell ? round_list_bytes(NT) : 4 * NW * kWaveCand;
        const bool in_lds = !BIG && 16 * c.n + 4 * cs_words + list_lds <= lds_bytes;
        const float4 *tpos = p.t_pos;
        const unsigned *cstart = p.cell_start;
        unsigned *list_area = reinterpret_cast<unsigned *>(s_dyn);
        if (in_lds) {
          fill_positions<NT>(s_dyn, p.t_pos, c.n);
          unsigned *s_cs = reinterpret_cast<unsigned *>(s_dyn + c.n);
          for (int q = tid; q <= c.ncell; q += NT) s_cs[q] = gload((const int *)p.cell_start, q);
          __syncthreads();
          tpos = s_dyn;
          cstart = s_cs;
          list_area = s_cs + cs_words;
        }
        unsigned *cand = list_area + wv * kWaveCand;
        // this piece's slots of the sorted arrays into place, coalesced (the list
        // build below only reads the sorted copies)
        for (int t = J.w * NT + tid; t < c.n; t += J.g * NT)
          place_sorted(p, cur, t, gload(p.t_pos, t));
        // one wave per cell (list_cell_particles), cells dealt round-robin over the waves
        // of all pieces, in a batch by rounds (list_rounds); or one wave per particle.  The
        // second half of the wave's window holds the counts.
        int kept = 0, longest = 0;
        int *wcnt = reinterpret_cast<int *>(cand + kCellWindow);
        auto direct = [&](int i, int kk, int, int jj) {
          if (kk < c.n_max) p.nbl[nbl_addr(i, kk, c)] = jj;
        };
        for (int t = J.w * NW + wv; !by_cell && t < c.n; t += J.g * NW) {
          const int kt = list_wave_one<false>(c, p, cur, t, cand, s_cs2, tpos, cstart, longest);
          if (lane == 0) kept += kt;
        }
        if constexpr (kRounds) {
          if (by_cell)
            list_rounds<TP, NT>(c, p, J.w, J.g, reinterpret_cast<unsigned short *>(list_area), s_cs2, tpos, cstart, kept,
                                longest);
        }
        for (int cell = J.w * NW + wv; !kRounds && by_cell && cell < c.ncell; cell += J.g * NW) {
          const unsigned e1 = min(cstart[cell + 1], (unsigned)c.n), e0 = min(cstart[cell], e1);
          const int ne = (int)(e1 - e0);
          if (ne == 0) continue;  // uniform over the wave
          if (ne > kWaveCand - kCellWindow) {  // more particles than count slots: one at a time
            for (unsigned t = e0; t < e1; ++t) {
              const int kt = list_wave_one<false>(c, p, cur, (int)t, cand, s_cs2, tpos, cstart, longest);
              if (lane == 0) kept += kt;
            }
            continue;
          }
          for (int l = lane; l < ne; l += 64) wcnt[l] = 0;
          int cx, cy, cz;
          cell_coords(tpos[e0], c, cx, cy, cz);
          list_cell_particles<BIG>(c, p, cx, cy, cz, (int)e0, (int)e1, cand, wcnt, s_cs2, tpos, cstart, direct);
          for (int l = lane; l < ne; l += 64) {
            const int cn = wcnt[l];
            p.nnb[e0 + l] = min(cn, c.n_max);
            kept += min(cn, c.n_max);
            longest = max(longest, cn);
          }
        }
        list_tally(kept, longest, c.n_max, p.ctl);
        if (!coop_barrier(p.bar_flags, J.g, J.w, ++k, 0, p.ctl, &s_ok, &s_any)) return;
      }
      if (!BIG && !prefilled) fill_positions<NT>(s_dyn, p.pos[cur], c.n);
      prefilled = false;
      __syncthreads();
      // positions of the step: the LDS copy, or device memory for a large system
      const float4 *spos = BIG ? (const float4 *)global_view(p.pos[cur]) : s_dyn;
      // this piece's wave units: unit q is wave q % wpv of owned block q / wpv; the
      // waves run their units without waiting for each other, and the wave partials
      // go to the system's partials buffer after the G block partials
      const int my_blocks = G > J.w ? (G - J.w + J.g - 1) / J.g : 0;
      const int my_units = my_blocks * wpv;
      // block partials alternate between two sets by step parity: a piece may write
      // the next step's partials while a slower piece still reads this step's
      BlockPartial *bpart = p.part + (step & 1) * G;
      // wave partials: in LDS (indexed by q) when this piece has few units, else in
      // the system's partials buffer (indexed by the unit)
      const bool wp_lds = my_units <= kLdsUnits;
      BlockPartial *wpart = p.part + 2 * G;
      for (int q = wv; q < my_units; q += NW) {
        const int b = J.w + (q / wpv) * J.g;
        const int u = b * wpv + q % wpv;
        const int gt = u * 64 + lane;
        const int i = gt / TP, t = gt % TP;
        const bool active = i < c.n;
        float fx = 0.f, fy = 0.f, fz = 0.f, uu = 0.f, w = 0.f;
        float4 pi = make_float4(0.f, 0.f, 0.f, 0.f);
        float4 vo = pi, l0 = pi, kc = pi;
        int4 im = make_int4(0, 0, 0, 0);
        const int ic = active ? i : c.n - 1;
        pi = BIG ? gload(p.pos[cur], ic) : s_dyn[ic];
        if (active) {
          if (t == 0) {
            vo = gload(p.vel, i);
            im = gload(p.img, i);
            l0 = gload(p.last, i);
          }
        }
        force_lane<TP, METHOD, kMultiBatch<TP, NT>::value, kMultiSlim<TP, BIG, NT>::value>(ic, t, active, pi, spos, nblg, nnbg, sp, c, fx, fy, fz,
                                                                  uu, w);
        fx = lane_sum<TP>(fx);
        fy = lane_sum<TP>(fy);
        fz = lane_sum<TP>(fz);
        uu = lane_sum<TP>(uu);
        w = lane_sum<TP>(w);
        BlockPartial v = zero_partial();
        if (active && t == 0)
          integrate_one<0>(c, p, cur, i, pi, vo, im, l0, kc, 0.0, 0.0, 0.0, xi, fx, fy, fz, uu, w, v);
        wave_reduce(v);
        if (lane == 0) {
          if (wp_lds)
            s_wp[q] = v;
          else
            wpart[u] = v;
          if (v.disp2 > c.half_skin2) s_bit = 1;
        }
      }
      __syncthreads();
      // owned block partials: each block's waves in index order (as group_reduce)
      for (int r = tid; r < my_blocks; r += NT) {
        const int b = J.w + r * J.g;
        BlockPartial a = wp_lds ? s_wp[r * wpv] : wpart[b * wpv];
        for (int q = 1; q < wpv; ++q) fold(a, wp_lds ? s_wp[r * wpv + q] : wpart[b * wpv + q]);
        bpart[b] = a;
      }
      if (!coop_barrier(p.bar_flags, J.g, J.w, ++k, s_bit, p.ctl, &s_ok, &s_any)) return;
      // piece 0 loads the control words now, beside the partials of the reduction
      CtlView cv{};
      if (J.w == 0 && tid == 0) cv = load_ctl(p.ctl);
      // every piece: the reduction of k_finish (1024 threads, each thread here
      // standing in for threads tid and tid + NT of that workgroup); with at most
      // 1024 blocks each thread's partials are loaded first, so that the positions
      // of the next step (loaded now when no rebuild is due and this is the
      // workgroup's only job) arrive in the same round trip
      BlockPartial a0 = zero_partial(), a1 = zero_partial();
      if (G <= 1024) {
        BlockPartial q0 = zero_partial(), q1 = zero_partial();
        if (tid < G) q0 = bpart[tid];
        if (NT < 1024 && tid + NT < G) q1 = bpart[tid + NT];
        prefilled = !BIG && nj == 1 && !s_any && step + 1 < nsteps;
        if (prefilled) fill_positions<NT>(s_dyn, p.pos[cur ^ 1], c.n);
        if (tid < G) fold(a0, q0);
        if (NT < 1024 && tid + NT < G) fold(a1, q1);
      } else {
        for (int b = tid; b < G; b += 1024) fold(a0, bpart[b]);
        for (int b = tid + NT; NT < 1024 && b < G; b += 1024) fold(a1, bpart[b]);
      }
      // a wave with no blocks holds zero partials, whose butterfly gives zeros again
      if (wv * 64 < G) wave_reduce(a0);
      if (NT < 1024 && NT + wv * 64 < G) wave_reduce(a1);
      if (lane == 0) {
        s_waves[wv] = a0;
        if (NT < 1024) s_waves[wv + NW] = a1;
      }
      __syncthreads();
      if (tid == 0) {
        // the waves of k_finish that hold data (as its group_reduce folds them)
        BlockPartial a = s_waves[0];
        const int used = min(16, (G + 63) / 64);
        for (int q = 1; q < used; ++q) fold(a, s_waves[q]);
        a.t0 = 0ull;
        a.t1 = 0ull;
        if (J.w == 0) {
          finish_step(c, p, a, cv);  // the one writer of the control block
          s_due = resort_due(c, cv.n_rebuilds) ? 1 : 0;
        }
        if (c.thermostat) s_xi[j] = xi_next(c, xi, a.ke_half);
        s_rebuild[j] = s_any;  // = (max displacement^2 > (skin/2)^2), as finish_step decides
      }
      __syncthreads();
      cur ^= 1;
      if (!BIG && s_rebuild[j]) {
        // spatial sort of the new positions by piece 0, as k_finish does
        if (J.w == 0) {
          if (c.list_kind == 4 && !s_due) {  // all-pairs lists sort only when a re-sort is due
            if (tid == 0) {
              begin_build(p.ctl);
              p.ctl->resorted = 0;
            }
          } else {
            unsigned *scnt = reinterpret_cast<unsigned *>(s_dyn);
            sort_small_shared<1>(c, p, cur, scnt, reinterpret_cast<int *>(scnt + kSmallCells + 1));
          }
        }
        // every piece learns whether the build ahead starts from a re-sort (its
        // decision depends on the build count, which piece 0 holds)
        if (step + 1 < nsteps && !coop_barrier(p.bar_flags, J.g, J.w, ++k, J.w == 0 ? s_due : 0, p.ctl, &s_ok, &s_any))
          return;
        if (tid == 0) s_resorted[j] = c.list_kind == 4 ? s_any : 1;
      }
      if (tid == 0) {
        s_cur[j] = cur;
        s_k[j] = k;
      }
    }
  }
}

template <int TP, bool BIG, int NT>
const void *multi_fn(int method) {
  return method == 0 ? (const void *)k_multi<TP, 0, BIG, NT>
         : method == 1 ? (const void *)k_multi<TP, 1, BIG, NT>
         : method == 2 ? (const void *)k_multi<TP, 2, BIG, NT>
         : method == 3 ? (const void *)k_multi<TP, 3, BIG, NT>
         : method == 4 ? (const void *)k_multi<TP, 4, BIG, NT>
                       : (const void *)k_multi<TP, 5, BIG, NT>;
}

// ---------------------------------------------------------------- start of a stepping call

// One launch at the start of srmd_step: the call's trace settings go into the
// control block, and the dynamic state the call starts from (positions, velocities,
// last-build positions, images and ids, precision residuals and the control block
// itself) is copied into the replay snapshot.
static __global__ __launch_bounds__(256) void k_call_begin(SysConst c, SysPtrs p, Snapshot snap, int cur, int thermo_every,
                                                           long long trace_cap, long long nsteps) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) {
    Control k = *p.ctl;
    k.thermo_every = thermo_every;
    k.trace_cap = trace_cap;
    k.n_records = 0;
    k.cur = cur;
    k.stop = k.step + nsteps;
    *p.ctl = k;
    *snap.ctl = k;
  }
  if (i < c.n) {
    snap.pos[i] = p.pos[cur][i];
    snap.vel[i] = p.vel[i];
    snap.last[i] = p.last[i];
    snap.img[i] = p.img[i];
    if (snap.kahan) snap.kahan[i] = p.kahan[i];
    if (snap.pos64) {
      snap.pos64[3 * i] = p.pos64[3 * i];
      snap.pos64[3 * i + 1] = p.pos64[3 * i + 1];
      snap.pos64[3 * i + 2] = p.pos64[3 * i + 2];
    }
  }
}

// The words of a run-ahead chain: the position buffer of the next step and the last step.
static __global__ void k_arm(Control *ctl, int cur, long long nsteps) {
  ctl->cur = cur;
  ctl->stop = ctl->step + nsteps;
}

// ---------------------------------------------------------------- state transfers

// The state in original particle order: slot k goes to entry img[k].w of the output
// arrays.  Bound by its scattered 12-byte writes; on one host thread the permutation
// made srmd_get_state take 31-34 ms at 1 024 000 particles, with it here 5.5 ms, which
// is the copies to the host.
static __global__ __launch_bounds__(256) void k_state_out(SysPtrs p, int n, int cur, StateXfer o) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int4 im = p.img[k];
  if (im.w < 0 || im.w >= n) {
    *o.bad = 1;
    return;
  }
  const size_t d = 3 * (size_t)im.w;
  const float4 r = p.pos[cur][k];
  if (o.pos) {
    o.pos[d] = r.x;
    o.pos[d + 1] = r.y;
    o.pos[d + 2] = r.z;
  }
  if (o.vel) {
    const float4 v = p.vel[k];
    o.vel[d] = v.x;
    o.vel[d + 1] = v.y;
    o.vel[d + 2] = v.z;
  }
  if (o.image) {
    o.image[d] = im.x;
    o.image[d + 1] = im.y;
    o.image[d + 2] = im.z;
  }
  if (o.force) {
    const float4 f = p.force[k];
    o.force[d] = f.x;
    o.force[d + 1] = f.y;
    o.force[d + 2] = f.z;
  }
  if (o.pos64) {
    const size_t e = 3 * (size_t)k;
    o.pos64[d] = p.pos64 ? p.pos64[e] : (double)r.x;
    o.pos64[d + 1] = p.pos64 ? p.pos64[e + 1] : (double)r.y;
    o.pos64[d + 2] = p.pos64 ? p.pos64[e + 2] : (double)r.z;
  }
}

// x wrapped into [-L/2, L/2) in float64, rounded to float32 (onto +L/2: the periodic
// twin), as the host wraps the positions of a new system.
__device__ __forceinline__ float wrap_side(float x, double Ld, float L, float halfL) {
  float f = (float)((double)x - Ld * floor((double)x / Ld + 0.5));
  if (f >= halfL) f -= L;
  if (f < -halfL) f += L;
  return f;
}

// A new state from the caller's arrays (in.pos and in.vel; nullptr keeps the current
// one), in two passes: k_state_order puts the current positions, types and velocities
// into original order (into the idle position buffer and the sort's velocity copy),
// and k_state_in writes the system's arrays in that order: wrapped positions, also as
// the last-build ones, identity ids, image counters and residuals cleared, errors
// cleared and a rebuild requested.
static __global__ __launch_bounds__(256) void k_state_order(SysPtrs p, int n, int cur) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int id = p.img[k].w;
  if (id < 0 || id >= n) return;
  p.pos[cur ^ 1][id] = p.pos[cur][k];
  p.t_vel[id] = p.vel[k];
}

static __global__ __launch_bounds__(256) void k_state_in(SysPtrs p, int n, int cur, float3 L, StateXfer in) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) {
    p.ctl->error = 0;
    p.ctl->rebuild = 1;
  }
  if (i >= n) return;
  float4 r = p.pos[cur ^ 1][i], v = p.t_vel[i];
  const size_t d = 3 * (size_t)i;
  if (in.pos) {
    r.x = in.pos[d];
    r.y = in.pos[d + 1];
    r.z = in.pos[d + 2];
  }
  if (in.vel) {
    v.x = in.vel[d];
    v.y = in.vel[d + 1];
    v.z = in.vel[d + 2];
  }
  v.w = 0.f;
  r.x = wrap_side(r.x, (double)L.x, L.x, 0.5f * L.x);
  r.y = wrap_side(r.y, (double)L.y, L.y, 0.5f * L.y);
  r.z = wrap_side(r.z, (double)L.z, L.z, 0.5f * L.z);
  p.pos[cur][i] = r;
  p.last[i] = r;
  p.vel[i] = v;
  p.img[i] = make_int4(0, 0, 0, i);
  if (p.pos64) {
    p.pos64[d] = (double)r.x;
    p.pos64[d + 1] = (double)r.y;
    p.pos64[d + 2] = (double)r.z;
  }
  if (p.kahan) p.kahan[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

// ---------------------------------------------------------------- stateless force evaluation

// The caller's arrays as the source of the sort: positions (x, y, z per particle) wrapped
// into [-L/2, L/2) as srmd_create wraps them, zero velocities and images, identity ids.  A
// type out of range is taken as 0 with its image x counter set to 1 (reported by
// k_direct_out), so that no table lookup leaves the pair tables.
struct SortDirect {
  const SysConst &c;
  const SysPtrs &p;
  const float *__restrict__ xyz;
  const int *__restrict__ type;
  __device__ void get(int i, float4 &q, int &id) const {
    float r[3];
    for (int d = 0; d < 3; ++d) {
      const double x = (double)xyz[3 * i + d], L = c.Ld[d];
      float f = (float)(x - L * floor(x / L + 0.5));
      if (f >= c.halfL[d]) f -= c.L[d];
      if (f < -c.halfL[d]) f += c.L[d];
      r[d] = f;
    }
    const int ty = type[i];
    q = make_float4(r[0], r[1], r[2], __int_as_float(ty < 0 || ty >= c.ntypes ? 0 : ty));
    id = i;
  }
  __device__ void put(int i, unsigned dst, int) const {
    const int ty = type[i];
    p.t_vel[dst] = make_float4(0.f, 0.f, 0.f, 0.f);
    p.t_img[dst] = make_int4(ty < 0 || ty >= c.ntypes ? 1 : 0, 0, 0, i);
  }
};

// Start of a stateless force evaluation in caller-provided scratch: the control block
// cleared with a list build requested, *status cleared, and the spatial sort straight from
// the caller's arrays.  A small system's evaluation is a chain of launches of a few
// microseconds each, so the set-up is not a launch of its own, nor the reduction
// (k_direct_out): 36.8 -> 31.5 us for 1500 particles.
static __global__ __launch_bounds__(1024) void k_direct_sort(SysConst c, SysPtrs p, const float *__restrict__ xyz,
                                                      const int *__restrict__ type, int *status) {
  __shared__ unsigned s_cnt[kSmallCells + 1];
  __shared__ int s_id[kSmallN];
  int *w = reinterpret_cast<int *>(p.ctl);
  if (threadIdx.x < sizeof(Control) / sizeof(int)) w[threadIdx.x] = 0;
  __syncthreads();
  if (threadIdx.x == 0) {
    p.ctl->rebuild = 1;
    *status = 0;
  }
  sort_small_from<1024>(c, p, s_cnt, s_id, SortDirect{c, p, xyz, type});
}

// End of a stateless force evaluation: forces in original particle order; block 0 also
// reduces the G block partials (as k_finish does) to the float64 potential energy and
// virial and writes into *status the error bits (bit 0 non-finite force, bit 1 list
// capacity exceeded); bit 2 of it stands for a type out of range.
static __global__ __launch_bounds__(1024) void k_direct_out(SysConst c, SysPtrs p, int G, float *__restrict__ force,
                                                     double *__restrict__ energy, int *status) {
  __shared__ BlockPartial s_waves[16];
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < c.n) {
    const int4 im = p.img[t];
    if (im.x != 0) atomicOr(status, 4);
    const int id = im.w;
    const float4 f = p.force[t];
    if (id >= 0 && id < c.n) {
      force[3 * id] = f.x;
      force[3 * id + 1] = f.y;
      force[3 * id + 2] = f.z;
    }
  }
  if (blockIdx.x != 0) return;
  BlockPartial a = zero_partial();
  for (int b = threadIdx.x; b < G; b += blockDim.x) {
    const BlockPartial q = p.part[b];
    a.pe += q.pe;
    a.w += q.w;
    a.nonfinite |= q.nonfinite;
  }
  group_reduce(a, s_waves, (int)blockDim.x, (G + 63) / 64);
  if (threadIdx.x == 0) {
    energy[0] = a.pe;
    energy[1] = a.w;
    const int e = (p.ctl->error | (a.nonfinite ? 1 : 0)) & 3;
    if (e) atomicOr(status, e);
  }
}

// ---------------------------------------------------------------- launchers

// Threads per particle for which the staged kernels exist.
constexpr bool staged_tp(int tp) { return tp <= 4; }

// Dynamic LDS of a step or force workgroup that copies its regions.
inline size_t stage_lds_bytes(const SysConst &c) { return sizeof(float4) * (size_t)c.stage_lds; }

// Allow a staged kernel the LDS it needs (raised once per size; a host call, not a
// stream operation, so it may run during a capture).
template <class F>
hipError_t allow_lds(F *fn, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

template <int TP>
hipError_t launch_step_tp(int method, int prec, dim3 g, dim3 b, hipStream_t st, const SysConst &c,
                                 const SysPtrs &p, int cur, int tail, size_t lds) {
#define SRMD_STEP_CASE(M, P)                                                                 \
  if (method == M && prec == P) {                                                            \
    if constexpr (staged_tp(TP)) {                                                           \
      if (c.stage) {                                                                         \
        const size_t region = stage_lds_bytes(c);                                            \
        const hipError_t e = allow_lds(k_step<TP, M, P, true>, region);                      \
        if (e != hipSuccess) return e;                                                       \
        hipLaunchKernelGGL((k_step<TP, M, P, true>), g, b, region, st, c, p, cur, tail);     \
        return hipGetLastError();                                                            \
      }                                                                                      \
    }                                                                                        \
    hipLaunchKernelGGL((k_step<TP, M, P, false>), g, b, lds, st, c, p, cur, tail);           \
    return hipGetLastError();                                                                \
  }
  SRMD_STEP_CASE(0, 0) SRMD_STEP_CASE(0, 1) SRMD_STEP_CASE(0, 2)
  SRMD_STEP_CASE(1, 0) SRMD_STEP_CASE(1, 1) SRMD_STEP_CASE(1, 2)
  SRMD_STEP_CASE(2, 0) SRMD_STEP_CASE(2, 1) SRMD_STEP_CASE(2, 2)
  SRMD_STEP_CASE(3, 0) SRMD_STEP_CASE(3, 1) SRMD_STEP_CASE(3, 2)
  SRMD_STEP_CASE(4, 0) SRMD_STEP_CASE(4, 1) SRMD_STEP_CASE(4, 2)
  SRMD_STEP_CASE(5, 0) SRMD_STEP_CASE(5, 1) SRMD_STEP_CASE(5, 2)
#undef SRMD_STEP_CASE
  return hipErrorInvalidValue;
}

template <int TP, int METHOD>
hipError_t launch_force_of(dim3 g, dim3 b, hipStream_t st, const SysConst &c, const SysPtrs &p, int cur) {
  if constexpr (staged_tp(TP)) {
    if (c.stage) {
      const size_t region = stage_lds_bytes(c);
      const hipError_t e = allow_lds(k_force<TP, METHOD, true>, region);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL((k_force<TP, METHOD, true>), g, b, region, st, c, p, cur);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((k_force<TP, METHOD, false>), g, b, 0, st, c, p, cur);
  return hipGetLastError();
}

template <int TP>
hipError_t launch_force_tp(int method, dim3 g, dim3 b, hipStream_t st, const SysConst &c, const SysPtrs &p, int cur) {
  switch (method) {
    case 0: return launch_force_of<TP, 0>(g, b, st, c, p, cur);
    case 1: return launch_force_of<TP, 1>(g, b, st, c, p, cur);
    case 2: return launch_force_of<TP, 2>(g, b, st, c, p, cur);
    case 3: return launch_force_of<TP, 3>(g, b, st, c, p, cur);
    case 4: return launch_force_of<TP, 4>(g, b, st, c, p, cur);
    case 5: return launch_force_of<TP, 5>(g, b, st, c, p, cur);
    default: return hipErrorInvalidValue;
  }
}

// The templated kernels are compiled once per threads-per-particle value in a
// translation unit of their own (this file with SRMD_TP defined), everything else in
// the one without it.
#define SRMD_KERNELS_OF(PREFIX, TP)                                                                                     \
  PREFIX template hipError_t launch_step_tp<TP>(int, int, dim3, dim3, hipStream_t, const SysConst &, const SysPtrs &,   \
                                                int, int, size_t);                                                      \
  PREFIX template hipError_t launch_force_tp<TP>(int, dim3, dim3, hipStream_t, const SysConst &, const SysPtrs &, int); \
  PREFIX template const void *multi_fn<TP, false, kPersistThreads>(int);
#define SRMD_KERNELS_TO_8(PREFIX, TP)                                     \
  PREFIX template const void *multi_fn<TP, true, kPersistThreads>(int);   \
  PREFIX template const void *multi_fn<TP, false, kBatchThreads>(int);
#ifdef SRMD_TP
SRMD_KERNELS_OF(, SRMD_TP)
#if SRMD_TP <= 8
SRMD_KERNELS_TO_8(, SRMD_TP)
#endif
#else
SRMD_KERNELS_OF(extern, 1)
SRMD_KERNELS_OF(extern, 2)
SRMD_KERNELS_OF(extern, 4)
SRMD_KERNELS_OF(extern, 8)
SRMD_KERNELS_OF(extern, 16)
SRMD_KERNELS_OF(extern, 32)
SRMD_KERNELS_OF(extern, 64)
SRMD_KERNELS_TO_8(extern, 1)
SRMD_KERNELS_TO_8(extern, 2)
SRMD_KERNELS_TO_8(extern, 4)
SRMD_KERNELS_TO_8(extern, 8)

// The persistent kernel for (tp, method) with a workgroup of threads; the large-system
// form exists for tp <= 8.
static const void *multi_fn_of(int tp, int method, bool big, int threads) {
  if (big) {
    switch (tp) {
      case 1: return multi_fn<1, true, kPersistThreads>(method);
      case 2: return multi_fn<2, true, kPersistThreads>(method);
      case 4: return multi_fn<4, true, kPersistThreads>(method);
      case 8: return multi_fn<8, true, kPersistThreads>(method);
      default: return nullptr;
    }
  }
  if (threads == kBatchThreads) {
    switch (tp) {
      case 1: return multi_fn<1, false, kBatchThreads>(method);
      case 2: return multi_fn<2, false, kBatchThreads>(method);
      case 4: return multi_fn<4, false, kBatchThreads>(method);
      case 8: return multi_fn<8, false, kBatchThreads>(method);
      default: return nullptr;
    }
  }
  switch (tp) {
    case 1: return multi_fn<1, false, kPersistThreads>(method);
    case 2: return multi_fn<2, false, kPersistThreads>(method);
    case 4: return multi_fn<4, false, kPersistThreads>(method);
    case 8: return multi_fn<8, false, kPersistThreads>(method);
    case 16: return multi_fn<16, false, kPersistThreads>(method);
    case 32: return multi_fn<32, false, kPersistThreads>(method);
    case 64: return multi_fn<64, false, kPersistThreads>(method);
    default: return nullptr;
  }
}

bool multi_big_supported(int tp) { return multi_fn_of(tp, 0, true, kPersistThreads) != nullptr; }

// Threads of a workgroup of the persistent kernel for a batch.
int batch_threads(int tp) { return tp <= kBatchMaxTp ? kBatchThreads : kPersistThreads; }

int persist_threads() { return kPersistThreads; }

// Launch k_multi over nwg workgroups.  cooperative: some system is split over
// several workgroups, which must then all be resident at once.
hipError_t launch_multi(int tp, int method, bool big, int threads, int nwg, size_t lds, hipStream_t st,
                        const ReplicaDesc *reps, const CoopJob *jobs, const int *job_off, int nsteps,
                        bool cooperative) {
  const void *fn = multi_fn_of(tp, method, big, threads);
  if (!fn || nwg < 1) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  int lds_bytes = (int)lds;
  void *args[] = {&reps, &jobs, &job_off, &nsteps, &lds_bytes};
  if (cooperative) return hipLaunchCooperativeKernel(fn, dim3(nwg), dim3(threads), args, (unsigned)lds, st);
  return hipLaunchKernel(fn, dim3(nwg), dim3(threads), args, lds, st);
}

// Workgroups of the persistent kernel the device holds at once (at most 256).
int multi_max_groups(int tp, int method, bool big, int threads, size_t lds) {
  const void *fn = multi_fn_of(tp, method, big, threads);
  if (!fn) return 0;
  if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) return 0;
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, lds) != hipSuccess) return 0;
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  return std::min(per_cu * cus, kCoopMaxGroups);
}

int multi_max_jobs() { return kMaxJobs; }

// Dynamic LDS of the persistent kernel: the positions of a step, the sort's scratch,
// and where it fits in 150 KiB, the list build's copies of the sorted positions and
// the cell starts beside the candidate windows (up to 4096 cells counted).
size_t multi_lds_bytes(int n_max_particles, int threads) {
  const size_t pos = 16 * (size_t)n_max_particles;
  const size_t scratch = 4 * (size_t)(kSmallCells + 1 + kSmallN);
  const size_t cand = 4 * (size_t)(threads / 64 * kWaveCand);
  size_t b = std::max(pos, std::max(scratch, cand));
  // a batch's workgroup has a compute unit to itself: as much as its other arrays leave
  if (threads == kBatchThreads)
    return std::max(b, std::min<size_t>(146 * 1024, pos + 4 * (size_t)(kSmallCells + 4) + cand));
  const size_t listing = pos + 4 * (size_t)(4096 + 4) + cand;
  if (listing <= 150 * 1024) b = std::max(b, listing);
  return b;
}

int batch_max_particles() { return kSmallN; }

// Dynamic LDS of the large-system persistent kernel: the list build's candidate windows.
size_t big_lds_bytes() { return 4 * (size_t)(kPersistThreads / 64 * kWaveCand); }

int stage_units(int n) { return (n + kStageSlots - 1) / kStageSlots; }

size_t stage_list_lds(const SysConst &c) { return stage_list_bytes(c.stage_cap); }

bool stage_supported(int tp) { return staged_tp(tp); }

hipError_t launch_stage_expand(hipStream_t st, const SysConst &c, const SysPtrs &p, bool drop) {
  hipLaunchKernelGGL(k_stage_expand, dim3(stage_units(c.n)), dim3(kStageSlots), 0, st, c, p, drop ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_direct_sort(hipStream_t st, const SysConst &c, const SysPtrs &p, const float *xyz, const int *type,
                              int *status) {
  hipLaunchKernelGGL(k_direct_sort, dim3(1), dim3(1024), 0, st, c, p, xyz, type, status);
  return hipGetLastError();
}

hipError_t launch_direct_out(hipStream_t st, const SysConst &c, const SysPtrs &p, int G, float *force, double *energy,
                             int *status) {
  hipLaunchKernelGGL(k_direct_out, dim3((c.n + 1023) / 1024), dim3(1024), 0, st, c, p, G, force, energy, status);
  return hipGetLastError();
}

hipError_t launch_arm(hipStream_t st, Control *ctl, int cur, long long nsteps) {
  hipLaunchKernelGGL(k_arm, dim3(1), dim3(1), 0, st, ctl, cur, nsteps);
  return hipGetLastError();
}

hipError_t launch_state_out(hipStream_t st, const SysPtrs &p, int n, int cur, const StateXfer &o) {
  hipLaunchKernelGGL(k_state_out, dim3((n + 255) / 256), dim3(256), 0, st, p, n, cur, o);
  return hipGetLastError();
}

hipError_t launch_state_in(hipStream_t st, const SysPtrs &p, int n, int cur, const float L[3], const StateXfer &in) {
  hipLaunchKernelGGL(k_state_order, dim3((n + 255) / 256), dim3(256), 0, st, p, n, cur);
  hipLaunchKernelGGL(k_state_in, dim3((n + 255) / 256), dim3(256), 0, st, p, n, cur, make_float3(L[0], L[1], L[2]), in);
  return hipGetLastError();
}

hipError_t launch_call_begin(hipStream_t st, const SysConst &c, const SysPtrs &p, const Snapshot &snap, int cur,
                             int thermo_every, long long trace_cap, long long nsteps) {
  hipLaunchKernelGGL(k_call_begin, dim3((c.n + 255) / 256), dim3(256), 0, st, c, p, snap, cur, thermo_every, trace_cap,
                     nsteps);
  return hipGetLastError();
}

// tail = 1: the step kernel ends the step in its last workgroup (no k_finish<0>
// launch); lds = tail_lds_bytes for small systems, else 0.
hipError_t launch_step(int tp, int method, int prec, int blocks, int threads, hipStream_t st, const SysConst &c,
                       const SysPtrs &p, int cur, int tail, size_t lds) {
  const dim3 g(blocks), b(threads);
  switch (tp) {
    case 1: return launch_step_tp<1>(method, prec, g, b, st, c, p, cur, tail, lds);
    case 2: return launch_step_tp<2>(method, prec, g, b, st, c, p, cur, tail, lds);
    case 4: return launch_step_tp<4>(method, prec, g, b, st, c, p, cur, tail, lds);
    case 8: return launch_step_tp<8>(method, prec, g, b, st, c, p, cur, tail, lds);
    case 16: return launch_step_tp<16>(method, prec, g, b, st, c, p, cur, tail, lds);
    case 32: return launch_step_tp<32>(method, prec, g, b, st, c, p, cur, tail, lds);
    case 64: return launch_step_tp<64>(method, prec, g, b, st, c, p, cur, tail, lds);
    default: return hipErrorInvalidValue;
  }
}

// Dynamic LDS of a step kernel with the tail: the spatial sort's arrays for small
// systems (sorted in the tail), none otherwise; with the list built in the step
// (tail 2), at least the wave builder's candidate windows (the two uses alias).
size_t tail_lds_bytes(const SysConst &c, int threads, int tail) {
  const size_t sort = c.small_sort ? tail_sort_lds(c.n, c.ncell) : 0;
  const size_t windows = tail == 2 && c.list_kind == 1 ? sizeof(unsigned) * kWaveCand * (size_t)(threads / 64) : 0;
  return std::max(sort, windows);
}

// Bytes of a system's arrival counters (zeroed at allocation).
size_t arrive_bytes() { return kArriveBytes; }

hipError_t launch_force(int tp, int method, int blocks, int threads, hipStream_t st, const SysConst &c,
                        const SysPtrs &p, int cur) {
  const dim3 g(blocks), b(threads);
  switch (tp) {
    case 1: return launch_force_tp<1>(method, g, b, st, c, p, cur);
    case 2: return launch_force_tp<2>(method, g, b, st, c, p, cur);
    case 4: return launch_force_tp<4>(method, g, b, st, c, p, cur);
    case 8: return launch_force_tp<8>(method, g, b, st, c, p, cur);
    case 16: return launch_force_tp<16>(method, g, b, st, c, p, cur);
    case 32: return launch_force_tp<32>(method, g, b, st, c, p, cur);
    case 64: return launch_force_tp<64>(method, g, b, st, c, p, cur);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_finish(int mode, int G, int next, hipStream_t st, const SysConst &c, const SysPtrs &p) {
  if (mode == 0) hipLaunchKernelGGL((k_finish<0>), dim3(1), dim3(1024), 0, st, c, p, G, next);
  else hipLaunchKernelGGL((k_finish<1>), dim3(1), dim3(1024), 0, st, c, p, G, next);
  return hipGetLastError();
}

// Sort requested by the host for a small system (the multi-kernel sort of large
// systems always runs at the start of the step, gated on the flag).
hipError_t launch_host_sort(hipStream_t st, const SysConst &c, const SysPtrs &p, int cur) {
  if (!c.small_sort) return hipSuccess;
  hipLaunchKernelGGL(k_sort_small, dim3(1), dim3(1024), 0, st, c, p, cur);
  return hipGetLastError();
}

// Start-of-step rebuild chain: list build (small systems; the sort ran earlier) or
// the multi-kernel sort followed by the list build (large systems).
hipError_t launch_rebuild(hipStream_t st, const SysConst &c, const SysPtrs &p, int cur) {
  const int tb = 256;
  const int gb = c.list_blocks;
  if (!c.small_sort) {
    hipLaunchKernelGGL(k_bin, dim3(gb), dim3(tb), 0, st, c, p, cur);
    hipLaunchKernelGGL(k_scan, dim3(scan_tiles(c.ncell)), dim3(256), 0, st, c, p, cur);
    hipLaunchKernelGGL(k_scatter, dim3(gb), dim3(tb), 0, st, c, p, cur);
    hipLaunchKernelGGL(k_gather, dim3(gb), dim3(tb), 0, st, c, p, cur);
  }
  if (c.list_kind == 4) {
    const int lb = (c.n + 3) / 4;
    hipLaunchKernelGGL(k_list_allpairs, dim3(lb), dim3(tb), 0, st, c, p, cur);
  } else if (c.list_kind == 1) {
    const int lb = (c.n + kListWaves - 1) / kListWaves;
    hipLaunchKernelGGL(k_list_wave, dim3(lb), dim3(64 * kListWaves), 0, st, c, p, cur);
  } else if (c.stage) {
    const hipError_t e = allow_lds(k_list_stage, stage_list_lds(c));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_list_stage, dim3(stage_units(c.n)), dim3(kStageThreads), stage_list_lds(c), st, c, p,
                       cur);
  } else if (c.list_kind == 2) {
    hipLaunchKernelGGL(k_list_thread, dim3(gb), dim3(tb), 0, st, c, p, cur);
  } else if (c.list_kind == 5) {
    hipLaunchKernelGGL(k_list_row, dim3(c.nc[1] * c.nc[2]), dim3(256), 0, st, c, p, cur);
  } else {
    const int lb = (c.n + kCellSlots - 1) / kCellSlots;
    hipLaunchKernelGGL(k_list_cell, dim3(lb), dim3(64 * kCellWaves), 0, st, c, p, cur);
  }
  return hipGetLastError();
}

#endif  // SRMD_TP

}  // namespace srmd
