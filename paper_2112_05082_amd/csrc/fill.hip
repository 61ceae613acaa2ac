// Unique displacement-block fill of the global matrix (Galerkin EFIE, RWG).
//
// Z(d)[m][n] couples observer macro RWG m of the unit at lattice offset d to
// source macro RWG n of the unit at the origin (eq. (1), Sec. II-A):
//   Z_mn = j k eta sum_{a,b in +-} s_a s_b l_m l_n / (A_p A_q)
//          int_p int_q [ (r - v_a).(r' - v_b)/4 - 1/k^2 ] G(|r - r'|) dS' dS
// with the 7-point degree-5 rule on both triangles.  For triangle pairs whose
// cells are within Chebyshev distance extract_radius (the cells of the two
// units, shifted by the triangles' own cell offsets for bases that bridge two
// cells, Sec. III-B), G = 1/(4 pi R) + (exp(-jkR) - 1)/(4 pi R):
// the first term is integrated in closed form over the source triangle
// (edge-sum formulas of Wilton et al. / Graglia), the second by quadrature.
// Triangles of different coding states in the same cell overlap (coexistent
// meshes of the macro unit, Sec. III-A): the closed-form inner integral then
// has kinks along the source triangle's edges inside the observer triangle,
// so for those pairs the outer integral takes the composite rule, the 7-point
// rule on each of the 64 triangles of three midpoint subdivisions of the
// observer triangle.  Everything in FP64.
//
// Work is per triangle pair, not per entry: the integrals of a pair
//   T[a][b] = int_p int_q [ (r - P_a).(r' - Q_b)/4 - 1/k^2 ] G dS' dS
// (a, b vertices) serve every basis pair that meets on it, up to nine, where
// one thread per entry evaluates each pair once per entry (per block of the
// 1-bit unit 196 x 6,400 Green's function values instead of 49 x 4,096).
// Basis functions are cut into tiles of consecutive RWG touching at most
// kTileTri triangles; a tile pair's integrals are assembled into its entries.
//  - Blocks with no extracted pair (all but the few near d = 0): one
//    workgroup per (d, tile pair), a pair per thread, integrals in LDS
//    (fill_far_kernel).  G is symmetric, so Z(-d) is the transpose of Z(d)
//    and one evaluation fills both.
//  - The others: a pair per 8 lanes (one outer point each), or per wave for
//    the composite rule, integrals in a context workspace
//    (pair_near_kernel), then assembled (assemble_near_kernel).  One thread
//    per entry spent 12 ms on the 25 workgroups of the d = 0 block alone.
// Bound by FP64 arithmetic: about 60 instructions per Green's function value,
// 0.62 ms of issue for the 3,969 blocks of the 1-bit unit (32x32 arrays, 406 MB
// written), which took 23.9 ms by entries and takes 1.25 ms: fill_far_kernel
// 1.1, pair_near_kernel 0.087 (composite) + 0.034, assemble_near_kernel 0.006.
#include <array>

#include "fp64_math.h"
#include "r3m_common.h"

namespace r3m {
namespace {

struct Quad7 {
  double b[7][3];
  double w[7];
};

__constant__ Quad7 c_quad;

// the composite outer rule for overlapping cross-state pairs
constexpr int kSubLevels = 3;
constexpr int kSubTris = 1 << (2 * kSubLevels);  // 64
constexpr int kCompPts = 7 * kSubTris;           // 448
struct QuadComp {
  double b[kCompPts][3];
  double w[kCompPts];
};
__constant__ QuadComp c_comp;

Quad7 make_quad7() {
  Quad7 q;
  const double s15 = std::sqrt(15.0);
  const double a1 = (6.0 - s15) / 21.0, b1 = 1.0 - 2.0 * a1;
  const double a2 = (6.0 + s15) / 21.0, b2 = 1.0 - 2.0 * a2;
  const double w0 = 9.0 / 40.0, w1 = (155.0 - s15) / 1200.0, w2 = (155.0 + s15) / 1200.0;
  const double pts[7][3] = {{1.0 / 3.0, 1.0 / 3.0, 1.0 / 3.0}, {b1, a1, a1}, {a1, b1, a1},
                            {a1, a1, b1}, {b2, a2, a2}, {a2, b2, a2}, {a2, a2, b2}};
  const double ws[7] = {w0, w1, w1, w1, w2, w2, w2};
  for (int i = 0; i < 7; ++i) {
    for (int c = 0; c < 3; ++c) q.b[i][c] = pts[i][c];
    q.w[i] = ws[i];
  }
  return q;
}

// 7-point rule on each triangle of kSubLevels midpoint subdivisions, in
// barycentric coordinates of the parent triangle (weights sum to one)
QuadComp make_composite(const Quad7& q7) {
  // corners of the sub-triangles, in barycentric coordinates
  std::vector<std::array<std::array<double, 3>, 3>> tris(1);
  for (int c = 0; c < 3; ++c)
    for (int d = 0; d < 3; ++d) tris[0][c][d] = c == d ? 1.0 : 0.0;
  for (int lev = 0; lev < kSubLevels; ++lev) {
    std::vector<std::array<std::array<double, 3>, 3>> next;
    for (const auto& t : tris) {
      std::array<double, 3> m[3];  // midpoints of the edges opposite corners 2, 0, 1
      for (int d = 0; d < 3; ++d) {
        m[0][d] = 0.5 * (t[0][d] + t[1][d]);
        m[1][d] = 0.5 * (t[1][d] + t[2][d]);
        m[2][d] = 0.5 * (t[2][d] + t[0][d]);
      }
      next.push_back({t[0], m[0], m[2]});
      next.push_back({m[0], t[1], m[1]});
      next.push_back({m[2], m[1], t[2]});
      next.push_back({m[1], m[2], m[0]});
    }
    tris.swap(next);
  }
  QuadComp q;
  int i = 0;
  for (const auto& t : tris)
    for (int j = 0; j < 7; ++j, ++i) {
      for (int d = 0; d < 3; ++d)
        q.b[i][d] = q7.b[j][0] * t[0][d] + q7.b[j][1] * t[1][d] + q7.b[j][2] * t[2][d];
      q.w[i] = q7.w[j] / kSubTris;
    }
  return q;
}

struct V3 {
  double x, y, z;
};
__device__ inline V3 operator-(V3 a, V3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ inline V3 operator+(V3 a, V3 b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ inline V3 operator*(double s, V3 a) { return {s * a.x, s * a.y, s * a.z}; }
__device__ inline double dot(V3 a, V3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ inline V3 cross(V3 a, V3 b) {
  return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
__device__ inline double norm(V3 a) { return sqrt(dot(a, a)); }

// int_T 1/R dS' (S) and int_T (r' - r)/R dS' (V) for the flat triangle (t0,t1,t2)
__device__ void static_potentials(V3 r, V3 t0, V3 t1, V3 t2, double& S, V3& V) {
  V3 nn = cross(t1 - t0, t2 - t0);
  V3 n = (1.0 / norm(nn)) * nn;
  const double d = dot(n, r - t0);
  const double ad = fabs(d);
  V3 rho = r - d * n;
  S = 0.0;
  V3 Vp = {0.0, 0.0, 0.0};
  V3 tv[3] = {t0, t1, t2};
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    V3 a = tv[e], b = tv[(e + 1) % 3];
    V3 ab = b - a;
    const double len = norm(ab);
    V3 lh = (1.0 / len) * ab;
    V3 uh = cross(lh, n);  // outward in-plane normal of the edge
    const double tt = dot(a - rho, uh);
    const double lm = dot(a - rho, lh);
    const double lp = dot(b - rho, lh);
    const double R0sq = tt * tt + d * d;
    const double Rm = sqrt(lm * lm + R0sq);
    const double Rp = sqrt(lp * lp + R0sq);
    double f = 0.0;
    if (sqrt(R0sq) > 1e-12 * len) {
      if (lm >= 0.0)
        f = log((Rp + lp) / (Rm + lm));
      else if (lp <= 0.0)
        f = log((Rm - lm) / (Rp - lp));
      else
        f = log((Rp + lp) * (Rm - lm) / R0sq);
    }
    double term = tt * f;
    if (ad > 0.0) term -= ad * (atan(tt * lp / (R0sq + ad * Rp)) - atan(tt * lm / (R0sq + ad * Rm)));
    S += term;
    const double c = 0.5 * (R0sq * f + lp * Rp - lm * Rm);
    Vp = Vp + c * uh;
  }
  V = Vp - (d * S) * n;
}

__device__ inline V3 load_vertex(const double* tv, int t, int a) {
  const double* p = tv + 9 * t + 3 * a;
  return {p[0], p[1], p[2]};
}

constexpr int kTileTri = 32;                       // triangles of a tile
constexpr int kTilePairs = kTileTri * kTileTri;    // pairs of a tile pair
constexpr int kNearWsBytes = 64 << 20;             // integrals of the near blocks held at once

// a tile: RWG [m0, m0 + count) and the triangles they touch
struct FillTile {
  int32_t m0, count, n_tri, pad;
  int32_t tri[kTileTri];
};
struct FillDev {
  const FillTile* tiles;  // [n_tiles]
  // per RWG: the tile's local index of its two triangles (bits 0-7, 8-15) and
  // the free vertex in each (bits 16-17, 18-19)
  const uint32_t* rwg;
  int32_t n_tiles;
};

struct C128 {
  double re, im;
};

// The 7-point rule on barycentric coordinates: point 0 is the centroid, point
// 1 + v (4 + v) has coordinate b1 (b2) at vertex v and a1 (a2) at the others.
// A sum over points of w b_v g is then one sum common to the three vertices
// (cA, cB, cC per point kind) plus vertex v's own points (dB, dC).
struct Rule7 {
  double cA, cB, cC, dB, dC;
};
__constant__ Rule7 c_rule;

// Entry (m, n) from a tile pair's integrals T [9][kTilePairs] (a b, then p q)
__device__ __forceinline__ C128 entry_of(const double2* T, const GeomDev& g, const FillDev& f, const FillTile& I,
                                         const FillTile& J, int m, int nn) {
  const uint32_t um = f.rwg[m], un = f.rwg[nn];
  const double lm = g.rwg_len[m], ln = g.rwg_len[nn];
  double re = 0.0, im = 0.0;
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const int p = (um >> (8 * a)) & 255, fa = (um >> (16 + 2 * a)) & 3;
    const double cm = (a == 0 ? lm : -lm) / g.tri_area[I.tri[p]];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int q = (un >> (8 * b)) & 255, fb = (un >> (16 + 2 * b)) & 3;
      const double cc = cm * ((b == 0 ? ln : -ln) / g.tri_area[J.tri[q]]);
      const double2 t = T[(fa * 3 + fb) * kTilePairs + p * kTileTri + q];
      re += cc * t.x;
      im += cc * t.y;
    }
  }
  return {re, im};
}

// z = j k eta v into out[idx]; non-finite entries set the flag
template <typename OutT>
__device__ __forceinline__ void store_entry(OutT* out, size_t idx, C128 v, double keta, int* flag) {
  const double z_re = -keta * v.im, z_im = keta * v.re;
  if (!(isfinite(z_re) && isfinite(z_im))) atomicOr(flag, 1);
  out[2 * idx] = (OutT)z_re;
  out[2 * idx + 1] = (OutT)z_im;
}

// Blocks without extracted pairs: displacement slot s of the first half and
// its mirror image nslots - 1 - s (-d), tile pair (I, J).  1,024 threads, one
// pair each; 147 KB of integrals and 11 KB of quadrature points in LDS, so one
// workgroup (four waves per SIMD) per CU.  Points and integrals are stored
// source-fastest: lanes read consecutive words.  A launch takes the workgroups
// from tile pair tp0 of slot slot0 on (see max_workgroups).
template <typename OutT>
__global__ void __launch_bounds__(kTilePairs)
fill_far_kernel(GeomDev g, FillDev f, double k, double px, double py, int Dx, int Dy, int near_x, int near_y,
                int slot0, int tp0, OutT* __restrict__ out, int* __restrict__ flag) {
  extern __shared__ double2 far_lds[];
  double2* T = far_lds;                                                   // [9][kTilePairs]
  double* Po = reinterpret_cast<double*>(far_lds + 9 * kTilePairs);       // [7][3][kTileTri]
  double* Qo = Po + 21 * kTileTri;
  const int n_tp = f.n_tiles * f.n_tiles;
  const int id = tp0 + (int)blockIdx.x, slot = slot0 + id / n_tp, tp = id % n_tp;
  const int dx = slot % (2 * Dx + 1) - Dx, dy = slot / (2 * Dx + 1) - Dy;
  if (abs(dx) <= near_x && abs(dy) <= near_y) return;  // uniform: a near block
  const FillTile& I = f.tiles[tp / f.n_tiles];
  const FillTile& J = f.tiles[tp % f.n_tiles];
  const V3 off = {dx * px, dy * py, 0.0};
  for (int t = threadIdx.x; t < 2 * 7 * kTileTri; t += blockDim.x) {
    const int side = t / (7 * kTileTri), i = t / kTileTri % 7, l = t % kTileTri;
    const FillTile& X = side ? J : I;
    if (l < X.n_tri) {
      const int tri = X.tri[l];
      V3 v0 = load_vertex(g.tri_v, tri, 0), v1 = load_vertex(g.tri_v, tri, 1), v2 = load_vertex(g.tri_v, tri, 2);
      if (!side) {
        v0 = v0 + off;
        v1 = v1 + off;
        v2 = v2 + off;
      }
      const V3 r = c_quad.b[i][0] * v0 + c_quad.b[i][1] * v1 + c_quad.b[i][2] * v2;
      double* o = (side ? Qo : Po) + i * 3 * kTileTri + l;
      o[0] = r.x;
      o[kTileTri] = r.y;
      o[2 * kTileTri] = r.z;
    }
  }
  __syncthreads();
  const int p = threadIdx.x / kTileTri, q = threadIdx.x % kTileTri;
  if (p < I.n_tri && q < J.n_tri) {
    const Rule7 w = c_rule;
    // M[c][c'] = sum over point pairs of w_i w_j b_ic b_jc' G
    C128 M[3][3];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int d = 0; d < 3; ++d) M[c][d] = {0.0, 0.0};
#pragma unroll 1
    for (int i = 0; i < 7; ++i) {
      // the source points are read again for every outer point (held over the
      // loop they would not fit the 128 registers of 1,024 threads)
      asm volatile("" ::: "memory");
      const V3 r = {Po[(3 * i) * kTileTri + p], Po[(3 * i + 1) * kTileTri + p], Po[(3 * i + 2) * kTileTri + p]};
      C128 t[3], tc = {0.0, 0.0};
#pragma unroll
      for (int c = 0; c < 3; ++c) t[c] = {0.0, 0.0};
#pragma unroll
      for (int j = 0; j < 7; ++j) {
        const double ex = r.x - Qo[(3 * j) * kTileTri + q], ey = r.y - Qo[(3 * j + 1) * kTileTri + q],
                     ez = r.z - Qo[(3 * j + 2) * kTileTri + q];
        const double R2 = fma(ez, ez, fma(ey, ey, ex * ex));
        const double iR = rsqrt64(R2);
        double R = R2 * iR;
        R = fma(0.5 * iR, fma(-R, R, R2), R);
        double c, s;
        cos_sin(k * R, c, s);
        const double gr = c * iR, gi = -s * iR;
        const double cw = j == 0 ? w.cA : j < 4 ? w.cB : w.cC;
        tc.re = fma(cw, gr, tc.re);
        tc.im = fma(cw, gi, tc.im);
        if (j > 0) {
          const double dw = j < 4 ? w.dB : w.dC;
          C128& tv = t[j < 4 ? j - 1 : j - 4];
          tv.re = fma(dw, gr, tv.re);
          tv.im = fma(dw, gi, tv.im);
        }
      }
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const double tr = t[d].re + tc.re, ti = t[d].im + tc.im;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const double wb = c_quad.w[i] * c_quad.b[i][c];
          M[c][d].re = fma(wb, tr, M[c][d].re);
          M[c][d].im = fma(wb, ti, M[c][d].im);
        }
      }
    }
    // T[a][b] = A_p A_q ( sum_cc' M[c][c'] (P_c - P_a).(Q_c' - Q_b) / 4 - S / k^2 ),
    // with vertices relative to each triangle's first
    const int tp_ = I.tri[p], tq = J.tri[q];
    V3 P[3], Q[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      P[c] = load_vertex(g.tri_v, tp_, c) - load_vertex(g.tri_v, tp_, 0);
      Q[c] = load_vertex(g.tri_v, tq, c) - load_vertex(g.tri_v, tq, 0);
    }
    double D[3][3];
    C128 row[3], col[3], S = {0.0, 0.0}, X = {0.0, 0.0};
#pragma unroll
    for (int c = 0; c < 3; ++c) row[c] = col[c] = {0.0, 0.0};
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        D[c][d] = dot(P[c], Q[d]);
        row[c].re += M[c][d].re;
        row[c].im += M[c][d].im;
        col[d].re += M[c][d].re;
        col[d].im += M[c][d].im;
        X.re = fma(M[c][d].re, D[c][d], X.re);
        X.im = fma(M[c][d].im, D[c][d], X.im);
      }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      S.re += row[c].re;
      S.im += row[c].im;
    }
    const double scale = g.tri_area[tp_] * g.tri_area[tq] * (1.0 / (4.0 * kPi)), invk2 = 1.0 / (k * k);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        double re = fma(S.re, D[a][b], X.re), im = fma(S.im, D[a][b], X.im);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          re = fma(-col[c].re, D[a][c], re);
          im = fma(-col[c].im, D[a][c], im);
          re = fma(-row[c].re, D[c][b], re);
          im = fma(-row[c].im, D[c][b], im);
        }
        T[(a * 3 + b) * kTilePairs + threadIdx.x] =
            make_double2(scale * fma(0.25, re, -invk2 * S.re), scale * fma(0.25, im, -invk2 * S.im));
      }
  }
  __syncthreads();
  const int n = g.n_rwg;
  const double keta = k * kEta0;
  const size_t at = (size_t)slot * n * n;
  const size_t mirror = ((size_t)(2 * Dx + 1) * (2 * Dy + 1) - 1 - slot) * n * n;
  for (int e = threadIdx.x; e < I.count * J.count; e += blockDim.x) {
    const int m = I.m0 + e / J.count, nn = J.m0 + e % J.count;
    store_entry(out, at + (size_t)m * n + nn, entry_of(T, g, f, I, J, m, nn), keta, flag);
  }
  for (int e = threadIdx.x; e < I.count * J.count; e += blockDim.x) {
    const int nn = J.m0 + e / I.count, m = I.m0 + e % I.count;
    store_entry(out, mirror + (size_t)nn * n + m, entry_of(T, g, f, I, J, m, nn), keta, flag);
  }
}

// a near work unit u: displacement (|dx| <= near_x, |dy| <= near_y) and tile pair
__device__ __forceinline__ void near_unit(int u, int n_tiles, int near_x, int near_y, int& dx, int& dy, int& ti,
                                          int& tj) {
  const int n_tp = n_tiles * n_tiles;
  const int s = u / n_tp, tp = u % n_tp;
  dx = s % (2 * near_x + 1) - near_x;
  dy = s / (2 * near_x + 1) - near_y;
  ti = tp / n_tiles;
  tj = tp % n_tiles;
}

// Integrals of the near blocks' pairs, units [u0, u0 + gridDim.y) into
// ws [unit][9][kTilePairs].  LP lanes per pair share its outer points: 8 for
// the 7-point rule (pairs that take the composite rule are left out), 64 for
// the composite rule (the others are left out).
template <int LP>
__global__ void __launch_bounds__(256)
pair_near_kernel(GeomDev g, FillDev f, double k, double px, double py, int near_x, int near_y, int extract_radius,
                 int u0, double2* __restrict__ ws) {
  constexpr bool COMP = LP == 64;
  int dx, dy, ti, tj;
  near_unit(u0 + blockIdx.y, f.n_tiles, near_x, near_y, dx, dy, ti, tj);
  const FillTile& I = f.tiles[ti];
  const FillTile& J = f.tiles[tj];
  const int pair = (blockIdx.x * 256 + threadIdx.x) / LP, sub = threadIdx.x % LP;
  const int lp = pair / kTileTri, lq = pair % kTileTri;
  if (lp >= I.n_tri || lq >= J.n_tri) return;  // uniform over the pair's lanes
  const int p = I.tri[lp], q = J.tri[lq];
  // cells of the two triangles (a bridging basis has a triangle in the
  // neighbouring cell)
  int cx = dx, cy = dy;
  if (g.tri_cell) {
    cx += g.tri_cell[2 * p] - g.tri_cell[2 * q];
    cy += g.tri_cell[2 * p + 1] - g.tri_cell[2 * q + 1];
  }
  const bool extract = abs(cx) <= extract_radius && abs(cy) <= extract_radius;
  const int sp = g.tri_state[p], sq = g.tri_state[q];
  const bool overlap = extract && cx == 0 && cy == 0 && sp >= 0 && sq >= 0 && sp != sq;
  if (overlap != COMP) return;
  const V3 off = {dx * px, dy * py, 0.0};
  V3 P[3], Q[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    P[c] = load_vertex(g.tri_v, p, c) + off;
    Q[c] = load_vertex(g.tri_v, q, c);
  }
  const double Ap = g.tri_area[p], Aq = g.tri_area[q];
  const double inv4pi = 1.0 / (4.0 * kPi), invk2 = 1.0 / (k * k);
  C128 T[3][3];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) T[a][b] = {0.0, 0.0};
#pragma unroll 1
  for (int i = sub; i < (COMP ? kCompPts : 7); i += LP) {
    const double* bi = COMP ? c_comp.b[i] : c_quad.b[i];
    const double wi = (COMP ? c_comp.w[i] : c_quad.w[i]) * Ap;
    const V3 r = bi[0] * P[0] + bi[1] * P[1] + bi[2] * P[2];
    // s = int_q g dS', m = int_q (r' - r) g dS' of the quadrature part
    double s_re = 0.0, s_im = 0.0;
    V3 m_re = {0.0, 0.0, 0.0}, m_im = {0.0, 0.0, 0.0};
#pragma unroll 1
    for (int j = 0; j < 7; ++j) {
      const V3 rp = c_quad.b[j][0] * Q[0] + c_quad.b[j][1] * Q[1] + c_quad.b[j][2] * Q[2];
      const double wj = c_quad.w[j] * Aq;
      const double R = norm(r - rp);
      const double kR = k * R;
      double g_re, g_im;
      if (extract) {
        // (exp(-jkR) - 1)/(4 pi R) = (-2 sin^2(kR/2) - j sin(kR)) / (4 pi R)
        if (R == 0.0) {
          g_re = 0.0;
          g_im = -k * inv4pi;
        } else {
          const double sh = sin(0.5 * kR);
          g_re = -2.0 * sh * sh / R * inv4pi;
          g_im = -sin(kR) / R * inv4pi;
        }
      } else {
        double s, c;
        sincos(kR, &s, &c);
        g_re = c / R * inv4pi;
        g_im = -s / R * inv4pi;
      }
      s_re += wj * g_re;
      s_im += wj * g_im;
      const V3 dr = rp - r;
      m_re = m_re + (wj * g_re) * dr;
      m_im = m_im + (wj * g_im) * dr;
    }
    if (extract) {
      double S;
      V3 V;
      static_potentials(r, Q[0], Q[1], Q[2], S, V);
      s_re += inv4pi * S;
      m_re = m_re + inv4pi * V;
    }
    // int_q (r' - Q_b) g dS' = m + (r - Q_b) s
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const V3 e = r - Q[b];
      const V3 ir = m_re + s_re * e, ii = m_im + s_im * e;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const V3 ra = r - P[a];
        T[a][b].re += wi * (0.25 * dot(ra, ir) - invk2 * s_re);
        T[a][b].im += wi * (0.25 * dot(ra, ii) - invk2 * s_im);
      }
    }
  }
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      for (int o = LP / 2; o >= 1; o >>= 1) {
        T[a][b].re += __shfl_xor(T[a][b].re, o);
        T[a][b].im += __shfl_xor(T[a][b].im, o);
      }
      if (sub == 0)
        ws[((size_t)blockIdx.y * 9 + a * 3 + b) * kTilePairs + pair] = make_double2(T[a][b].re, T[a][b].im);
    }
}

template <typename OutT>
__global__ void __launch_bounds__(256)
assemble_near_kernel(GeomDev g, FillDev f, double k, int Dx, int Dy, int near_x, int near_y, int u0,
                     const double2* __restrict__ ws, OutT* __restrict__ out, int* __restrict__ flag) {
  int dx, dy, ti, tj;
  near_unit(u0 + blockIdx.y, f.n_tiles, near_x, near_y, dx, dy, ti, tj);
  const FillTile& I = f.tiles[ti];
  const FillTile& J = f.tiles[tj];
  const int n = g.n_rwg;
  const size_t at = (size_t)((dy + Dy) * (2 * Dx + 1) + dx + Dx) * n * n;
  for (int e = blockIdx.x * 256 + threadIdx.x; e < I.count * J.count; e += gridDim.x * 256) {
    const int m = I.m0 + e / J.count, nn = J.m0 + e % J.count;
    store_entry(out, at + (size_t)m * n + nn,
                entry_of(ws + (size_t)blockIdx.y * 9 * kTilePairs, g, f, I, J, m, nn), k * kEta0, flag);
  }
}

// Tiles of consecutive RWG touching at most kTileTri triangles, and the
// per-RWG words of FillDev, as one table (tiles first).
std::vector<char> make_tiles(const r3m_unit_geom* geom, int& n_tiles) {
  std::vector<FillTile> tiles;
  std::vector<uint32_t> words(geom->n_rwg);
  std::vector<int> local(geom->n_tri, -1);
  for (int m = 0; m < geom->n_rwg; ++m) {
    const int32_t* r = geom->rwg + 4 * m;
    auto fresh = [&] { return (local[r[0]] < 0 ? 1 : 0) + (local[r[1]] < 0 ? 1 : 0); };
    if (tiles.empty() || tiles.back().n_tri + fresh() > kTileTri) {
      std::fill(local.begin(), local.end(), -1);
      FillTile t{};
      t.m0 = m;
      tiles.push_back(t);
    }
    FillTile& t = tiles.back();
    ++t.count;
    uint32_t w = 0;
    for (int a = 0; a < 2; ++a) {
      if (local[r[a]] < 0) {
        local[r[a]] = t.n_tri;
        t.tri[t.n_tri++] = r[a];
      }
      int free = 0;
      for (int c = 0; c < 3; ++c) {
        const int v = geom->tri[3 * r[a] + c];
        if (v != r[2] && v != r[3]) free = c;
      }
      w |= (uint32_t)local[r[a]] << (8 * a) | (uint32_t)free << (16 + 2 * a);
    }
    words[m] = w;
  }
  n_tiles = (int)tiles.size();
  std::vector<char> host(tiles.size() * sizeof(FillTile) + words.size() * 4);
  std::memcpy(host.data(), tiles.data(), tiles.size() * sizeof(FillTile));
  std::memcpy(host.data() + tiles.size() * sizeof(FillTile), words.data(), words.size() * 4);
  return host;
}

constexpr size_t kFarLds = 9 * kTilePairs * sizeof(double2) + 2 * 21 * kTileTri * sizeof(double);
static_assert(kFarLds <= 160 * 1024, "a tile pair's integrals fit the LDS of a CU");

template <typename OutT>
void launch_fill(r3m_ctx ctx, const r3m_unit_geom* geom, const GeomDev& g, const FillDev& f, int Dx, int Dy, OutT* out,
                 hipStream_t stream) {
  const double k = 2.0 * kPi * geom->freq_hz / kC0;
  const int n_tp = f.n_tiles * f.n_tiles;
  int* flag = (int*)ctx->flag.ptr;
  // blocks that may hold an extracted pair
  const int64_t reach = (int64_t)geom->extract_radius + (geom->tri_cell ? 2 : 0);
  const int near_x = (int)std::min<int64_t>(Dx, reach), near_y = (int)std::min<int64_t>(Dy, reach);
  const int64_t half = ((int64_t)(2 * Dx + 1) * (2 * Dy + 1) - 1) / 2;
  if (near_x < Dx || near_y < Dy) {
    R3M_CHECK_HIP(hipFuncSetAttribute((const void*)fill_far_kernel<OutT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)kFarLds));
    const int64_t all = half * n_tp, most = max_workgroups(kTilePairs);
    for (int64_t w0 = 0; w0 < all; w0 += most) {
      hipLaunchKernelGGL(fill_far_kernel<OutT>, dim3((unsigned)std::min(most, all - w0)), dim3(kTilePairs), kFarLds,
                         stream, g, f, k, geom->period_x, geom->period_y, Dx, Dy, near_x, near_y, (int)(w0 / n_tp),
                         (int)(w0 % n_tp), out, flag);
      R3M_CHECK_HIP(hipGetLastError());
    }
  }
  const int64_t units = (int64_t)(2 * near_x + 1) * (2 * near_y + 1) * n_tp;
  const size_t per = 9 * kTilePairs * sizeof(double2);
  const int64_t chunk = std::min<int64_t>(units, kNearWsBytes / per);
  ctx->fill_ws.ensure((size_t)chunk * per);
  double2* ws = (double2*)ctx->fill_ws.ptr;
  for (int64_t u0 = 0; u0 < units; u0 += chunk) {
    const unsigned cnt = (unsigned)std::min<int64_t>(chunk, units - u0);
    hipLaunchKernelGGL(pair_near_kernel<64>, dim3(kTilePairs * 64 / 256, cnt), dim3(256), 0, stream, g, f, k,
                       geom->period_x, geom->period_y, near_x, near_y, geom->extract_radius, (int)u0, ws);
    hipLaunchKernelGGL(pair_near_kernel<8>, dim3(kTilePairs * 8 / 256, cnt), dim3(256), 0, stream, g, f, k,
                       geom->period_x, geom->period_y, near_x, near_y, geom->extract_radius, (int)u0, ws);
    hipLaunchKernelGGL(assemble_near_kernel<OutT>, dim3(7, cnt), dim3(256), 0, stream, g, f, k, Dx, Dy, near_x, near_y,
                       (int)u0, ws, out, flag);
    R3M_CHECK_HIP(hipGetLastError());
  }
}

}  // namespace
}  // namespace r3m

using namespace r3m;

extern "C" {

size_t r3m_blocks_bytes(int32_t n, int32_t Dx, int32_t Dy, r3m_dtype dtype) {
  if (n <= 0 || Dx < 0 || Dy < 0) return 0;
  return (size_t)(2 * Dx + 1) * (2 * Dy + 1) * n * n * dtype_size(dtype);
}

int r3m_fill_unique_blocks(r3m_ctx ctx, const r3m_unit_geom* geom, int32_t Dx, int32_t Dy,
                           r3m_dtype dtype, void* blocks_dev, size_t blocks_bytes,
                           hipStream_t stream) {
  return guarded(ctx, [&] {
    R3M_REQUIRE(ctx, R3M_ERR_INVALID_ARG, "ctx is NULL");
    R3M_REQUIRE(Dx >= 0 && Dy >= 0, R3M_ERR_INVALID_ARG, "Dx, Dy must be >= 0");
    R3M_REQUIRE(dtype == R3M_C128 || dtype == R3M_C64, R3M_ERR_UNSUPPORTED, "fill dtype must be C128 or C64");
    R3M_REQUIRE(blocks_dev, R3M_ERR_INVALID_ARG, "blocks_dev is NULL");
    validate_geom(geom);
    const size_t need = r3m_blocks_bytes(geom->n_rwg, Dx, Dy, dtype);
    R3M_REQUIRE(blocks_bytes >= need, R3M_ERR_BUFFER_TOO_SMALL, "blocks buffer too small");
    R3M_CHECK_HIP(hipSetDevice(ctx->device));
    static bool quad_ready = false;
    static std::mutex quad_mu;
    {
      std::lock_guard<std::mutex> lk(quad_mu);
      if (!quad_ready) {
        Quad7 q = make_quad7();
        R3M_CHECK_HIP(hipMemcpyToSymbol(HIP_SYMBOL(c_quad), &q, sizeof(q)));
        QuadComp qc = make_composite(q);
        R3M_CHECK_HIP(hipMemcpyToSymbol(HIP_SYMBOL(c_comp), &qc, sizeof(qc)));
        const Rule7 rule{q.w[0] / 3.0, q.w[1] * q.b[1][1], q.w[4] * q.b[4][1], q.w[1] * (q.b[1][0] - q.b[1][1]),
                         q.w[4] * (q.b[4][0] - q.b[4][1])};
        R3M_CHECK_HIP(hipMemcpyToSymbol(HIP_SYMBOL(c_rule), &rule, sizeof(rule)));
        quad_ready = true;
      }
    }
    GeomDev g = upload_geom(ctx, geom, stream);
    int n_tiles = 0;
    const std::vector<char> tab = make_tiles(geom, n_tiles);
    ctx->fill_tab.ensure(tab.size());
    R3M_CHECK_HIP(hipMemcpyAsync(ctx->fill_tab.ptr, tab.data(), tab.size(), hipMemcpyHostToDevice, stream));
    const char* base = (const char*)ctx->fill_tab.ptr;
    const FillDev f{(const FillTile*)base, (const uint32_t*)(base + (size_t)n_tiles * sizeof(FillTile)), n_tiles};
    R3M_CHECK_HIP(hipMemsetAsync(ctx->flag.ptr, 0, sizeof(int), stream));
    if (dtype == R3M_C128)
      launch_fill(ctx, geom, g, f, Dx, Dy, (double*)blocks_dev, stream);
    else
      launch_fill(ctx, geom, g, f, Dx, Dy, (float*)blocks_dev, stream);
    int flag = 0;
    R3M_CHECK_HIP(hipMemcpyAsync(&flag, ctx->flag.ptr, sizeof(int), hipMemcpyDeviceToHost, stream));
    R3M_CHECK_HIP(hipStreamSynchronize(stream));
    R3M_REQUIRE(flag == 0, R3M_ERR_NONFINITE, "non-finite entry in the filled blocks");
  });
}

}  // extern "C"
