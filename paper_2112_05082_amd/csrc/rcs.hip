// Plane-wave excitation U_k of eq. (1) and bistatic RCS of the retrieved
// currents (post-processing of Sec. IV-A), FP64.
//
// Excitation: U_m = int f_m . E_inc dS, E_inc = e0 e_hat exp(-j k k_hat . r),
// 7-point rule.  A unit at c sees the wave of the unit at the origin times
// exp(-j k k_hat . c): the integrals of the macro RWG are taken once per RHS
// (plane_wave_base_kernel) and a thread per (RHS, unit, active RWG) applies
// the phase, so that the 163 MB of 96 right-hand sides are written at 0.04
// ms instead of 0.43 with 14 sincos per entry.  Connected geometries
// (Sec. III-B): a unit's entries are its state's bases, then the shared ones;
// a bridging basis integrates over both of its triangles at their own
// positions, and D_k's masked extended bases get zero.
// RCS: radiation vectors of the macro RWGs of the unit at the origin,
// F_m(r_hat) = int f_m exp(j k r_hat . r) dS, are formed once per direction;
// then N(r_hat) = sum_u exp(j k r_hat . c_u) sum_{m in A(s_u)} I_{u,m} F_m and
// sigma = (k^2 eta^2 / 4 pi) |N - (N . r_hat) r_hat|^2 / |e0|^2.
#include "fp64_math.h"
#include "r3m_common.h"

#include <algorithm>

namespace r3m {
namespace {

// Scratch of one call: the context's buffer (kept for the next call) up to
// kPostKeep bytes, else an allocation of its own, released with the call.
// The calls that use it synchronise before they return.
constexpr size_t kPostKeep = 128 << 20;
struct PostBuf {
  DevBuf own;
  void* ptr;
  PostBuf(r3m_ctx ctx, size_t bytes) {
    DevBuf& b = bytes <= kPostKeep ? ctx->post : own;
    b.ensure(bytes);
    ptr = b.ptr;
  }
  ~PostBuf() { own.release(); }
};

struct IncDev {
  double kx, ky, kz;  // propagation direction k_hat
  double ex, ey, ez;  // polarisation e_hat (theta_hat)
  double e0;
  double pad;
};

// U of macro RWG mm of the unit whose origin is (cx, cy, 0), without e0
__device__ double2 plane_wave_value(const GeomDev& g, int mm, double cx, double cy, const IncDev& I, double k) {
  double re = 0.0, im = 0.0;
  for (int a = 0; a < 2; ++a) {
    const int t = g.rwg_tri[2 * mm + a];
    const int fv = g.rwg_free[2 * mm + a];
    const double* v = g.tri_v + 9 * t;
    const double A = g.tri_area[t];
    const double c = (a == 0 ? 1.0 : -1.0) * g.rwg_len[mm] / (2.0 * A);
    const double vx = v[3 * fv] + cx, vy = v[3 * fv + 1] + cy, vz = v[3 * fv + 2];
    for (int i = 0; i < 7; ++i) {
      double b0, b1, b2, w;
      quad7_point(i, b0, b1, b2, w);
      const double rx = b0 * v[0] + b1 * v[3] + b2 * v[6] + cx;
      const double ry = b0 * v[1] + b1 * v[4] + b2 * v[7] + cy;
      const double rz = b0 * v[2] + b1 * v[5] + b2 * v[8];
      const double proj = (rx - vx) * I.ex + (ry - vy) * I.ey + (rz - vz) * I.ez;
      double sn, cs;
      sincos(-k * (I.kx * rx + I.ky * ry + I.kz * rz), &sn, &cs);
      re += c * w * A * proj * cs;
      im += c * w * A * proj * sn;
    }
  }
  return make_double2(re, im);
}

// base[b][mm]: U of macro RWG mm of the unit at the origin, with e0
__global__ void __launch_bounds__(64)
plane_wave_base_kernel(GeomDev g, const IncDev* __restrict__ inc, double k, double2* __restrict__ base) {
  const int mm = blockIdx.x * 64 + threadIdx.x, b = blockIdx.y;
  if (mm >= g.n_rwg) return;
  const IncDev I = inc[b];
  const double2 v = plane_wave_value(g, mm, 0.0, 0.0, I, k);
  base[(size_t)b * g.n_rwg + mm] = make_double2(I.e0 * v.x, I.e0 * v.y);
}

// exp(-j k k_hat . c) of the unit at (ix px, iy py, 0)
__device__ __forceinline__ double2 unit_phase(const IncDev& I, int64_t ix, int64_t iy, double k, double px, double py) {
  double c, s;
  cos_sin(k * (I.kx * ((double)ix * px) + I.ky * ((double)iy * py)), c, s);
  return make_double2(c, -s);
}

__global__ void __launch_bounds__(256)
plane_wave_kernel(GeomDev g, const RhsDev* __restrict__ rhs, const IncDev* __restrict__ inc,
                  const double2* __restrict__ base, const uint8_t* __restrict__ states, int n_a, int n_v,
                  int n_states, double k, double px, double py, double2* __restrict__ out) {
  const int b = blockIdx.y;
  const RhsDev R = rhs[b];
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t units = (int64_t)R.Lx * R.Ly;
  if (e >= units * n_v) return;
  const int64_t u = e / n_v;
  const int r = (int)(e % n_v);
  int s = states[R.state_off + u];
  s = s < n_states ? s : n_states - 1;
  const int64_t ix = u % R.Lx, iy = u / R.Lx;
  const int mm = compact_to_macro(g, n_a, s, r, ix, iy);
  double2 v = make_double2(0.0, 0.0);
  if (mm >= 0) {
    const double2 w = base[(size_t)b * g.n_rwg + mm], ph = unit_phase(inc[b], ix, iy, k, px, py);
    v = make_double2(w.x * ph.x - w.y * ph.y, w.x * ph.y + w.y * ph.x);
  }
  out[R.unit_off * n_v + e] = v;
}

// Relaxed codebook (weights w [unit][n_states]): macro == 0 writes the blended
// excitation U_k(w)[u][m] = sum_s w[u][s] U[u][s n_a + m] ([unit][n_a]);
// macro != 0 writes every macro row U[u][mm] ([unit][n]), weights unused.
__global__ void plane_wave_relaxed_kernel(GeomDev g, const RhsDev* __restrict__ rhs, const IncDev* __restrict__ inc,
                                          const double* __restrict__ wts, int n_a, int n_states, int macro, double k,
                                          double px, double py, double2* __restrict__ out) {
  const int b = blockIdx.y;
  const RhsDev R = rhs[b];
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int per = macro ? n_a * n_states : n_a;
  if (e >= (int64_t)R.Lx * R.Ly * per) return;
  const int64_t u = e / per;
  const int m = (int)(e - u * per);
  const double cx = (double)(u % R.Lx) * px, cy = (double)(u / R.Lx) * py;
  const IncDev I = inc[b];
  double2 acc = make_double2(0.0, 0.0);
  if (macro) {
    acc = plane_wave_value(g, m, cx, cy, I, k);
  } else {
    for (int st = 0; st < n_states; ++st) {
      const double w = wts[(R.unit_off + u) * n_states + st];
      const double2 v = plane_wave_value(g, st * n_a + m, cx, cy, I, k);
      acc.x += w * v.x;
      acc.y += w * v.y;
    }
  }
  out[R.unit_off * per + e] = make_double2(I.e0 * acc.x, I.e0 * acc.y);
}

// F[dir][m][3] for the macro unit at the origin, or (DIR_FAST) F[m][3][dir],
// for readers whose lanes are directions, with the directions' unit vectors
// in rhat[dir][3]
template <bool DIR_FAST>
__global__ void macro_radiation_kernel(GeomDev g, const double* __restrict__ dirs, int n_dir, double k,
                                       double2* __restrict__ F, double* __restrict__ rhat) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n_dir * g.n_rwg) return;
  const int d = e / g.n_rwg, m = e % g.n_rwg;
  const double th = dirs[2 * d], ph = dirs[2 * d + 1];
  const double rx = sin(th) * cos(ph), ry = sin(th) * sin(ph), rz = cos(th);
  if (DIR_FAST && m == 0) {
    rhat[3 * d] = rx;
    rhat[3 * d + 1] = ry;
    rhat[3 * d + 2] = rz;
  }
  double acc[6] = {0, 0, 0, 0, 0, 0};
  for (int a = 0; a < 2; ++a) {
    const int t = g.rwg_tri[2 * m + a];
    const int fv = g.rwg_free[2 * m + a];
    const double* v = g.tri_v + 9 * t;
    const double A = g.tri_area[t];
    const double c = (a == 0 ? 1.0 : -1.0) * g.rwg_len[m] / (2.0 * A);
    for (int i = 0; i < 7; ++i) {
      double b0, b1, b2, w;
      quad7_point(i, b0, b1, b2, w);
      double p[3];
      for (int q = 0; q < 3; ++q) p[q] = b0 * v[q] + b1 * v[3 + q] + b2 * v[6 + q];
      double sn, cs;
      sincos(k * (rx * p[0] + ry * p[1] + rz * p[2]), &sn, &cs);
      for (int q = 0; q < 3; ++q) {
        const double f = c * w * A * (p[q] - v[3 * fv + q]);
        acc[2 * q] += f * cs;
        acc[2 * q + 1] += f * sn;
      }
    }
  }
  for (int q = 0; q < 3; ++q)
    F[DIR_FAST ? ((size_t)m * 3 + q) * n_dir + d : (size_t)e * 3 + q] = make_double2(acc[2 * q], acc[2 * q + 1]);
}

constexpr int kRcsThreads = 256;
constexpr int kRcsWaves = kRcsThreads / 64;
// Radiation sums on the FP64 matrix cores.  The sum over units is taken first,
// per compact entry r and coding state s (array factor):
//   A_{s,r}(d) = sum_{u in state s} exp(j k r_hat_d . c_u) I_{u,r},
// then N(d) = sum_{s,r} A_{s,r}(d) F_{macro(s,r)}(d) (a shared basis of a
// connected geometry has one A, over the units where D_k keeps it).  A is a
// real product of (entry, re | im) rows x units and units x directions (cos |
// sin): 16x16x4 tiles, five row tiles (40 entries, no padding for the patches'
// 40 bases) x two direction tiles per wave, so that a step of four units is
// 20 matrix instructions on five 8-byte loads and two phases per lane.  The
// units of a state are listed 256 at a time (ballots, in unit order), so no
// step multiplies by a mask.  The four waves of a workgroup take a quarter of
// its unit chunk each and are summed in wave order, then the chunks in theirs.
// Bound by the matrix cores, then by the passes' ends (reading F): 96
// right-hand sides of 32x32 to 64x64 units x 360 directions are 0.38 ms of
// matrix-core issue and take 0.85 ms (0.28 of it outside the unit steps); with
// lane = direction on the vector units and a scalar load per unit they took
// 3.5 ms.
constexpr int kRcsRowTiles = 5;                    // (entry, part) row tiles of a pass
constexpr int kRcsRows = 8 * kRcsRowTiles;         // entries of a pass
constexpr int kRcsDirTiles = 2;
constexpr int kRcsDirs = 16 * kRcsDirTiles;        // directions per workgroup
constexpr int kRcsList = 256;                      // units listed at a time by a wave
constexpr int kRcsUnits = kRcsWaves * kRcsList;    // smallest unit chunk
constexpr size_t kRcsWgs = 2048;
constexpr size_t kRcsPartialBytes = 64 << 20;      // radiation sums of the chunks
typedef double f64x4 __attribute__((ext_vector_type(4)));

// sigma of one direction from the radiation vector N (3 complex)
__device__ __forceinline__ double rcs_value(const double (&N)[6], double rx, double ry, double rz, double scale) {
  const double rr[3] = {rx, ry, rz};
  const double dre = N[0] * rx + N[2] * ry + N[4] * rz;
  const double dim = N[1] * rx + N[3] * ry + N[5] * rz;
  double p2 = 0.0;
  for (int q = 0; q < 3; ++q) {
    const double qr = N[2 * q] - dre * rr[q], qi = N[2 * q + 1] - dim * rr[q];
    p2 += qr * qr + qi * qi;
  }
  return scale * p2;
}

// The listed units' contributions to a pass: steps of four units, the next
// step's currents in flight.  p: the pass's first entry in unit 0; rows: its
// (entry, part) rows.  FULL: all 80 rows, none masked.  c0 >= 0: shared
// entries from c0 on, zero where D_k masks them.  Units past the list's end
// get a zero phase (their currents are those of a listed unit).
template <bool FULL>
__device__ __forceinline__ void rcs_steps(const GeomDev& g, const int2* list, int cnt, const double* __restrict__ p,
                                          int Lx, int n_v, int rows, int c0, int lane,
                                          const double (&kx)[kRcsDirTiles], const double (&ky)[kRcsDirTiles],
                                          double px, double py, f64x4 (&ac)[kRcsRowTiles][kRcsDirTiles],
                                          f64x4 (&as)[kRcsRowTiles][kRcsDirTiles]) {
  const int col = lane & 15, kq = lane >> 4;
  double a[kRcsRowTiles];
  int2 at = make_int2(0, 0);
  bool in = false;
  auto load = [&](int j) {
    in = j + kq < cnt;
    at = list[in ? j + kq : 0];
    const double* pu = p + ((int64_t)at.y * Lx + at.x) * n_v * 2;
#pragma unroll
    for (int t = 0; t < kRcsRowTiles; ++t) {
      if (FULL) {
        a[t] = pu[t * 16 + col];
      } else {
        const int row = min(t * 16 + col, rows - 1);
        a[t] = pu[row];
        if (c0 >= 0) {
          const int e = g.common_ext[c0 + row / 2];
          if ((e == 1 && at.x == 0) || (e == 2 && at.y == 0)) a[t] = 0.0;
        }
      }
    }
  };
  double bn[2 * kRcsDirTiles];  // cos and sin of the loaded units' phases
  auto phases = [&] {
    const double cx = (double)at.x * px, cy = (double)at.y * py;
#pragma unroll
    for (int e = 0; e < kRcsDirTiles; ++e) {
      double c, s;
      cos_sin(kx[e] * cx + ky[e] * cy, c, s);
      bn[2 * e] = in ? c : 0.0;
      bn[2 * e + 1] = in ? s : 0.0;
    }
  };
  if (cnt == 0) return;
  load(0);
  phases();
#pragma unroll 1
  for (int j = 0; j < cnt; j += 4) {
    double av[kRcsRowTiles], bv[2 * kRcsDirTiles];
#pragma unroll
    for (int t = 0; t < kRcsRowTiles; ++t) av[t] = a[t];
#pragma unroll
    for (int e = 0; e < 2 * kRcsDirTiles; ++e) bv[e] = bn[e];
    load(j + 4);  // past the end: unit list[0] again, with zero phases
    phases();
#pragma unroll
    for (int t = 0; t < kRcsRowTiles; ++t) {
      if (FULL || t * 16 < rows) {  // uniform
#pragma unroll
        for (int e = 0; e < kRcsDirTiles; ++e) {
          ac[t][e] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[t], bv[2 * e], ac[t][e], 0, 0, 0);
          as[t][e] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[t], bv[2 * e + 1], as[t][e], 0, 0, 0);
        }
      }
    }
    // the next step's phases in the shadow of the matrix instructions (64
    // cycles each)
    if (FULL) {
#pragma unroll
      for (int t = 0; t < 4 * kRcsRowTiles; ++t) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
      }
    }
  }
}

// One workgroup per (RHS, unit chunk, 32 directions); the direction groups of
// a chunk share one XCD (and its L2 copy of the currents).  partial (n_chunks
// > 1): [chunk][b][dir][6]; else sigma is written.  FULL: n_a a multiple of 40
// and no shared entries.  A launch takes the workgroups from id0 (a multiple of
// 8) on (see max_workgroups).
template <bool FULL>
__global__ void __launch_bounds__(kRcsThreads, 2)
rcs_kernel(GeomDev g, const RhsDev* __restrict__ rhs, const uint8_t* __restrict__ states,
           const double2* __restrict__ I, const double2* __restrict__ F, const double* __restrict__ rhat, int n_dir,
           int n_a, int n_v, int n_states, int B, int n_dgrp, int n_chunks, int64_t chunk_units, int64_t id0, double k,
           double px, double py, double scale, double* __restrict__ partial, double* __restrict__ sigma) {
  __shared__ int2 list_s[kRcsWaves][kRcsList];
  __shared__ double sum_s[kRcsWaves][6][kRcsDirs];
  const int64_t id = id0 + blockIdx.x;
  const int64_t slot = id / 8, grp = (slot / n_dgrp) * 8 + id % 8;
  if (grp >= (int64_t)B * n_chunks) return;
  // chunk-major: the XCDs then share the arrays' first chunks and their last,
  // of which small arrays have none
  const int chunk = (int)(grp / B), b = (int)(grp % B), dgrp = (int)(slot % n_dgrp);
  const RhsDev R = rhs[b];
  const int64_t units = (int64_t)R.Lx * R.Ly;
  const int lane = threadIdx.x & 63, col = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int2* list = list_s[wave];
  int d[kRcsDirTiles];
  double kx[kRcsDirTiles], ky[kRcsDirTiles];  // phase per metre along x and y
#pragma unroll
  for (int t = 0; t < kRcsDirTiles; ++t) {
    d[t] = min(dgrp * kRcsDirs + t * 16 + col, n_dir - 1);
    kx[t] = k * rhat[3 * d[t]];
    ky[t] = k * rhat[3 * d[t] + 1];
  }
  const double* Ir = reinterpret_cast<const double*>(I + R.unit_off * n_v);
  // the wave's radiation sums stay in LDS between passes (registers are the
  // accumulators')
  for (int t = lane; t < 6 * kRcsDirs; t += 64) sum_s[wave][t / kRcsDirs][t % kRcsDirs] = 0.0;
  // passes: (state, block of 40 entries), then the shared entries' blocks
  const int sb = (n_a + kRcsRows - 1) / kRcsRows, cb = (n_v - n_a + kRcsRows - 1) / kRcsRows;
  const int n_pass = n_states * sb + cb;
  const int64_t c_lo = (int64_t)chunk * chunk_units, c_hi = min(units, c_lo + chunk_units);
  // units of one list would keep one wave busy and leave the others their
  // passes' ends: the waves take the passes in turn instead (us a call, units
  // split / passes in turn: 6x6 with four states 136 / 85, 12x12 154 / 94, 16
  // states of one basis 214 / 99, 12x12 of two states x 64 right-hand sides x
  // 360 directions 183 / 136)
  const bool by_pass = c_hi - c_lo <= kRcsList;
  const int64_t u_lo = c_lo + (by_pass ? 0 : wave * kRcsList);
  for (int pass = by_pass ? wave : 0; pass < n_pass; pass += by_pass ? kRcsWaves : 1) {
    const bool shared = !FULL && pass >= n_states * sb;
    const int s = shared ? -1 : pass / sb;
    const int r0 = shared ? n_a + (pass - n_states * sb) * kRcsRows : (pass % sb) * kRcsRows;
    const int rows = 2 * min(kRcsRows, (shared ? n_v : n_a) - r0);  // (entry, part) rows
    f64x4 ac[kRcsRowTiles][kRcsDirTiles], as[kRcsRowTiles][kRcsDirTiles];  // sums with cos and with sin
#pragma unroll
    for (int t = 0; t < kRcsRowTiles; ++t)
#pragma unroll
      for (int e = 0; e < kRcsDirTiles; ++e) ac[t][e] = as[t][e] = f64x4{0, 0, 0, 0};
    for (int64_t u0 = u_lo; u0 < c_hi; u0 += kRcsUnits) {
      // the state's units among the next 256, in order
      int cnt = 0;
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int h = 0; h < kRcsList / 64; ++h) {
        const int64_t u = u0 + h * 64 + lane;
        bool in = u < c_hi;
        if (in && !shared) {
          int su = states[R.state_off + u];
          su = su < n_states ? su : n_states - 1;
          in = su == s;
        }
        const unsigned long long m = __ballot(in);
        if (in) {
          const int y = units < 1ll << 31 ? (int)u / R.Lx : (int)(u / R.Lx);
          list[cnt + __popcll(m & ((1ull << lane) - 1))] = make_int2((int)(u - (int64_t)y * R.Lx), y);
        }
        cnt += __popcll(m);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      rcs_steps<FULL>(g, list, cnt, Ir + 2 * r0, R.Lx, n_v, rows, shared ? r0 - n_a : -1, lane, kx, ky, px, py, ac, as);
    }
    // N = A F: result entry i of a lane is row 4 i + lane / 16 of its tile; a
    // real part's row adds (cos, sin), an imaginary part's (-sin, cos)
#pragma unroll
    for (int e = 0; e < kRcsDirTiles; ++e) {
      double N[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
      for (int t = 0; t < kRcsRowTiles; ++t) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = t * 16 + 4 * i + kq;
          const bool in = FULL || row < rows;  // a row past the pass adds zero
          const int r = r0 + (FULL ? row : min(row, rows - 1)) / 2;
          const int mm = shared ? g.n_st + (r - n_a) : s * n_a + r;
          const double xr = !in ? 0.0 : row & 1 ? -as[t][e][i] : ac[t][e][i];
          const double xi = !in ? 0.0 : row & 1 ? ac[t][e][i] : as[t][e][i];
#pragma unroll
          for (int q = 0; q < 3; ++q) {
            const double2 f = F[((size_t)mm * 3 + q) * n_dir + d[e]];
            N[2 * q] += xr * f.x - xi * f.y;
            N[2 * q + 1] += xr * f.y + xi * f.x;
          }
        }
        // the sums are formed tile by tile (the compiler would move each
        // below, to where it is used, and spill all of the tiles' loads)
        asm volatile("" : "+v"(N[0]), "+v"(N[1]), "+v"(N[2]), "+v"(N[3]), "+v"(N[4]), "+v"(N[5]));
      }
#pragma unroll
      for (int q = 0; q < 6; ++q) {
        N[q] += __shfl_xor(N[q], 16);
        N[q] += __shfl_xor(N[q], 32);
        if (kq == 0) sum_s[wave][q][e * 16 + col] += N[q];
      }
    }
  }
  __syncthreads();
  const int dd = dgrp * kRcsDirs + threadIdx.x;
  if (threadIdx.x < kRcsDirs && dd < n_dir) {
    double T[6];
    for (int q = 0; q < 6; ++q) {
      T[q] = sum_s[0][q][threadIdx.x];
      for (int w = 1; w < kRcsWaves; ++w) T[q] += sum_s[w][q][threadIdx.x];
    }
    if (n_chunks == 1) {
      sigma[(size_t)b * n_dir + dd] = rcs_value(T, rhat[3 * dd], rhat[3 * dd + 1], rhat[3 * dd + 2], scale);
    } else {
      double* o = partial + (((size_t)chunk * B + b) * n_dir + dd) * 6;
      for (int q = 0; q < 6; ++q) o[q] = T[q];
    }
  }
}

// sigma from the chunks' radiation sums, added in chunk order
__global__ void __launch_bounds__(256)
rcs_finish_kernel(const double* __restrict__ partial, const double* __restrict__ rhat, int n_dir, int B, int n_chunks,
                  double scale, double* __restrict__ sigma) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= (int64_t)B * n_dir) return;
  double N[6] = {0, 0, 0, 0, 0, 0};
  for (int c = 0; c < n_chunks; ++c)
    for (int q = 0; q < 6; ++q) N[q] += partial[((size_t)c * B * n_dir + e) * 6 + q];
  const int d = (int)(e % n_dir);
  sigma[e] = rcs_value(N, rhat[3 * d], rhat[3 * d + 1], rhat[3 * d + 2], scale);
}

// Radiation vector of the blended current I~[u][s n_a + r] = w[u][s] I[u][r]
// (relaxed codebook) for direction d and RHS b: sigma as rcs_kernel, and the
// transverse part N_perp (3 complex) kept for the objective's gradient.
__global__ void __launch_bounds__(kRcsThreads)
rcs_relaxed_kernel(const RhsDev* __restrict__ rhs, const double* __restrict__ wts, const double2* __restrict__ I,
                   const double2* __restrict__ F, const double* __restrict__ dirs, int n_dir, int n, int n_a,
                   int n_states, double k, double px, double py, double scale, double* __restrict__ sigma,
                   double2* __restrict__ nperp) {
  __shared__ double sh[kRcsThreads / 64][6];
  const int d = blockIdx.x, b = blockIdx.y;
  const RhsDev R = rhs[b];
  const double th = dirs[2 * d], ph = dirs[2 * d + 1];
  const double rx = sin(th) * cos(ph), ry = sin(th) * sin(ph), rz = cos(th);
  const int64_t units = (int64_t)R.Lx * R.Ly;
  double acc[6] = {0, 0, 0, 0, 0, 0};
  const double2* Fd = F + (size_t)d * n * 3;
  for (int64_t u = threadIdx.x; u < units; u += blockDim.x) {
    const double cx = (double)(u % R.Lx) * px, cy = (double)(u / R.Lx) * py;
    double sn, cs;
    sincos(k * (rx * cx + ry * cy), &sn, &cs);
    double loc[6] = {0, 0, 0, 0, 0, 0};
    const double2* Iu = I + (R.unit_off + u) * n_a;
    for (int st = 0; st < n_states; ++st) {
      const double w = wts[(R.unit_off + u) * n_states + st];
      for (int m = 0; m < n_a; ++m) {
        const double2 cur = make_double2(w * Iu[m].x, w * Iu[m].y);
        const double2* f = Fd + (size_t)(st * n_a + m) * 3;
        for (int q = 0; q < 3; ++q) {
          loc[2 * q] += cur.x * f[q].x - cur.y * f[q].y;
          loc[2 * q + 1] += cur.x * f[q].y + cur.y * f[q].x;
        }
      }
    }
    for (int q = 0; q < 3; ++q) {
      acc[2 * q] += loc[2 * q] * cs - loc[2 * q + 1] * sn;
      acc[2 * q + 1] += loc[2 * q] * sn + loc[2 * q + 1] * cs;
    }
  }
  for (int q = 0; q < 6; ++q)
    for (int o = 32; o >= 1; o >>= 1) acc[q] += __shfl_xor(acc[q], o);
  if ((threadIdx.x & 63) == 0)
    for (int q = 0; q < 6; ++q) sh[threadIdx.x >> 6][q] = acc[q];
  __syncthreads();
  if (threadIdx.x == 0) {
    double N[6];
    for (int q = 0; q < 6; ++q) {
      N[q] = sh[0][q];
      for (int w = 1; w < kRcsThreads / 64; ++w) N[q] += sh[w][q];
    }
    const double rr[3] = {rx, ry, rz};
    const double dre = N[0] * rx + N[2] * ry + N[4] * rz;
    const double dim = N[1] * rx + N[3] * ry + N[5] * rz;
    double p2 = 0.0;
    for (int q = 0; q < 3; ++q) {
      const double pr = N[2 * q] - dre * rr[q], pi = N[2 * q + 1] - dim * rr[q];
      p2 += pr * pr + pi * pi;
      nperp[((size_t)b * n_dir + d) * 3 + q] = make_double2(pr, pi);
    }
    sigma[(size_t)b * n_dir + d] = scale * p2;
  }
}

// J[b] = mean over directions of sigma[b][:] (fixed order)
__global__ void mean_dirs_kernel(const double* __restrict__ sigma, int n_dir, int B, double* __restrict__ J) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  double t = 0.0;
  for (int d = 0; d < n_dir; ++d) t += sigma[(size_t)b * n_dir + d];
  J[b] = t / n_dir;
}

// G[u][mm] = dJ/dI~[u][mm] = (scale / n_dir) sum_d conj(N_perp(d)) . F_mm(d)
// exp(j k r_hat_d . c_u) (Wirtinger derivative of the mean RCS), macro layout
__global__ void relaxed_dj_kernel(const RhsDev* __restrict__ rhs, const double2* __restrict__ F,
                                  const double* __restrict__ dirs, const double2* __restrict__ nperp, int n_dir, int n,
                                  double k, double px, double py, double scale, double2* __restrict__ G) {
  const int b = blockIdx.y;
  const RhsDev R = rhs[b];
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)R.Lx * R.Ly * n) return;
  const int64_t u = e / n;
  const int mm = (int)(e - u * n);
  const double cx = (double)(u % R.Lx) * px, cy = (double)(u / R.Lx) * py;
  double gr = 0.0, gi = 0.0;
  for (int d = 0; d < n_dir; ++d) {
    const double th = dirs[2 * d], ph = dirs[2 * d + 1];
    double sn, cs;
    sincos(k * (sin(th) * cos(ph) * cx + sin(th) * sin(ph) * cy), &sn, &cs);
    const double2* f = F + ((size_t)d * n + mm) * 3;
    const double2* np_ = nperp + ((size_t)b * n_dir + d) * 3;
    double tr = 0.0, ti = 0.0;  // conj(N_perp) . F_mm
    for (int q = 0; q < 3; ++q) {
      tr += np_[q].x * f[q].x + np_[q].y * f[q].y;
      ti += np_[q].x * f[q].y - np_[q].y * f[q].x;
    }
    gr += tr * cs - ti * sn;
    gi += tr * sn + ti * cs;
  }
  G[R.unit_off * n + e] = make_double2(scale / n_dir * gr, scale / n_dir * gi);
}

// a[u][r] = sum_s w[u][s] G[u][s n_a + r]: P(w)^T G, the adjoint right-hand side
__global__ void blend_transpose_kernel(const RhsDev* __restrict__ rhs, const double* __restrict__ wts,
                                       const double2* __restrict__ G, int n_a, int n_states, double2* __restrict__ a) {
  const int b = blockIdx.y;
  const RhsDev R = rhs[b];
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)R.Lx * R.Ly * n_a) return;
  const int64_t u = e / n_a;
  const int r = (int)(e - u * n_a);
  double xr = 0.0, xi = 0.0;
  for (int st = 0; st < n_states; ++st) {
    const double w = wts[(R.unit_off + u) * n_states + st];
    const double2 g = G[(R.unit_off + u) * n_a * n_states + st * n_a + r];
    xr += w * g.x;
    xi += w * g.y;
  }
  a[R.unit_off * n_a + e] = make_double2(xr, xi);
}

}  // namespace
}  // namespace r3m

using namespace r3m;

extern "C" {

int r3m_plane_wave_rhs(r3m_ctx ctx, const r3m_unit_geom* geom, const r3m_batch* batch,
                       const double* inc_host, void* b_dev, hipStream_t stream) {
  return guarded(ctx, [&] {
    R3M_REQUIRE(ctx, R3M_ERR_INVALID_ARG, "ctx is NULL");
    validate_geom(geom);
    require_extension_classes(geom);
    validate_batch(batch, 1 << 20, 1 << 20);
    if (batch->B == 0) return;
    R3M_REQUIRE(inc_host && b_dev, R3M_ERR_INVALID_ARG, "NULL argument");
    R3M_CHECK_HIP(hipSetDevice(ctx->device));
    const int n_a = geom->state_off[1] - geom->state_off[0];
    GeomDev g = upload_geom(ctx, geom, stream);
    const BatchDesc& bd = get_batch(ctx, batch, 4, 4, stream);
    std::vector<IncDev> inc(bd.B);
    for (int b = 0; b < bd.B; ++b) {
      const double th = inc_host[3 * b], ph = inc_host[3 * b + 1];
      R3M_REQUIRE(std::isfinite(th) && std::isfinite(ph) && std::isfinite(inc_host[3 * b + 2]),
                  R3M_ERR_INVALID_ARG, "non-finite incidence");
      inc[b] = IncDev{-std::sin(th) * std::cos(ph), -std::sin(th) * std::sin(ph), -std::cos(th),
                      std::cos(th) * std::cos(ph), std::cos(th) * std::sin(ph), -std::sin(th),
                      inc_host[3 * b + 2], 0.0};
    }
    const size_t ib = (inc.size() * sizeof(IncDev) + 255) / 256 * 256;
    PostBuf tmp(ctx, ib + (size_t)bd.B * geom->n_rwg * sizeof(double2));
    const IncDev* inc_dev = (const IncDev*)tmp.ptr;
    double2* base = (double2*)((char*)tmp.ptr + ib);
    R3M_CHECK_HIP(hipMemcpyAsync(tmp.ptr, inc.data(), inc.size() * sizeof(IncDev), hipMemcpyHostToDevice, stream));
    int64_t maxU = 0;
    for (int b = 0; b < bd.B; ++b) maxU = std::max<int64_t>(maxU, bd.n_units[b]);
    const double k = 2.0 * kPi * geom->freq_hz / kC0;
    const int n_v = vec_per_unit(geom);
    dim3 grid(ceil_div((size_t)maxU * n_v, 256), bd.B);
    check_states(bd, batch->states, geom->n_states, deferred_word(ctx), kDeferredBadState, stream);
    hipLaunchKernelGGL(plane_wave_base_kernel, dim3(ceil_div((size_t)geom->n_rwg, 64), bd.B), dim3(64), 0, stream, g,
                       inc_dev, k, base);
    hipLaunchKernelGGL(plane_wave_kernel, grid, dim3(256), 0, stream, g, bd.rhs, inc_dev, (const double2*)base,
                       batch->states, n_a, n_v, geom->n_states, k, geom->period_x, geom->period_y, (double2*)b_dev);
    R3M_CHECK_HIP(hipGetLastError());
    take_deferred(ctx, stream);  // synchronises
  });
}

int r3m_rcs(r3m_ctx ctx, const r3m_unit_geom* geom, const r3m_batch* batch, const void* I_dev,
            int32_t n_dir, const double* dirs_host, double e0, double* sigma_dev, hipStream_t stream) {
  return guarded(ctx, [&] {
    R3M_REQUIRE(ctx, R3M_ERR_INVALID_ARG, "ctx is NULL");
    validate_geom(geom);
    require_extension_classes(geom);
    validate_batch(batch, 1 << 20, 1 << 20);
    R3M_REQUIRE(n_dir >= 0, R3M_ERR_INVALID_ARG, "n_dir < 0");
    R3M_REQUIRE(e0 != 0.0 && std::isfinite(e0), R3M_ERR_INVALID_ARG, "e0 must be finite and non-zero");
    if (batch->B == 0 || n_dir == 0) return;
    R3M_REQUIRE(I_dev && dirs_host && sigma_dev, R3M_ERR_INVALID_ARG, "NULL argument");
    for (int d = 0; d < 2 * n_dir; ++d)
      R3M_REQUIRE(std::isfinite(dirs_host[d]), R3M_ERR_INVALID_ARG, "non-finite direction");
    R3M_CHECK_HIP(hipSetDevice(ctx->device));
    const int n_a = geom->state_off[1] - geom->state_off[0];
    GeomDev g = upload_geom(ctx, geom, stream);
    const BatchDesc& bd = get_batch(ctx, batch, 4, 4, stream);
    const double k = 2.0 * kPi * geom->freq_hz / kC0;
    // unit chunks: the smallest (four lists) for few right-hand sides, doubled
    // while there are more than kRcsWgs workgroups (a pass's end costs the same
    // for every chunk: 96 right-hand sides took 1.17, 1.09 and 1.07 ms with
    // chunks of 1,024, 2,048 and 4,096 units, 4,608 to 1,152 workgroups) or
    // the radiation sums exceed their buffer; a single chunk writes sigma
    int64_t maxU = 1, chunk_units = kRcsUnits;
    for (int b = 0; b < bd.B; ++b) maxU = std::max<int64_t>(maxU, bd.n_units[b]);
    auto chunks = [&] { return (maxU + chunk_units - 1) / chunk_units; };
    const int n_dgrp = ceil_div((size_t)n_dir, kRcsDirs);
    while (chunks() > 1 && ((size_t)chunks() * bd.B * n_dgrp > kRcsWgs ||
                            (size_t)chunks() * bd.B * n_dir * 6 * sizeof(double) > kRcsPartialBytes))
      chunk_units *= 2;
    const int n_chunks = (int)chunks();
    const size_t fbytes = (size_t)n_dir * geom->n_rwg * 3 * sizeof(double2);
    const size_t pbytes = n_chunks > 1 ? (size_t)n_chunks * bd.B * n_dir * 6 * sizeof(double) : 0;
    PostBuf tmp(ctx, fbytes + pbytes + (size_t)n_dir * 40);
    double2* F = (double2*)tmp.ptr;
    double* part = (double*)((char*)tmp.ptr + fbytes);
    double* ddev = (double*)((char*)tmp.ptr + fbytes + pbytes);
    double* rhat = ddev + 2 * (size_t)n_dir;
    R3M_CHECK_HIP(hipMemcpyAsync(ddev, dirs_host, (size_t)n_dir * 16, hipMemcpyHostToDevice, stream));
    hipLaunchKernelGGL(macro_radiation_kernel<true>, dim3(ceil_div((size_t)n_dir * geom->n_rwg, 128)), dim3(128), 0,
                       stream, g, (const double*)ddev, n_dir, k, F, rhat);
    const double scale = k * k * kEta0 * kEta0 / (4.0 * kPi) / (e0 * e0);
    check_states(bd, batch->states, geom->n_states, deferred_word(ctx), kDeferredBadState, stream);
    R3M_REQUIRE((size_t)ceil_div((size_t)bd.B, 8) * 8 * ceil_div((size_t)n_dir, 64) < (1ull << 31),
                R3M_ERR_INVALID_ARG, "too many right-hand sides x directions for one RCS call");
    const int64_t n_wg = ((int64_t)bd.B * n_chunks + 7) / 8 * 8 * n_dgrp, most = max_workgroups(kRcsThreads);
    auto launch = [&](auto kern) {
      for (int64_t id0 = 0; id0 < n_wg; id0 += most) {
        hipLaunchKernelGGL(kern, dim3((unsigned)std::min(most, n_wg - id0)), dim3(kRcsThreads), 0, stream, g, bd.rhs,
                           batch->states, (const double2*)I_dev, (const double2*)F, (const double*)rhat, n_dir, n_a,
                           vec_per_unit(geom), geom->n_states, bd.B, n_dgrp, n_chunks, chunk_units, id0, k,
                           geom->period_x, geom->period_y, scale, part, sigma_dev);
        R3M_CHECK_HIP(hipGetLastError());
      }
    };
    if (n_a % kRcsRows == 0 && vec_per_unit(geom) == n_a)
      launch(rcs_kernel<true>);
    else
      launch(rcs_kernel<false>);
    if (n_chunks > 1)
      hipLaunchKernelGGL(rcs_finish_kernel, dim3(ceil_div((size_t)bd.B * n_dir, 256)), dim3(256), 0, stream,
                         (const double*)part, (const double*)rhat, n_dir, bd.B, n_chunks, scale, sigma_dev);
    R3M_CHECK_HIP(hipGetLastError());
    take_deferred(ctx, stream);  // synchronises
  });
}

int r3m_relaxed_rhs(r3m_ctx ctx, const r3m_unit_geom* geom, const r3m_batch* batch, const double* weights_dev,
                    const double* inc_host, int32_t macro, void* b_dev, hipStream_t stream) {
  return guarded(ctx, [&] {
    R3M_REQUIRE(ctx, R3M_ERR_INVALID_ARG, "ctx is NULL");
    validate_geom(geom);
    require_isolated(geom);
    validate_batch(batch, 1 << 20, 1 << 20);
    if (batch->B == 0) return;
    R3M_REQUIRE(inc_host && b_dev && (macro || weights_dev), R3M_ERR_INVALID_ARG, "NULL argument");
    R3M_CHECK_HIP(hipSetDevice(ctx->device));
    const int n_a = geom->state_off[1] - geom->state_off[0];
    GeomDev g = upload_geom(ctx, geom, stream);
    const BatchDesc& bd = get_batch(ctx, batch, 4, 4, stream);
    std::vector<IncDev> inc(bd.B);
    for (int b = 0; b < bd.B; ++b) {
      const double th = inc_host[3 * b], ph = inc_host[3 * b + 1];
      R3M_REQUIRE(std::isfinite(th) && std::isfinite(ph) && std::isfinite(inc_host[3 * b + 2]),
                  R3M_ERR_INVALID_ARG, "non-finite incidence");
      inc[b] = IncDev{-std::sin(th) * std::cos(ph), -std::sin(th) * std::sin(ph), -std::cos(th),
                      std::cos(th) * std::cos(ph), std::cos(th) * std::sin(ph), -std::sin(th),
                      inc_host[3 * b + 2], 0.0};
    }
    DevBuf tmp;
    tmp.ensure(inc.size() * sizeof(IncDev));
    R3M_CHECK_HIP(hipMemcpyAsync(tmp.ptr, inc.data(), inc.size() * sizeof(IncDev), hipMemcpyHostToDevice, stream));
    int64_t maxU = 0;
    for (int b = 0; b < bd.B; ++b) maxU = std::max<int64_t>(maxU, bd.n_units[b]);
    const double k = 2.0 * kPi * geom->freq_hz / kC0;
    const int per = macro ? n_a * geom->n_states : n_a;
    hipLaunchKernelGGL(plane_wave_relaxed_kernel, dim3(ceil_div((size_t)maxU * per, 256), bd.B), dim3(256), 0,
                       stream, g, bd.rhs, (const IncDev*)tmp.ptr, weights_dev, n_a, geom->n_states, macro ? 1 : 0, k,
                       geom->period_x, geom->period_y, (double2*)b_dev);
    R3M_CHECK_HIP(hipGetLastError());
    R3M_CHECK_HIP(hipStreamSynchronize(stream));
    tmp.release();
  });
}

int r3m_relaxed_objective(r3m_ctx ctx, const r3m_unit_geom* geom, const r3m_batch* batch, const double* weights_dev,
                          const void* I_dev, int32_t n_dir, const double* dirs_host, double e0, double* J_dev,
                          double* sigma_dev, void* G_dev, void* adj_dev, hipStream_t stream) {
  return guarded(ctx, [&] {
    R3M_REQUIRE(ctx, R3M_ERR_INVALID_ARG, "ctx is NULL");
    validate_geom(geom);
    require_isolated(geom);
    validate_batch(batch, 1 << 20, 1 << 20);
    R3M_REQUIRE(n_dir >= 1, R3M_ERR_INVALID_ARG, "n_dir < 1");
    R3M_REQUIRE(e0 != 0.0 && std::isfinite(e0), R3M_ERR_INVALID_ARG, "e0 must be finite and non-zero");
    if (batch->B == 0) return;
    R3M_REQUIRE(weights_dev && I_dev && dirs_host && J_dev && sigma_dev && G_dev && adj_dev, R3M_ERR_INVALID_ARG,
                "NULL argument");
    for (int d = 0; d < 2 * n_dir; ++d)
      R3M_REQUIRE(std::isfinite(dirs_host[d]), R3M_ERR_INVALID_ARG, "non-finite direction");
    R3M_CHECK_HIP(hipSetDevice(ctx->device));
    const int n_a = geom->state_off[1] - geom->state_off[0];
    GeomDev g = upload_geom(ctx, geom, stream);
    const BatchDesc& bd = get_batch(ctx, batch, 4, 4, stream);
    const double k = 2.0 * kPi * geom->freq_hz / kC0;
    DevBuf tmp;
    const size_t fbytes = (size_t)n_dir * geom->n_rwg * 3 * sizeof(double2);
    const size_t npbytes = (size_t)bd.B * n_dir * 3 * sizeof(double2);
    tmp.ensure(fbytes + npbytes + (size_t)n_dir * 16 + 512);
    double2* F = (double2*)tmp.ptr;
    double2* np_ = (double2*)((char*)tmp.ptr + fbytes);
    double* ddev = (double*)((char*)tmp.ptr + fbytes + npbytes);
    R3M_CHECK_HIP(hipMemcpyAsync(ddev, dirs_host, (size_t)n_dir * 16, hipMemcpyHostToDevice, stream));
    hipLaunchKernelGGL(macro_radiation_kernel<false>, dim3(ceil_div((size_t)n_dir * geom->n_rwg, 128)), dim3(128), 0,
                       stream, g, ddev, n_dir, k, F, (double*)nullptr);
    const double scale = k * k * kEta0 * kEta0 / (4.0 * kPi) / (e0 * e0);
    hipLaunchKernelGGL(rcs_relaxed_kernel, dim3(n_dir, bd.B), dim3(kRcsThreads), 0, stream, bd.rhs, weights_dev,
                       (const double2*)I_dev, (const double2*)F, (const double*)ddev, n_dir, geom->n_rwg, n_a,
                       geom->n_states, k, geom->period_x, geom->period_y, scale, sigma_dev, np_);
    hipLaunchKernelGGL(mean_dirs_kernel, dim3(ceil_div((size_t)bd.B, 64)), dim3(64), 0, stream,
                       (const double*)sigma_dev, n_dir, bd.B, J_dev);
    int64_t maxU = 0;
    for (int b = 0; b < bd.B; ++b) maxU = std::max<int64_t>(maxU, bd.n_units[b]);
    hipLaunchKernelGGL(relaxed_dj_kernel, dim3(ceil_div((size_t)maxU * geom->n_rwg, 256), bd.B), dim3(256), 0,
                       stream, bd.rhs, (const double2*)F, (const double*)ddev, (const double2*)np_, n_dir,
                       geom->n_rwg, k, geom->period_x, geom->period_y, scale, (double2*)G_dev);
    hipLaunchKernelGGL(blend_transpose_kernel, dim3(ceil_div((size_t)maxU * n_a, 256), bd.B), dim3(256), 0, stream,
                       bd.rhs, weights_dev, (const double2*)G_dev, n_a, geom->n_states, (double2*)adj_dev);
    R3M_CHECK_HIP(hipGetLastError());
    R3M_CHECK_HIP(hipStreamSynchronize(stream));
    tmp.release();
  });
}

}  // extern "C"
