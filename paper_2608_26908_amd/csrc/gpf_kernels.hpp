// gpf_kernels.hpp -- HIP kernels of the coupled GP phase-field / LBM step.
//
// One step = two launches over tiles of cells:
//   k_phi    phi^n, mu^n              -> phi^{n+1}          (Eq. PhfGrand, Sec. 2.1)
//   k_mulbm  phi^n, phi^{n+1}, mu^n, U^{n-1}, f*^{n-1}
//                                     -> mu^{n+1}, U^n, f*^n (Eq. conc; Eqs. LBMEq_1,
//                                        f^eq, discreteForce, buoyancy, rhovel)
// or one, k_step2, on 2D grids of up to 3 MiB per component.
// f buffers hold post-collision, pre-streaming populations as deviations
// f - w_k rho0; streaming is a pull at the start of k_mulbm, with half-way
// bounce-back where the source lies behind a wall.  All buffers are A-B:
// every kernel reads one copy and writes the other.
#pragma once
#include "gpf_device.hpp"

namespace gpf {

// Population k of f^n at cell (x, y, z) = P, as a deviation from w_k rho0:
// pulled from the stored post-collision f* of the upstream cell P - c_k, or,
// when that cell lies behind a wall, the reflected f*_{opp k}(P) (half-way
// bounce-back; the wall sits on the zero-flux face of phi and mu).  The
// test-only moving upper wall of axis 1 adds 6 w_k rho0 c_k . U_wall.
template <int D, int Q, class R>
__device__ __forceinline__ R pull_f(const KP<R>& p, const R* __restrict__ fin, int x, int y, int z,
                                    int64_t P, int k) {
  using L = Lat<Q>;
  int src[3] = {x - L::c(k, 0), y - L::c(k, 1), z - L::c(k, 2)};
  bool in = true;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    if (L::c(k, a) == 0) continue;
    if (src[a] < 0 || src[a] >= p.n[a]) {
      if (p.per[a])
        src[a] = (src[a] + p.n[a]) % p.n[a];
      else
        in = false;
    }
  }
  // each post-collision value is pulled once per step: a streaming
  // (nontemporal) load, as the stores of the new state are streaming stores
  if (in)
    return __builtin_nontemporal_load(&fin[k * p.cells + (int64_t)src[2] * p.sz + (int64_t)src[1] * p.sy + src[0]]);
  R val = fin[Lat<Q>::opp(k) * p.cells + P];
  if (L::c(k, 1) < 0 && !p.per[1] && y - L::c(k, 1) >= p.n[1])
    val += R(6 * L::w(k)) * p.rho0 * R(L::c(k, 0)) * p.lid_u;
  return val;
}

// Element u + l of a buffer, u wave-uniform and l a lane's own non-negative
// offset: the uniform part is formed in scalar registers and the access is a
// global load or store with a scalar base and a 32-bit lane offset.
template <class T>
__device__ __forceinline__ T* lane_at(T* base, int64_t u, int l) {
  using C = typename std::conditional<std::is_const<T>::value, const char, char>::type;
  return reinterpret_cast<T*>(reinterpret_cast<C*>(base + u) + (uint32_t)l * (uint32_t)sizeof(T));
}

// A scalar pointer that the compiler may not re-derive: stepping it from one
// component to the next costs two scalar additions, where forming every
// component's address anew costs a 64-bit multiplication each.
template <class T> __device__ __forceinline__ void opaque_ptr(T*& q) { asm volatile("" : "+s"(q)); }

// How a kernel reads the populations and writes the new state, each read once
// and read again only in the next step: streaming (nontemporal), cached, or as
// p.cached says (both forms in the code, which a kernel of a few microseconds
// pays for: 495 -> 517 us in 50 steps of 144 x 700).
enum Access { STREAM, CACHED, EITHER };

// Stores of the C components v of one cell, element u + l of each.
template <int C, Access AC, class R>
__device__ __forceinline__ void store_comps(const KP<R>& p, R* __restrict__ out, int64_t u, int l, const R (&v)[C]) {
  auto put = [&](auto stream) {
    R* q = out + u;
    opaque_ptr(q);
#pragma unroll
    for (int k = 0; k < C; ++k) {
      if constexpr (decltype(stream)::value)
        __builtin_nontemporal_store(v[k], lane_at(q, 0, l));
      else
        *lane_at(q, 0, l) = v[k];
      if (k + 1 < C) {
        q += p.cells;
        opaque_ptr(q);
      }
    }
  };
  if (AC == CACHED || (AC == EITHER && p.cached))
    put(std::false_type());
  else
    put(std::true_type());
}

// Source cells of the pulls of one lane, as element offsets: xs, ys, zs at
// index 1 - c is the cell P - c_k's part along that axis (wrapped on a
// periodic axis, clamped at a wall); w*: the source with c = +1 (index 0) or
// c = -1 (index 2) lies behind a wall.  With ROW a wave's lanes share their
// row, so ys joins zs in the scalar part of the address.
template <bool ROW> struct PullAt {
  using YS = typename std::conditional<ROW, int64_t, int>::type;
  int xs[3];
  YS ys[3];
  int64_t zs[3];
  bool wx[3], wy[3], wz[3];
};
template <int D, bool ROW, class R>
__device__ __forceinline__ PullAt<ROW> pull_at(const KP<R>& p, int x, int y, int z) {
  PullAt<ROW> q;
  auto axis = [](int v, int n, int per, int (&s)[3], bool (&w)[3]) {
    s[1] = v;
    w[1] = false;
    w[0] = !per && v - 1 < 0;
    w[2] = !per && v + 1 >= n;
    s[0] = (v - 1 < 0) ? (per ? v - 1 + n : 0) : v - 1;
    s[2] = (v + 1 >= n) ? (per ? v + 1 - n : n - 1) : v + 1;
  };
  int ys[3], zs[3] = {0, 0, 0};
  q.wz[0] = q.wz[1] = q.wz[2] = false;
  axis(x, p.n[0], p.per[0], q.xs, q.wx);
  axis(y, p.n[1], p.per[1], ys, q.wy);
  if constexpr (D == 3) axis(z, p.n[2], p.per[2], zs, q.wz);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    q.ys[i] = (typename PullAt<ROW>::YS)ys[i] * (typename PullAt<ROW>::YS)p.sy;
    q.zs[i] = (int64_t)zs[i] * p.sz;
  }
  return q;
}

// The populations f^n of the cell (x, y, z) (what pull_f does cell by cell)
// for a wave whose lanes share the plane z and, with ROW, the row y: each
// access is a scalar base plus the lane's 32-bit offset.  (The bases come from
// PullAt's own values, so they are formed per lane where lanes share neither, as
// in k_partial: slower, and the same cells with ROW, whose lane part is x alone.)
// Every source is
// loaded first (clamped at walls); then the cells at a wall, in tiles at the
// grid's faces only, take the reflected population f*_{opp k}(P) instead
// (half-way bounce-back).
template <int D, int Q, bool ROW, Access AC, class R>
__device__ __forceinline__ void pull_cell(const KP<R>& p, const R* __restrict__ fin, const PullAt<ROW>& px,
                                          R (&f)[Q]) {
  using L = Lat<Q>;
  auto get = [&](auto stream) {
    const R* q = fin;
    opaque_ptr(q);
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      const int ix = 1 - L::c(k, 0), iy = 1 - L::c(k, 1), iz = 1 - L::c(k, 2);
      const R* at = lane_at(q, px.zs[iz] + (ROW ? (int64_t)px.ys[iy] : 0), px.xs[ix] + (ROW ? 0 : (int)px.ys[iy]));
      if constexpr (decltype(stream)::value)
        f[k] = __builtin_nontemporal_load(at);
      else
        f[k] = *at;
      if (k + 1 < Q) {
        q += p.cells;
        opaque_ptr(q);
      }
    }
  };
  if (AC == CACHED || (AC == EITHER && p.cached))
    get(std::false_type());
  else
    get(std::true_type());
  auto bounce = [&](int k) -> R {
    R val = *lane_at(fin, (int64_t)L::opp(k) * p.cells + px.zs[1] + (ROW ? (int64_t)px.ys[1] : 0),
                     px.xs[1] + (ROW ? 0 : (int)px.ys[1]));
    // the moving lid: sources above the upper y wall
    if (L::c(k, 1) < 0 && px.wy[2]) val += R(6 * L::w(k)) * p.rho0 * R(L::c(k, 0)) * p.lid_u;
    return val;
  };
#pragma unroll
  for (int a = 0; a < D; ++a)
#pragma unroll
    for (int side = 0; side < 3; side += 2)
      if (a == 0 ? px.wx[side] : (a == 1 ? px.wy[side] : px.wz[side])) {
#pragma unroll
        for (int k = 0; k < Q; ++k)
          if (1 - L::c(k, a) == side) f[k] = bounce(k);
      }
}

// ---------------------------------------------------------------------------
// Phase field: active set, right-hand side, projection.
// ---------------------------------------------------------------------------
// Active set of a cell: bit b set when phase b is non-zero somewhere in the
// 9/19-point neighbourhood v[phase][dz+1][dy+1][dx+1].
// Phase b is non-zero somewhere exactly when its largest value over the
// neighbourhood is positive (one max per value instead of a compare and a
// select).
template <int D, int N, class R>
__device__ __forceinline__ unsigned active_of(const R (&v)[N][3][3][3]) {
  unsigned active = 0u;
#pragma unroll
  for (int b = 0; b < N; ++b) {
    R m = v[b][1][1][1];
#pragma unroll
    for (int dz = (D == 3 ? -1 : 0); dz <= (D == 3 ? 1 : 0); ++dz)
#pragma unroll
      for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
        for (int dx = -1; dx <= 1; ++dx) {
          if (dx != 0 && dy != 0 && dz != 0) continue;
          if (dx == 0 && dy == 0 && dz == 0) continue;
          m = fmax(m, v[b][dz + 1][dy + 1][dx + 1]);
        }
    if (m > R(0)) active |= 1u << b;
  }
  return active;
}

// Right-hand side R_a of Eq. (PhfGrand) (tau eps dphi_a/dt = R_a before the
// constraint) for every phase, from phi^n on the neighbourhood v (walls
// mirrored, periodic axes wrapped; the cube corners are not used) and mu^n:
//   R_a = eps [div J_a - sum_b dA_ab/dq(q_ab) . grad phi_b] - dW/dphi_a / eps
//         - sum_b psi^b dh_b/dphi_a,
// J_a = -sum_b phi_b,f dA_ab/dq(q_ab,f) on faces (none on wall faces).
// mu: mu^n as stored.  ISO: no pair has an anisotropy, so a face flux needs
// the normal derivative only (the general form's values, bit for bit).
template <int D, int N, int NC, class R, bool ISO>
__device__ __forceinline__ void pf_rhs(const KP<R>& p, const R (&v)[N][3][3][3], const R (&mu)[NC], int x, int y,
                                       int z, R tshift, R (&Rv)[N]) {
  const int pos[3] = {x, y, z};
  const R idx = R(1) / p.dx;
  const R ih2 = R(0.5) / p.dx;
  // central difference along e at X = P + o (o within the neighbourhood)
  auto gc = [&](int b, int ox, int oy, int oz, int e) -> R {
    int op[3] = {ox, oy, oz}, om[3] = {ox, oy, oz};
    op[e] += 1;
    om[e] -= 1;
    return (v[b][op[2] + 1][op[1] + 1][op[0] + 1] - v[b][om[2] + 1][om[1] + 1][om[0] + 1]) * ih2;
  };

  R div[N];
#pragma unroll
  for (int b = 0; b < N; ++b) div[b] = R(0);

  // face fluxes J_a = -sum_b phi_b,f dA_ab/dq(q_ab,f), q = phi_a grad phi_b - phi_b grad phi_a
#pragma unroll
  for (int a = 0; a < D; ++a) {
#pragma unroll
    for (int s = -1; s <= 1; s += 2) {
      const bool wall = !p.per[a] && ((s < 0 && pos[a] == 0) || (s > 0 && pos[a] == p.n[a] - 1));
      if (wall) continue;
      int o[3] = {0, 0, 0};
      o[a] = s;
      R pf[N], gf[N][D];
#pragma unroll
      for (int b = 0; b < N; ++b) {
        const R vP = v[b][1][1][1];
        const R vQ = v[b][o[2] + 1][o[1] + 1][o[0] + 1];
        pf[b] = R(0.5) * (vP + vQ);
#pragma unroll
        for (int e = 0; e < D; ++e) {
          if (e == a)
            gf[b][e] = R(s) * (vQ - vP) * idx;
          else if constexpr (!ISO)
            gf[b][e] = R(0.5) * (gc(b, 0, 0, 0, e) + gc(b, o[0], o[1], o[2], e));
        }
      }
      R J[N];
#pragma unroll
      for (int b = 0; b < N; ++b) J[b] = R(0);
#pragma unroll
      for (int al = 0; al < N; ++al)
#pragma unroll
        for (int be = al + 1; be < N; ++be) {
          R q[D], g[D];
          if constexpr (ISO) {
            g[a] = R(2) * p.gamma[al][be] * (pf[al] * gf[be][a] - pf[be] * gf[al][a]);
          } else {
#pragma unroll
            for (int e = 0; e < D; ++e) q[e] = pf[al] * gf[be][e] - pf[be] * gf[al][e];
            dAdq<D, R, R>(q, p.gamma[al][be], p.delta[al][be], p.qmin2, g);
          }
          J[al] -= pf[be] * g[a];
          J[be] += pf[al] * g[a];
        }
#pragma unroll
      for (int b = 0; b < N; ++b) div[b] += R(s) * J[b] * idx;
    }
  }

  // cell-centre terms
  R ph[N], g0[N][D];
#pragma unroll
  for (int b = 0; b < N; ++b) {
    ph[b] = v[b][1][1][1];
#pragma unroll
    for (int e = 0; e < D; ++e) g0[b][e] = gc(b, 0, 0, 0, e);
  }
  R cell[N];
#pragma unroll
  for (int b = 0; b < N; ++b) cell[b] = R(0);
#pragma unroll
  for (int al = 0; al < N; ++al)
#pragma unroll
    for (int be = al + 1; be < N; ++be) {
      R q[D], g[D];
#pragma unroll
      for (int e = 0; e < D; ++e) q[e] = ph[al] * g0[be][e] - ph[be] * g0[al][e];
      if constexpr (ISO) {
#pragma unroll
        for (int e = 0; e < D; ++e) g[e] = R(2) * p.gamma[al][be] * q[e];
      } else {
        dAdq<D, R, R>(q, p.gamma[al][be], p.delta[al][be], p.qmin2, g);
      }
#pragma unroll
      for (int e = 0; e < D; ++e) {
        cell[al] += g[e] * g0[be][e];
        cell[be] -= g[e] * g0[al][e];
      }
    }

  // grand potentials psi^b(mu, T) = -1/2 mu.chi.mu - mu.(c0[b] + mT[b] (T - T_E)) + dS[b] (T - T_E)
  R m[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) m[i] = p.mu_ref[i] + mu[i];
  const R tdev = (p.G != R(0)) ? p.G * (R(pos[p.pull_axis]) - tshift) : p.tdev_iso;
  R ps[N];
#pragma unroll
  for (int b = 0; b < N; ++b) {
    R r = R(0);
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      R chimu = R(0);
#pragma unroll
      for (int j = 0; j < NC; ++j) chimu += p.chi[i][j] * m[j];
      r += -R(0.5) * m[i] * chimu - m[i] * (p.c0[b][i] + p.mT[b][i] * tdev);
    }
    ps[b] = r + p.dS[b] * tdev;
  }

#pragma unroll
  for (int al = 0; al < N; ++al) {
    R dW = R(0);
#pragma unroll
    for (int be = 0; be < N; ++be) {
      if (be == al) continue;
      if (p.potential == 0)
        dW += R(1.6211389382774044) * p.gamma[al][be] * ph[be];  // 16 / pi^2
      else
        dW += R(18) * p.gamma[al][be] * ph[al] * ph[be] * ph[be];
    }
    R drive = R(0);
#pragma unroll
    for (int be = 0; be < N; ++be) drive += ps[be] * dh<N, R>(ph, be, al);
    Rv[al] = p.eps * (div[al] - cell[al]) - dW * p.ieps - drive;
  }
}

// phi^{n+1} of a cell from its neighbourhood v and mu^n: unchanged when one
// phase is active (bulk, returned true), else the projection of
// phi + dt/(tau eps) R over the active phases onto the simplex.  act_out, if
// not null, receives the cell's active set.
template <int D, int N, int NC, class R, bool ISO>
__device__ __forceinline__ bool phi_from_stencil(const KP<R>& p, const R (&v)[N][3][3][3],
                                                 const R (&mu)[NC], int x, int y, int z,
                                                 R tshift, R (&res)[N], uint8_t* __restrict__ act_out) {
  const unsigned active = active_of<D, N, R>(v);
  if (act_out) *act_out = (uint8_t)active;
  if (__builtin_popcount(active) <= 1) {  // bulk: phi unchanged
#pragma unroll
    for (int b = 0; b < N; ++b) res[b] = v[b][1][1][1];
    return true;
  }
  R Rv[N], vv[N];
  pf_rhs<D, N, NC, R, ISO>(p, v, mu, x, y, z, tshift, Rv);
#pragma unroll
  for (int b = 0; b < N; ++b) vv[b] = v[b][1][1][1] + p.rate * Rv[b];
  R theta;
  project_masked<N, R>(active, vv, res, theta);
  return false;
}

// T - T_E of a cell at pull-axis coordinate c, step shift ts
template <class R>
__device__ __forceinline__ R tdev_at(const KP<R>& p, int c, R ts) {
  return (p.G != R(0)) ? p.G * (R(c) - ts) : p.tdev_iso;
}

// C^b_i(mu, T) of one cell, mu as stored; MT: the equilibrium compositions
// depend on T (some mT != 0; an instance of its own keeps the registers of
// the common case)
template <int N, int NC, class R, bool MT>
__device__ __forceinline__ R comp_of(const KP<R>& p, int b, int i, const R (&m)[NC], R td) {
  R C = p.c0s[b][i];
  if constexpr (MT) C += p.mT[b][i] * td;
#pragma unroll
  for (int k = 0; k < NC; ++k) C += p.chi[i][k] * m[k];
  return C;
}

// What a face of the chemical-potential update takes from one of its two
// cells besides mu: the mixture composition c*_i = sum_b h_b(phi^{n+1})
// C^b_i(mu^n, T^n) and the diffusivity d_i = sum_b phi_b D^b_i (the mobility
// is M_ik = d_i chi_ik).
template <int N, int NC, class R, bool MT>
__device__ __forceinline__ void face_quant(const KP<R>& p, const R (&ph)[N], const R (&m)[NC], R td, R (&cs)[NC],
                                           R (&d)[NC]) {
  R h[N];
  interp_h<N, R>(ph, h);
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    cs[i] = R(0);
    d[i] = R(0);
#pragma unroll
    for (int b = 0; b < N; ++b) {
      cs[i] += h[b] * comp_of<N, NC, R, MT>(p, b, i, m, td);
      d[i] += ph[b] * p.D[b][i];
    }
  }
}

// ---------------------------------------------------------------------------
// Forces, moments and collision of one cell from its streamed populations f
// (deviations): U^n and the post-collision populations, stored at element
// u + l of each component.  phi^n, phi^{n+1}, mu^{n+1} at the cell; g1: the
// differences phi^{n+1}_b(P + e_a) - phi^{n+1}_b(P - e_a) that the shrinkage
// force (SH) takes its normals from; td0: T^n - T_E.
// ---------------------------------------------------------------------------
template <int D, int Q, int N, int NC, class R, bool SH, bool MT, Access AC>
__device__ __forceinline__ void collide_cell(const KP<R>& p, int64_t u0, int l0, const R (&f)[Q], const R (&ph0)[N],
                                             const R (&ph1)[N], const R (&mn)[NC], const R (&g1)[SH ? N : 1][D],
                                             R td0, R* __restrict__ u_out, R* __restrict__ fout,
                                             R* __restrict__ dr_out) {
  using L = Lat<Q>;
  // moments (deviation storage: rho = rho0 + sum f~, momentum = sum f~ c)
  R dr = R(0), mom[D];
#pragma unroll
  for (int a = 0; a < D; ++a) mom[a] = R(0);
#pragma unroll
  for (int k = 0; k < L::Q; ++k) {
    dr += f[k];
#pragma unroll
    for (int a = 0; a < D; ++a)
      if (L::c(k, a) != 0) mom[a] += R(L::c(k, a)) * f[k];
  }
  const R rho = p.rho0 + dr;
  if (dr_out) *lane_at(dr_out, u0, l0) = dr;  // kept for the adjoint sweep
  const R phil = ph1[N - 1];
  R bsum = R(0);
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    // the liquid at T^{n+1}
    const R Cl = comp_of<N, NC, R, MT>(p, N - 1, i, mn, td0 + p.dtdev);
    bsum += p.gbeta[i] * (Cl - p.c_ref[i]);
  }
  R FB[D];
#pragma unroll
  for (int a = 0; a < D; ++a) FB[a] = R(0);
  FB[p.grav_axis] = -rho * phil * bsum * p.grav_sign;
  if constexpr (SH) {
    // shrinkage, Eq. (shrinkage): eta_b (phi^{n+1}_b - phi^n_b) along the unit
    // normal of phi^{n+1}_b (central differences, walls mirrored), per lattice
    // step
#pragma unroll
    for (int b = 0; b < N; ++b) {
      if (p.eta[b] == R(0)) continue;
      R g[D], gg = R(0);
#pragma unroll
      for (int a = 0; a < D; ++a) {
        g[a] = g1[b][a] / (R(2) * p.dx);
        gg += g[a] * g[a];
      }
      if (gg > p.qmin2) {
        const R s = p.eta[b] * (ph1[b] - ph0[b]) / gsqrt(gg);
#pragma unroll
        for (int a = 0; a < D; ++a) FB[a] += s * g[a];
      }
    }
  }
  const R sol = (R(1) - phil) * (R(1) - phil);
  R u[D], F[D];
  const R iu = (phil != R(0)) ? R(1) / (rho * (R(1) + R(0.5) * p.kappa * sol)) : R(0);
#pragma unroll
  for (int a = 0; a < D; ++a) {
    u[a] = (mom[a] + R(0.5) * FB[a]) * iu;
    F[a] = FB[a] - p.kappa * rho * sol * u[a];
  }
  R uu = R(0), uF = R(0);
#pragma unroll
  for (int a = 0; a < D; ++a) {
    uu += u[a] * u[a];
    uF += u[a] * F[a];
  }
  // f*_k = f_k + omega (feq_k - f_k) + S_k, written per pair of opposite
  // velocities as keep f_k + w_k (even +- odd):
  //   even = omega dr - 3/2 omega rho u.u - 3 guo u.F + (c.u) (c.h),
  //   odd = c.g,  g = 3 (omega rho u + guo F),  h = 9/2 omega rho u + 9 guo F
  // (10 operations per pair instead of 30; 1 - omega is exact for tau <= 2)
  const R orho = p.omega * rho;
  const R keep = R(1) - p.omega;
  const R e0 = p.omega * dr - R(1.5) * orho * uu - R(3) * p.guo * uF;
  R g[D], h[D];
#pragma unroll
  for (int a = 0; a < D; ++a) {
    g[a] = R(3) * (orho * u[a] + p.guo * F[a]);
    h[a] = R(4.5) * orho * u[a] + R(9) * p.guo * F[a];
  }
  R fp[L::Q];
  fp[0] = keep * f[0] + R(L::w(0)) * e0;
#pragma unroll
  for (int k = 1; k < L::Q; ++k) {
    constexpr auto opp = [](int q) { return L::opp(q); };
    const int kb = opp(k);
    if (kb < k) continue;
    R cu = R(0), cg = R(0), ch = R(0);
#pragma unroll
    for (int a = 0; a < D; ++a) {
      if (L::c(k, a) != 0) {
        cu += R(L::c(k, a)) * u[a];
        cg += R(L::c(k, a)) * g[a];
        ch += R(L::c(k, a)) * h[a];
      }
    }
    const R even = R(L::w(k)) * (e0 + cu * ch), odd = R(L::w(k)) * cg;
    fp[k] = keep * f[k] + (even + odd);
    fp[kb] = keep * f[kb] + (even - odd);
  }
  store_comps<L::Q, AC, R>(p, fout, u0, l0, fp);
  store_comps<D, AC, R>(p, u_out, u0, l0, u);
}

// coordinate along one axis of a tile-halo cell, v >= -1: periodic axes wrap,
// walls clamp (values across a wall are never used: wall faces carry no
// flux).  Beyond n, the first cell past a periodic grid, nothing is used
// either: those cells only have to lie inside.
__device__ __forceinline__ int wrap_or_clamp(int v, int n, int per) {
  if (v < 0) return per ? v + n : 0;
  return v >= n ? (per ? min(v - n, n - 1) : n - 1) : v;
}

// the same for v >= -2 and up to n + 1, two cells past the grid
__device__ __forceinline__ int wrap2_or_clamp(int v, int n, int per) {
  if (v < 0) return per ? (v + n < 0 ? v + 2 * n : v + n) : 0;
  return v >= n ? (per ? min(v - n < n ? v - n : v - 2 * n, n - 1) : n - 1) : v;
}

// Tile of a phase-field block.  Work-groups are dealt to the 8 XCDs
// round-robin; renumbering gives each XCD a contiguous range of tiles, so
// tiles that are neighbours in y and z share its L2.
struct Tile {
  int x0, y0, z0;
  unsigned lb;  // tile index: x fastest, then y, then z
};
template <int D, int TX, int TY, int TZ> struct PhiTile {
  static constexpr int HC = (TX + 2) * (TY + 2) * (D == 3 ? TZ + 2 : 1);  // cells with the halo
};
template <int TX, int TY, int TZ>
__device__ __forceinline__ Tile tile_at(unsigned lb, int tiles_x, int tiles_y) {
  Tile t;
  t.lb = lb;
  const unsigned q = lb / (unsigned)tiles_x;
  t.x0 = (int)(lb - q * (unsigned)tiles_x) * TX;
  t.z0 = (int)(q / (unsigned)tiles_y) * TZ;
  t.y0 = (int)(q % (unsigned)tiles_y) * TY;
  return t;
}
__device__ __forceinline__ unsigned xcd_block() {
  const unsigned nb = gridDim.x, b = blockIdx.x, per8 = nb / 8u;
  return (b < per8 * 8u) ? (b % 8u) * per8 + b / 8u : b;
}

// ---------------------------------------------------------------------------
// Phase field over TX x TY x TZ tiles, one cell per thread: phi^n of the tile
// and its one-cell halo goes to LDS (all of a block's loads in flight
// together, the cell's own mu^n with them), one barrier, then the 9/19-point
// stencil reads LDS.  Bound by the latency of one such tile where few are
// walked (dendrites), by VALU issue on lamellar solids.  The form before this
// one walked 4 or 16 planes of a 64 x 4 column with a barrier per plane; us
// per step of the phase field (todo list and walk), then and now: 28 -> 17
// (256^3 dendrite), 24 -> 17 (64^3), 28 -> 18 (FP64 150 x 131 x 117), 81 -> 42
// (192^3, three phases; 14 of these from ISO), 67 -> 22 (96^3, three phases),
// 91 -> 26 (96 x 96 x 128, four phases).  Tiles of 32 x 4 x 4 cells took 46
// and 30 us in the 192^3 and the four-phase case, 16 x 4 x 4 43 and 27,
// 32 x 8 x 4 49 and 29.
// ---------------------------------------------------------------------------
// One tile.  was_bulk: phi_out, which still holds phi^{n-1}, already holds
// phi^n on every cell of T.  Ends in a barrier after the last read of sh.
// act_out (null: none) receives each cell's active set of phases.
template <int D, int N, int NC, class R, int TX, int TY, int TZ, bool ISO>
__device__ __forceinline__ void phi_tile(const KP<R>& p, const R* __restrict__ phi, const R* __restrict__ mu,
                                         R* __restrict__ phi_out, bool was_bulk, uint8_t* __restrict__ bulk_out,
                                         uint8_t* __restrict__ act_out, R tshift, const Tile& T,
                                         R (&sh)[N][PhiTile<D, TX, TY, TZ>::HC]) {
  constexpr int HX = TX + 2, HY = TY + 2, HC = PhiTile<D, TX, TY, TZ>::HC;
  constexpr int NT = TX * TY * TZ, PER = (HC + NT - 1) / NT;  // halo-tile cells per thread
  const int tid = threadIdx.x;
  const int lx = tid % TX, ly = (tid / TX) % TY, lz = tid / (TX * TY);
  const int x = T.x0 + lx, y = T.y0 + ly, z = T.z0 + lz;
  const bool own = x < p.n[0] && y < p.n[1] && (D == 2 || z < p.n[2]);
  const int64_t P = (int64_t)z * p.sz + (int64_t)y * p.sy + x;
  R pre[PER][N], m[NC];
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const int i = tid + r * NT;
    if (i < HC) {
      const int gx = wrap_or_clamp(T.x0 - 1 + i % HX, p.n[0], p.per[0]);
      const int gy = wrap_or_clamp(T.y0 - 1 + (i / HX) % HY, p.n[1], p.per[1]);
      const int gz = (D == 3) ? wrap_or_clamp(T.z0 - 1 + i / (HX * HY), p.n[2], p.per[2]) : 0;
      const int64_t o = (int64_t)gz * p.sz + (int64_t)gy * p.sy + gx;
#pragma unroll
      for (int q = 0; q < N; ++q) pre[r][q] = phi[q * p.cells + o];
    }
  }
#pragma unroll
  for (int i = 0; i < NC; ++i) m[i] = own ? mu[i * p.cells + P] : R(0);
#pragma unroll
  for (int r = 0; r < PER; ++r)
    if (tid + r * NT < HC)
#pragma unroll
      for (int q = 0; q < N; ++q) sh[q][tid + r * NT] = pre[r][q];
  block_sync_lds();
  int all_bulk = 1;
  if (own) {
    const int c0 = ((D == 3 ? lz + 1 : 0) * HY + ly + 1) * HX + lx + 1;
    R v[N][3][3][3];
#pragma unroll
    for (int dz = (D == 3 ? -1 : 0); dz <= (D == 3 ? 1 : 0); ++dz)
#pragma unroll
      for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
        for (int dx = -1; dx <= 1; ++dx) {
          if (dx != 0 && dy != 0 && dz != 0) continue;
#pragma unroll
          for (int q = 0; q < N; ++q) v[q][dz + 1][dy + 1][dx + 1] = sh[q][c0 + (dz * HY + dy) * HX + dx];
        }
    R res[N];
    const bool bulk =
        phi_from_stencil<D, N, NC, R, ISO>(p, v, m, x, y, z, tshift, res, act_out ? act_out + P : nullptr);
    all_bulk = bulk ? 1 : 0;
    if (!(was_bulk && bulk))
#pragma unroll
      for (int q = 0; q < N; ++q) phi_out[q * p.cells + P] = res[q];
  }
  const int b = __syncthreads_and(all_bulk);
  if (bulk_out && tid == 0) bulk_out[T.lb] = (uint8_t)b;
}

// Bulk flag of the tile at neighbour offset i (0..26: dx, dy, dz in -1..1,
// x fastest) of logical tile lb in a grid of nt[0] x nt[1] x nt[2] tiles;
// periodic axes wrap, and a tile beyond a wall counts as bulk (no stencil
// reaches across a wall).
__device__ __forceinline__ int bulk_flag_at(const uint8_t* __restrict__ bulk, unsigned lb, int i, const int nt[3],
                                            const int per[3], int D) {
  const int d[3] = {i % 3 - 1, (i / 3) % 3 - 1, i / 9 - 1};
  int t3[3] = {(int)(lb % (unsigned)nt[0]), (int)((lb / (unsigned)nt[0]) % (unsigned)nt[1]),
               (int)(lb / (unsigned)(nt[0] * nt[1]))};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    t3[a] += d[a];
    if (t3[a] < 0 || t3[a] >= nt[a]) {
      if (a < D && per[a])
        t3[a] += (t3[a] < 0) ? nt[a] : -nt[a];
      else
        return 1;
    }
  }
  return bulk[t3[0] + nt[0] * (t3[1] + nt[1] * t3[2])];
}

// Bulk history (both null when phi_out is not the buffer that held phi^{n-1}),
// one flag per tile: bulk_in[tile] says every cell of the tile was bulk in the
// step that produced phi^n from phi^{n-1}, so phi_out, which still holds
// phi^{n-1}, already holds phi^n there, and a cell that is bulk again (phi^{n+1}
// = phi^n) need not be stored.  bulk_out[tile] records the same for this step.
// If a tile and every tile its stencils reach (the 26 around it, none beyond a
// wall) were bulk in that step, phi^n = phi^{n-1} on every stencil the tile
// evaluates, so each cell has its previous active set and is bulk again:
// phi_out already holds phi^{n+1} = phi^n, nothing to do.
//
// On a 3D grid that is mostly bulk nearly every tile of a launch is of that
// kind, and dispatching a block for each costs more than the others' work.
// There k_phi, launched with a grid of resident blocks, walks a list of the
// other tiles, which the step before made: once its k_phi has set every flag,
// phi_todo (on blocks of its own in the step's k_mulbm, one thread per tile)
// checks every tile's neighbourhood, sets the next step's flag of each tile that
// will be skipped and appends the others.  Each XCD walks a contiguous part of
// the list (whose waves append in about the order of the tiles), so tiles that
// are neighbours share its L2.  Two list lengths take turns: a k_mulbm counts
// into one, zero until then, and clears the other, which its step's k_phi has
// read.  (A launch of its own for the list cost 6 to 7 us per step: 25 us of a
// 64^3 step, now 20.)
// ---------------------------------------------------------------------------
// What a k_mulbm is to list: nb tiles of flags `in` (x fastest, nt per axis);
// no blocks: nothing.
struct Todo {
  const uint8_t* in;
  uint8_t* out;
  unsigned *list, *count, *clear;
  int nt[3];
  unsigned nb, blocks;
};
template <int D, int NT>
__device__ __forceinline__ void phi_todo(const Todo& t, const int (&per)[3]) {
  const unsigned lb = blockIdx.x * (unsigned)NT + threadIdx.x;
  bool need = false;
  if (lb < t.nb) {
    int ok = 1;
#pragma unroll
    for (int i = 0; i < 27; ++i) ok &= bulk_flag_at(t.in, lb, i, t.nt, per, D);
    if (ok)
      t.out[lb] = 1;
    else
      need = true;
  }
  // one atomic per wave; the wave's listed tiles take consecutive slots
  const unsigned long long m = __ballot(need);
  const unsigned lane = __lane_id();
  unsigned base = 0;
  if (m && lane == 0) base = atomicAdd(t.count, (unsigned)__popcll(m));
  base = __shfl(base, 0);
  const unsigned slot = base + (unsigned)__popcll(m & ((1ull << lane) - 1ull));
  if (need && slot < t.nb) t.list[slot] = lb;
}

// list null: every tile, each checked for the skip above where bulk_in is given.
// One kernel for both: the compiler's choice of
// fused multiply-adds is the same, so a run resumed from a checkpoint, whose
// first step has no history, continues bit for bit.  gridDim.x is a multiple
// of 8: XCD k (blocks b = k mod 8) takes part k of the tiles.
template <int D, int N, int NC, class R, int TX, int TY, int TZ, bool ISO>
__global__ void __launch_bounds__(TX * TY * TZ)
k_phi(KP<R> p, const R* __restrict__ phi, const R* __restrict__ mu, R* __restrict__ phi_out,
      const uint8_t* __restrict__ bulk_in, uint8_t* __restrict__ bulk_out, uint8_t* __restrict__ act_out,
      const unsigned* __restrict__ list, const unsigned* __restrict__ count, R tshift, int tiles_x, int tiles_y,
      int tiles_z) {
  __shared__ R sh[N][PhiTile<D, TX, TY, TZ>::HC];
  const unsigned nb = (unsigned)tiles_x * (unsigned)tiles_y * (unsigned)tiles_z;
  const unsigned cnt = list ? min(*count, nb) : nb;
  const bool check = !list && bulk_in;
  const unsigned g8 = gridDim.x / 8u, k = blockIdx.x % 8u;
  const unsigned hi = (unsigned)(((unsigned long long)cnt * (k + 1u)) / 8u);
  for (unsigned w = (unsigned)(((unsigned long long)cnt * k) / 8u) + blockIdx.x / 8u; w < hi; w += g8) {
    const unsigned lb = list ? list[w] : w;
    // listed entries are tile indices (the list starts zeroed); the test keeps
    // a count that disagrees with the list inside the grid (uniform per block)
    if (lb >= nb) continue;
    // the parameter block (first kernel argument), read anew for every tile:
    // carried through the loop it took 20 to 50 vector registers
    using KPc = const __attribute__((address_space(4))) KP<R>*;
    KPc kp = (KPc)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(kp));
    const KP<R>& q = *(const KP<R>*)kp;
    if (check) {
      int ok = 1;
      if (threadIdx.x < 27) {
        const int nt[3] = {tiles_x, tiles_y, tiles_z};
        ok = bulk_flag_at(bulk_in, lb, (int)threadIdx.x, nt, q.per, D);
      }
      if (__syncthreads_and(ok)) {
        if (bulk_out && threadIdx.x == 0) bulk_out[lb] = 1;
        continue;
      }
    }
    phi_tile<D, N, NC, R, TX, TY, TZ, ISO>(q, phi, mu, phi_out, bulk_in && bulk_in[lb], bulk_out, act_out, tshift,
                                           tile_at<TX, TY, TZ>(lb, tiles_x, tiles_y), sh);
  }
}

// ---------------------------------------------------------------------------
// Chemical potential + LBM over TX x TY x TZ tiles, one cell per thread.
// Each thread loads phi^{n+1}, mu^n and U of its own cell and of about one
// cell of the tile's face halo, forms from them what the faces of the mu
// update need (face_quant) once per cell, and shares it through LDS; the
// populations are pulled meanwhile.  One barrier per block, no loop: a wave
// has all of its loads in flight at once and many blocks per CU overlap
// their loads with each other's arithmetic and stores.
// Order of the tiles: strips of `strip` tile rows, walked layer by layer along
// z, so that a layer's halo planes are read again while the strip's own are
// still in L2; each XCD takes a contiguous part of that order.  With an eighth
// of the rows per strip every XCD owns one strip and all eight walk the same
// planes together (192^3 FP32: 259 us, strips of 8 tile rows 280; three phases
// 273 and 294; 256^3: 630, and 640 to 708 with strips of a quarter or half).
// Threads past the grid's edge hold the wrapped (periodic) or clamped (wall)
// cell, which only serves as a neighbour.
// ---------------------------------------------------------------------------
// HBM bound in 3D (FP32, 256^3: 197 B/cell moved of the 168 that the state
// needs), VALU issue beside it for three and four phases.  The form before
// this one walked 64 x 4 columns plane by plane, held the next plane's values
// in registers (127 to 186 of them, 2 to 4 waves per SIMD) and formed
// face_quant at all seven cells: 50 to 81 registers now.  us per launch, then
// and now: 675 -> 631 (256^3, two phases, FP32), 1407 -> 1236 (FP64), 357 ->
// 293 (192^3, three phases, two solutes), 117 -> 67 (96 x 96 x 128, four
// phases), 35 -> 19 (64^3); tiles of 32 x 4 x 2 and 32 x 4 x 4 cells took 646
// and 673 on 256^3, 64 x 2 x 2 took 664 and 64 x 4 x 1 632.  Two phases in FP32
// gain from tiles of whole 1 KiB rows (256 x 2 x 1), whose x-shifted pulls share
// their lines within a CU: 629 -> 603 us on 256^3, 265 -> 246 on 250 x 200 x
// 128, though 95 -> 109 on 128^3, where half of their lanes idle; in FP64 (1224
// and 1228) and with more phases (176 and 178) they gain nothing.
// Tiles of 32 x 4 x 2 on rows of up to 32 and of 65 to 96 cells, of whose lanes 64
// columns leave a quarter and more without a cell; us per step with 64 and with 32
// columns: 49.1 and 45.8 (96^3, two phases, FP32), 83.8 and 78.8 (FP64), 48.8 and
// 44.7 (three phases), 23.9 and 18.1 (24 x 80 x 80), 47.1 and 40.1 (66 x 70 x 60,
// FP64).  Rows of 129 to 160 cells, of whose lanes 64 columns leave 17 to 33 %, keep
// 64: 129 x 128 x 96 83 and 85, three phases 101 and 105, 27 velocities on 129 x 160 x
// 96 136 and 141, 150 x 128 x 96 84 and 86; in FP64 144 and 140, but three phases 216
// and 171.
// LDS-shared slots of a tile: its T cells (slot = thread), then the halo of
// each face: z-, z+ (TX x TY cells each), y-, y+ (TX x TZ), x-, x+ (TY x TZ).
template <int D, int TX, int TY, int TZ> struct MuTile {
  static constexpr int T = TX * TY * TZ;
  static constexpr int HZ = (D == 3) ? TX * TY : 0, HY = TX * TZ, HX = TY * TZ;
  static constexpr int H = 2 * (HZ + HY + HX);
  // first halo slot of axis a, relative to T
  static constexpr int base(int a) { return a == 2 ? 0 : (a == 1 ? 2 * HZ : 2 * (HZ + HY)); }
  static constexpr int face(int a) { return a == 2 ? HZ : (a == 1 ? HY : HX); }
};

// mu^{n+1} (mn) of a thread's cell from the tile's shared slots: sv holds mu^n,
// c*, d (and with SH phi^{n+1}) per slot, su U_a of the tile's cells axis after
// axis, then of the halo of the faces along a.  pos, lpos: the cell in the grid
// and in the tile (slot tid).  g1 (SH): the differences of phi^{n+1} across the
// cell that its normals are taken from.
template <int D, int N, int NC, class R, int TX, int TY, int TZ, bool SH, bool MT, int NV, int NS, int NU>
__device__ __forceinline__ void mu_update(const KP<R>& p, const int (&pos)[3], const int (&lpos)[3], int tid,
                                          const R (&sv)[NV][NS], const R (&su)[NU], const R (&ph0)[N],
                                          const R (&ph1)[N], const R (&m0)[NC], const R (&uc)[D], const R (&cs0)[NC],
                                          const R (&d0)[NC], R td0, R (&mn)[NC], R (&g1)[SH ? N : 1][D]) {
  using M = MuTile<D, TX, TY, TZ>;
  constexpr int T = M::T;
  // divergence of the face fluxes (diffusion and advection)
  R divJ[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) divJ[i] = R(0);
  const int text[3] = {TX, TY, TZ}, tstr[3] = {1, TX, TX * TY};
#pragma unroll
  for (int a = 0; a < D; ++a) {
    // index of the cell's column within a face of the tile across axis a
    const int fi = a == 0 ? lpos[2] * TY + lpos[1] : (a == 1 ? lpos[2] * TX + lpos[0] : lpos[1] * TX + lpos[0]);
#pragma unroll
    for (int si = 0; si < 2; ++si) {
      const int s = si ? 1 : -1;
      const bool inner = si ? lpos[a] + 1 < text[a] : lpos[a] > 0;
      const int h = M::base(a) + si * M::face(a) + fi;
      const int slot = inner ? tid + s * tstr[a] : T + h;
      if constexpr (SH) {
        // (the slot beyond a wall holds the cell at the wall itself)
#pragma unroll
        for (int b = 0; b < N; ++b) g1[b][a] = si ? sv[3 * NC + b][slot] - g1[b][a] : sv[3 * NC + b][slot];
      }
      const bool wall = !p.per[a] && ((s < 0 && pos[a] == 0) || (s > 0 && pos[a] == p.n[a] - 1));
      if (wall) continue;
      const R uf = R(0.5) * (uc[a] + su[inner ? a * T + slot : D * T + h]) * p.conv;
      R dm[NC];
#pragma unroll
      for (int k = 0; k < NC; ++k) dm[k] = R(s) * (sv[k][slot] - m0[k]) * p.idx;
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        const R df = -R(0.5) * (d0[i] + sv[2 * NC + i][slot]);
        R JD = R(0);
#pragma unroll
        for (int k = 0; k < NC; ++k) JD += df * p.chi[i][k] * dm[k];
        const R JA = uf * R(0.5) * (cs0[i] + sv[NC + i][slot]);
        divJ[i] += R(s) * (JD + JA) * p.idx;
      }
    }
  }
  R h0[N], h1[N];
  interp_h<N, R>(ph0, h0);
  interp_h<N, R>(ph1, h1);
  R Dl[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) Dl[i] = -p.dt * divJ[i];
  // dh/dt source with C at T^n, and the dT/dt term of Eq. (conc) over the
  // step, -sum_b h_b^{n+1} (C^b(mu^n, T^{n+1}) - C^b(mu^n, T^n)) = -sum_b
  // h_b^{n+1} mT[b] (T^{n+1} - T^n)
  R sh = R(0);
#pragma unroll
  for (int b = 0; b < N; ++b) {
    sh += h1[b];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      Dl[i] -= comp_of<N, NC, R, MT>(p, b, i, m0, td0) * (h1[b] - h0[b]);
      if constexpr (MT) Dl[i] -= h1[b] * (p.mT[b][i] * p.dtdev);
    }
  }
  if (NC == 1) {
    mn[0] = m0[0] + Dl[0] / (sh * p.chi[0][0]);
  } else {
    const R a11 = sh * p.chi[0][0], a12 = sh * p.chi[0][1];
    const R a21 = sh * p.chi[1][0], a22 = sh * p.chi[1][NC - 1];
    const R det = a11 * a22 - a12 * a21;
    mn[0] = m0[0] + (a22 * Dl[0] - a12 * Dl[NC - 1]) / det;
    mn[NC - 1] = m0[NC - 1] + (-a21 * Dl[0] + a11 * Dl[NC - 1]) / det;
  }
}

template <int D, int Q, int N, int NC, class R, int TX, int TY, int TZ, bool SH, bool MT>
__global__ void __launch_bounds__(TX * TY * TZ)
k_mulbm(KP<R> p, const R* __restrict__ phi0, const R* __restrict__ phi1, const R* __restrict__ mu,
        const R* __restrict__ uold, const R* __restrict__ fin, R* __restrict__ mu_out, R* __restrict__ u_out,
        R* __restrict__ fout, R* __restrict__ dr_out, const uint8_t* __restrict__ phi_bulk, int phi_lx, int phi_ly,
        int phi_lz, R tshift, int tiles_x, int tiles_y, int strip, Todo todo) {
  using M = MuTile<D, TX, TY, TZ>;
  // Two phases stream whatever p.cached says.  With both forms in the code, which
  // also changes how the compiler orders the loads, us per step were 46 -> 37 on 96^3
  // (FP32, in the cache) and 95 -> 92 on 128^3, but 20.5 -> 21.6 on 64^3 and, FP64 and 27
  // velocities, 343 -> 373 on 200 x 160 x 96.
  constexpr Access AC = N == 2 ? STREAM : EITHER;
  constexpr bool ROW = TX % 64 == 0;
  static_assert(TX * TY >= 64 && (ROW || 64 % TX == 0), "a wave's lanes share a plane, and with ROW a row");
  static_assert(D == 3 || TZ == 1, "one plane in 2D");
  constexpr int T = M::T, H = M::H, HI = (H + T - 1) / T;
  constexpr int NV = 3 * NC + (SH ? N : 0);  // mu, c*, d (and phi^{n+1}) per slot
  __shared__ R sv[NV][T + H];
  __shared__ R su[D * T + H];  // U_a of the cells, axis after axis, then of the halo of the faces along a
  if (blockIdx.x < todo.blocks) {
    phi_todo<D, T>(todo, p.per);
    return;
  }
  int x0, y0, z0;
  {
    // contiguous part of the tile order per XCD (todo.blocks is a multiple of
    // 8), then strips
    const unsigned nb = gridDim.x - todo.blocks, b = blockIdx.x - todo.blocks, per8 = nb / 8u;
    const unsigned lb = (b < per8 * 8u) ? (b % 8u) * per8 + b / 8u : b;
    const unsigned tx = (unsigned)tiles_x, ty = (unsigned)tiles_y, layers = nb / (tx * ty);
    const unsigned sfull = (unsigned)strip * tx * layers;  // tiles of a full strip
    const unsigned s = lb / sfull, r = lb % sfull;
    const unsigned hs = min((unsigned)strip, ty - s * (unsigned)strip);
    const unsigned z = r / (hs * tx), q = r % (hs * tx);
    x0 = (int)(q % tx) * TX;
    y0 = (int)(s * (unsigned)strip + q / tx) * TY;
    z0 = (int)z * TZ;
  }
  const int tid = threadIdx.x;
  // the step's k_phi, which read this list length, has finished
  if (todo.clear && blockIdx.x == todo.blocks && tid == 0) atomicExch(todo.clear, 0u);
  const int lx = tid % TX;
  const int ly = ROW ? __builtin_amdgcn_readfirstlane((tid / TX) % TY) : (tid / TX) % TY;
  const int lz = (D == 3) ? __builtin_amdgcn_readfirstlane(tid / (TX * TY)) : 0;
  const int x = x0 + lx, y = y0 + ly, z = z0 + lz;
  // the padding of a row is computed and stored too (from the wrapped or
  // clamped cell): its last line leaves the chip whole
  const bool own = x < (int)p.sy && y < p.n[1] && (D == 2 || z < p.n[2]);
  const int xw = wrap_or_clamp(x, p.n[0], p.per[0]), yw = wrap_or_clamp(y, p.n[1], p.per[1]);
  const int zw = (D == 3) ? wrap_or_clamp(z, p.n[2], p.per[2]) : 0;
  // the thread's cell: scalar part and lane part of its element offset
  const int64_t cu = (int64_t)zw * p.sz + (ROW ? (int64_t)yw * p.sy : 0);
  const int cl = xw + (ROW ? 0 : (int)((uint32_t)yw * (uint32_t)p.sy));
  const int cs = cl + (x - xw);  // where the cell is stored
  // phi_bulk (the phase field's flags of this step, null when there are none):
  // where the phase-field tile (2^phi_lx x 2^phi_ly x 2^phi_lz cells) that
  // holds this cell was left bulk, phi^n =
  // phi^{n+1}, so phi^n is not read
  bool same0 = false;
  if (phi_bulk) {
    const int ptx = ((p.n[0] - 1) >> phi_lx) + 1, pty = ((p.n[1] - 1) >> phi_ly) + 1;
    same0 = phi_bulk[(xw >> phi_lx) + ptx * ((yw >> phi_ly) + pty * (D == 3 ? zw >> phi_lz : 0))] != 0;
  }
  R ph1[N], m0[NC], uc[D], ph0[N];
#pragma unroll
  for (int q = 0; q < N; ++q) ph1[q] = *lane_at(phi1, q * p.cells + cu, cl);
#pragma unroll
  for (int q = 0; q < NC; ++q) m0[q] = *lane_at(mu, q * p.cells + cu, cl);
#pragma unroll
  for (int a = 0; a < D; ++a) uc[a] = *lane_at(uold, a * p.cells + cu, cl);
  // halo cells of this thread: slots T + tid, T + tid + T, ...
  R hph[HI][N], hm[HI][NC], hu[HI];
  int hpa[HI];  // their pull-axis coordinate
#pragma unroll
  for (int i = 0; i < HI; ++i) {
    const int j = tid + i * T;
    if (j < H) {
      int hx, hy, hz, a;
      if (j < 2 * M::HZ) {
        const int r = j % (TX * TY);
        a = 2;
        hx = x0 + r % TX;
        hy = y0 + r / TX;
        hz = (j >= M::HZ) ? z0 + TZ : z0 - 1;
      } else if (j < 2 * (M::HZ + M::HY)) {
        const int q = j - 2 * M::HZ, r = q % M::HY;
        a = 1;
        hx = x0 + r % TX;
        hz = z0 + r / TX;
        hy = (q >= M::HY) ? y0 + TY : y0 - 1;
      } else {
        const int q = j - 2 * (M::HZ + M::HY), r = q % M::HX;
        a = 0;
        hy = y0 + r % TY;
        hz = z0 + r / TY;
        hx = (q >= M::HX) ? x0 + TX : x0 - 1;
      }
      hx = wrap_or_clamp(hx, p.n[0], p.per[0]);
      hy = wrap_or_clamp(hy, p.n[1], p.per[1]);
      hz = (D == 3) ? wrap_or_clamp(hz, p.n[2], p.per[2]) : 0;
      const int64_t o = (int64_t)hz * p.sz + (int64_t)hy * p.sy + hx;
#pragma unroll
      for (int q = 0; q < N; ++q) hph[i][q] = phi1[q * p.cells + o];
#pragma unroll
      for (int q = 0; q < NC; ++q) hm[i][q] = mu[q * p.cells + o];
      hu[i] = uold[a * p.cells + o];
      hpa[i] = (p.pull_axis == 0) ? hx : (p.pull_axis == 1 ? hy : hz);
    }
  }
  R f[Q];
  const PullAt<ROW> px = pull_at<D, ROW, R>(p, xw, yw, zw);
  if (own) pull_cell<D, Q, ROW, AC, R>(p, fin, px, f);
  if (!same0) {
#pragma unroll
    for (int q = 0; q < N; ++q) ph0[q] = *lane_at(phi0, q * p.cells + cu, cl);
  }
  const int pa = p.pull_axis;
  const R td0 = MT ? tdev_at(p, pa == 0 ? xw : (pa == 1 ? yw : zw), tshift) : R(0);
  R cs0[NC], d0[NC];
  face_quant<N, NC, R, MT>(p, ph1, m0, td0, cs0, d0);
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    sv[q][tid] = m0[q];
    sv[NC + q][tid] = cs0[q];
    sv[2 * NC + q][tid] = d0[q];
  }
  if constexpr (SH)
#pragma unroll
    for (int q = 0; q < N; ++q) sv[3 * NC + q][tid] = ph1[q];
#pragma unroll
  for (int a = 0; a < D; ++a) su[a * T + tid] = uc[a];
#pragma unroll
  for (int i = 0; i < HI; ++i) {
    const int j = tid + i * T;
    if (j < H) {
      R cq[NC], d[NC];
      face_quant<N, NC, R, MT>(p, hph[i], hm[i], MT ? tdev_at(p, hpa[i], tshift) : R(0), cq, d);
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        sv[q][T + j] = hm[i][q];
        sv[NC + q][T + j] = cq[q];
        sv[2 * NC + q][T + j] = d[q];
      }
      if constexpr (SH)
#pragma unroll
        for (int q = 0; q < N; ++q) sv[3 * NC + q][T + j] = hph[i][q];
      su[D * T + j] = hu[i];
    }
  }
  block_sync_lds();
  if (!own) return;

  if (same0) {
#pragma unroll
    for (int q = 0; q < N; ++q) ph0[q] = ph1[q];
  }
  R mn[NC], g1[SH ? N : 1][D];
  const int pos[3] = {x, y, z}, lpos[3] = {lx, ly, lz};
  mu_update<D, N, NC, R, TX, TY, TZ, SH, MT>(p, pos, lpos, tid, sv, su, ph0, ph1, m0, uc, cs0, d0, td0, mn, g1);
  store_comps<NC, AC, R>(p, mu_out, cu, cs, mn);
  collide_cell<D, Q, N, NC, R, SH, MT, AC>(p, cu, cs, f, ph0, ph1, mn, g1, td0, u_out, fout, dr_out);
}

// ---------------------------------------------------------------------------
// One step of a 2D grid in one launch.  A block owns TX x TY cells, one per
// thread, and has a thread more for every cell of the tile's face halo: each
// computes phi^{n+1} of its cell from phi^n of the tile and two halo cells (in
// LDS) and from it the face quantities that the tile shares; then the tile's
// threads update mu and the populations as k_mulbm does.
// Up to some 10^5 cells a 2D step is bound by latency: the launch (1.5 to 2
// us), a chain of loads (1.5), the phase field of an interface cell (0.8), the
// rest (0.8).  One launch for both halves and the halo's phase field on waves
// of its own shorten that chain; a grid of some 10^5 cells and more gains from
// reading the phase fields once.  us per step in a run, k_phi and k_mulbm in
// turn and this kernel: 9.1 and 5.6 (256^2, FP32), 9.7 and 6.0 (128^2, FP64),
// 13.5 and 8.4 (144 x 700, four phases), 19.7 and 17.0 (1024 x 512, three
// phases, FP32); but 33.9 and 36 (the same in FP64) and 98 and 109 (2048^2,
// two phases, FP32), where the halo's share of the work counts and the bulk
// history spares k_phi most of its tiles.  An instance of its own without
// anisotropy (ISO), and the populations' loads sent off before the wait for the
// phase field's: 2 to 3 % of a step of three and four phases without it, 1 % of
// two (before, the instance chose at run time).
// ---------------------------------------------------------------------------
template <int TX, int TY> struct StepTile {
  static constexpr int T = TX * TY, H = 2 * (TX + TY), NT = T + (H + 63) / 64 * 64;
};

template <int Q, int N, int NC, class R, int TX, int TY, bool SH, bool MT, bool ISO>
__global__ void __launch_bounds__((StepTile<TX, TY>::NT))
k_step2(KP<R> p, const R* __restrict__ phi0, R* __restrict__ phi1, const R* __restrict__ mu,
        const R* __restrict__ uold, const R* __restrict__ fin, R* __restrict__ mu_out, R* __restrict__ u_out,
        R* __restrict__ fout, R* __restrict__ dr_out, uint8_t* __restrict__ act_out, R tshift, int tiles_x) {
  constexpr int D = 2;
  using M = MuTile<D, TX, TY, 1>;
  // the wide tile is that of grids above 2^18 cells whose two states fit the
  // last-level cache
  constexpr Access AC = TX == 64 ? CACHED : STREAM;
  constexpr bool ROW = TX == 64;
  constexpr int T = StepTile<TX, TY>::T, H = StepTile<TX, TY>::H, NT = StepTile<TX, TY>::NT;
  static_assert(T % 64 == 0 && H == M::H, "tile threads fill their waves; slots as in MuTile");
  constexpr int FX = TX + 4, FY = TY + 4, FC = FX * FY, FP = (FC + NT - 1) / NT;
  constexpr int NV = 3 * NC + (SH ? N : 0);
  __shared__ R sp[N][FC];  // phi^n of the tile and two halo cells, walls repeating the last cell
  __shared__ R sv[NV][T + H];
  __shared__ R su[D * T + H];
  const unsigned lb = xcd_block();
  const int x0 = (int)(lb % (unsigned)tiles_x) * TX, y0 = (int)(lb / (unsigned)tiles_x) * TY;
  const int tid = threadIdx.x;
  R fpre[FP][N];
#pragma unroll
  for (int r = 0; r < FP; ++r) {
    const int i = min(tid + r * NT, FC - 1);
    const int64_t o = (int64_t)wrap2_or_clamp(y0 - 2 + i / FX, p.n[1], p.per[1]) * p.sy +
                      wrap2_or_clamp(x0 - 2 + i % FX, p.n[0], p.per[0]);
#pragma unroll
    for (int q = 0; q < N; ++q) fpre[r][q] = phi0[q * p.cells + o];
  }
  // the thread's cell: of the tile (slot tid < T), or of the halo of a face
  // along axis ha (slot tid = T + j)
  const bool tile = __builtin_amdgcn_readfirstlane(tid) < T;
  int lx = tid % TX, ly = tid / TX, ha = 0;
  if (!tile) {
    const int j = min(tid - T, H - 1);
    if (j < 2 * TX) {
      ha = 1;
      lx = j % TX;
      ly = (j >= TX) ? TY : -1;
    } else {
      ly = (j - 2 * TX) % TY;
      lx = (j - 2 * TX >= TY) ? TX : -1;
    }
  }
  const int x = x0 + lx, y = y0 + ly;
  const int xw = wrap_or_clamp(x, p.n[0], p.per[0]), yw = wrap_or_clamp(y, p.n[1], p.per[1]);
  // its place in sp: on a periodic axis the cell itself, at a wall the cell it repeats
  const int c0 = ((p.per[1] ? y : yw) - y0 + 2) * FX + (p.per[0] ? x : xw) - x0 + 2;
  const int64_t P = (int64_t)yw * p.sy + xw;
  R m0[NC], uc[D];
#pragma unroll
  for (int q = 0; q < NC; ++q) m0[q] = mu[q * p.cells + P];
  if (tile) {
#pragma unroll
    for (int a = 0; a < D; ++a) uc[a] = uold[a * p.cells + P];
  } else {
    uc[0] = uold[ha * p.cells + P];
    uc[1] = R(0);
  }
  // the padding of a row is computed and stored too, as in k_mulbm
  const bool own = tile && x < (int)p.sy && y < p.n[1];
  // (with ROW a wave of the tile shares its row)
  const PullAt<ROW> px = pull_at<D, ROW, R>(p, xw, ROW ? __builtin_amdgcn_readfirstlane(yw) : yw, 0);
  R f[Q];
  if (own) pull_cell<D, Q, ROW, AC, R>(p, fin, px, f);
#pragma unroll
  for (int r = 0; r < FP; ++r)
    if (tid + r * NT < FC)
#pragma unroll
      for (int q = 0; q < N; ++q) sp[q][tid + r * NT] = fpre[r][q];
  block_sync_lds();
  R ph0[N], ph1[N];
  {
    R v[N][3][3][3];
#pragma unroll
    for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
      for (int dx = -1; dx <= 1; ++dx)
#pragma unroll
        for (int q = 0; q < N; ++q) v[q][1][dy + 1][dx + 1] = sp[q][c0 + dy * FX + dx];
#pragma unroll
    for (int q = 0; q < N; ++q) ph0[q] = v[q][1][1][1];
    uint8_t* act = (act_out && tile && x < p.n[0] && y < p.n[1]) ? act_out + P : nullptr;
    phi_from_stencil<D, N, NC, R, ISO>(p, v, m0, xw, yw, 0, tshift, ph1, act);
  }
  const R td0 = MT ? tdev_at(p, p.pull_axis == 0 ? xw : yw, tshift) : R(0);
  R cs0[NC], d0[NC];
  face_quant<N, NC, R, MT>(p, ph1, m0, td0, cs0, d0);
  if (tid < T + H) {
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      sv[q][tid] = m0[q];
      sv[NC + q][tid] = cs0[q];
      sv[2 * NC + q][tid] = d0[q];
    }
    if constexpr (SH)
#pragma unroll
      for (int q = 0; q < N; ++q) sv[3 * NC + q][tid] = ph1[q];
    if (tile) {
#pragma unroll
      for (int a = 0; a < D; ++a) su[a * T + tid] = uc[a];
    } else {
      su[(D - 1) * T + tid] = uc[0];
    }
  }
  block_sync_lds();
  if (!own) return;
  const int64_t cu = ROW ? (int64_t)__builtin_amdgcn_readfirstlane(y) * p.sy : 0;
  const int cs = x + (ROW ? 0 : y * (int)p.sy);
  store_comps<N, AC, R>(p, phi1, cu, cs, ph1);
  R mn[NC], g1[SH ? N : 1][D];
  const int pos[3] = {x, y, 0}, lpos[3] = {lx, ly, 0};
  mu_update<D, N, NC, R, TX, TY, 1, SH, MT>(p, pos, lpos, tid, sv, su, ph0, ph1, m0, uc, cs0, d0, td0, mn, g1);
  store_comps<NC, AC, R>(p, mu_out, cu, cs, mn);
  collide_cell<D, Q, N, NC, R, SH, MT, AC>(p, cu, cs, f, ph0, ph1, mn, g1, td0, u_out, fout, dr_out);
}

// ---------------------------------------------------------------------------
// Auxiliary kernels (read, write, totals, health).  One thread per cell on a
// 1D grid.
// ---------------------------------------------------------------------------

// Moving frame (Case 2 follows the growth front with a moving frame; the
// paper gives no details, the reading is stated with the host code).
// k_front: the largest pull-axis index of a cell whose liquid fraction is at
// most 1/2 (-1 if none), max-reduced over each wave, then one atomic per wave.
template <int N, class R>
__global__ void __launch_bounds__(256) k_front(KP<R> p, const R* __restrict__ phi, int* __restrict__ front) {
  int v = -1, x, y, z;
  int64_t P;
  if (dense_cell(p, (int64_t)blockIdx.x * blockDim.x + threadIdx.x, x, y, z, P) &&
      phi[(N - 1) * p.cells + P] <= R(0.5))
    v = (p.pull_axis == 0) ? x : (p.pull_axis == 1) ? y : z;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off, 64));
  if ((threadIdx.x & 63) == 0 && v >= 0) atomicMax(front, v);
}

// k_shift: out = in moved down axis ax by d cells (all components); the last
// d planes repeat the last plane of `in`.
template <class R>
__global__ void k_shift(KP<R> p, const R* __restrict__ in, R* __restrict__ out, int ncomp, int ax, int64_t d) {
  int x, y, z;
  int64_t P;
  if (!dense_cell(p, (int64_t)blockIdx.x * blockDim.x + threadIdx.x, x, y, z, P)) return;
  const int64_t c = ax == 0 ? x : (ax == 1 ? y : z), stride = ax == 0 ? 1 : (ax == 1 ? p.sy : p.sz);
  const int64_t o = (min(c + d, (int64_t)p.n[ax] - 1) - c) * stride;
  for (int k = 0; k < ncomp; ++k) out[k * p.cells + P] = in[k * p.cells + P + o];
}

// f^n_k(P) = stored f*_k(P - c_k) (+ bounce-back), plus w_k rho0 in FP64: the
// full f in dense order, as T.  A block owns 4 rows of 64 cells.  HBM bound
// (one read and one write of the populations: 166 us a call on FP64 150 x 131 x
// 117, through an FP64 copy and a conversion 277).
template <int D, int Q, class R, class T>
__global__ void __launch_bounds__(256) k_gather_f(KP<R> p, const R* __restrict__ fin, T* __restrict__ out, int tiles_x,
                                                  int tiles_y) {
  using L = Lat<Q>;
  const Tile t = tile_at<64, 4, 1>(xcd_block(), tiles_x, tiles_y);
  const int x = t.x0 + (int)threadIdx.x % 64;
  const int y = t.y0 + __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64), z = (D == 3) ? t.z0 : 0;
  if (x >= p.n[0] || y >= p.n[1]) return;
  R f[Q];
  pull_cell<D, Q, true, STREAM, R>(p, fin, pull_at<D, true, R>(p, x, y, z), f);
  T* q = out + ((int64_t)z * p.n[1] + y) * p.n[0];
  opaque_ptr(q);
#pragma unroll
  for (int k = 0; k < L::Q; ++k) {
    *lane_at(q, 0, x) = (T)((double)f[k] + L::w(k) * (double)p.rho0);
    if (k + 1 < L::Q) {
      q += p.live;
      opaque_ptr(q);
    }
  }
}

// inverse of k_gather_f: the stored pre-streaming f* that streams to f^n.
// With d > 0 it inverts the pull of f^n moved down axis `ax` by d cells (the
// moving frame): every read of f^n at coordinate c along ax reads c + d,
// clamped to the last plane.
template <int D, int Q, class R>
__global__ void k_scatter_f(KP<R> p, const double* __restrict__ fn, R* __restrict__ fst, int ax, int d) {
  using L = Lat<Q>;
  int64_t Qc;
  int x, y, z;
  if (!dense_cell(p, (int64_t)blockIdx.x * blockDim.x + threadIdx.x, x, y, z, Qc)) return;
  auto at = [&](int c0, int c1, int c2) -> int64_t {  // fn is in dense order
    int c[3] = {c0, c1, c2};
    c[ax] = min(c[ax] + d, p.n[ax] - 1);
    return ((int64_t)c[2] * p.n[1] + c[1]) * p.n[0] + c[0];
  };
  for (int k = 0; k < L::Q; ++k) {
    int dst[3] = {x + L::c(k, 0), y + L::c(k, 1), z + L::c(k, 2)};
    bool in = true;
    for (int a = 0; a < D; ++a)
      if (dst[a] < 0 || dst[a] >= p.n[a]) {
        if (p.per[a])
          dst[a] = (dst[a] + p.n[a]) % p.n[a];
        else
          in = false;
      }
    double val;
    if (in) {
      val = fn[k * p.live + at(dst[0], dst[1], dst[2])] - L::w(k) * (double)p.rho0;
    } else {
      const int kb = L::opp(k);
      val = fn[kb * p.live + at(x, y, z)] - L::w(kb) * (double)p.rho0;
      if (L::c(kb, 1) < 0 && !p.per[1] && y - L::c(kb, 1) >= p.n[1])
        val -= 6.0 * L::w(kb) * (double)p.rho0 * L::c(kb, 0) * (double)p.lid_u;
    }
    fst[k * p.cells + Qc] = (R)val;
  }
}

// Copies between the stored form (precision R) and a dense array of T, and the
// loss seed.  HBM bound, or by the host's call on small grids: they take the few
// sizes they need instead of the parameter block (0.4 us per call).  A block
// takes copy_cells(C) * 256 consecutive cells of the dense array, whose lines it fills
// (64 x 4 tiles leave partial lines at every row's end); rows are sy apart in every
// plane, so a cell's stored element is its dense one and its row's number times
// the padding.  All of a thread's loads are in flight before its first store.
// us per phi read to the device, FP32, 150 x 131 x 117, the host's 8 among them:
// 9.1, with one cell per thread 11.2, with tiles 11.7.
constexpr int copy_cells(int comps) { return comps <= 4 ? 4 : 1; }
struct Rows {
  int n0, pad;  // cells of a row, padding behind it
  int64_t cells, live;
};
__device__ __forceinline__ int64_t stored_at(const Rows& g, int64_t i) {
  if (g.pad == 0) return i;
  // 32-bit divisions are a quarter of the 64-bit ones
  const int64_t row = g.live <= (int64_t)0xffffffff ? (int64_t)((unsigned)i / (unsigned)g.n0) : i / g.n0;
  return i + row * g.pad;
}
// get(P, i, v) and put(P, i, v) of the cells of a thread: P stored, i dense
template <class V, int CELLS, class GET, class PUT>
__device__ __forceinline__ void copy_block(const Rows& g, GET&& get, PUT&& put) {
  V v[CELLS];
  int64_t P[CELLS];
  const int64_t i0 = (int64_t)blockIdx.x * (CELLS * 256) + threadIdx.x;
#pragma unroll
  for (int j = 0; j < CELLS; ++j) {
    const int64_t i = i0 + j * 256;
    P[j] = stored_at(g, i);
    if (i < g.live) get(P[j], i, v[j]);
  }
#pragma unroll
  for (int j = 0; j < CELLS; ++j)
    if (i0 + j * 256 < g.live) put(P[j], i0 + j * 256, v[j]);
}
template <class T, int C> struct CellOf {
  T c[C];
};
// MU: component i is stored less r0 (i = 0) or r1, the reference chemical
// potentials.
template <class R, class T, bool MU, int C>
__global__ void __launch_bounds__(256) k_unpack(Rows g, const R* __restrict__ in, T* __restrict__ out, T r0, T r1) {
  using V = CellOf<R, C>;
  copy_block<V, copy_cells(C)>(
      g,
      [&](int64_t P, int64_t, V& v) {
#pragma unroll
        for (int k = 0; k < C; ++k) v.c[k] = in[k * g.cells + P];
      },
      [&](int64_t, int64_t i, const V& v) {
#pragma unroll
        for (int k = 0; k < C; ++k) out[k * g.live + i] = MU ? (T)v.c[k] + (k == 0 ? r0 : r1) : (T)v.c[k];
      });
}
template <class R, class T, bool MU, int C>
__global__ void __launch_bounds__(256) k_pack(Rows g, const T* __restrict__ in, R* __restrict__ out, T r0, T r1) {
  using V = CellOf<T, C>;
  copy_block<V, copy_cells(C)>(
      g,
      [&](int64_t, int64_t i, V& v) {
#pragma unroll
        for (int k = 0; k < C; ++k) v.c[k] = in[k * g.live + i];
      },
      [&](int64_t P, int64_t, const V& v) {
#pragma unroll
        for (int k = 0; k < C; ++k) out[k * g.cells + P] = (R)(MU ? v.c[k] - (k == 0 ? r0 : r1) : v.c[k]);
      });
}
// derived per-cell fields in FP64: 0 rho (out may be fgathered: a cell's sum goes
// over its own first population), 1 mixture composition C (nc comps), 2
// temperature, 3 active-set bitmask
template <int D, int Q, int N, int NC, class R>
__global__ void k_derived(KP<R> p, int which, const R* __restrict__ phi, const R* __restrict__ mu,
                          const double* fgathered, double tshift_d, double* out) {
  using L = Lat<Q>;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t P;
  int x, y, z;
  if (!dense_cell(p, i, x, y, z, P)) return;
  if (which == 0) {
    double r = 0.0;
    for (int k = 0; k < L::Q; ++k) r += fgathered[k * p.live + i];
    out[i] = r;
  } else if (which == 1) {
    double ph[N], h[N], m[NC];
    for (int b = 0; b < N; ++b) ph[b] = (double)phi[b * p.cells + P];
    for (int q = 0; q < NC; ++q) m[q] = (double)mu[q * p.cells + P];
    interp_h<N, double>(ph, h);
    const int pos[3] = {x, y, z};
    const double td = (p.G != R(0)) ? (double)p.G * ((double)pos[p.pull_axis] - tshift_d) : (double)p.tdev_iso;
    for (int q = 0; q < NC; ++q) {
      double c = 0.0;
      for (int b = 0; b < N; ++b) {
        double C = p.c0s_d[b][q] + (double)p.mT[b][q] * td;
        for (int k = 0; k < NC; ++k) C += (double)p.chi[q][k] * m[k];
        c += h[b] * C;
      }
      out[q * p.live + i] = c;
    }
  } else if (which == 2) {
    const int pos[3] = {x, y, z};
    out[i] = (double)p.T_E + ((p.G != R(0)) ? (double)p.G * ((double)pos[p.pull_axis] - tshift_d)
                                              : (double)p.tdev_iso);
  } else {
    unsigned mask = 0u;
    for (int k = 0; k < L::Q; ++k) {
      const int xx = nb_field(x, L::c(k, 0), p.n[0], p.per[0]);
      const int yy = nb_field(y, L::c(k, 1), p.n[1], p.per[1]);
      const int zz = (D == 3) ? nb_field(z, L::c(k, 2), p.n[2], p.per[2]) : 0;
      const int64_t j = (int64_t)zz * p.sz + (int64_t)yy * p.sy + xx;
      for (int b = 0; b < N; ++b)
        if (phi[b * p.cells + j] > R(0)) mask |= 1u << b;
    }
    out[i] = (double)mask;
  }
}

// FP64 block partial sums in a fixed order: solute (NC values, which 0),
// mass (which 1) or the loss 1/2 sum_a (phi_a - target_a)^2 (which 2).  The mass
// reads all populations: all of a cell's are loaded before the first is added
// (us per call, added as each came and now: 449 and 270 on 256^3, FP32, 95 and 60
// on 96^3, 27 velocities, FP64; some 25 of them are the host's).
constexpr int RED_BLOCK = 256;
template <int D, int Q, int N, int NC, class R>
__global__ void __launch_bounds__(RED_BLOCK)
k_partial(KP<R> p, int which, const R* __restrict__ phi, const R* __restrict__ mu,
          const R* __restrict__ f, const double* __restrict__ target, double tshift_d,
          double* __restrict__ partial) {
  using L = Lat<Q>;
  __shared__ double sh[NC][RED_BLOCK];
  const int t = threadIdx.x;
  double acc[NC];
  for (int i = 0; i < NC; ++i) acc[i] = 0.0;
  for (int64_t j = (int64_t)blockIdx.x * RED_BLOCK + t; j < p.live; j += (int64_t)gridDim.x * RED_BLOCK) {
    int64_t P;
    int x, y, z;
    dense_cell(p, j, x, y, z, P);
    if (which == 0) {
      double ph[N], h[N], m[NC];
      for (int b = 0; b < N; ++b) ph[b] = (double)phi[b * p.cells + P];
      for (int i = 0; i < NC; ++i) m[i] = (double)mu[i * p.cells + P];
      interp_h<N, double>(ph, h);
      const int pos[3] = {x, y, z};
      const double td = (p.G != R(0)) ? (double)p.G * ((double)pos[p.pull_axis] - tshift_d) : (double)p.tdev_iso;
      for (int i = 0; i < NC; ++i) {
        double c = 0.0;
        for (int b = 0; b < N; ++b) {
          double C = p.c0s_d[b][i] + (double)p.mT[b][i] * td;
          for (int k = 0; k < NC; ++k) C += (double)p.chi[i][k] * m[k];
          c += h[b] * C;
        }
        acc[i] += c;
      }
    } else if (which == 1) {
      R g[Q];
      // (a wave's cells lie in rows of their own here: bases per lane, see pull_cell)
      pull_cell<D, Q, true, STREAM, R>(p, f, pull_at<D, true, R>(p, x, y, z), g);
      double r = 0.0;
#pragma unroll
      for (int k = 0; k < L::Q; ++k) r += (double)g[k] + L::w(k) * (double)p.rho0;
      acc[0] += r;
    } else {
      double r = 0.0;
      for (int b = 0; b < N; ++b) {
        const double d = (double)phi[b * p.cells + P] - target[b * p.live + j];
        r += d * d;
      }
      acc[0] += 0.5 * r;
    }
  }
  for (int i = 0; i < NC; ++i) sh[i][t] = acc[i];
  __syncthreads();
  for (int s = RED_BLOCK / 2; s > 0; s >>= 1) {
    if (t < s)
      for (int i = 0; i < NC; ++i) sh[i][t] += sh[i][t + s];
    __syncthreads();
  }
  // one value per block and component of this total, in the stride
  // k_final_sum reads: NC for the solute, 1 for the mass and the loss
  const int ncomp = (which == 0) ? NC : 1;
  if (t == 0)
    for (int i = 0; i < ncomp; ++i) partial[blockIdx.x * ncomp + i] = sh[i][0];
}

__global__ void k_final_sum(const double* __restrict__ partial, int nblocks, int ncomp,
                            double* __restrict__ out) {
  __shared__ double sh[RED_BLOCK];
  for (int i = 0; i < ncomp; ++i) {
    double acc = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += RED_BLOCK) acc += partial[b * ncomp + i];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = RED_BLOCK / 2; s > 0; s >>= 1) {
      if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
      __syncthreads();
    }
    if (threadIdx.x == 0) out[i] = sh[0];
    __syncthreads();
  }
}

// dL/dphi of the loss 1/2 sum (phi - target)^2: phi - target in FP64, dense
template <class R, int C>
__global__ void __launch_bounds__(256) k_loss_seed(Rows g, const R* __restrict__ phi, const double* __restrict__ target,
                                                   double* __restrict__ out) {
  using V = CellOf<double, C>;
  copy_block<V, copy_cells(C)>(
      g,
      [&](int64_t P, int64_t i, V& v) {
#pragma unroll
        for (int k = 0; k < C; ++k) v.c[k] = (double)phi[k * g.cells + P] - target[k * g.live + i];
      },
      [&](int64_t, int64_t i, const V& v) {
#pragma unroll
        for (int k = 0; k < C; ++k) out[k * g.live + i] = v.c[k];
      });
}

// ---------------------------------------------------------------------------
// Bandwidth probes (measurement only): the memory access patterns of the
// population update without its arithmetic, on 19 FP32 arrays of an
// n0 x n1 x n2 grid (all axes periodic).  k_probe_copy19: out_k(P) = in_k(P);
// k_probe_pull19: out_k(P) = in_k(P - c_k) with the D3Q19 velocities, one
// thread per cell in 256-cell blocks; k_probe_pull19_z: the same pull by
// 64 x TY tiles that walk ZC planes (XCD-aware tile order).  Streaming (nontemporal) loads and stores as in the step kernels.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_probe_copy19(const float* __restrict__ in, float* __restrict__ out,
                                                      int64_t cells) {
  const int64_t P = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (P >= cells) return;
#pragma unroll
  for (int k = 0; k < 19; ++k)
    __builtin_nontemporal_store(__builtin_nontemporal_load(&in[k * cells + P]), &out[k * cells + P]);
}

__device__ __forceinline__ void probe_pull_cell(const float* __restrict__ in, float* __restrict__ out, int x, int y,
                                                int z, int n0, int n1, int n2, int64_t cells) {
  using L = Lat<19>;
  const int64_t P = ((int64_t)z * n1 + y) * n0 + x;
  float v[19];
#pragma unroll
  for (int k = 0; k < 19; ++k) {
    const int xs = (x - L::c(k, 0) + n0) % n0, ys = (y - L::c(k, 1) + n1) % n1, zs = (z - L::c(k, 2) + n2) % n2;
    v[k] = __builtin_nontemporal_load(&in[k * cells + ((int64_t)zs * n1 + ys) * n0 + xs]);
  }
#pragma unroll
  for (int k = 0; k < 19; ++k) __builtin_nontemporal_store(v[k], &out[k * cells + P]);
}

__global__ void __launch_bounds__(256) k_probe_pull19(const float* __restrict__ in, float* __restrict__ out, int n0,
                                                      int n1, int n2) {
  const int64_t cells = (int64_t)n0 * n1 * n2;
  const int64_t P = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (P >= cells) return;
  probe_pull_cell(in, out, (int)(P % n0), (int)((P / n0) % n1), (int)(P / ((int64_t)n0 * n1)), n0, n1, n2, cells);
}

template <int TY>
__global__ void __launch_bounds__(64 * TY) k_probe_pull19_z(const float* __restrict__ in, float* __restrict__ out,
                                                            int n0, int n1, int n2, int zc) {
  const int64_t cells = (int64_t)n0 * n1 * n2;
  const Tile T = tile_at<64, TY, 1>(xcd_block(), n0 / 64, n1 / TY);
  const int x = T.x0 + (int)threadIdx.x % 64, y = T.y0 + (int)threadIdx.x / 64;
  for (int z = T.z0 * zc; z < min((T.z0 + 1) * zc, n2); ++z) probe_pull_cell(in, out, x, y, z, n0, n1, n2, cells);
}

// health: NaN/Inf in phi or mu, or rho <= 0, records the smallest step seen
template <int D, int Q, int N, int NC, class R>
__global__ void k_health(KP<R> p, const R* __restrict__ phi, const R* __restrict__ mu,
                         const R* __restrict__ f, unsigned long long step,
                         unsigned long long* __restrict__ bad_step) {
  using L = Lat<Q>;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t P;
  int x, y, z;
  if (!dense_cell(p, i, x, y, z, P)) return;
  bool bad = false;
  for (int b = 0; b < N; ++b) bad |= !isfinite(phi[b * p.cells + P]);
  for (int i = 0; i < NC; ++i) bad |= !isfinite(mu[i * p.cells + P]);
  R r = p.rho0;
  for (int k = 0; k < L::Q; ++k) r += pull_f<D, Q, R>(p, f, x, y, z, P, k);
  bad |= !(r > R(0));
  if (bad) atomicMin(bad_step, step);
}

}  // namespace gpf
