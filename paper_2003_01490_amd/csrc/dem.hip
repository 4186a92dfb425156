// Discrete element part of one time step (Alg. 1, DEM sub-cycles), FP64.
//
// Prologue: per-sphere sum of the momentum-exchange partials written by the
// boundary kernel (fixed order), averaging with the previous step (Sec. 4.2;
// the first step averages with itself), copy of the positions the mapping
// starts from, and a neighbour list per sphere (candidates whose gap is below
// the largest lubrication cut-off plus a skin, ascending ids).  Then n_sub
// sub-cycles with dt_p = 1/n_sub and F_fp held constant:
//   release of prescribed spheres below their gap; velocity-Verlet start force
//   for newly free spheres; Eq. (velocity_verlet_1); lubrication (Sec. 3.1,
//   step function on the raw gap, magnitude on max(gap, delta_min)), contacts
//   (Eqs. normalCollisionForce, tangentialCollisionForce with the spring
//   projected, rescaled and reset as in Sec. 4.1.2), external force
//   V (rho_p - rho_f) g; Eq. (velocity_verlet_2) and its rotational analogue.
// Forces are gathered per sphere (each sphere sums over its own partners), so
// nothing is scattered and the pair terms come out antisymmetric exactly.
//
// Few spheres: one workgroup, eight lanes per sphere, state in LDS, sub-cycles
// separated by workgroup barriers (beyond DEM_LDS_MAX spheres, where it is asked
// for explicitly, one thread per sphere on global memory).  Many spheres: eight
// lanes per sphere over a chain of launches; neighbours are found by all pairs
// (up to DEM_PAIRS_MAX spheres) or through uniform bins, and x, u, w alternate between two buffers every sub-cycle
// (positions are advanced into the other buffer, then forces read the new
// positions and the old velocities and write the new velocities into the other
// buffer), so each sub-cycle needs only two launches.  All give the same bits.
#include "internal.hpp"

#include <algorithm>
#include <climits>

namespace lbmdem {

constexpr double PI_D = 3.14159265358979323846;

// one of three values (all read first: choosing between fields of the
// by-value descriptor would place it in scratch memory)
template <typename T>
__device__ __forceinline__ T sel3(int k, T a, T b, T c) {
  return k == 0 ? a : (k == 1 ? b : c);
}

struct Partner {
  int code;        // sphere id >= 0, wall -1 - (2 axis + side)
  int j;           // sphere id or -1
  double n[3];     // unit normal from partner to i
  double delta;    // signed gap
  double xcp[3];   // contact point
  double rj[3];    // xcp - x_j
};

__device__ inline void cross3(const double* a, const double* b, double* o) {
  o[0] = a[1] * b[2] - a[2] * b[1];
  o[1] = a[2] * b[0] - a[0] * b[2];
  o[2] = a[0] * b[1] - a[1] * b[0];
}
__device__ inline double dot3(const double* a, const double* b) {
  return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}
__device__ inline double norm3(const double* a) { return sqrt(dot3(a, a)); }

// rigid-body surface velocity u + w x r (r = point - centre)
__device__ inline void body_vel(const double* u, const double* w, const double* r, double* U) {
  double wr[3];
  cross3(w, r, wr);
  U[0] = u[0] + wr[0];
  U[1] = u[1] + wr[1];
  U[2] = u[2] + wr[2];
}

// sphere partner at xj: gap first (most listed partners are out of reach), the
// rest of the geometry on demand
__device__ __forceinline__ double sphere_offset(const DevDomain& d, const double* xi, double Ri, const double* xj,
                                                double Rj, double* dd, double* dist) {
  const int n[3] = {d.nx, d.ny, d.nz};
  for (int a = 0; a < 3; ++a) dd[a] = min_image(xi[a] - xj[a], n[a], d.walls[a]);
  *dist = norm3(dd);
  return *dist - (Ri + Rj);
}

__device__ __forceinline__ void make_sphere_partner(const double* xi, int j, const double* dd, double dist,
                                                    double delta, Partner& pt) {
  pt.code = j;
  pt.j = j;
  pt.delta = delta;
  for (int a = 0; a < 3; ++a) {
    pt.n[a] = dd[a] / dist;
    pt.xcp[a] = xi[a] - 0.5 * dd[a];
    pt.rj[a] = 0.5 * dd[a];
  }
}

// gap to the wall plane of an axis and side
__device__ __forceinline__ double wall_gap(const DevDomain& d, const double* xi, double R, int a, int side) {
  const double xa = sel3(a, xi[0], xi[1], xi[2]);
  const int na = sel3(a, d.nx, d.ny, d.nz);
  return side ? (((double)na - 1.0) - xa) - R : (xa - 1.0) - R;
}

__device__ __forceinline__ void make_wall_partner(const double* xi, double R, int a, int side, double delta,
                                                  Partner& pt) {
  // selects instead of indexing local arrays with the runtime axis, so that
  // nothing spills to scratch memory
  const double s = side ? -1.0 : 1.0;
  pt.code = -1 - (2 * a + side);
  pt.j = -1;
  pt.n[0] = a == 0 ? s : 0.0;
  pt.n[1] = a == 1 ? s : 0.0;
  pt.n[2] = a == 2 ? s : 0.0;
  pt.delta = delta;
  const double h = R + 0.5 * delta;
  for (int k = 0; k < 3; ++k) pt.xcp[k] = xi[k] - h * pt.n[k];
  pt.rj[0] = pt.rj[1] = pt.rj[2] = 0.0;
}

// axis and side of the wk-th wall plane (walled axes in order, lower side first)
__device__ __forceinline__ void wall_of(const DevDomain& d, int wk, int* a, int* side) {
  const int w0 = d.walls[0] ? 2 : 0, w1 = d.walls[1] ? 2 : 0;
  *a = wk < w0 ? 0 : (wk < w0 + w1 ? 1 : 2);
  *side = wk - (*a == 0 ? 0 : (*a == 1 ? w0 : w0 + w1));
}

__device__ inline double collision_time(const DevDomain& d, double D) {
  return d.tc > 0.0 ? d.tc : 2.31 * D * sqrt(3.0);  // Eq. (collisionTimeChoice)
}
__device__ inline double min_lub_gap(const DevDomain& d, double R) {
  return d.dmin >= 0.0 ? d.dmin : (0.001 + 0.00007 * R) * R;  // Eq. (lubricationGapSize)
}

__device__ __forceinline__ void lubrication(const DevDomain& d, double dmin, const double* n, double delta,
                            const double* ui, const double* wi, double Ri, const double* uj,
                            const double* wj, double Rj, bool wall, double* F, double* T) {
  const double mu = d.nu;
  const double dl = delta > dmin ? delta : dmin;
  double uij[3], un[3], ut[3];
  for (int a = 0; a < 3; ++a) uij[a] = ui[a] - (wall ? 0.0 : uj[a]);
  const double uijn = dot3(uij, n);
  for (int a = 0; a < 3; ++a) {
    un[a] = uijn * n[a];
    ut[a] = uij[a] - un[a];
  }
  const double k = wall ? 0.0 : Rj / Ri;
  double L = 0.0;
  if ((d.lub_mask & 1) && delta > 0.0 && delta < d.cut_n) {
    const double coef = wall ? 1.0 : (k * k) / ((1.0 + k) * (1.0 + k));
    const double mag = -6.0 * PI_D * mu * Ri * Ri * coef * (1.0 / dl - d.inv_cut_n);
    for (int a = 0; a < 3; ++a) F[a] += mag * un[a];
  }
  if ((d.lub_mask & 2) && delta > 0.0 && delta < d.cut_tt) {
    L = log(dl / d.cut_tt);
    const double cf = wall ? 8.0 / 15.0
                           : 4.0 * k * (2.0 + k + 2.0 * k * k) / (15.0 * (1.0 + k) * (1.0 + k) * (1.0 + k));
    const double ct = wall ? 0.1 : k * (4.0 + k) / (10.0 * (1.0 + k) * (1.0 + k));
    const double fm = 6.0 * PI_D * mu * Ri * cf * L;
    const double tm = 8.0 * PI_D * mu * Ri * Ri * ct * L;
    double uxn[3];
    cross3(uij, n, uxn);
    for (int a = 0; a < 3; ++a) {
      F[a] += fm * ut[a];
      T[a] += tm * uxn[a];
    }
  }
  if ((d.lub_mask & 4) && delta > 0.0 && delta < d.cut_tr) {
    if (!((d.lub_mask & 2) && d.cut_tr == d.cut_tt)) L = log(dl / d.cut_tr);  // else as above
    const double cf = wall ? 2.0 / 15.0 : 2.0 * k * k / (15.0 * (1.0 + k) * (1.0 + k));
    const double ct = wall ? 0.4 : 2.0 * k / (5.0 * (1.0 + k));
    double wv[3], av[3], wxn[3];
    for (int a = 0; a < 3; ++a) {
      wv[a] = wall ? wi[a] : (wi[a] + wj[a]) + (4.0 / k) * wi[a] + 4.0 * k * wj[a];
      av[a] = wall ? wi[a] : wi[a] + 0.25 * k * wj[a];
    }
    cross3(wv, n, wxn);
    const double an = dot3(av, n);
    const double fm = -6.0 * PI_D * mu * Ri * Ri * cf * L;
    const double tm = 8.0 * PI_D * mu * Ri * Ri * Ri * ct * L;
    for (int a = 0; a < 3; ++a) {
      F[a] += fm * wxn[a];
      T[a] += tm * (av[a] - an * n[a]);
    }
  }
}

__device__ __forceinline__ double longest_cut(const DevDomain& d) {
  return fmax(d.cut_n, fmax(d.cut_tt, d.cut_tr));
}

// What one partner does to sphere i: c[0..2] lubrication force, c[3..5] its
// torque, c[6..8] contact force, c[9..11] its torque.  hv: the pair's
// tangential spring (zero for a new contact); returns whether the two touch
// (and contacts are evaluated), with the new spring in hv.
__device__ __forceinline__ bool pair_terms(const DevDomain& d, bool contact, const Partner& pt, const double* xi,
                                           const double* ui, const double* wi, double Ri, double mi,
                                           const double* uj, const double* wj, double Rj, double mj, double dtp,
                                           double* hv, double* c) {
  const bool is_wall = pt.j < 0;
  const bool touch = contact && pt.delta < 0.0;
  if (touch) {
    double uij[3], un[3], Ui[3], Uj[3], ut[3], ri[3];
    for (int a = 0; a < 3; ++a) {
      uij[a] = ui[a] - uj[a];
      ri[a] = pt.xcp[a] - xi[a];
    }
    const double uijn = dot3(uij, pt.n);
    for (int a = 0; a < 3; ++a) un[a] = uijn * pt.n[a];
    body_vel(ui, wi, ri, Ui);
    if (is_wall) {
      Uj[0] = Uj[1] = Uj[2] = 0.0;
    } else {
      body_vel(uj, wj, pt.rj, Uj);
    }
    for (int a = 0; a < 3; ++a) ut[a] = (Ui[a] - Uj[a]) - un[a];
    const double meff = is_wall ? mi : mi * mj / (mi + mj);
    const double D = is_wall ? 2.0 * Ri : Ri + Rj;
    const double Tc = collision_time(d, D);
    const double le = d.log_e;
    const double kn = meff * (PI_D * PI_D + le * le) / (Tc * Tc);  // Eq. (normalDEMparameters)
    const double dn = -2.0 * meff * le / Tc;
    const double kt = d.kappa * kn;  // Eq. (tangentialCollisionParameters)
    const double dt = d.sqrt_kappa * dn;
    double Fn[3];
    for (int a = 0; a < 3; ++a) Fn[a] = -kn * pt.delta * pt.n[a] - dn * un[a];
    const double hn = dot3(hv, pt.n);
    double ht[3];
    for (int a = 0; a < 3; ++a) ht[a] = hv[a] - hn * pt.n[a];
    const double lh = norm3(hv), lht = norm3(ht);
    if (lht > 0.0)
      for (int a = 0; a < 3; ++a) hv[a] = (lh / lht) * ht[a];
    else
      for (int a = 0; a < 3; ++a) hv[a] = ht[a];
    double Fsd[3];
    for (int a = 0; a < 3; ++a) Fsd[a] = -kt * hv[a] - dt * ut[a];
    const double fsd = norm3(Fsd);
    const double fmax = d.friction * norm3(Fn);
    double Ft[3];
    if (fsd < fmax || fsd == 0.0) {
      for (int a = 0; a < 3; ++a) {
        Ft[a] = Fsd[a];
        hv[a] = hv[a] + dtp * ut[a];
      }
    } else {
      for (int a = 0; a < 3; ++a) {
        const double tv = Fsd[a] / fsd;
        Ft[a] = fmax * tv;
        hv[a] = -(fmax * tv + dt * ut[a]) / kt;
      }
    }
    double Tt[3];
    cross3(ri, Ft, Tt);
    for (int a = 0; a < 3; ++a) {
      c[6 + a] += Fn[a] + Ft[a];
      c[9 + a] += Tt[a];
    }
  }
  if (pt.delta > 0.0 && pt.delta < longest_cut(d)) {
    const double Rh = is_wall ? Ri : 2.0 * Ri * Rj / (Ri + Rj);
    lubrication(d, min_lub_gap(d, Rh), pt.n, pt.delta, ui, wi, Ri, uj, wj, Rj, is_wall, c, c + 3);
  }
  return touch;
}

// total force (k < 3) or torque component from the partner sums
__device__ __forceinline__ double total_term(double ffp, double lub, double col, double fext, bool force) {
  return force ? ((ffp + lub) + col) + fext : (ffp + lub) + col;
}

// V (rho_p - rho_f), the mass the external force acts on
__device__ __forceinline__ double buoyant_mass(double R, double rho) {
  const double V = (4.0 / 3.0) * PI_D * R * R * R;
  return V * (rho - 1.0);
}

// forces on sphere i at the current state, one thread: the terms of its
// partners, each formed from zero, added in list order (neighbours, then
// walls).  contact: evaluate contacts; upd: write the tangential-spring
// history
__device__ __forceinline__ void eval_forces(const DevDomain& d, const DevParticles& p, int i, bool contact,
                                            bool upd, double dtp, double* Fout, double* Tout) {
  double sum[12] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  const double maxcut = longest_cut(d);
  const double xi[3] = {p.x[3 * i], p.x[3 * i + 1], p.x[3 * i + 2]};
  const double ui[3] = {p.u[3 * i], p.u[3 * i + 1], p.u[3 * i + 2]};
  const double wi[3] = {p.w[3 * i], p.w[3 * i + 1], p.w[3 * i + 2]};
  const double Ri = p.R[i];
  int* hid = p.hist_id + (size_t)i * HIST_SLOTS;
  double* hd = p.hist_d + (size_t)i * HIST_SLOTS * 3;
  const int nn = p.nbr_n[i];
  const int nwalls = 2 * (d.walls[0] + d.walls[1] + d.walls[2]);
  bool any = false;
  for (int s = 0; s < HIST_SLOTS; ++s) any = any || hid[s] != INT_MIN;
  for (int pi = 0; pi < nn + nwalls; ++pi) {
    const bool wall = pi >= nn;
    int j = -1, a = 0, side = 0;
    double dd[3] = {0, 0, 0}, dist = 0.0, delta;
    if (!wall) {
      j = p.nbr[(size_t)i * NBR_MAX + pi];
      delta = sphere_offset(d, xi, Ri, p.x + 3 * j, p.R[j], dd, &dist);
    } else {
      wall_of(d, pi - nn, &a, &side);
      delta = wall_gap(d, xi, Ri, a, side);
    }
    const int code = wall ? -1 - (2 * a + side) : j;
    int slot = -1;
    if (any)
      for (int s = 0; s < HIST_SLOTS; ++s)
        if (hid[s] == code) slot = s;
    if (!(delta < maxcut) && slot < 0) continue;
    Partner pt;
    if (wall)
      make_wall_partner(xi, Ri, a, side, delta, pt);
    else
      make_sphere_partner(xi, j, dd, dist, delta, pt);
    const double zero[3] = {0, 0, 0};
    const double* uj = wall ? zero : p.u + 3 * j;
    const double* wj = wall ? zero : p.w + 3 * j;
    double hv[3] = {0, 0, 0}, c[12] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    if (slot >= 0)
      for (int k = 0; k < 3; ++k) hv[k] = hd[slot * 3 + k];
    const bool touch = pair_terms(d, contact, pt, xi, ui, wi, Ri, p.m[i], uj, wj, wall ? 0.0 : p.R[j],
                                  wall ? 0.0 : p.m[j], dtp, hv, c);
    if (upd && touch) {
      if (slot < 0)
        for (int s = 0; s < HIST_SLOTS && slot < 0; ++s)
          if (hid[s] == INT_MIN) slot = s;
      if (slot < 0) {
        atomicOr(d.status, ST_HIST_FULL);
      } else {
        hid[slot] = code;
        any = true;
        for (int k = 0; k < 3; ++k) hd[slot * 3 + k] = hv[k];
      }
    } else if (upd && slot >= 0) {
      hid[slot] = INT_MIN;
    }
    for (int k = 0; k < 12; ++k) sum[k] += c[k];
  }
  const double bm = buoyant_mass(Ri, p.rho[i]);
  const double* Ffp = p.Ffp + 6 * i;
  double* dg = p.diag + 18 * i;
  for (int a = 0; a < 3; ++a) {
    Fout[a] = total_term(Ffp[a], sum[a], sum[6 + a], bm * d.gravity[a], true);
    Tout[a] = total_term(Ffp[3 + a], sum[3 + a], sum[9 + a], 0.0, false);
  }
  for (int k = 0; k < 12; ++k) dg[6 + k] = sum[k];
}

// ---- eight lanes per sphere --------------------------------------------------
// The sub-cycles are chains of dependent FP64 work and memory round trips, so
// the partners of a sphere are taken by the eight lanes of a group at once:
// lane g forms the terms of partners g, g + 8, ..., and the terms of those in
// reach are then added in list order (shuffles over the set bits of the
// group's ballot), the same order and bits as eval_forces.  The group's lanes
// 0-2 and 3-5 hold the components of force, velocity and torque, spin.
constexpr int GROUP = 8;

// state arrays of the spheres, in LDS or in global memory
struct GroupState {
  const double *x, *u, *w;  // [P][3]
  const double *R, *m;      // [P]
};

// Sums of the terms of all partners of sphere i: component g (< 6) of the
// lubrication and of the contact force and torque into *lub and *col of lane
// g; nbr(k): the k-th listed neighbour.  Every lane of the wavefront
// calls it (`on`: the group has a sphere).  hid: the sphere's 24 history codes;
// hd: its springs.  A round's ended contacts free their slots and its new ones
// take the first free slot one after the other in list order, as eval_forces
// does: which slot, and whether there is one, is the same in every kernel.
template <typename NBR>
__device__ __forceinline__ void group_forces(const DevDomain& d, const GroupState& s, int i, bool on, int nn,
                                             NBR nbr, int* hid, double* hd, bool contact, bool upd, double dtp,
                                             double* lub, double* col) {
  const int lane = threadIdx.x & 63, g = lane & (GROUP - 1), base = lane & ~(GROUP - 1);
  const double maxcut = longest_cut(d);
  double xi[3] = {0, 0, 0}, Ri = 0.0;
  unsigned mine = 0;  // bit k: slot g + 8 k is taken
  if (on) {
    for (int a = 0; a < 3; ++a) xi[a] = s.x[3 * i + a];
    Ri = s.R[i];
#pragma unroll
    for (int k = 0; k < HIST_SLOTS / GROUP; ++k) mine |= (unsigned)(hid[g + GROUP * k] != INT_MIN) << k;
  }
  const bool any = ((__ballot(mine != 0) >> base) & 0xFFull) != 0;  // the sphere has a spring
  const int nwalls = 2 * (d.walls[0] + d.walls[1] + d.walls[2]);
  const int tot = on ? nn + nwalls : 0;
  double sl = 0.0, sc = 0.0;
  for (int p0 = 0; __any(p0 < tot); p0 += GROUP) {
    const int pi = p0 + g;
    double c[12] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}, hv[3] = {0, 0, 0};
    bool reach = false, starts = false, ends = false;
    int code = 0, slot = -1;
    if (pi < tot) {
      const bool wall = pi >= nn;
      int j = -1, a = 0, side = 0;
      double dd[3] = {0, 0, 0}, dist = 0.0, delta, Rj = 0.0;
      if (!wall) {
        j = nbr(pi);
        Rj = s.R[j];
        delta = sphere_offset(d, xi, Ri, s.x + 3 * j, Rj, dd, &dist);
      } else {
        wall_of(d, pi - nn, &a, &side);
        delta = wall_gap(d, xi, Ri, a, side);
      }
      code = wall ? -1 - (2 * a + side) : j;
      if (any)
        for (int q = 0; q < HIST_SLOTS; ++q)
          if (hid[q] == code) slot = q;
      reach = delta < maxcut || slot >= 0;
      if (reach) {
        Partner pt;
        if (wall)
          make_wall_partner(xi, Ri, a, side, delta, pt);
        else
          make_sphere_partner(xi, j, dd, dist, delta, pt);
        double ui[3], wi[3], uj[3] = {0, 0, 0}, wj[3] = {0, 0, 0}, mj = 0.0;
        for (int q = 0; q < 3; ++q) {
          ui[q] = s.u[3 * i + q];
          wi[q] = s.w[3 * i + q];
        }
        if (!wall) {
          for (int q = 0; q < 3; ++q) {
            uj[q] = s.u[3 * j + q];
            wj[q] = s.w[3 * j + q];
          }
          mj = s.m[j];
        }
        if (slot >= 0)
          for (int q = 0; q < 3; ++q) hv[q] = hd[slot * 3 + q];
        const bool touch = pair_terms(d, contact, pt, xi, ui, wi, Ri, s.m[i], uj, wj, Rj, mj, dtp, hv, c);
        starts = upd && touch && slot < 0;
        ends = upd && !touch && slot >= 0;
        if (upd && touch && slot >= 0)
          for (int q = 0; q < 3; ++q) hd[slot * 3 + q] = hv[q];
      }
    }
    unsigned in = (unsigned)((__ballot(reach) >> base) & 0xFFull);
    if (!__any(in != 0)) continue;
    if (__builtin_expect(__any(starts || ends), 0)) {
      const unsigned es = (unsigned)((__ballot(starts) >> base) & 0xFFull),
                     ee = (unsigned)((__ballot(ends) >> base) & 0xFFull);
      unsigned free_slots = 0;  // the same in the group's lanes
#pragma unroll 1
      for (int k = 0; k < HIST_SLOTS / GROUP; ++k)
        free_slots |= (unsigned)((__ballot(!((mine >> k) & 1u)) >> base) & 0xFFull) << (GROUP * k);
#pragma unroll 1
      for (int e = 0; e < GROUP; ++e) {
        const int se = __shfl(slot, base + e, 64);
        if ((ee >> e) & 1u) {
          free_slots |= 1u << se;
        } else if ((es >> e) & 1u) {
          const int f = __ffs(free_slots) - 1;  // -1: none left
          if (g == e) slot = f;
          free_slots &= free_slots - 1u;
        }
      }
      mine = 0;
#pragma unroll 1
      for (int k = 0; k < HIST_SLOTS / GROUP; ++k) mine |= (~free_slots >> (g + GROUP * k) & 1u) << k;
      if (ends && ((free_slots >> slot) & 1u)) hid[slot] = INT_MIN;  // (not taken again)
      if (starts && slot < 0) {
        atomicOr(d.status, ST_HIST_FULL);
      } else if (starts) {
        hid[slot] = code;
        for (int q = 0; q < 3; ++q) hd[slot * 3 + q] = hv[q];
      }
    }
    while (__any(in != 0)) {
      const int src = in ? base + __ffs(in) - 1 : lane;
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        const double vl = __shfl(c[k], src, 64), vc = __shfl(c[6 + k], src, 64);
        if (in && g == k) {
          sl += vl;
          sc += vc;
        }
      }
      in &= in - 1u;
    }
  }
  *lub = sl;
  *col = sc;
}

// component g (< 6) of the total force or torque
__device__ __forceinline__ double group_total(const DevDomain& d, int g, double lub, double col, double ffp,
                                              double bm) {
  const double grav = sel3(g, d.gravity[0], d.gravity[1], d.gravity[2]);
  return total_term(ffp, lub, col, bm * grav, g < 3);
}

// Momentum-exchange sum of sphere i by one wavefront: lane l adds the
// partials l, l + 64, ... in order, then a fixed shuffle tree combines the
// lanes, so the result does not depend on scheduling.  Lane c < 6 then averages
// its component with the previous step (into Ffp, and copy if given), and lanes
// 0-2 pin the position the mapping starts from.  (Everything the wave needs is
// loaded before the tree: one memory round trip; the tree's steps stay a loop:
// beside the sweep every new line of code is a fetch of its own.)
__device__ __forceinline__ void resolved_force(const DevDomain& d, const DevParticles& p, int i, int lane,
                                               double* copy = nullptr) {
  const int nb = d.ZB * d.RB;
  const int c = lane < 6 ? lane : 0;
  double prev = p.Fprev[6 * i + c];
  const double x = p.x[3 * i + (lane < 3 ? lane : 0)];
  const bool valid = p.prev_valid[i] != 0;
  double F[6] = {0, 0, 0, 0, 0, 0};
  for (int b = lane; b < nb; b += 64)
    for (int k = 0; k < 6; ++k) F[k] += d.partial[((size_t)i * nb + b) * 6 + k];
#pragma unroll 1
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int k = 0; k < 6; ++k) F[k] += __shfl_down(F[k], off, 64);
  double f = 0.0;
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const double v = __shfl(F[k], 0, 64);
    if (lane == k) f = v;
  }
  if (lane >= 6) return;
  const int k = 6 * i + lane;
  p.Fraw[k] = f;
  double m = f;
  if (d.force_averaging) {
    if (!valid) prev = f;
    m = 0.5 * (f + prev);
    p.Fprev[k] = f;
    if (lane == 0) p.prev_valid[i] = 1;
  }
  p.Ffp[k] = m;
  if (copy) copy[k] = m;
  if (lane < 3) p.xmap[3 * i + lane] = x;
}

// gap between spheres i and j (minimum image); the neighbour test of all
// kernels, so that they list the same partners
__device__ __forceinline__ double pair_gap(const DevDomain& d, const DevParticles& p, int i, int j) {
  double dd[3], dist;
  return sphere_offset(d, p.x + 3 * i, p.R[i], p.x + 3 * j, p.R[j], dd, &dist);
}

__device__ __forceinline__ double list_range(const DevDomain& d) {
  return longest_cut(d) + d.skin;
}

// Gap of a prescribed sphere to the wall plane it approaches: the plane ahead
// along its target velocity on every walled axis where that is nonzero
// (Sec. 4.4.2 switches the acceleration off near the wall the sphere moves
// to); large if there is none.
__device__ __forceinline__ double axis_gap_ahead(double x, double R, double ut, int wall, double n) {
  if (!wall || ut == 0.0) return 1e300;
  return ut < 0.0 ? (x - 1.0) - R : ((n - 1.0) - x) - R;
}
__device__ inline double gap_ahead(const DevDomain& d, const double* x, double R, const double* presc) {
  double g = 1e300;
  const int n[3] = {d.nx, d.ny, d.nz};
#pragma unroll
  for (int a = 0; a < 3; ++a) g = fmin(g, axis_gap_ahead(x[a], R, presc[a], d.walls[a], (double)n[a]));
  return g;
}

// release of a prescribed sphere below its gap; start force of a newly free one
__device__ __forceinline__ void release_and_start(const DevDomain& d, const DevParticles& p, int i, double dtp) {
  if (p.mode[i] == MODE_PRESCRIBED && gap_ahead(d, p.x + 3 * i, p.R[i], p.presc + 6 * i) < p.presc[6 * i + 5]) {
    p.mode[i] = MODE_FREE;
    p.old_valid[i] = 0;
  }
  if (p.mode[i] == MODE_FREE && !p.old_valid[i]) {
    eval_forces(d, p, i, false, false, dtp, p.Fold + 6 * i, p.Fold + 6 * i + 3);
    p.old_valid[i] = 1;
  }
}

// Factors of Eqs. (velocity_verlet_1) and (velocity_verlet_2) of a mass (or
// moment of inertia) m
__device__ __forceinline__ double position_factor(double m, double dtp) { return dtp * dtp / (2.0 * m); }
__device__ __forceinline__ double velocity_factor(double m, double dtp) { return dtp / (2.0 * m); }

// One component of Eq. (velocity_verlet_1) (free), x + dt_p u (prescribed),
// unchanged (fixed); periodic axes wrap
__device__ __forceinline__ double next_position(int mode, double x, double u, double fold, double c2, double dtp,
                                                double L, int wall) {
  double xo = x;
  if (mode == MODE_FREE)
    xo = (x + dtp * u) + c2 * fold;
  else if (mode == MODE_PRESCRIBED)
    xo = x + dtp * u;
  if (!wall) {
    if (xo < 0.0)
      xo += L;
    else if (xo >= L)
      xo -= L;
  }
  return xo;
}

// one component of Eq. (velocity_verlet_2) or its rotational analogue
__device__ __forceinline__ double next_velocity(double v, double fold, double fnew, double cu) {
  return v + cu * (fold + fnew);
}

// the ramp of Eq. (artificial_acceleration)
__device__ __forceinline__ double prescribed_velocity(double u_target, double c_acc, double t_st, double t) {
  const double ramp = 1.0 - exp(-c_acc * t / t_st);
  return u_target * ramp;
}

// the position of sphere i after a sub-cycle; xo may alias p.x + 3 i
__device__ __forceinline__ void advance_position(const DevDomain& d, const DevParticles& p, int i, double dtp,
                                                 double* xo) {
  const int n[3] = {d.nx, d.ny, d.nz};
  for (int a = 0; a < 3; ++a)
    xo[a] = next_position(p.mode[i], p.x[3 * i + a], p.u[3 * i + a], p.Fold[6 * i + a],
                          position_factor(p.m[i], dtp), dtp, (double)n[a],
                          d.walls[a]);
}

// velocities of sphere i from F_old and the new force in p.Fnew; uo, wo may
// alias p.u + 3 i, p.w + 3 i.
__device__ __forceinline__ void advance_velocity(const DevDomain& d, const DevParticles& p, int i, double dtp,
                                                 double* uo, double* wo) {
  const double* Fn = p.Fnew + 6 * i;
  double* dg = p.diag + 18 * i;
  for (int k = 0; k < 6; ++k) dg[k] = Fn[k];
  if (p.mode[i] == MODE_FREE) {
    for (int a = 0; a < 3; ++a) {
      uo[a] = next_velocity(p.u[3 * i + a], p.Fold[6 * i + a], Fn[a], velocity_factor(p.m[i], dtp));
      wo[a] = next_velocity(p.w[3 * i + a], p.Fold[6 * i + 3 + a], Fn[3 + a], velocity_factor(p.I[i], dtp));
      p.Fold[6 * i + a] = Fn[a];
      p.Fold[6 * i + 3 + a] = Fn[3 + a];
    }
  } else if (p.mode[i] == MODE_PRESCRIBED) {
    p.tpresc[i] += dtp;
    for (int a = 0; a < 3; ++a) {
      uo[a] = prescribed_velocity(p.presc[6 * i + a], p.presc[6 * i + 3], p.presc[6 * i + 4], p.tpresc[i]);
      wo[a] = 0.0;
    }
  } else {
    for (int a = 0; a < 3; ++a) {
      uo[a] = p.u[3 * i + a];
      wo[a] = p.w[3 * i + a];
    }
  }
}

__device__ __forceinline__ void health_check(const DevDomain& d, const DevParticles& p, int i) {
  bool ok = true;
  for (int a = 0; a < 3; ++a)
    ok = ok && isfinite(p.x[3 * i + a]) && isfinite(p.u[3 * i + a]) && isfinite(p.w[3 * i + a]);
  if (!ok) atomicOr(d.status, ST_NONFINITE);
}

__device__ __forceinline__ void dem_body(const DevDomain& d, const DevParticles& p) {
  const int P = d.P;
  {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwave = blockDim.x >> 6;
    for (int i = wave; i < P; i += nwave) resolved_force(d, p, i, lane);
  }
  __syncthreads();
  // neighbour list for this step by all pairs, partners ascending
  const double range = list_range(d);
  for (int i = threadIdx.x; i < P; i += blockDim.x) {
    int cnt = 0;
    for (int j = 0; j < P; ++j) {
      if (j == i || !(pair_gap(d, p, i, j) < range)) continue;
      if (cnt < NBR_MAX)
        p.nbr[(size_t)i * NBR_MAX + cnt] = j;
      else
        atomicOr(d.status, ST_NBR_FULL);
      cnt++;
    }
    p.nbr_n[i] = cnt < NBR_MAX ? cnt : NBR_MAX;
  }
  __syncthreads();
  const double dtp = 1.0 / (double)d.n_sub;
  for (int sub = 0; sub < d.n_sub; ++sub) {
    for (int i = threadIdx.x; i < P; i += blockDim.x) release_and_start(d, p, i, dtp);
    __syncthreads();
    for (int i = threadIdx.x; i < P; i += blockDim.x) advance_position(d, p, i, dtp, p.x + 3 * i);
    __syncthreads();
    for (int i = threadIdx.x; i < P; i += blockDim.x)
      eval_forces(d, p, i, true, true, dtp, p.Fnew + 6 * i, p.Fnew + 6 * i + 3);
    __syncthreads();
    for (int i = threadIdx.x; i < P; i += blockDim.x) advance_velocity(d, p, i, dtp, p.u + 3 * i, p.w + 3 * i);
    __syncthreads();
  }
  for (int i = threadIdx.x; i < P; i += blockDim.x) health_check(d, p, i);
}

// ---- step control -----------------------------------------------------------

// At the start of the step's DEM kernel: true if the domain does not step (it
// is frozen, or the stop rule was met at the end of the last step; the step
// control kernel then freezes it).
__device__ __forceinline__ bool dem_stopped(const DevDomain& d) { return !step_live(d.ctl); }

__global__ void k_advance(DevDomain d) { step_control(d); }

__global__ void k_advance_batch(const DevDomain* __restrict__ tab, int ndom) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < ndom) step_control(tab[k]);
}

// one workgroup, state in global memory
__device__ __forceinline__ void dem_global_run(const DevDomain& d) {
  dem_body(d, d.p);
}

__global__ __launch_bounds__(256) void k_dem(DevDomain d) {
  __builtin_amdgcn_s_setprio(3);
  if (dem_stopped(d)) return;
  dem_global_run(d);
}

// Few spheres: one workgroup, a group of eight lanes per sphere.  Lane g < 6 of
// a group keeps its component of position and velocity (0-2) or spin (3-5) with
// its force and coefficients in registers for the whole step; what partners
// read (x, u, w in two buffers, R, m), the histories and the lists live in LDS.
// Bound by the latency of its dependent FP64 chain, not by any rate.  Against
// one thread per sphere with the whole state in memory arrays: 1 sphere 37 ->
// 18 us alone and 93 -> 44 us beside the 128x128x256 FP32 sweep (where every
// memory access of a sub-cycle costs microseconds: none is left in the quiet
// path), 40 agitated spheres 253 -> 78 us (72 since the pair terms' constants come
// with the domain), 16 requests of a batch 73 -> 27 us.
// LDS bytes of P spheres
__host__ __device__ inline size_t dem_lds_bytes(int P) {
  return (size_t)P * (8 * (3 + 6 + 6 + 6 + 2 + 3 * HIST_SLOTS) + 4 * HIST_SLOTS + NBR_MAX);
}
static_assert(DEM_LDS_MAX * (8 * 95 + 4 * HIST_SLOTS + NBR_MAX) <= 65536 && DEM_LDS_MAX <= 255,
              "few-sphere DEM state exceeds 64 KB of LDS");

__device__ __forceinline__ void dem_lds_run(const DevDomain& d, unsigned char* lds) {
  const int P = d.P, T = (int)blockDim.x, tid = (int)threadIdx.x;
  const int g = tid & (GROUP - 1), i = tid / GROUP;  // T >= GROUP P
  const int lane = tid & 63, base = lane & ~(GROUP - 1);
  const bool on = i < P, own = on && g < 6;
  const DevParticles& p = d.p;
  double* sx = (double*)lds;
  double *su = sx + 3 * P, *sw = su + 6 * P, *sFfp = sw + 6 * P, *sR = sFfp + 6 * P, *sm = sR + P, *shd = sm + P;
  int* shid = (int*)(shd + 3 * HIST_SLOTS * P);
  uint8_t* snbr = (uint8_t*)(shid + HIST_SLOTS * P);
  __shared__ int s_phase0;

  const double dtp = 1.0 / (double)d.n_sub;
  const int c = g < 3 ? g : g - 3;  // component of this lane
  double x = 0.0, v = 0.0, fold = 0.0, cpos = 0.0, cvel = 0.0, fext = 0.0, ut = 0.0, t = 0.0;
  double c_acc = 0.0, t_st = 1.0, gap = 0.0, R = 0.0;
  int mode = MODE_FIXED, old = 1;
  if (tid == 0) s_phase0 = 0;
  if (on) {
    const double m = p.m[i], rho = p.rho[i];
    R = p.R[i];
    mode = p.mode[i];
    old = p.old_valid[i];
    t = p.tpresc[i];
    if (own) {
      v = g < 3 ? p.u[3 * i + c] : p.w[3 * i + c];
      fold = p.Fold[6 * i + g];
      const double in = g < 3 ? m : p.I[i];
      if (g < 3) {
        x = p.x[3 * i + g];
        ut = p.presc[6 * i + g];
        fext = buoyant_mass(R, rho) * sel3(g, d.gravity[0], d.gravity[1], d.gravity[2]);
        sx[3 * i + g] = x;
        su[3 * i + g] = v;
      } else {
        sw[3 * i + c] = v;
      }
      cpos = position_factor(m, dtp);
      cvel = velocity_factor(in, dtp);
    }
    if (mode == MODE_PRESCRIBED) {
      c_acc = p.presc[6 * i + 3];
      t_st = p.presc[6 * i + 4];
      gap = p.presc[6 * i + 5];
    }
    if (g == 0) {
      sR[i] = R;
      sm[i] = m;
    }
  }
  for (int k = tid; k < HIST_SLOTS * P; k += T) shid[k] = p.hist_id[k];
  for (int k = tid; k < 3 * HIST_SLOTS * P; k += T) shd[k] = p.hist_d[k];
  // the momentum-exchange sums, one wavefront per sphere
  for (int k = tid >> 6; k < P; k += T >> 6) resolved_force(d, p, k, lane, sFfp);
  __syncthreads();
  const double ffp = own ? sFfp[6 * i + g] : 0.0;
  if (mode == MODE_PRESCRIBED || (mode == MODE_FREE && !old)) s_phase0 = 1;

  // neighbour list for this step by all pairs, partners ascending
  int nn = 0;
  const double range = list_range(d);
  for (int j0 = 0; j0 < P; j0 += GROUP) {
    const int j = j0 + g;
    bool near = false;
    if (on && j < P && j != i) {
      double dd[3], dist;
      near = sphere_offset(d, sx + 3 * i, R, sx + 3 * j, sR[j], dd, &dist) < range;
    }
    const unsigned m = (unsigned)((__ballot(near) >> base) & 0xFFull);
    if (near) {
      const int at = nn + __popc(m & ((1u << g) - 1u));
      if (at < NBR_MAX)
        snbr[NBR_MAX * i + at] = (uint8_t)j;
      else
        atomicOr(d.status, ST_NBR_FULL);
    }
    nn += __popc(m);
  }
  nn = nn < NBR_MAX ? nn : NBR_MAX;
  __syncthreads();
  const bool phase0 = s_phase0 != 0;  // some sphere can start or be released

  const double L = (double)sel3(g, d.nx, d.ny, d.nz);
  const int wall = sel3(g, d.walls[0], d.walls[1], d.walls[2]);
  for (int sub = 0; sub < d.n_sub; ++sub) {
    double *u1 = su + (sub & 1 ? 0 : 3 * P), *w1 = sw + (sub & 1 ? 0 : 3 * P);
    const GroupState s = {sx, su + (sub & 1 ? 3 * P : 0), sw + (sub & 1 ? 3 * P : 0), sR, sm};
    // phase 0: release below the gap, start force of newly free spheres; phase
    // 1 (after the positions): forces and velocities.  One loop, so that the
    // force code is there once.
    for (int phase = phase0 ? 0 : 1; phase < 2; ++phase) {
      bool act = on;
      if (phase == 0) {
        // lanes 0-2 each take one axis of gap_ahead
        const bool near = own && g < 3 && fmin(1e300, axis_gap_ahead(x, R, ut, wall, L)) < gap;
        if (mode == MODE_PRESCRIBED && ((__ballot(near) >> base) & 0xFFull)) {
          mode = MODE_FREE;
          old = 0;
        }
        act = on && mode == MODE_FREE && !old;
        old = act ? 1 : old;
      } else {
        if (own && g < 3) {
          x = next_position(mode, x, v, fold, cpos, dtp, L, wall);
          sx[3 * i + g] = x;
        }
        __syncthreads();
      }
      if (__any(act)) {
        double lub, col;
        group_forces(d, s, i, act, nn, [&](int k) { return (int)snbr[NBR_MAX * i + k]; }, shid + HIST_SLOTS * i,
                     shd + 3 * HIST_SLOTS * i, phase == 1, phase == 1, dtp, &lub, &col);
        if (act && g < 6) {
          const double F = total_term(ffp, lub, col, fext, g < 3);
          if (phase == 1) {
            if (mode == MODE_FREE) {
              v = next_velocity(v, fold, F, cvel);
            } else if (mode == MODE_PRESCRIBED) {
              t += dtp;
              v = g < 3 ? prescribed_velocity(ut, c_acc, t_st, t) : 0.0;
            }
            if (g < 3)
              u1[3 * i + c] = v;
            else
              w1[3 * i + c] = v;
            if (sub == d.n_sub - 1) {
              p.diag[18 * i + g] = F;
              p.diag[18 * i + 6 + g] = lub;
              p.diag[18 * i + 12 + g] = col;
            }
          }
          if (mode == MODE_FREE) fold = F;
        }
      }
      __syncthreads();
    }
  }

  if (own) {
    if (g < 3) p.x[3 * i + g] = x;
    (g < 3 ? p.u : p.w)[3 * i + c] = v;
    p.Fold[6 * i + g] = fold;
    if (!(isfinite(v) && isfinite(x))) atomicOr(d.status, ST_NONFINITE);
    if (g == 0) {
      p.tpresc[i] = t;
      p.mode[i] = mode;
      p.old_valid[i] = old;
    }
  }
  for (int k = tid; k < HIST_SLOTS * P; k += T) p.hist_id[k] = shid[k];
  for (int k = tid; k < 3 * HIST_SLOTS * P; k += T) p.hist_d[k] = shd[k];
}

// threads of the few-sphere kernel: one wavefront, whose barriers cost nothing,
// up to eight spheres
constexpr int DEM_LDS_THREADS = GROUP * DEM_LDS_MAX;
static unsigned dem_lds_threads(int P) { return P <= 8 ? 64u : (P <= 32 ? 256u : (unsigned)DEM_LDS_THREADS); }

// The one-workgroup kernels run beside the sweep in an overlapped step: they
// are a chain of dependent FP64 work, so their waves take the highest issue
// priority on the CUs they share with the sweep's waves.
extern __shared__ double dem_smem[];

__global__ __launch_bounds__(DEM_LDS_THREADS) void k_dem_lds(DevDomain d) {
  __builtin_amdgcn_s_setprio(3);
  if (dem_stopped(d)) return;
  dem_lds_run(d, (unsigned char*)dem_smem);
}

// many domains, one workgroup each (the few-sphere kernels above)
__global__ __launch_bounds__(DEM_LDS_THREADS) void k_dem_batch(const DevDomain* __restrict__ tab, int ndom) {
  const DevDomain& d = tab[blockIdx.x];
  if (dem_stopped(d) || d.P <= 0) return;
  if (d.P <= DEM_LDS_MAX)
    dem_lds_run(d, (unsigned char*)dem_smem);
  else
    dem_global_run(d);
}

void launch_dem_batch(const BatchTables& b, hipStream_t s) {
  // threads for the largest few-sphere domain there can be (domains with more
  // spheres take any number)
  const int P = b.max_P < DEM_LDS_MAX ? b.max_P : DEM_LDS_MAX;
  if (b.ndom > 0 && b.max_P > 0)
    hipLaunchKernelGGL(k_dem_batch, dim3(b.ndom), dim3(dem_lds_threads(P)), dem_lds_bytes(P), s, b.tab, b.ndom);
}

void launch_advance(const DevDomain& d, hipStream_t s) { hipLaunchKernelGGL(k_advance, dim3(1), dim3(1), 0, s, d); }

void launch_advance_batch(const BatchTables& b, hipStream_t s) {
  if (b.ndom > 0) hipLaunchKernelGGL(k_advance_batch, dim3((b.ndom + 63) / 64), dim3(64), 0, s, b.tab, b.ndom);
}

// ---------------------------------------------------------------------------
// Grid-wide kernel for many spheres.

__device__ __forceinline__ int bin_index(const DevDomain& d, const double* x, int* b) {
  const int n[3] = {d.nx, d.ny, d.nz};
  for (int a = 0; a < 3; ++a) {
    const int nb = d.bins.n[a];
    int k = (int)floor(x[a] * (double)nb / (double)n[a]);
    b[a] = k < 0 ? 0 : (k >= nb ? nb - 1 : k);
  }
  return b[0] + d.bins.n[0] * (b[1] + d.bins.n[1] * b[2]);
}

__device__ __forceinline__ void bin_insert(const DevDomain& d, const DevParticles& p, int i) {
  const double* x = p.x + 3 * i;
  if (!(isfinite(x[0]) && isfinite(x[1]) && isfinite(x[2]))) {
    atomicOr(d.status, ST_NONFINITE);
    return;
  }
  int b[3];
  int* c = d.bins.cell + (size_t)bin_index(d, x, b) * (1 + BIN_CAP);
  const int k = atomicAdd(c, 1);
  if (k < BIN_CAP)
    c[1 + k] = i;
  else
    atomicOr(d.status, ST_NBR_FULL);
}

// The neighbour test of dem_body by 32 lanes per sphere.  With bins lane e takes
// the e-th of the 27 around the sphere, so their counts and ids are read in two
// round trips instead of 27 one after the other (10,000 spheres beside the 384^3
// sweep: 253 -> 23 us); without, spheres e, e + 32, ...  The partners are collected
// in LDS in any order and then written by rank (ids are distinct), so every
// kernel produces the same list.
constexpr int NBR_LANES = 32;
__device__ __forceinline__ void lane_neighbours(const DevDomain& d, const DevParticles& p, int i, bool bins, int* cand,
                                                int* ncand) {
  const int e = threadIdx.x & (NBR_LANES - 1);
  const bool on = i < d.P;
  if (e == 0) *ncand = 0;
  __syncthreads();
  const double range = list_range(d);
  auto test = [&](int j) {
    if (j == i || !(pair_gap(d, p, i, j) < range)) return;
    const int at = atomicAdd(ncand, 1);
    if (at < NBR_MAX)
      cand[at] = j;
    else
      atomicOr(d.status, ST_NBR_FULL);
  };
  const double* x = p.x + 3 * (on ? i : 0);
  if (on && !bins) {
    for (int j = e; j < d.P; j += NBR_LANES) test(j);
  } else if (on && isfinite(x[0]) && isfinite(x[1]) && isfinite(x[2])) {
    int b[3];
    bin_index(d, x, b);
    const int n0 = d.bins.n[0], n1 = d.bins.n[1], n2 = d.bins.n[2];
    const int a0 = axis_count(n0), a1 = axis_count(n1), a2 = axis_count(n2);
    int kx, ky, kz;
    if (e < a0 * a1 * a2 && axis_bin(b[0], n0, d.walls[0], e % a0, &kx) &&
        axis_bin(b[1], n1, d.walls[1], e / a0 % a1, &ky) && axis_bin(b[2], n2, d.walls[2], e / (a0 * a1), &kz)) {
      const int* c = d.bins.cell + (size_t)(kx + n0 * (ky + n1 * kz)) * (1 + BIN_CAP);
      const int m = min(c[0], BIN_CAP);
      for (int k = 0; k < m; ++k) test(c[1 + k]);
    }
  }
  __syncthreads();
  const int n = min(*ncand, NBR_MAX);
  if (!on) return;
  int* out = p.nbr + (size_t)i * NBR_MAX;
  for (int k = e; k < n; k += NBR_LANES) {
    const int j = cand[k];
    int rank = 0;
    for (int q = 0; q < n; ++q) rank += cand[q] < j;
    out[rank] = j;
  }
  if (e == 0) p.nbr_n[i] = n;
}

// Many spheres: a group of lanes per sphere, the sub-cycles as a chain of ordinary
// launches (a kernel boundary wherever every sphere must see the others'
// state): the momentum-exchange sums and the bins, the neighbour lists, then
// per sub-cycle the positions (into the other buffer) and the forces and
// velocities (into the other buffer).  Ordinary launches can run beside the
// sweep on a second stream, where a cooperative grid could not be sure of
// having all its blocks resident.  Per sphere the arithmetic and its order are
// those of the one-workgroup kernels (identical bits).
__global__ __launch_bounds__(DEM_GRID_THREADS) void k_demg_prologue(DevDomain d, int bins) {
  if (dem_stopped(d)) return;
  const int lane = threadIdx.x & 63;
  const int i = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  if (i >= d.P) return;
  resolved_force(d, d.p, i, lane);
  if (bins && lane == 0) bin_insert(d, d.p, i);
}

// the same where each sphere has one partial (one block per sphere in the
// boundary pass): lane g < 6 of its group takes component g
__global__ __launch_bounds__(DEM_GRID_THREADS) void k_demg_prologue_one(DevDomain d, int bins) {
  if (dem_stopped(d)) return;
  const int g = threadIdx.x & (GROUP - 1);
  const int i = (int)((blockIdx.x * blockDim.x + threadIdx.x) / GROUP);
  if (i >= d.P) return;
  const DevParticles& p = d.p;
  if (g < 6) {
    const int k = 6 * i + g;
    const double F = 0.0 + d.partial[k];
    p.Fraw[k] = F;
    if (d.force_averaging) {
      const double prev = p.prev_valid[i] ? p.Fprev[k] : F;
      p.Ffp[k] = 0.5 * (F + prev);
      p.Fprev[k] = F;
    } else {
      p.Ffp[k] = F;
    }
  }
  if (g < 3) p.xmap[3 * i + g] = p.x[3 * i + g];
  if (bins && g == 7) bin_insert(d, p, i);
  if (g == 0 && d.force_averaging) p.prev_valid[i] = 1;
}

__global__ __launch_bounds__(DEM_GRID_THREADS) void k_demg_neighbours(DevDomain d, int bins) {
  if (dem_stopped(d)) return;
  constexpr int PER = DEM_GRID_THREADS / NBR_LANES;
  __shared__ int cand[PER][NBR_MAX], ncand[PER];
  const int s = threadIdx.x / NBR_LANES;
  lane_neighbours(d, d.p, (int)blockIdx.x * PER + s, bins != 0, cand[s], &ncand[s]);
}

// state of sub-cycle `sub` (even: the first buffers), and the other buffer
__device__ __forceinline__ void subcycle_buffers(const DevParticles& p, int sub, DevParticles& a, double** x1,
                                                 double** u1, double** w1) {
  const bool odd = sub & 1;
  a = p;
  a.x = odd ? p.x2 : p.x;
  a.u = odd ? p.u2 : p.u;
  a.w = odd ? p.w2 : p.w;
  *x1 = odd ? p.x : p.x2;
  *u1 = odd ? p.u : p.u2;
  *w1 = odd ? p.w : p.w2;
}

__global__ __launch_bounds__(DEM_GRID_THREADS) void k_demg_position(DevDomain d, int sub, int bins) {
  if (dem_stopped(d)) return;
  const int gtid = blockIdx.x * blockDim.x + threadIdx.x;
  if (bins && sub == 0) {  // the lists are built: clear the bins for the next step
    const int nbins = d.bins.n[0] * d.bins.n[1] * d.bins.n[2];
    for (int k = gtid; k < nbins; k += gridDim.x * blockDim.x) d.bins.cell[(size_t)k * (1 + BIN_CAP)] = 0;
  }
  if (gtid >= d.P) return;
  DevParticles a;
  double *x1, *u1, *w1;
  subcycle_buffers(d.p, sub, a, &x1, &u1, &w1);
  const double dtp = 1.0 / (double)d.n_sub;
  release_and_start(d, a, gtid, dtp);
  advance_position(d, a, gtid, dtp, x1 + 3 * gtid);
}

// forces at the new positions with the old velocities, new velocities into
// the other buffer, by a group of eight lanes per sphere (one thread per
// sphere walked its partners one after the other, a chain of memory round
// trips per partner: 10,000 spheres beside the 384^3 sweep 77 -> 41 us per
// sub-cycle); after the last sub-cycle the state is
// copied back if it ended in the second buffers (odd n_sub, a kernel of its
// own) and checked.  With `fuse` the group then advances its own sphere's
// position of the next sub-cycle: nothing in this launch reads the buffer that
// goes into, and that step reads only the sphere's own state -- valid when no
// sphere can be released from a prescribed motion (a release evaluates forces
// on every partner's state, which needs the sub-cycle's launch boundary).
__global__ __launch_bounds__(DEM_GRID_THREADS) void k_demg_velocity(DevDomain d, int sub, int fuse) {
  if (dem_stopped(d)) return;
  const int g = threadIdx.x & (GROUP - 1);
  const int gi = (int)((blockIdx.x * blockDim.x + threadIdx.x) / GROUP);
  const bool on = gi < d.P;  // every lane stays for the group's shuffles
  const int i = on ? gi : 0;
  DevParticles a;
  double *x1, *u1, *w1;
  subcycle_buffers(d.p, sub, a, &x1, &u1, &w1);
  const double dtp = 1.0 / (double)d.n_sub;
  const GroupState s = {x1, a.u, a.w, a.R, a.m};
  const int* nbr = a.nbr + (size_t)i * NBR_MAX;
  double lub, col;
  group_forces(d, s, i, on, a.nbr_n[i], [&](int k) { return nbr[k]; }, a.hist_id + (size_t)i * HIST_SLOTS,
               a.hist_d + (size_t)i * HIST_SLOTS * 3, true, true, dtp, &lub, &col);
  if (!on || g >= 6) return;
  const int c = g < 3 ? g : g - 3, k = 6 * i + g;
  const double F = group_total(d, g, lub, col, a.Ffp[k], buoyant_mass(a.R[i], a.rho[i]));
  const int mode = a.mode[i];
  const double v0 = g < 3 ? a.u[3 * i + c] : a.w[3 * i + c];
  double v1 = v0, fold = 0.0;
  if (mode == MODE_FREE) {
    fold = F;
    v1 = next_velocity(v0, a.Fold[k], F, velocity_factor(g < 3 ? a.m[i] : a.I[i], dtp));
    a.Fold[k] = F;
  } else if (mode == MODE_PRESCRIBED) {
    const double t = a.tpresc[i] + dtp;
    v1 = g < 3 ? prescribed_velocity(a.presc[6 * i + c], a.presc[6 * i + 3], a.presc[6 * i + 4], t) : 0.0;
    if (g == 0) a.tpresc[i] = t;
  }
  (g < 3 ? u1 : w1)[3 * i + c] = v1;
  const bool last = sub == d.n_sub - 1;
  if (last) {
    a.diag[18 * i + g] = F;
    a.diag[18 * i + 6 + g] = lub;
    a.diag[18 * i + 12 + g] = col;
    if (!(d.n_sub & 1) && !(isfinite(v1) && (g >= 3 || isfinite(x1[3 * i + c])))) atomicOr(d.status, ST_NONFINITE);
  }
  if (fuse && g < 3) {
    // position of the next sub-cycle, into the buffer x came from
    double* xn = sub & 1 ? d.p.x2 : d.p.x;
    const int n = sel3(g, d.nx, d.ny, d.nz);
    xn[3 * i + g] = next_position(mode, x1[3 * i + g], v1, fold, position_factor(a.m[i], dtp), dtp, (double)n,
                                 sel3(g, d.walls[0], d.walls[1], d.walls[2]));
  }
}

__global__ __launch_bounds__(DEM_GRID_THREADS) void k_demg_epilogue(DevDomain d) {
  if (dem_stopped(d)) return;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d.P) return;
  const DevParticles& p = d.p;
  for (int a = 0; a < 3; ++a) {
    p.x[3 * i + a] = p.x2[3 * i + a];
    p.u[3 * i + a] = p.u2[3 * i + a];
    p.w[3 * i + a] = p.w2[3 * i + a];
  }
  health_check(d, p, i);
}

bool dem_many(const DevDomain& d, int kernel) { return kernel == 2 || (kernel == 0 && d.P > DEM_LDS_MAX); }

hipError_t launch_dem(const DevDomain& d, int kernel, bool no_release, hipStream_t s) {
  if (d.P <= 0) return hipSuccess;
  if (!dem_many(d, kernel)) {
    if (d.P <= DEM_LDS_MAX)
      hipLaunchKernelGGL(k_dem_lds, dim3(1), dim3(dem_lds_threads(d.P)), dem_lds_bytes(d.P), s, d);
    else
      hipLaunchKernelGGL(k_dem, dim3(1), dim3(256), 0, s, d);
    return hipGetLastError();
  }
  const unsigned T = DEM_GRID_THREADS;
  auto grid = [&](int lanes) { return dim3((unsigned)(((long long)d.P * lanes + T - 1) / T)); };
  // Lists by all pairs up to DEM_PAIRS_MAX spheres: a bin holds BIN_CAP of them,
  // which a cluster of few spheres in a wide lattice (bins grow until their number
  // is a few per sphere), or of small ones beside a large max_radius, exceeds.
  const int bins = kernel == 2 || d.P > DEM_PAIRS_MAX ? 1 : 0;
  if (d.ZB * d.RB == 1)
    hipLaunchKernelGGL(k_demg_prologue_one, grid(GROUP), dim3(T), 0, s, d, bins);
  else
    hipLaunchKernelGGL(k_demg_prologue, grid(64), dim3(T), 0, s, d, bins);
  hipLaunchKernelGGL(k_demg_neighbours, grid(NBR_LANES), dim3(T), 0, s, d, bins);
  // (its threads also clear the bins, a few each: with only the threads of 156
  // spheres that alone took 20 us)
  const long long clear = bins ? ((long long)d.bins.n[0] * d.bins.n[1] * d.bins.n[2] + 4 * T - 1) / (4 * T) : 0;
  hipLaunchKernelGGL(k_demg_position, dim3(std::max(grid(1).x, (unsigned)clear)), dim3(T), 0, s, d, 0, bins);
  for (int sub = 0; sub < d.n_sub; ++sub) {
    const int fuse = no_release && sub + 1 < d.n_sub ? 1 : 0;
    hipLaunchKernelGGL(k_demg_velocity, grid(GROUP), dim3(T), 0, s, d, sub, fuse);
    if (!fuse && sub + 1 < d.n_sub) hipLaunchKernelGGL(k_demg_position, grid(1), dim3(T), 0, s, d, sub + 1, bins);
  }
  if (d.n_sub & 1) hipLaunchKernelGGL(k_demg_epilogue, grid(1), dim3(T), 0, s, d);
  return hipGetLastError();
}

}  // namespace lbmdem
