// Explicit step of the Rykov diatomic model (Sec. 2.3 in its explicit limit
// with the equilibrium of Eqs. GHR_equ, equ11-equ13 and the rotational
// source of Eq. equ19), FP64, in 2-D and 3-D, and the adaptation of the
// velocity tree it drives (Secs. 3.2-3.4).  Three reduced distributions per
// cell and leaf, [3][cell][leaf]: G, H (the 3 - D hidden translational
// degrees of freedom; identically zero in 3-D) and R (rotational energy,
// two degrees of freedom); D + 3 conserved variables (rho, rho U, rho E,
// rho E_rot).  One pass per stage, written for clarity rather than speed:
//   k_dg_recon   limited least-squares reconstruction at x_f - xi h into the
//                interface rows (boundary Maxwellian triples on incoming leaves)
//   k_dg_face    interface moments, rotational and heat-flux relaxation over h,
//                Rykov equilibrium, characteristic blend in place, flux F_f
//   k_dg_macro   W* = W - dt/V sum sigma A F, point-implicit rotational exchange
//   k_dg_target  closure coefficients of the Rykov target ((D+3)^2 system)
//   k_dg_update  flux divergence, relaxation, heat fluxes of phi^{n+1}
// Part of the library's single translation unit, after avs_kernels.hip.

namespace avs {

template <int D>
struct Dg {
  static constexpr int NW = D + 3;           // rho, rho U, rho E, rho E_rot
  static constexpr int NQ = 2 * D;           // q_t, q_r
  // record: rho, U[D], T_t, T_r, q_t[D], q_r[D], dt/tau, E_rot target, T
  static constexpr int IT = 1 + D, IR = 2 + D, IQT = 3 + D, IQR = 3 + 2 * D, IDT = 3 + 3 * D, IER = 4 + 3 * D,
                       IT0 = 5 + 3 * D, NT = 6 + 3 * D;
  static constexpr int MAXF = Cfg<D>::MAXF;
  static constexpr int NACC = NW * (1 + NW);   // moments of the base and of the NW closure directions
};

struct DiaGas {
  double R, Z, delta, omega0, omega1;
};

// rho (2 pi R T)^(-D/2)
template <int D>
__device__ __forceinline__ double dg_norm(double rho, double RT) {
  return D == 2 ? rho / (2.0 * M_PI * RT) : rho * pow(2.0 * M_PI * RT, -0.5 * D);
}

// Rykov equilibrium triple at one leaf (c = xi - U), or, with t_only, the
// translational part at (T_t, T_r) with zero heat fluxes; gt and g are the
// Maxwellians at T_t and at T = (3 T_t + 2 T_r)/5.
template <int D>
__device__ __forceinline__ void dg_equilibrium(const DiaGas& gp, double rho, const double (&c)[D], double Tt, double Tr,
                                               const double* qt, const double* qr, bool t_only, double gt, double g,
                                               double& G, double& H, double& Rr) {
  const double R = gp.R;
  const double T = (3.0 * Tt + 2.0 * Tr) / 5.0;
  double c2 = 0.0, cqt = 0.0, cqr = 0.0;
#pragma unroll
  for (int d = 0; d < D; ++d) c2 += c[d] * c[d];
  const double RTt = R * Tt, RT = R * T;
  const double hid = 3 - D;
  if (t_only) {
    G = gt;
    H = hid * RTt * gt;
    Rr = R * Tr * gt;
    return;
  }
#pragma unroll
  for (int d = 0; d < D; ++d) {
    cqt += c[d] * qt[d];
    cqr += c[d] * qr[d];
  }
  const double pt = rho * RTt, p = rho * RT;
  const double at = cqt / (15.0 * pt * RTt), ar = gp.omega0 * cqt / (15.0 * p * RT);
  const double Gt = gt * (1.0 + at * (c2 / RTt - (D + 2.0)));
  const double Gr = g * (1.0 + ar * (c2 / RT - (D + 2.0)));
  const double Ht = hid * RTt * gt * (1.0 + at * (c2 / RTt - D));
  const double Hr = hid * RT * g * (1.0 + ar * (c2 / RT - D));
  const double Rt = R * Tr * (Gt + (1.0 - gp.delta) * cqr / (pt * RTt) * gt);
  const double Rq = RT * (Gr + gp.omega1 * (1.0 - gp.delta) * cqr / (p * RT) * g);
  const double wt = 1.0 - 1.0 / gp.Z, wr = 1.0 / gp.Z;
  G = wt * Gt + wr * Gr;
  H = wt * Ht + wr * Hr;
  Rr = wt * Rt + wr * Rq;
}

// Separable per-axis tables of the Maxwellians at T_t and at T (the
// half-finest grid carries every leaf centre), built by the whole block
// from a record r = (rho, U[D], T_t, T_r, ...); followed by a barrier.
template <int D>
__device__ __forceinline__ void dg_tables(const double* r, double R, const VGrid& vg, double* tabt, double* tabr,
                                          double* part, double* parr) {
  if (threadIdx.x == 0) {
    const double Tt = r[Dg<D>::IT], T = (3.0 * r[Dg<D>::IT] + 2.0 * r[Dg<D>::IR]) / 5.0;
    part[P_COEF] = dg_norm<D>(r[0], R * Tt);
    parr[P_COEF] = dg_norm<D>(r[0], R * T);
    for (int d = 0; d < 3; ++d) part[P_U + d] = parr[P_U + d] = d < D ? r[1 + d] : 0.0;
    part[P_I2RT] = 0.5 / (R * Tt);
    parr[P_I2RT] = 0.5 / (R * T);
  }
  __syncthreads();
  build_tab<D>(tabt, part, vg);
  build_tab<D>(tabr, parr, vg);
  __syncthreads();
}

// rho, U, T_t, T_r, T from W = (rho, rho U, rho E, rho E_rot).
template <int D>
__device__ __forceinline__ bool dg_temps(const double* w, double R, double& rho, double (&U)[D], double& Tt, double& Tr,
                                         double& T) {
  rho = w[0];
  double uu = 0.0;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    U[d] = w[1 + d] / rho;
    uu += U[d] * U[d];
  }
  Tr = w[2 + D] / (rho * R);
  Tt = (w[1 + D] - 0.5 * rho * uu - w[2 + D]) / (1.5 * rho * R);
  T = (3.0 * Tt + 2.0 * Tr) / 5.0;
  return rho > 0.0 && Tt > 0.0 && Tr > 0.0;
}

// moments (rho, rho U, rho E, rho E_rot) contribution of one leaf
template <int D>
__device__ __forceinline__ void dg_mom(double* m, double A, const double (&xi)[D], double G, double H, double Rr) {
  double xi2 = 0.0;
#pragma unroll
  for (int d = 0; d < D; ++d) xi2 += xi[d] * xi[d];
  m[0] += A * G;
#pragma unroll
  for (int d = 0; d < D; ++d) m[1 + d] += A * G * xi[d];
  m[1 + D] += A * (0.5 * (xi2 * G + H) + Rr);
  m[2 + D] += A * Rr;
}

template <int D>
__global__ __launch_bounds__(BLOCK) void k_dg_recon(Geo g, Leaves L, double h, const double* __restrict__ vin,
                                                   double* __restrict__ fv, DiaGas gp, int chunk) {
  constexpr int MAXF = Dg<D>::MAXF;
  const int i = xcd_cell(g, blockIdx.x);
  if (i < 0) return;
  const int k0 = blockIdx.y * chunk, k1 = min(L.n, k0 + chunk);
  const int ns = g.nslot[i];
  const size_t cs = (size_t)g.nc * L.ld, fs = (size_t)g.nf * L.ld;
  // neighbour rows (a slot without an interior neighbour reads the cell's
  // own row and is skipped), so that every load of a leaf is issued before
  // any is used
  size_t nb[MAXF];
  unsigned mask = 0;
#pragma unroll
  for (int s = 0; s < MAXF; ++s) {
    const int j = s < ns ? g.s_nbr[i * MAXF + s] : -1;
    if (j >= 0) mask |= 1u << s;
    nb[s] = (size_t)(j >= 0 ? j : i) * L.ld;
  }
  // the cell's LSQ coefficients and face offsets, held for the leaf loop
  double cf[MAXF][D], dd[MAXF][D];
#pragma unroll
  for (int s = 0; s < MAXF; ++s)
#pragma unroll
    for (int d = 0; d < D; ++d) {
      cf[s][d] = s < ns ? g.s_lsq[(size_t)(i * MAXF + s) * D + d] : 0.0;
      dd[s][d] = s < ns ? g.s_d[(size_t)(i * MAXF + s) * D + d] : 0.0;
    }
  const double eps2 = g.eps2[i];
  for (int k = k0 + threadIdx.x; k < k1; k += BLOCK) {
    double xi[D], A;
    int u[D];
    leaf_load<D>(L, k, xi, A, u);
    double ph[3], gr[3][D], pmax[3], pmin[3], nv[MAXF][3];
#pragma unroll
    for (int p = 0; p < 3; ++p) ph[p] = vin[p * cs + (size_t)i * L.ld + k];
#pragma unroll
    for (int s = 0; s < MAXF; ++s)
#pragma unroll
      for (int p = 0; p < 3; ++p) nv[s][p] = vin[p * cs + nb[s] + k];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
#pragma unroll
      for (int d = 0; d < D; ++d) gr[p][d] = 0.0;
      pmax[p] = pmin[p] = ph[p];
    }
#pragma unroll
    for (int s = 0; s < MAXF; ++s) {
      if (!(mask & (1u << s))) continue;
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        const double v = nv[s][p];
        const double dv = v - ph[p];
#pragma unroll
        for (int d = 0; d < D; ++d) gr[p][d] += dv * cf[s][d];
        pmax[p] = fmax(pmax[p], v);
        pmin[p] = fmin(pmin[p], v);
      }
    }
    // Venkatakrishnan psi_f = N/Dn with a = |D2|, b = |D1| (same sign),
    // N = b^2 + eps^2 + 2ab, Dn = b^2 + 2a^2 + ab + eps^2 (psi = 1 for
    // D2 = 0); a, b and eps scaled by the power of two above the largest of
    // them, the minimum over faces kept as a fraction by cross-multiplication
    // and ended by one division
    double lg[3][D];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      double d2s[MAXF];
      const double up0 = pmax[p] - ph[p], dn0 = ph[p] - pmin[p];
      double mx = fmax(up0, dn0);
#pragma unroll
      for (int s = 0; s < MAXF; ++s) {
        double d2 = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) d2 += gr[p][d] * dd[s][d];
        d2s[s] = d2;
        if (s < ns) mx = fmax(fabs(d2), mx);
      }
      double lim = 1.0;
      // below the smallest normal number the differences carry no
      // information: the slope stays unlimited
      if (ns > 0 && mx > 1e-300) {
        int ex;
        (void)frexp(mx, &ex);
        const double inv = ldexp(1.0, -ex);
        const double e2 = fmin(eps2 * inv * inv, 1e30);
        const double up = up0 * inv, dn = dn0 * inv;
        double Nm = 1.0, Dm = 0.0;
#pragma unroll
        for (int s = 0; s < MAXF; ++s) {
          if (s < ns) {
            const double a = fabs(d2s[s]) * inv;
            const double b = d2s[s] > 0.0 ? up : dn;
            const double c = b * b + e2 + 1e-300;
            const double Nn = c + 2.0 * a * b;
            const double Dd = c + a * (2.0 * a + b);
            if (Nn * Dm < Nm * Dd) {
              Nm = Nn;
              Dm = Dd;
            }
          }
        }
        lim = Nm / Dm;
      }
#pragma unroll
      for (int d = 0; d < D; ++d) lg[p][d] = lim * gr[p][d];
    }
    for (int s = 0; s < ns; ++s) {
      const int f = g.s_face[i * MAXF + s];
      const double sig = g.s_sig[i * MAXF + s];
      const double sn = normal_speed<D>(xi, g.f_nrm + (size_t)f * D);
      const bool upwind = sig > 0.0 ? sn >= 0.0 : sn < 0.0;
      const int Rc = g.f_R[f];
      const size_t o = (size_t)f * L.ld + k;
      if (upwind) {
        double r[D];
#pragma unroll
        for (int d = 0; d < D; ++d) r[d] = g.s_d[(size_t)(i * MAXF + s) * D + d] - xi[d] * h;
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          double x = 0.0;
#pragma unroll
          for (int d = 0; d < D; ++d) x += lg[p][d] * r[d];
          fv[p * fs + o] = ph[p] + x;
        }
      } else if (Rc < 0) {
        // incoming leaf of a boundary face: the equilibrium triple of the
        // wall (unit density, scaled by the wall density later) or of the far field
        const int b = -1 - Rc;
        const double* st = g.bc_prim + (size_t)b * (D + 2);
        const double rho = g.bc_kind[b] == 0 ? 1.0 : st[0];
        double c2 = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) {
          const double c = xi[d] - st[1 + d];
          c2 += c * c;
        }
        const double RT = gp.R * st[1 + D];
        const double gv = dg_norm<D>(rho, RT) * exp(-c2 / (2.0 * RT));
        fv[o] = gv;
        fv[fs + o] = (3 - D) * RT * gv;
        fv[2 * fs + o] = RT * gv;
      }
    }
  }
}

// block sum of NN doubles per thread; every thread gets the sums
template <int NN>
__device__ __forceinline__ void dg_sum(double* v, double* red) {
  for (int m = 0; m < NN; ++m) {
    double x = v[m];
    for (int o = 32; o > 0; o >>= 1) x += __shfl_down(x, o);
    if ((threadIdx.x & 63) == 0) red[(threadIdx.x >> 6) * NN + m] = x;
  }
  __syncthreads();
  if (threadIdx.x < NN) {
    double x = 0.0;
    for (int w = 0; w < BLOCK / 64; ++w) x += red[w * NN + threadIdx.x];
    red[BLOCK / 64 * NN + threadIdx.x] = x;
  }
  __syncthreads();
  for (int m = 0; m < NN; ++m) v[m] = red[BLOCK / 64 * NN + m];
  __syncthreads();
}

// With rf (the implicit step), also r_f = |U.n| + a + 2 mu/(rho dl) of the
// predictor: interior faces from the interface moment state (rho, U, T_t of
// the reconstructed rows, its tau), boundary faces from the cell's W^n and
// dl = 2 (x_f - x_i).n; a = sqrt(5/3 R T_t), mu/rho = tau R T_t.
template <int D>
__global__ __launch_bounds__(BLOCK) void k_dg_face(Geo g, Leaves L, VGrid vg, GasP vgas, DiaGas gp, double h,
                                                  double* __restrict__ fv, double* __restrict__ F, int* __restrict__ bad,
                                                  const double* __restrict__ W, double* __restrict__ rf) {
  using C = Dg<D>;
  constexpr int NW = C::NW;
  extern __shared__ double lds_d[];
  __shared__ double red[(BLOCK / 64 + 1) * (Dg<D>::NW + 2 * D + D * (D + 1) / 2)];
  __shared__ double rec[C::NT], part[NPAR], parr[NPAR];
  const int f = blockIdx.x;
  const int Rc = g.f_R[f];
  const size_t fs = (size_t)g.nf * L.ld;
  double n[D];
#pragma unroll
  for (int d = 0; d < D; ++d) n[d] = g.f_nrm[(size_t)f * D + d];
  double* row0 = fv + (size_t)f * L.ld;
  if (Rc >= 0) {
    // one pass of raw moments: the conserved moments, then
    // e1_d = sum A (xi^2 G + H)/2 xi_d, p_de = sum A G xi_d xi_e (d <= e) and
    // r1_d = sum A R xi_d, from which the heat fluxes about U follow
    constexpr int NP = D * (D + 1) / 2, NS = NW + 2 * D + NP;
    double m[NS];
    for (int t = 0; t < NS; ++t) m[t] = 0.0;
    for (int k = threadIdx.x; k < L.n; k += BLOCK) {
      double xi[D], A;
      int u[D];
      leaf_load<D>(L, k, xi, A, u);
      const double Gv = row0[k], Hv = row0[fs + k], Rv = row0[2 * fs + k];
      dg_mom<D>(m, A, xi, Gv, Hv, Rv);
      double xi2 = 0.0;
#pragma unroll
      for (int d = 0; d < D; ++d) xi2 += xi[d] * xi[d];
      const double ek = A * 0.5 * (xi2 * Gv + Hv), ag = A * Gv, ar = A * Rv;
      int t = NW + 2 * D;
#pragma unroll
      for (int d = 0; d < D; ++d) {
        m[NW + d] += ek * xi[d];
        m[NW + D + d] += ar * xi[d];
#pragma unroll
        for (int e = d; e < D; ++e) m[t++] += ag * xi[d] * xi[e];
      }
    }
    dg_sum<NS>(m, red);
    double rho, U[D], Ttb, Trb, T;
    const bool ok = dg_temps<D>(m, gp.R, rho, U, Ttb, Trb, T);
    // q_t = sum A (|c|^2 G + H)/2 c and q_r = sum A R c with c = xi - U,
    // expanded in the raw moments
    double q[C::NQ];
    {
      double uu = 0.0, um = 0.0, pu[D];
#pragma unroll
      for (int d = 0; d < D; ++d) {
        uu += U[d] * U[d];
        um += U[d] * m[1 + d];
      }
#pragma unroll
      for (int d = 0; d < D; ++d) {
        pu[d] = 0.0;
#pragma unroll
        for (int e = 0; e < D; ++e) {
          const int a = d < e ? d : e, b = d < e ? e : d;
          pu[d] += U[e] * m[NW + 2 * D + a * D - a * (a - 1) / 2 + (b - a)];
        }
      }
      const double e0 = m[1 + D] - m[2 + D];
#pragma unroll
      for (int d = 0; d < D; ++d) {
        q[d] = m[NW + d] - U[d] * e0 - pu[d] + U[d] * um + 0.5 * uu * (m[1 + d] - U[d] * m[0]);
        q[D + d] = m[NW + D + d] - U[d] * m[2 + D];
      }
    }
    if (threadIdx.x == 0) {
      if (!ok) atomicMin(bad, g.nc + f);
      const double tf = ok ? tau_of(rho, Ttb, vgas) : 1.0;
      if (rf) {
        constexpr int MAXF = Dg<D>::MAXF;
        const size_t so = (size_t)g.f_L[f] * MAXF + g.f_sL[f];
        double un = 0.0, dl2 = 0.0;
        for (int d = 0; d < D; ++d) {
          un += U[d] * n[d];
          dl2 += g.s_dx[so * D + d] * g.s_dx[so * D + d];
        }
        const double RTt = gp.R * Ttb;
        rf[f] = fabs(un) + sqrt(5.0 / 3.0 * RTt) + 2.0 * tf * RTt / sqrt(dl2);
      }
      const double kz = h / (gp.Z * tf);
      const double ER = (m[2 + D] + kz * (rho * gp.R * T)) / (1.0 + kz);
      const double Tr = ER / (rho * gp.R);
      const double Tt = Ttb + (2.0 / 3.0) * (Trb - Tr);
      const double lt = (1.0 - 1.0 / gp.Z) / 3.0 + gp.omega0 / (3.0 * gp.Z);
      const double lr = (1.0 - gp.delta) * ((1.0 - 1.0 / gp.Z) * Tr / Tt + gp.omega1 / gp.Z);
      rec[0] = rho;
      for (int d = 0; d < D; ++d) {
        rec[1 + d] = U[d];
        rec[C::IQT + d] = q[d] / (1.0 + (1.0 - lt) * h / tf);
        rec[C::IQR + d] = q[D + d] / (1.0 + (1.0 - lr) * h / tf);
      }
      rec[C::IT] = Tt;
      rec[C::IR] = Tr;
      rec[C::IDT] = tf / (tf + h);      // blend weights a, b in the dt/tau and E_rot slots
      rec[C::IER] = h / (tf + h);
    }
    __syncthreads();
    double* tabt = lds_d;
    double* tabr = lds_d + D * vg.numax;
    dg_tables<D>(rec, gp.R, vg, tabt, tabr, part, parr);
    const double a = rec[C::IDT], b = rec[C::IER];
    double fl[NW];
    for (int t = 0; t < NW; ++t) fl[t] = 0.0;
    for (int k = threadIdx.x; k < L.n; k += BLOCK) {
      double xi[D], A;
      int u[D];
      leaf_load<D>(L, k, xi, A, u);
      double c[D];
#pragma unroll
      for (int d = 0; d < D; ++d) c[d] = xi[d] - rec[1 + d];
      double Ge, He, Re;
      dg_equilibrium<D>(gp, rec[0], c, rec[C::IT], rec[C::IR], rec + C::IQT, rec + C::IQR, false,
                        maxw<D>(part, tabt, vg.numax, u), maxw<D>(parr, tabr, vg.numax, u), Ge, He, Re);
      const double Gv = a * row0[k] + b * Ge;
      const double Hv = a * row0[fs + k] + b * He;
      const double Rv = a * row0[2 * fs + k] + b * Re;
      row0[k] = Gv;
      row0[fs + k] = Hv;
      row0[2 * fs + k] = Rv;
      dg_mom<D>(fl, A * normal_speed<D>(xi, n), xi, Gv, Hv, Rv);
    }
    dg_sum<NW>(fl, red);
    if (threadIdx.x < NW) F[(size_t)f * NW + threadIdx.x] = fl[threadIdx.x];
    return;
  }
  const int bc = -1 - Rc;
  const bool wall = g.bc_kind[bc] == 0;
  if (rf && threadIdx.x == 0) {
    constexpr int MAXF = Dg<D>::MAXF;
    const int c = g.f_L[f];
    const size_t so = (size_t)c * MAXF + g.f_sL[f];
    double rho, U[D], Tt, Tr, T;
    if (!dg_temps<D>(W + (size_t)c * NW, gp.R, rho, U, Tt, Tr, T)) atomicMin(bad, c);
    double un = 0.0, dn = 0.0;
    for (int d = 0; d < D; ++d) {
      un += U[d] * n[d];
      dn += g.s_d[so * D + d] * n[d];
    }
    const double RTt = gp.R * Tt;
    rf[f] = fabs(un) + sqrt(5.0 / 3.0 * RTt) + 2.0 * tau_of(rho, Tt, vgas) * RTt / (2.0 * dn);
  }
  double sc = 1.0;
  if (wall) {
    double nd[2] = {0.0, 0.0};
    for (int k = threadIdx.x; k < L.n; k += BLOCK) {
      double xi[D], A;
      int u[D];
      leaf_load<D>(L, k, xi, A, u);
      const double s = normal_speed<D>(xi, n);
      if (s > 0.0) nd[0] += A * s * row0[k];
      if (s < 0.0) nd[1] += A * (-s) * row0[k];
    }
    dg_sum<2>(nd, red);
    sc = nd[0] / nd[1];
  }
  double fl[NW];
  for (int t = 0; t < NW; ++t) fl[t] = 0.0;
  for (int k = threadIdx.x; k < L.n; k += BLOCK) {
    double xi[D], A;
    int u[D];
    leaf_load<D>(L, k, xi, A, u);
    const double s = normal_speed<D>(xi, n);
    double Gv = row0[k], Hv = row0[fs + k], Rv = row0[2 * fs + k];
    if (wall && s < 0.0) {
      Gv *= sc;
      Hv *= sc;
      Rv *= sc;
      row0[k] = Gv;
      row0[fs + k] = Hv;
      row0[2 * fs + k] = Rv;
    }
    dg_mom<D>(fl, A * s, xi, Gv, Hv, Rv);
  }
  dg_sum<NW>(fl, red);
  if (threadIdx.x < NW) F[(size_t)f * NW + threadIdx.x] = fl[threadIdx.x];
}

// W* = W - dt/V sum sigma A F; rotational exchange point-implicit with tau
// of W*; target record of W^{n+1} with the heat fluxes q of phi^n.
template <int D>
__global__ void k_dg_macro(Geo g, GasP vgas, DiaGas gp, double dt, const double* __restrict__ F,
                           const double* __restrict__ W, double* __restrict__ Wn, const double* __restrict__ q,
                           double* __restrict__ tp, int* __restrict__ bad) {
  using C = Dg<D>;
  constexpr int MAXF = C::MAXF, NW = C::NW;
  const int i = blockIdx.x * BLOCK + threadIdx.x;
  if (i >= g.nc) return;
  double Fs[NW];
  for (int m = 0; m < NW; ++m) Fs[m] = 0.0;
  for (int s = 0; s < g.nslot[i]; ++s) {
    const int f = g.s_face[i * MAXF + s];
    const double sa = g.s_sigA[i * MAXF + s];
    for (int m = 0; m < NW; ++m) Fs[m] += sa * F[(size_t)f * NW + m];
  }
  double w[NW];
  const double dtv = g.dtv[i];
  for (int m = 0; m < NW; ++m) w[m] = W[(size_t)i * NW + m] - dtv * Fs[m];
  double rho, U[D], Tt, Tr, T;
  if (!dg_temps<D>(w, gp.R, rho, U, Tt, Tr, T)) {
    atomicMin(bad, i);
    rho = 1.0; Tt = Tr = T = 1.0;
  }
  const double tt = tau_of(rho, Tt, vgas);
  const double k = dt / (gp.Z * tt);
  w[2 + D] = (w[2 + D] + k * (rho * gp.R * T)) / (1.0 + k);
  for (int m = 0; m < NW; ++m) Wn[(size_t)i * NW + m] = w[m];
  dg_temps<D>(w, gp.R, rho, U, Tt, Tr, T);
  double* r = tp + (size_t)i * C::NT;
  r[0] = rho;
  for (int d = 0; d < D; ++d) r[1 + d] = U[d];
  r[C::IT] = Tt;
  r[C::IR] = Tr;
  for (int d = 0; d < C::NQ; ++d) r[C::IQT + d] = q[(size_t)i * C::NQ + d];
  r[C::IDT] = dt / tt;
  r[C::IER] = (1.0 - 1.0 / gp.Z) * w[2 + D] + rho * gp.R * T / gp.Z;
  r[C::IT0] = T;
}

// Closure accumulators of one leaf: the base triple's moments, then those
// of the D + 3 directions (1, c, |c|^2) x (g, (3-D) R T g, R T g) at T and
// (0, 0, R T g).
template <int D>
__device__ __forceinline__ void dg_close_acc(double* acc, double A, const double (&xi)[D], const double (&c)[D],
                                             double RT, double gv, double G, double H, double Rr) {
  constexpr int NW = Dg<D>::NW;
  dg_mom<D>(acc, A, xi, G, H, Rr);
  double c2 = 0.0;
#pragma unroll
  for (int d = 0; d < D; ++d) c2 += c[d] * c[d];
  const double hid = 3 - D;
  dg_mom<D>(acc + NW, A, xi, gv, hid * RT * gv, RT * gv);
#pragma unroll
  for (int d = 0; d < D; ++d) dg_mom<D>(acc + NW * (2 + d), A, xi, c[d] * gv, hid * RT * c[d] * gv, RT * c[d] * gv);
  dg_mom<D>(acc + NW * (2 + D), A, xi, c2 * gv, hid * RT * c2 * gv, RT * c2 * gv);
  dg_mom<D>(acc + NW * (3 + D), A, xi, 0.0, 0.0, RT * gv);
}

// Reduce the closure accumulators and solve J lambda = target - M[base].
template <int D>
__device__ __forceinline__ void dg_close_solve(double* acc, double* red, double* Jm, double* bv, double* xv,
                                               const double* target, double* lam_out, int i, int* bad) {
  constexpr int NW = Dg<D>::NW, NA = Dg<D>::NACC;
  for (int g0 = 0; g0 < NA; g0 += 8) {
    double v[8];
    for (int m = 0; m < 8; ++m) v[m] = g0 + m < NA ? acc[g0 + m] : 0.0;
    dg_sum<8>(v, red);
    for (int m = 0; m < 8; ++m)
      if (g0 + m < NA) acc[g0 + m] = v[m];
  }
  if (threadIdx.x == 0) {
    for (int l = 0; l < NW; ++l) {
      for (int e = 0; e < NW; ++e) Jm[l * NW + e] = acc[NW + NW * e + l];
      bv[l] = target[l] - acc[l];
    }
    if (!solve_small<NW>(Jm, bv, xv)) atomicMin(bad, i);
    if (lam_out)
      for (int e = 0; e < NW; ++e) lam_out[e] = xv[e];
  }
  __syncthreads();
}

// Closure coefficients: the Rykov target (or, with init, the translational
// part with zero heat fluxes) plus sum_m lambda_m e_m has the moments
// (rho, rho U, rho E, E_rot target) of W.
template <int D>
__global__ __launch_bounds__(BLOCK) void k_dg_target(Geo g, Leaves L, VGrid vg, DiaGas gp, const double* __restrict__ tp,
                                                    const double* __restrict__ Wt, double* __restrict__ lam, int init,
                                                    int* __restrict__ bad) {
  using C = Dg<D>;
  constexpr int NW = C::NW;
  extern __shared__ double lds_d[];
  __shared__ double red[(BLOCK / 64 + 1) * 8];
  __shared__ double Jm[NW * NW], bv[NW], xv[NW], part[NPAR], parr[NPAR], tg[NW];
  const int i = blockIdx.x;
  const double* r = tp + (size_t)i * C::NT;
  double* tabt = lds_d;
  double* tabr = lds_d + D * vg.numax;
  if (threadIdx.x < NW)
    tg[threadIdx.x] = (threadIdx.x < 2 + D || init) ? Wt[(size_t)i * NW + threadIdx.x] : r[C::IER];
  dg_tables<D>(r, gp.R, vg, tabt, tabr, part, parr);
  const double rho = r[0], Tt = r[C::IT], Tr = r[C::IR], RT = gp.R * r[C::IT0];
  double acc[C::NACC];
  for (int m = 0; m < C::NACC; ++m) acc[m] = 0.0;
  for (int k = threadIdx.x; k < L.n; k += BLOCK) {
    double xi[D], A;
    int u[D];
    leaf_load<D>(L, k, xi, A, u);
    double c[D];
#pragma unroll
    for (int d = 0; d < D; ++d) c[d] = xi[d] - r[1 + d];
    const double gv = maxw<D>(parr, tabr, vg.numax, u);
    double Ge, He, Re;
    dg_equilibrium<D>(gp, rho, c, Tt, Tr, r + C::IQT, r + C::IQR, init != 0, maxw<D>(part, tabt, vg.numax, u), gv,
                      Ge, He, Re);
    dg_close_acc<D>(acc, A, xi, c, RT, gv, Ge, He, Re);
  }
  dg_close_solve<D>(acc, red, Jm, bv, xv, tg, lam + (size_t)i * NW, i, bad);
}

// phi^{n+1} = (phi^n + dt/tau g~ - dt/V sum sigma A xi.n phi_f) / (1 + dt/tau)
// (init = 0), the closed initial state (init = 1), or the right-hand side of
// the implicit micro system scaled by dt/V, dt/tau (g~ - phi^n) - dt/V sum
// sigma A xi.n phi_f (init = 2); heat fluxes of the result about U (not for
// a right-hand side).
template <int D>
__global__ __launch_bounds__(BLOCK) void k_dg_update(Geo g, Leaves L, VGrid vg, DiaGas gp, const double* __restrict__ vin,
                                                    const double* __restrict__ fv, double* __restrict__ vout,
                                                    const double* __restrict__ tp, const double* __restrict__ lam,
                                                    double* __restrict__ q, int init) {
  using C = Dg<D>;
  constexpr int MAXF = C::MAXF, NW = C::NW;
  extern __shared__ double lds_d[];
  __shared__ double red[(BLOCK / 64 + 1) * 8];
  __shared__ double part[NPAR], parr[NPAR];
  const int i = blockIdx.x;
  const double* r = tp + (size_t)i * C::NT;
  double* tabt = lds_d;
  double* tabr = lds_d + D * vg.numax;
  dg_tables<D>(r, gp.R, vg, tabt, tabr, part, parr);
  const double rho = r[0], Tt = r[C::IT], Tr = r[C::IR], dtt = r[C::IDT];
  const double RT = gp.R * r[C::IT0], dtv = g.dtv[i], hid = 3 - D;
  double la[NW];
  for (int e = 0; e < NW; ++e) la[e] = lam[(size_t)i * NW + e];
  const int ns = g.nslot[i];
  const size_t cs = (size_t)g.nc * L.ld, fs = (size_t)g.nf * L.ld;
  double qa[C::NQ];
  for (int t = 0; t < C::NQ; ++t) qa[t] = 0.0;
  for (int k = threadIdx.x; k < L.n; k += BLOCK) {
    double xi[D], A;
    int u[D];
    leaf_load<D>(L, k, xi, A, u);
    double c[D], c2 = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      c[d] = xi[d] - r[1 + d];
      c2 += c[d] * c[d];
    }
    const double gv = maxw<D>(parr, tabr, vg.numax, u);
    double Ge, He, Re;
    dg_equilibrium<D>(gp, rho, c, Tt, Tr, r + C::IQT, r + C::IQR, init == 1, maxw<D>(part, tabt, vg.numax, u), gv,
                      Ge, He, Re);
    double poly = la[0];
#pragma unroll
    for (int d = 0; d < D; ++d) poly += la[1 + d] * c[d];
    poly += la[1 + D] * c2;
    const double tg[3] = {Ge + poly * gv, He + poly * hid * RT * gv, Re + poly * RT * gv + la[2 + D] * RT * gv};
    double nv[3];
    if (init == 1) {
      for (int p = 0; p < 3; ++p) nv[p] = tg[p];
    } else {
      double div[3] = {0, 0, 0};
      for (int s = 0; s < ns; ++s) {
        const int f = g.s_face[i * MAXF + s];
        const double w = g.s_sigA[i * MAXF + s] * normal_speed<D>(xi, g.f_nrm + (size_t)f * D);
        for (int p = 0; p < 3; ++p) div[p] += w * fv[p * fs + (size_t)f * L.ld + k];
      }
      for (int p = 0; p < 3; ++p) {
        const double ph = vin[p * cs + (size_t)i * L.ld + k];
        nv[p] = init == 2 ? dtt * (tg[p] - ph) - dtv * div[p] : (ph + dtt * tg[p] - dtv * div[p]) / (1.0 + dtt);
      }
    }
    for (int p = 0; p < 3; ++p) vout[p * cs + (size_t)i * L.ld + k] = nv[p];
    const double et = A * 0.5 * (c2 * nv[0] + nv[1]), er = A * nv[2];
#pragma unroll
    for (int d = 0; d < D; ++d) {
      qa[d] += et * c[d];
      qa[D + d] += er * c[d];
    }
  }
  if (init == 2) return;   // a residual: the heat fluxes follow the micro sweeps
  dg_sum<C::NQ>(qa, red);
  if (threadIdx.x < C::NQ) q[(size_t)i * C::NQ + threadIdx.x] = qa[threadIdx.x];
}

// Record from W (no exchange, zero heat fluxes): the initial state and the
// heat fluxes after a remap.
template <int D>
__global__ void k_dg_initrec(int nc, DiaGas gp, const double* __restrict__ W, double* __restrict__ tp,
                             int* __restrict__ bad) {
  using C = Dg<D>;
  const int i = blockIdx.x * BLOCK + threadIdx.x;
  if (i >= nc) return;
  double rho, U[D], Tt, Tr, T;
  if (!dg_temps<D>(W + (size_t)i * C::NW, gp.R, rho, U, Tt, Tr, T)) atomicMin(bad, i);
  double* r = tp + (size_t)i * C::NT;
  r[0] = rho;
  for (int d = 0; d < D; ++d) r[1 + d] = U[d];
  r[C::IT] = Tt;
  r[C::IR] = Tr;
  for (int d = 0; d < C::NQ; ++d) r[C::IQT + d] = 0.0;
  r[C::IDT] = 0.0;
  r[C::IER] = W[(size_t)i * C::NW + 2 + D];
  r[C::IT0] = T;
}

// Heat fluxes q_t, q_r of the state about the U of the record tp.
template <int D>
__global__ __launch_bounds__(BLOCK) void k_dg_heat(Geo g, Leaves L, const double* __restrict__ v,
                                                  const double* __restrict__ tp, double* __restrict__ q) {
  using C = Dg<D>;
  __shared__ double red[(BLOCK / 64 + 1) * 8];
  const int i = blockIdx.x;
  const double* r = tp + (size_t)i * C::NT;
  const size_t cs = (size_t)g.nc * L.ld;
  double qa[C::NQ];
  for (int t = 0; t < C::NQ; ++t) qa[t] = 0.0;
  for (int k = threadIdx.x; k < L.n; k += BLOCK) {
    double xi[D], A;
    int u[D];
    leaf_load<D>(L, k, xi, A, u);
    const size_t o = (size_t)i * L.ld + k;
    double c[D], c2 = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      c[d] = xi[d] - r[1 + d];
      c2 += c[d] * c[d];
    }
    const double et = A * 0.5 * (c2 * v[o] + v[cs + o]), er = A * v[2 * cs + o];
#pragma unroll
    for (int d = 0; d < D; ++d) {
      qa[d] += et * c[d];
      qa[D + d] += er * c[d];
    }
  }
  dg_sum<C::NQ>(qa, red);
  if (threadIdx.x < C::NQ) q[(size_t)i * C::NQ + threadIdx.x] = qa[threadIdx.x];
}

// --------------------------------------------- adaptation of the state
// Criterion partials over groups of CRIT_CELLS cells: M1 = A G / rho,
// M2 = A (1/2 (|c|^2 G + H) + R) / (rho E - rho |U|^2/2), max over the group,
// in a fixed operation order (no contraction) so that the flags are
// reproducible bit for bit.
// The first group also takes the nprobe probe states (rho, U, T) with the
// equilibrium triple (g, (3-D) R T g, R T g).  Their criterion constants
// (rho, U and the internal energy from the probe's conserved state, which
// holds 5/2 rho R T) come from the host; the triple is evaluated in the
// oracle's association.  exp and pow are this library's, so probe values of
// M_k agree with the oracle's to rounding, not bit for bit: flags are equal
// away from ties with C1 and C2.
template <int D>
__global__ __launch_bounds__(BLOCK) void k_dg_crit_partial(Leaves L, int nc, const double* __restrict__ vdf,
                                                          const double* __restrict__ W, double* __restrict__ part,
                                                          int nprobe, const double* __restrict__ probe_cc,
                                                          const double* __restrict__ probe_prim, double R) {
#pragma clang fp contract(off)
  constexpr int NW = Dg<D>::NW;
  const int k = blockIdx.x * BLOCK + threadIdx.x;
  const int grp = blockIdx.y;
  if (k >= L.n) return;
  const size_t cs = (size_t)nc * L.ld;
  double xi[D], A;
  int u[D];
  leaf_load<D>(L, k, xi, A, u);
  double m = -INFINITY;
  const int i1 = min(nc, (grp + 1) * CRIT_CELLS);
  for (int i = grp * CRIT_CELLS; i < i1; ++i) {
    const double* w = W + (size_t)i * NW;
    const double rho = w[0];
    double U[D];
    for (int d = 0; d < D; ++d) U[d] = w[1 + d] / rho;
    double ke = U[0] * U[0];
    for (int d = 1; d < D; ++d) ke = ke + U[d] * U[d];
    const double eint = w[1 + D] - 0.5 * rho * ke;
    double c = xi[0] - U[0];
    double c2 = c * c;
    for (int d = 1; d < D; ++d) {
      c = xi[d] - U[d];
      c2 = c2 + c * c;
    }
    const size_t o = (size_t)i * L.ld + k;
    const double G = vdf[o], H = vdf[cs + o], Rr = vdf[2 * cs + o];
    const double M1 = (A * G) / rho;
    const double M2 = (A * (0.5 * (c2 * G + H) + Rr)) / eint;
    m = fmax(m, fmax(M1, M2));
  }
  if (grp == 0) {
    for (int p = 0; p < nprobe; ++p) {
      const double* pr = probe_prim + (size_t)p * (D + 2);
      const double* cc = probe_cc + (size_t)p * (D + 2);
      const double rho = pr[0], T = pr[1 + D];
      // the triple about the probe's own U
      double c = xi[0] - pr[1];
      double cg2 = c * c;
      for (int d = 1; d < D; ++d) {
        c = xi[d] - pr[1 + d];
        cg2 = cg2 + c * c;
      }
      const double G = rho * pow(2.0 * M_PI * R * T, -0.5 * D) * exp(-cg2 / (2.0 * R * T));
      const double H = (double)(3 - D) * R * T * G, Rr = R * T * G;
      // the criterion about U of the conserved state
      c = xi[0] - cc[1];
      double c2 = c * c;
      for (int d = 1; d < D; ++d) {
        c = xi[d] - cc[1 + d];
        c2 = c2 + c * c;
      }
      const double M1 = (A * G) / cc[0];
      const double M2 = (A * (0.5 * (c2 * G + H) + Rr)) / cc[1 + D];
      m = fmax(m, fmax(M1, M2));
    }
  }
  part[(size_t)grp * L.cap + k] = m;
}

// Consanguinity reconstruction of G, H, R onto the new leaves: a kept or
// split leaf copies its source, a merged parent is the balanced pairwise
// mean of its 2^D children.
template <int D>
__global__ __launch_bounds__(BLOCK) void k_dg_gather(int nc, Leaves Lo, Leaves Ln, const int* __restrict__ kind,
                                                    const int* __restrict__ src, const double* __restrict__ vin,
                                                    double* __restrict__ vout) {
#pragma clang fp contract(off)
  const int i = blockIdx.x;
  const size_t cso = (size_t)nc * Lo.ld, csn = (size_t)nc * Ln.ld;
  for (int j = threadIdx.x; j < Ln.n; j += BLOCK) {
    const int k = src[j];
    for (int p = 0; p < 3; ++p) {
      const double* a = vin + p * cso + (size_t)i * Lo.ld + k;
      double v;
      if (kind[j] == 2) {
        v = D == 2 ? ((a[0] + a[1]) + (a[2] + a[3])) * 0.25
                   : (((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]))) * 0.125;
      } else {
        v = a[0];
      }
      vout[p * csn + (size_t)i * Ln.ld + j] = v;
    }
  }
}

// Closure of the state onto W in place: f + sum_m lambda_m e_m with the
// directions of the target's closure at T of W.
template <int D>
__global__ __launch_bounds__(BLOCK) void k_dg_close(Geo g, Leaves L, VGrid vg, DiaGas gp, const double* __restrict__ W,
                                                   double* __restrict__ v, int* __restrict__ bad) {
  using C = Dg<D>;
  constexpr int NW = C::NW;
  extern __shared__ double lds_d[];
  __shared__ double red[(BLOCK / 64 + 1) * 8];
  __shared__ double Jm[NW * NW], bv[NW], xv[NW], part[NPAR], parr[NPAR], rec[C::NT], tg[NW];
  const int i = blockIdx.x;
  if (threadIdx.x == 0) {
    double rho, U[D], Tt, Tr, T;
    if (!dg_temps<D>(W + (size_t)i * NW, gp.R, rho, U, Tt, Tr, T)) atomicMin(bad, i);
    rec[0] = rho;
    for (int d = 0; d < D; ++d) rec[1 + d] = U[d];
    rec[C::IT] = Tt;
    rec[C::IR] = Tr;
    rec[C::IT0] = T;
  }
  if (threadIdx.x < NW) tg[threadIdx.x] = W[(size_t)i * NW + threadIdx.x];
  __syncthreads();
  double* tabt = lds_d;
  double* tabr = lds_d + D * vg.numax;
  dg_tables<D>(rec, gp.R, vg, tabt, tabr, part, parr);
  const double RT = gp.R * rec[C::IT0], hid = 3 - D;
  const size_t cs = (size_t)g.nc * L.ld;
  double acc[C::NACC];
  for (int m = 0; m < C::NACC; ++m) acc[m] = 0.0;
  for (int k = threadIdx.x; k < L.n; k += BLOCK) {
    double xi[D], A;
    int u[D];
    leaf_load<D>(L, k, xi, A, u);
    const size_t o = (size_t)i * L.ld + k;
    double c[D];
#pragma unroll
    for (int d = 0; d < D; ++d) c[d] = xi[d] - rec[1 + d];
    dg_close_acc<D>(acc, A, xi, c, RT, maxw<D>(parr, tabr, vg.numax, u), v[o], v[cs + o], v[2 * cs + o]);
  }
  dg_close_solve<D>(acc, red, Jm, bv, xv, tg, nullptr, i, bad);
  double la[NW];
  for (int e = 0; e < NW; ++e) la[e] = xv[e];
  for (int k = threadIdx.x; k < L.n; k += BLOCK) {
    double xi[D], A;
    int u[D];
    leaf_load<D>(L, k, xi, A, u);
    double c[D], c2 = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      c[d] = xi[d] - rec[1 + d];
      c2 += c[d] * c[d];
    }
    const double gv = maxw<D>(parr, tabr, vg.numax, u);
    double poly = la[0];
#pragma unroll
    for (int d = 0; d < D; ++d) poly += la[1 + d] * c[d];
    poly += la[1 + D] * c2;
    const size_t o = (size_t)i * L.ld + k;
    v[o] = v[o] + poly * gv;
    v[cs + o] = v[cs + o] + poly * hid * RT * gv;
    v[2 * cs + o] = v[2 * cs + o] + (poly * RT * gv + la[2 + D] * RT * gv);
  }
}

// ------------------------------------------------- implicit step (IUGKS)
// out = vin + dphi over the three components (cells as blocks).
__global__ void k_dgi_finish(int nc, Leaves L, const double* __restrict__ vin, const double* __restrict__ dphi,
                             double* __restrict__ out) {
  const int i = blockIdx.x;
  const size_t cs = (size_t)nc * L.ld;
  for (int k = threadIdx.x; k < L.n; k += BLOCK)
    for (int p = 0; p < 3; ++p) {
      const size_t o = p * cs + (size_t)i * L.ld + k;
      out[o] = vin[o] + dphi[o];
    }
}

}  // namespace avs
