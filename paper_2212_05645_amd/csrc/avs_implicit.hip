// Implicit step (IUGKS, Sec. 2.3.1-2.3.2 of arXiv 2212.05645): Roe-type
// macroscopic predictor solved by point-relaxation symmetric Gauss-Seidel
// sweeps (Eqs. equ_delw, delta_Flux, Roe, SGS_w) and the upwind microscopic
// increment solved by symmetric Gauss-Seidel sweeps (Eqs. delta_phi,
// SGS_phi).  Both sweep the cells colour by colour: the cells of one colour
// of a greedy colouring of the face-neighbour graph share no face, so one
// launch updates a whole colour and the result is the sequential
// Gauss-Seidel sweep in colour-major cell order.  Interface VDFs, fluxes,
// the target and the closure are those of the explicit step.
// The predictor is shared with the diatomic gas.
// Part of the library's single translation unit, after avs_kernels.hip.

namespace avs {

// r_ij = |U.n| + a + 2 mu / (rho dl) per face.  Interior
// faces take the interface state of Eq. w_interface (its record: U, RT and
// tau = h a / b with a = tau/(tau+h), b = h/(tau+h); mu/rho = tau R T);
// boundary faces take the cell's W^n and the mirrored distance
// dl = 2 (x_f - x_i) . n.  gamma = 5/3.
template <int D>
__global__ void k_imp_rface(Geo g, GasP gas, double h, const double* __restrict__ W, const double* __restrict__ fpar,
                            double* __restrict__ rf) {
  constexpr int MAXF = Cfg<D>::MAXF;
  const int f = blockIdx.x * BLOCK + threadIdx.x;
  if (f >= g.nf) return;
  const int L = g.f_L[f], R = g.f_R[f], sl = g.f_sL[f];
  const size_t so = (size_t)L * MAXF + sl;
  const double* n = g.f_nrm + (size_t)f * D;
  double un = 0.0, RT, nu_over_dl;
  if (R >= 0) {
    const double* par = fpar + (size_t)f * NPAR;
    for (int d = 0; d < D; ++d) un += par[P_U + d] * n[d];
    RT = par[P_RT];
    const double tf = h * par[P_A] / par[P_B];
    double dl2 = 0.0;
    for (int d = 0; d < D; ++d) dl2 += g.s_dx[so * D + d] * g.s_dx[so * D + d];
    nu_over_dl = tf * RT / sqrt(dl2);
  } else {
    double rho, U[D], T;
    prim_from_W<D>(W + (size_t)L * (D + 2), gas, rho, U, T);
    for (int d = 0; d < D; ++d) un += U[d] * n[d];
    RT = gas.R * T;
    double dn = 0.0;
    for (int d = 0; d < D; ++d) dn += g.s_d[so * D + d] * n[d];
    nu_over_dl = tau_of(rho, T, gas) * RT / (2.0 * dn);
  }
  rf[f] = fabs(un) + sqrt(5.0 / 3.0 * RT) + 2.0 * nu_over_dl;
}

// ---- predictor (Eqs. equ_delw, SGS_w; with ROT the rotational row of Eq.
// SGS_wrot), monatomic W = (rho, rho U, rho E) and diatomic W = (rho, rho U,
// rho E, rho E_rot).  The sweeps are chains of short dependent launches (a
// colour of a 64 x 64 mesh is 32 waves), so what counts is the latency of
// one turn.  Everything a turn needs that does not change during the sweeps
// is therefore formed once per step, in the sweeps' own (colour-major) cell
// order, and the sweeps carry W~ = W + dW with 1/rho and p beside dW: a turn
// is one load of the cell's record, one gather of its neighbours' rows and
// about 110 FP64 instructions with a single division.
template <int D, bool ROT>
struct Pred {
  static constexpr int N = D + 2 + (ROT ? 1 : 0);
  static constexpr int SR = 2 * N + 2;           // state row: W~, 1/rho, p, dW
  static constexpr int MAXF = Cfg<D>::MAXF;
  static constexpr int REC = D + 2 + N;          // per slot: (A/2) n (outward), A/2, (A/2) r, (A/2) G(W_j)
};

// slot types of the sweeps' neighbour table beside a cell index >= 0
constexpr int PRED_NONE = -1, PRED_WALL = -2, PRED_SELF = -3;

// 1/rho and p of a state: p = rho R T (T_t with ROT) = 2/3 of the internal
// translational energy density.
template <int D, bool ROT, int N = Pred<D, ROT>::N>
__device__ __forceinline__ void pred_aux(const double (&w)[N], double& ir, double& p) {
  ir = 1.0 / w[0];
  double mm = 0.0;
#pragma unroll
  for (int d = 0; d < D; ++d) mm += w[1 + d] * w[1 + d];
  p = w[1 + D] - 0.5 * mm * ir;
  if constexpr (ROT) p -= w[2 + D];
  p *= 1.0 / 1.5;
}

// Euler flux (rho U.n, rho U U.n + p n, (rho E + p) U.n[, rho E_rot U.n])
// through hn, a multiple of the normal.
template <int D, bool ROT, int N = Pred<D, ROT>::N>
__device__ __forceinline__ void pred_flux(const double (&w)[N], double ir, double p, const double (&hn)[D],
                                          double (&G)[N]) {
  double mn = 0.0;
#pragma unroll
  for (int d = 0; d < D; ++d) mn += w[1 + d] * hn[d];
  const double un = mn * ir;
  G[0] = mn;
#pragma unroll
  for (int d = 0; d < D; ++d) G[1 + d] = w[1 + d] * un + p * hn[d];
  G[1 + D] = (w[1 + D] + p) * un;
  if constexpr (ROT) G[2 + D] = w[2 + D] * un;
}

// W reflected in a wall of unit normal n (normal momentum reversed; 1/rho
// and p are the cell's own).
template <int N, int D>
__device__ __forceinline__ void mirror_state(const double (&w)[N], const double (&n)[D], double (&o)[N]) {
  double mn = 0.0;
#pragma unroll
  for (int d = 0; d < D; ++d) mn += w[1 + d] * n[d];
#pragma unroll
  for (int m = 0; m < N; ++m) o[m] = w[m];
#pragma unroll
  for (int d = 0; d < D; ++d) o[1 + d] -= 2.0 * mn * n[d];
}

// Records of the sweeps, one thread per cell in colour-major order: slot
// records rec[slot][REC][nc] and neighbours nb[slot][nc], the right-hand side
// rhs[N][nc] = -sum_f sigma A F_f^n, inv[nc] = 1 / (V/dt + 1/2 sum_f A r),
// and the state rows st[nc] by cell index at dW = 0.
template <int D, bool ROT>
__global__ void k_pred_setup(Geo g, const int* __restrict__ cells, const double* __restrict__ F,
                             const double* __restrict__ rf, const double* __restrict__ W, double* __restrict__ rec,
                             int* __restrict__ nb, double* __restrict__ rhs, double* __restrict__ inv,
                             double* __restrict__ st) {
  using C = Pred<D, ROT>;
  constexpr int MAXF = C::MAXF, N = C::N;
  const int t = blockIdx.x * BLOCK + threadIdx.x;
  if (t >= g.nc) return;
  const int i = cells[t];
  const int ns = g.nslot[i];
  const size_t nc = g.nc;
  double acc[N], wi[N], ar = 0.0, iri, pi;
#pragma unroll
  for (int m = 0; m < N; ++m) {
    acc[m] = 0.0;
    wi[m] = W[(size_t)i * N + m];
  }
  pred_aux<D, ROT>(wi, iri, pi);
#pragma unroll
  for (int s = 0; s < MAXF; ++s) {
    int kind = PRED_NONE;
    double hn[D], G0[N], ha = 0.0, ra = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) hn[d] = 0.0;
#pragma unroll
    for (int m = 0; m < N; ++m) G0[m] = 0.0;
    if (s < ns) {
      const int f = g.s_face[i * MAXF + s], j = g.s_nbr[i * MAXF + s];
      const double sa = g.s_sigA[i * MAXF + s], sig = g.s_sig[i * MAXF + s];
      for (int m = 0; m < N; ++m) acc[m] -= sa * F[(size_t)f * N + m];
      ar += (sa * sig) * rf[f];
      const bool wall = j < 0 && g.bc_kind[-1 - g.f_R[f]] == 0;
      if (j >= 0 || wall) {
        kind = wall ? PRED_WALL : (j == i ? PRED_SELF : j);
        ha = 0.5 * (sa * sig);
        ra = ha * rf[f];
        double n[D], w0[N];
#pragma unroll
        for (int d = 0; d < D; ++d) {
          n[d] = sig * g.f_nrm[(size_t)f * D + d];
          hn[d] = ha * n[d];
        }
        double ir = iri, p = pi;
        if (wall) {
          mirror_state<N, D>(wi, n, w0);
        } else {
#pragma unroll
          for (int m = 0; m < N; ++m) w0[m] = W[(size_t)j * N + m];
          pred_aux<D, ROT>(w0, ir, p);
        }
        pred_flux<D, ROT>(w0, ir, p, hn, G0);
      }
    }
    nb[s * nc + t] = kind;
    double* r = rec + (size_t)s * C::REC * nc + t;
#pragma unroll
    for (int d = 0; d < D; ++d) r[d * nc] = hn[d];
    r[D * nc] = ha;
    r[(D + 1) * nc] = ra;
#pragma unroll
    for (int m = 0; m < N; ++m) r[(D + 2 + m) * nc] = G0[m];
  }
#pragma unroll
  for (int m = 0; m < N; ++m) {
    rhs[m * nc + t] = acc[m];
    st[(size_t)i * C::SR + m] = wi[m];
    st[(size_t)i * C::SR + N + 2 + m] = 0.0;
  }
  st[(size_t)i * C::SR + N] = iri;
  st[(size_t)i * C::SR + N + 1] = pi;
  inv[t] = 1.0 / (1.0 / g.dtv[i] + 0.5 * ar);
}

// Workgroups of the sweeps: one wave, so that the few thousand cells of a
// colour spread over as many CUs as there are.
constexpr int PRED_BLOCK = 64;

// One turn of a colour of a PRSGS sweep on Eq. SGS_w: for each cell i of the
// colour, dW_i = (rhs_i - sum_j A/2 [G(W_j + dW_j) - G(W_j)] + sum_j A r/2
// dW_j) / diag_i over interior neighbours j and wall faces (whose outside is
// the mirror of the cell's own W and current dW), with the outward normal
// of i; a far-field face holds the outside increment at zero.  With ROT the
// rotational row gains k = V/(Z tau) on its diagonal and k (rho R T - rho
// E_rot^n) on its right-hand side, tau and rho R T at the cell's current
// iterate (zr = Z, Rg = R).
// reps > 1: the colour's turn comes reps times in a row (a symmetric sweep
// ends and the next begins on the same colour).  No cell of the colour
// reads another one's increment, so the neighbours' part is summed once and
// only what reads the cell's own iterate (a wall's mirror state, a periodic
// cell that is its own neighbour, the rotational source) is iterated; any
// other cell would form the same value again.
// Bound by latency: 2048 cells (a colour of 64 x 64, FP64) 6.9 -> 4.9 us a
// turn against four dependent loads and four divisions per flux, and 121
// instead of 240 turns in 60 sweeps.
template <int D, bool ROT>
__global__ __launch_bounds__(PRED_BLOCK) void k_pred_turn(Geo g, GasP vgas, double zr, double dt,
                                                          const int* __restrict__ cells, int t0, int cnt, int reps,
                                                          const double* __restrict__ W, const double* __restrict__ rec,
                                                          const int* __restrict__ nb, const double* __restrict__ rhs,
                                                          const double* __restrict__ inv, double* __restrict__ st,
                                                          int* __restrict__ bad) {
  using C = Pred<D, ROT>;
  constexpr int MAXF = C::MAXF, N = C::N, SR = C::SR;
  const int l = blockIdx.x * PRED_BLOCK + threadIdx.x;
  if (l >= cnt) return;
  const int t = t0 + l;
  const size_t nc = g.nc;
  const int i = cells[t];
  int j[MAXF];
  double hn[MAXF][D], ra[MAXF], G0[MAXF][N], acc[N], wi[N];
  unsigned own = 0;
#pragma unroll
  for (int s = 0; s < MAXF; ++s) {
    j[s] = nb[s * nc + t];
    const double* r = rec + (size_t)s * C::REC * nc + t;
#pragma unroll
    for (int d = 0; d < D; ++d) hn[s][d] = r[d * nc];
    ra[s] = r[(D + 1) * nc];
#pragma unroll
    for (int m = 0; m < N; ++m) G0[s][m] = r[(D + 2 + m) * nc];
  }
#pragma unroll
  for (int m = 0; m < N; ++m) acc[m] = rhs[m * nc + t];
  const double iv = inv[t];
#pragma unroll
  for (int m = 0; m < N; ++m) wi[m] = W[(size_t)i * N + m];
  double w[MAXF][SR];
#pragma unroll
  for (int s = 0; s < MAXF; ++s) {
    const double* row = st + (size_t)(j[s] >= 0 ? j[s] : i) * SR;
#pragma unroll
    for (int m = 0; m < SR; ++m) w[s][m] = row[m];
  }
#pragma unroll
  for (int s = 0; s < MAXF; ++s) {
    double ws[N], G1[N];
#pragma unroll
    for (int m = 0; m < N; ++m) ws[m] = w[s][m];
    if (j[s] >= 0) {
      pred_flux<D, ROT>(ws, w[s][N], w[s][N + 1], hn[s], G1);
#pragma unroll
      for (int m = 0; m < N; ++m) acc[m] += ra[s] * w[s][N + 2 + m] - (G1[m] - G0[s][m]);
    } else if (j[s] < PRED_NONE) {
      own |= 1u << s;
    }
  }
  double wc[N], dc[N], ir, p;
  if (!ROT && !own) {
#pragma unroll
    for (int m = 0; m < N; ++m) {
      dc[m] = acc[m] * iv;
      wc[m] = wi[m] + dc[m];
    }
    pred_aux<D, ROT>(wc, ir, p);
  } else {
#pragma unroll
    for (int m = 0; m < N; ++m) {
      wc[m] = st[(size_t)i * SR + m];
      dc[m] = st[(size_t)i * SR + N + 2 + m];
    }
    ir = st[(size_t)i * SR + N];
    p = st[(size_t)i * SR + N + 1];
    for (int q = 0; q < reps; ++q) {
      double a[N];
#pragma unroll
      for (int m = 0; m < N; ++m) a[m] = acc[m];
#pragma unroll
      for (int s = 0; s < MAXF; ++s) {
        if (!((own >> s) & 1u)) continue;
        double ws[N], ds[N], h[D], G1[N];
        const double ha = rec[((size_t)s * C::REC + D) * nc + t];
#pragma unroll
        for (int d = 0; d < D; ++d) h[d] = hn[s][d] / ha;
        if (j[s] == PRED_WALL && ha > 0.0) {
          mirror_state<N, D>(wc, h, ws);
          mirror_state<N, D>(dc, h, ds);
        } else {
#pragma unroll
          for (int m = 0; m < N; ++m) { ws[m] = wc[m]; ds[m] = dc[m]; }
        }
        pred_flux<D, ROT>(ws, ir, p, hn[s], G1);
#pragma unroll
        for (int m = 0; m < N; ++m) a[m] += ra[s] * ds[m] - (G1[m] - G0[s][m]);
      }
      double k = 0.0;
      if constexpr (ROT) {
        const double rho = wc[0], Tr = wc[2 + D] / (rho * vgas.R), Tt = p / (rho * vgas.R);
        if (rho > 0.0 && Tt > 0.0 && Tr > 0.0) {
          k = dt / g.dtv[i] / (zr * tau_of(rho, Tt, vgas));
          a[2 + D] += k * (rho * vgas.R * ((3.0 * Tt + 2.0 * Tr) / 5.0) - wi[2 + D]);
        } else {
          atomicMin(bad, i);
        }
      }
#pragma unroll
      for (int m = 0; m < N; ++m) {
        dc[m] = ROT && m == 2 + D ? a[m] / (1.0 / iv + k) : a[m] * iv;
        wc[m] = wi[m] + dc[m];
      }
      pred_aux<D, ROT>(wc, ir, p);
    }
  }
#pragma unroll
  for (int m = 0; m < N; ++m) {
    st[(size_t)i * SR + m] = wc[m];
    st[(size_t)i * SR + N + 2 + m] = dc[m];
  }
  st[(size_t)i * SR + N] = ir;
  st[(size_t)i * SR + N + 1] = p;
}

// Implicit flux of a face, in place over F^n (Eqs. delta_Flux, Roe):
// F_f + 1/2 [G(W~_L) - G(W_L) + G(W~_R) - G(W_R)] + 1/2 r (dW_L - dW_R)
// through the face normal, the outside of a boundary face as in the
// predictor (mirror state at a wall, so that no mass crosses it; increment 0
// at the far field).  The explicit macro update then gives W^{n+1} in flux
// form: exactly conservative after any number of sweeps.
template <int D, bool ROT>
__global__ void k_pred_flux(Geo g, const double* __restrict__ W, const double* __restrict__ st,
                            const double* __restrict__ rf, double* __restrict__ F) {
  using C = Pred<D, ROT>;
  constexpr int N = C::N, SR = C::SR;
  const int f = blockIdx.x * BLOCK + threadIdx.x;
  if (f >= g.nf) return;
  const int L = g.f_L[f], R = g.f_R[f];
  const bool wall = R < 0 && g.bc_kind[-1 - R] == 0;
  double n[D], hn[D], v[N];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    n[d] = g.f_nrm[(size_t)f * D + d];
    hn[d] = 0.5 * n[d];
  }
  const double hr = 0.5 * rf[f];
#pragma unroll
  for (int m = 0; m < N; ++m) v[m] = F[(size_t)f * N + m];
  for (int side = 0; side < 2; ++side) {
    if (side == 1 && R < 0 && !wall) continue;
    const int c = side == 1 && R >= 0 ? R : L;
    double w0[N], w1[N], dw[N], ir0, p0;
#pragma unroll
    for (int m = 0; m < N; ++m) {
      w0[m] = W[(size_t)c * N + m];
      w1[m] = st[(size_t)c * SR + m];
      dw[m] = st[(size_t)c * SR + N + 2 + m];
    }
    pred_aux<D, ROT>(w0, ir0, p0);
    const double ir1 = st[(size_t)c * SR + N], p1 = st[(size_t)c * SR + N + 1];
    if (side == 1 && wall) {
      double t0[N], t1[N], td[N];
      mirror_state<N, D>(w0, n, t0);
      mirror_state<N, D>(w1, n, t1);
      mirror_state<N, D>(dw, n, td);
#pragma unroll
      for (int m = 0; m < N; ++m) { w0[m] = t0[m]; w1[m] = t1[m]; dw[m] = td[m]; }
    }
    // both fluxes by the same expression, so that a zero increment changes
    // nothing bit for bit
    double e1[N], e0[N];
    pred_flux<D, ROT>(w1, ir1, p1, hn, e1);
    pred_flux<D, ROT>(w0, ir0, p0, hn, e0);
    const double sr = side == 0 ? hr : -hr;
#pragma unroll
    for (int m = 0; m < N; ++m) v[m] = v[m] + ((e1[m] - e0[m]) + sr * dw[m]);
  }
#pragma unroll
  for (int m = 0; m < N; ++m) F[(size_t)f * N + m] = v[m];
}

template <int D, typename T>
__global__ __launch_bounds__(BLOCK, (waves_hint<D, T>())) void k_passC_res(Geo g, Leaves L, VGrid vg,
                                                                          const T* __restrict__ vin,
                                                                          const T* __restrict__ fv, T* __restrict__ res,
                                                                          const double* __restrict__ fpar,
                                                                          const double* __restrict__ tpar,
                                                                          const double* __restrict__ lam) {
  d_passC<D, T, true>(g, L, vg, vin, fv, res, fpar, tpar, lam, nullptr, nullptr, blockIdx.x);
}

// x[p][i][k] = 0 for every component and leaf k < n of cell i = block.
template <typename T>
__global__ void k_imp_zero(int P, int nc, Leaves L, T* __restrict__ x) {
  const int i = blockIdx.x;
  const size_t cs = (size_t)nc * L.ld;
  for (int k = threadIdx.x; k < L.n; k += BLOCK)
    for (int p = 0; p < P; ++p) x[p * cs + (size_t)i * L.ld + k] = (T)0;
}

// One colour of a symmetric Gauss-Seidel sweep on Eq. SGS_phi, scaled by
// dt/V: per leaf, dphi_i = (res_i - dt/V sum_{xi.n<0} sigma A xi.n dphi_j)
// / (1 + dt/tau~ + dt/V sum_{xi.n>=0} sigma A xi.n), res the right-hand side
// from pass C.  Boundary faces hold the outside increment at zero.
// P components; dt/tau~ of cell i is tpar[i * tstride + toff].  With out
// (the cell's last visit of the last sweep, when its increment is final),
// also out = vin + dphi; out may be the buffer of res, which only the cell
// itself reads.  reps > 1: the colour's turn comes reps times in a row; only
// a cell that is its own (periodic) neighbour forms another value then.
template <int D, typename T, int P = Cfg<D>::P>
__global__ __launch_bounds__(BLOCK) void k_imp_micro(Geo g, Leaves L, const int* __restrict__ cells,
                                                     const T* res, T* __restrict__ dphi,
                                                     const double* __restrict__ tpar, int tstride, int toff, int reps,
                                                     const T* __restrict__ vin = nullptr, T* out = nullptr) {
  constexpr int MAXF = Cfg<D>::MAXF;
  __shared__ double snrm[MAXF][D];
  __shared__ double ssa[MAXF];
  __shared__ int snbr[MAXF];
  const int i = cells[blockIdx.x];
  const int ns = g.nslot[i];
  if (threadIdx.x < MAXF) {
    const int s = threadIdx.x;
    const int f = s < ns ? g.s_face[i * MAXF + s] : 0;
    snbr[s] = s < ns ? g.s_nbr[i * MAXF + s] : -1;
    ssa[s] = s < ns ? g.s_sigA[i * MAXF + s] : 0.0;
    for (int d = 0; d < D; ++d) snrm[s][d] = g.f_nrm[(size_t)f * D + d];
  }
  __syncthreads();
  const double dtt = tpar[(size_t)i * tstride + toff], dtv = g.dtv[i];
  const size_t cs = (size_t)g.nc * L.ld;
  bool self = false;
  for (int s = 0; s < ns; ++s) self = self || snbr[s] == i;
  const int nrep = self ? reps : 1;
  for (int r = 0; r < nrep; ++r)
  for (int k = threadIdx.x; k < L.n; k += BLOCK) {
    double xi[D], A;
    int u[D];
    leaf_load<D>(L, k, xi, A, u);
    double dg = 1.0 + dtt;
    T off[P];
#pragma unroll
    for (int p = 0; p < P; ++p) off[p] = 0;
    for (int s = 0; s < ns; ++s) {
      const double w = ssa[s] * normal_speed<D>(xi, snrm[s]);
      if (w >= 0.0) {
        dg += dtv * w;
      } else if (snbr[s] >= 0) {
        const size_t o = (size_t)snbr[s] * L.ld + k;
#pragma unroll
        for (int p = 0; p < P; ++p) off[p] += (T)w * dphi[p * cs + o];
      }
    }
    const size_t o = (size_t)i * L.ld + k;
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const T x = (res[p * cs + o] - (T)dtv * off[p]) / (T)dg;
      dphi[p * cs + o] = x;
      if (out && r == nrep - 1) out[p * cs + o] = vin[p * cs + o] + x;
    }
  }
}

// phi^{n+1} = phi^n (no micro sweeps: the increment is zero).
template <typename T>
__global__ void k_imp_copy(int P, int nc, Leaves L, const T* __restrict__ vin, T* __restrict__ out) {
  const int i = blockIdx.x;
  const size_t cs = (size_t)nc * L.ld;
  for (int k = threadIdx.x; k < L.n; k += BLOCK)
    for (int p = 0; p < P; ++p) {
      const size_t o = p * cs + (size_t)i * L.ld + k;
      out[o] = vin[o];
    }
}

}  // namespace avs

namespace avs {

// ------------------------------------------- Rykov diatomic equilibrium
// g^phi = (1 - 1/Z) phi^t + (1/Z) phi^r for phi = G, H, R (Eqs. GHR_equ,
// equ11-equ13) at every leaf, for one state per block: st = (rho, U[D],
// T_t, T_r, q_t[D], q_r[D]).  T = (3 T_t + 2 T_r)/5, p_t = rho R T_t,
// p = rho R T; H carries the 3 - D hidden translational degrees of freedom
// (zero in 3-D).  Out: [3][n][ld] in T.
struct RykovP {
  double R, Z, delta, omega0, omega1;
};

template <int D, typename T>
__global__ __launch_bounds__(BLOCK) void k_rykov_eq(Leaves L, VGrid vg, RykovP gp, int n, const double* __restrict__ states,
                                                   T* __restrict__ out) {
  // the two Maxwellians (at T_t and at T) from separable per-axis tables of
  // the half-finest grid (exact products of one-dimensional factors)
  extern __shared__ double lds_d[];
  double* tabt = lds_d;
  double* tabr = lds_d + D * vg.numax;
  __shared__ double part[NPAR], parr[NPAR];
  const int i = blockIdx.x;
  if (i >= n) return;
  const double* st = states + (size_t)i * (3 + 3 * D);
  const double rho = st[0], Tt = st[1 + D], Tr = st[2 + D];
  double U[D], qt[D], qr[D];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    U[d] = st[1 + d];
    qt[d] = st[3 + D + d];
    qr[d] = st[3 + 2 * D + d];
  }
  const double R = gp.R;
  const double Teq = (3.0 * Tt + 2.0 * Tr) / 5.0;
  const double RTt = R * Tt, RT = R * Teq;
  const double pt = rho * RTt, p = rho * RT;
  if (threadIdx.x == 0) {
    part[P_COEF] = rho * pow(2.0 * M_PI * RTt, -0.5 * D);
    parr[P_COEF] = rho * pow(2.0 * M_PI * RT, -0.5 * D);
    for (int d = 0; d < 3; ++d) {
      part[P_U + d] = d < D ? U[d] : 0.0;
      parr[P_U + d] = d < D ? U[d] : 0.0;
    }
    part[P_I2RT] = 0.5 / RTt;
    parr[P_I2RT] = 0.5 / RT;
  }
  __syncthreads();
  build_tab<D>(tabt, part, vg);
  build_tab<D>(tabr, parr, vg);
  __syncthreads();
  const double wt = 1.0 - 1.0 / gp.Z, wr = 1.0 / gp.Z;
  const double kt = 1.0 / (15.0 * pt * RTt), kr = gp.omega0 / (15.0 * p * RT);
  const double irt_t = 1.0 / RTt, irt = 1.0 / RT;
  const double mt = (1.0 - gp.delta) / (pt * RTt), mr = gp.omega1 * (1.0 - gp.delta) / (p * RT);
  const double RTr = R * Tr;
  const size_t cs = (size_t)n * L.ld;
  for (int k = threadIdx.x; k < L.n; k += BLOCK) {
    double xi[D], A;
    int u[D];
    leaf_load<D>(L, k, xi, A, u);
    double c2 = 0.0, cqt = 0.0, cqr = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const double c = xi[d] - U[d];
      c2 += c * c;
      cqt += c * qt[d];
      cqr += c * qr[d];
    }
    const double gt = maxw<D>(part, tabt, vg.numax, u);
    const double g = maxw<D>(parr, tabr, vg.numax, u);
    const double at = cqt * kt, ar = cqt * kr;
    const double Gt = gt * (1.0 + at * (c2 * irt_t - D - 2));
    const double Gr = g * (1.0 + ar * (c2 * irt - D - 2));
    const double Ht = RTt * gt * (3 - D) * (1.0 + at * (c2 * irt_t - D));
    const double Hr = RT * g * (3 - D) * (1.0 + ar * (c2 * irt - D));
    const double Rt = RTr * (Gt + mt * cqr * gt);
    const double Rr = RT * (Gr + mr * cqr * g);
    const size_t o = (size_t)i * L.ld + k;
    out[o] = (T)(wt * Gt + wr * Gr);
    out[cs + o] = (T)(wt * Ht + wr * Hr);
    out[2 * cs + o] = (T)(wt * Rt + wr * Rr);
  }
}

}  // namespace avs
