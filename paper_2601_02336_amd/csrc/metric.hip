// Per-particle local metric (arXiv:2601.02336, Sec. 5, "Exploitation of
// local geometry"): at the start of an SMC iteration every particle gets its
// own mass matrix, the Hessian of the tempered posterior's negative log
// density at the particle, held fixed during the mutation.  Read here as the
// Gauss-Newton form
//   M = beta F + diag(prior precision),
//   F_kl = <dh/dtheta_k | dh/dtheta_l> = sum_d sum_j w_dj Re(conj(dh_dj/dk) dh_dj/dl),
// which is positive semi-definite by construction and equals the expected
// Hessian of -log L.
//
// No bin loop per particle: with h_dj = P'_d a_j e^{-2 pi i Phi_dj},
// a_j = f_j^-7/6 / u_scale and Phi_dj = sum_a gamma_a g_a(f_j) a combination
// of the phase functions g (constant, the basis rows, f),
//   dh_dj/dk = a_j e^{-2 pi i Phi_dj} (D_dk - 2 pi i P'_d dPhi_dj/dk),
//   D_dk = dP'_d/dk,
// so
//   F_kl = sum_d [ W_d00 Re(conj D_dk D_dl)
//                + 2 pi (s_dk (W_d g_l)_0 + s_dl (W_d g_k)_0)
//                + 4 pi^2 |P'_d|^2 g_kd^T W_d g_ld ],
//   s_dk = Im(conj(D_dk) P'_d),  g_kd[a] = dgamma_a/dtheta_k (detector d),
// with W_d the per-event moments sum_j w_dj a_j^2 g_a(f_j) g_b(f_j) built once
// with the bin tables.  Then, per particle, the lower Cholesky factor of
// M^{-1} that the NUTS kernel takes.
#include "coeffs.h"
#include "common.h"
#include "context.h"

namespace smcgw {

// Four particles per wavefront, 16 lanes each: a lane is a tangent or a detector in
// the prologue, a row of W_d, a column of F and a row of the factor in turn.  Nothing
// crosses the groups and a workgroup is one wavefront, so there are no barriers, and
// the matrices stay in registers but for the column that a step of the factorisation
// broadcasts.  What bounds it is the chain of one particle (29000 cycles: prologue 9800,
// F 9400, factor 3300, inverse 2300, the rest loads and stores), so particles in flight
// are what counts: eight workgroups fit a compute unit, 32 particles, where a workgroup of
// two wavefronts for each held 12 and spent most instructions on a few lanes.  Event of
// 3 x 8033 bins, 11 parameters, 6144 particles: 71.5 -> 20 us a call, 64: 21.2 -> 14.3
// (of which 9 are the call).  Every entry is rounded as it was there.
constexpr int SUB_LANES = 16;
constexpr int MET_SUBS = 64 / SUB_LANES;
static_assert(SUB_LANES == MAXDIM && NPAR <= SUB_LANES && NGEO <= SUB_LANES && 2 * MAXDET < SUB_LANES, "lane roles");

struct PrecDesc {
    double prec[MAXDIM];   // prior precision of each sampled coordinate
};

// What F is formed from.
struct MetricInput {
    double th[NPAR], cb[CB_SIZE];
    double wg[NPAR][NGEO];   // W_d gamma_k of the current detector
    double dr[NPAR], di[NPAR], s[NPAR];
    ExtAngles ang;
};

struct MetricState {
    union {
        MetricInput in;
        double Rt[MAXDIM][MAXDIM];   // the factor's columns
    };
    union {
        double F[MAXDIM][MAXDIM];
        double out[MAXDIM * MAXDIM];
    };
    double diag[MAXDIM];
};

// Groups start 16 of the 64 banks apart: each reads its own copy of an entry.
struct MetricSub : MetricState {
    double pad[8 + (256 - (sizeof(MetricState) + 64) % 256 + 64) % 256 / 8];
};
static_assert(sizeof(MetricSub) % 256 == 64, "bank offset of the groups");

// M = beta F + diag(prior precision) over the sampled coordinates (coordinate a of
// the sample being row idx[a] of F), then the lower Cholesky factor of M^{-1} into
// chol[p], or the fallback where M or the factor is not numerically positive definite.
// The factor comes from the order-reversed matrix: with J the reversal permutation and
// J M J = R R^T, M^{-1} = (J R^-T J)(J R^-T J)^T and J R^-T J is lower triangular with
// a positive diagonal, so it is that factor; it needs one Cholesky and one triangular
// inverse.  Lane i holds row i of J M J, then column i of R^{-1}.  An entry takes its
// products with the finished columns in column order, as in the textbook's row-by-row
// form (see cholesky_rows).
// N >= D rows and columns are factored: those beyond D are the identity's, so the steps
// need no branches and the reads of the next ones are under way early.  own: coordinate
// D-1-lane's row of F, prec: its prior precision.
template <int N>
__device__ __forceinline__ void finish_metric(MetricSub& S, const int* idx, int D, double beta, int own, double prec,
                                              const double* __restrict__ fallback, double* __restrict__ chol,
                                              double* __restrict__ fisher, int32_t* __restrict__ status, int p,
                                              int lane) {
    if (fisher)
        for (int i = lane; i < D * D; i += SUB_LANES) fisher[(size_t)p * D * D + i] = S.F[idx[i / D]][idx[i % D]];
    double A[N];   // row `lane`
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const double f = S.F[own][idx[max(D - 1 - j, 0)]];
        const double v = fma(beta, f, j == lane ? prec : 0.0);
        A[j] = j < D && lane < D ? v : j == lane ? 1.0 : 0.0;
    }
    bool ok = cholesky_rows(A, S.Rt, S.diag, lane);
    // X = R^{-1}, lane c column c by forward substitution
    double X[N];
#pragma unroll
    for (int r = 0; r < N; ++r) X[r] = r == lane ? 1.0 : 0.0;
    bool finite = true;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        X[k] = k < lane ? 0.0 : X[k] / S.Rt[k][k];
        finite = finite && isfinite(X[k]);
#pragma unroll
        for (int r = k + 1; r < N; ++r) X[r] = fma(-S.Rt[k][r], X[k], X[r]);
    }
    // a non-finite entry takes the fallback too
    const unsigned long long bad = __ballot(lane < D && !finite);
    ok = ok && !(bad >> (threadIdx.x & ~(SUB_LANES - 1)) & ((1ull << SUB_LANES) - 1));
    if (status && lane == 0) status[p] = ok ? 0 : 1;
    // factor L[i][j] = X[D-1-j][D-1-i]: lane c holds row D-1-c
    if (lane < D) {
#pragma unroll
        for (int r = 0; r < N; ++r)
            if (r < D) S.out[(D - 1 - lane) * D + D - 1 - r] = X[r];
    }
    wave_lds_fence();
    double* o = chol + (size_t)p * D * D;
    if (ok) {
#pragma unroll
        for (int i = 0; i < N * N; i += SUB_LANES)
            if (i + lane < D * D) o[i + lane] = S.out[i + lane];
    } else {
        for (int i = lane; i < D * D; i += SUB_LANES) o[i] = fallback ? fallback[i] : (i / D == i % D ? 1.0 : 0.0);
    }
}

// The coefficient block is built as in the NUTS leaf: the intrinsic part with one
// tangent per lane, shared sin / cos in parallel lanes, then one detector and tangent
// per lane.
__global__ __launch_bounds__(64) void local_metric_kernel(const DevEvent* __restrict__ evs, int n_events,
                                                          const int32_t* __restrict__ ev_of_p, ParamMap pm,
                                                          PrecDesc pd, int P, const double* __restrict__ theta,
                                                          double beta_host, const double* __restrict__ beta_dev,
                                                          const double* __restrict__ fallback,
                                                          double* __restrict__ chol, double* __restrict__ fisher,
                                                          int32_t* __restrict__ status,
                                                          const double* __restrict__ st, int run_size) {
    __shared__ MetricSub sub[MET_SUBS];
    const int lane = threadIdx.x % SUB_LANES;
    MetricSub& S = sub[threadIdx.x / SUB_LANES];
    const int p = blockIdx.x * MET_SUBS + threadIdx.x / SUB_LANES;
    const int D = pm.dim;
    if (p >= P) return;
    // independent runs: particle p belongs to run p / run_size, whose state gives beta; a finished run is skipped
    const int run = st ? p / run_size : 0;
    if (st && st[(size_t)run * SMCGW_STATE_SIZE + SMCGW_ST_DONE] != 0.0) return;
    if (st && fallback) fallback += (size_t)run * D * D;
    const DevEvent& ev = evs[event_index(ev_of_p, p, n_events)];
    const int n_det = ev.n_det;
    const double* wmom = ev.wmom;
    MetricInput& in = S.in;
    // coordinate D-1-lane, as the factorisation orders them (read here, ahead of its use)
    const int own = lane < D ? pm.idx[D - 1 - lane] : 0;
    const double prec = lane < D ? pd.prec[D - 1 - lane] : 0.0;

    int from = -1;   // the coordinate that sets parameter `lane` (the last one that names it)
    for (int k = 0; k < D; ++k) from = pm.idx[k] == lane ? k : from;
    const double x = theta[(size_t)p * D + min(lane, D - 1)], xp = __shfl(x, max(from, 0), SUB_LANES);
    if (lane < NPAR) in.th[lane] = from >= 0 ? xp : pm.fixed[lane];
    wave_lds_fence();
    if (lane < 4) prep_intrinsic_n<1>(ev, in.th, in.cb, lane, lane == 0);
    if (lane < ANG_COUNT) {
        double sn, cs;
        sincos(extrinsic_angle(ev, in.th, lane), &sn, &cs);
        in.ang.sc[lane][0] = sn;
        in.ang.sc[lane][1] = cs;
    }
    wave_lds_fence();
    if (lane < 2 * MAXDET) {
        const ExtAngles ang = in.ang;
        const int k = lane / MAXDET;
        prep_extrinsic_det_n<1>(ev, in.th, ang, in.cb, lane - k * MAXDET, k, k == 0);
    } else if (lane == 2 * MAXDET) {
        prep_extrinsic_common(ev, in.th, in.cb);
    }
    wave_lds_fence();
    const double* cb = in.cb;
    const double amp = cb[CB_AMP];

    // gamma_a derives the phase c_0 + sum_b c_{1+b} B_b(f) + f tau_d, with c_0 containing
    // -phi_c / (2 pi) and tau_d = t_c + delay_d(ra, dec), so it is sparse: the coefficients' derivatives for the four intrinsic
    // parameters, one entry for ra, dec, t_c (of f) and phi_c (constant), none for d_L, iota and psi.
    // Lane a takes row a of W, then lane l the column F_kl, k <= l.  The coefficients' derivatives are read from
    // LDS both times: held in registers a call is 1 us shorter, but a wavefront's 224 registers then wait for two
    // of another stream's NUTS workgroups to leave a SIMD instead of one (2.2 ms a launch there against 1.1).
    const int la = min(lane, NGEO - 1), l = min(lane, NPAR - 1);
    double acc[NPAR], wnext[NGEO];   // the next detector's row is under way
#pragma unroll
    for (int k = 0; k < NPAR; ++k) acc[k] = 0.0;
#pragma unroll
    for (int b = 0; b < NGEO; ++b) wnext[b] = wmom[la * NGEO + b];
#pragma unroll 1
    for (int d = 0; d < n_det; ++d) {
        double w[NGEO];
#pragma unroll
        for (int b = 0; b < NGEO; ++b) {
            w[b] = wnext[b];
            wnext[b] = wmom[(min(d + 1, n_det - 1) * NGEO + la) * NGEO + b];
        }
        const double W0 = __shfl(w[0], 0, SUB_LANES);
        const double qr = amp * cb[CB_PR + d], qi = amp * cb[CB_PI + d];
        const double tra = cb[CB_DTAU + 2 * d], tdec = cb[CB_DTAU + 2 * d + 1];
        constexpr double GPHIC = -1.0 / TWO_PI;
        double gk[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int b = 0; b < NCOEF; ++b)
#pragma unroll
            for (int k = 0; k < 4; ++k) gk[k] = fma(w[b], cb[CB_DC + 4 * b + k], gk[k]);
        if (lane < NGEO) {
#pragma unroll
            for (int k = 0; k < 4; ++k) in.wg[k][lane] = gk[k];
            in.wg[P_DL][lane] = 0.0;
            in.wg[P_IOTA][lane] = 0.0;
            in.wg[P_PSI][lane] = 0.0;
            in.wg[P_RA][lane] = w[NGEO - 1] * tra;
            in.wg[P_DEC][lane] = w[NGEO - 1] * tdec;
            in.wg[P_TC][lane] = w[NGEO - 1];
            in.wg[P_PHIC][lane] = w[0] * GPHIC;
        }
        {
            const bool cam = lane == P_MC || lane == P_DL, proj = lane >= P_IOTA && lane <= P_DEC;
            const double g = cb[lane == P_MC ? CB_DLNCA_MC : CB_DLNCA_DL];
            const int m = proj ? lane - P_IOTA : 0;
            const double xr = cam ? g * qr : proj ? amp * cb[CB_DPR + 4 * d + m] : 0.0;
            const double xi = cam ? g * qi : proj ? amp * cb[CB_DPI + 4 * d + m] : 0.0;
            if (lane < NPAR) {
                in.dr[lane] = xr;
                in.di[lane] = xi;
                in.s[lane] = xr * qi - xi * qr;
            }
        }
        wave_lds_fence();
        double wl[NGEO];
#pragma unroll
        for (int b = 0; b < NGEO; ++b) wl[b] = in.wg[l][b];
        const double drl = in.dr[l], dil = in.di[l], sl = in.s[l];
#pragma unroll
        for (int k = 0; k < NPAR; ++k) {
            double gwg = 0.0;
            if (k < 4) {
#pragma unroll
                for (int b = 0; b < NCOEF; ++b) gwg = fma(cb[CB_DC + 4 * b + k], wl[b], gwg);
            } else if (k == P_RA || k == P_DEC || k == P_TC) {
                gwg = (k == P_RA ? tra : k == P_DEC ? tdec : 1.0) * wl[NGEO - 1];
            } else if (k == P_PHIC) {
                gwg = GPHIC * wl[0];
            }
            const double wgl0 = wl[0], wgk0 = in.wg[k][0], drk = in.dr[k], dik = in.di[k], sk = in.s[k];
            acc[k] += W0 * (drk * drl + dik * dil)
                    + TWO_PI * fma(sk, wgl0, sl * wgk0)
                    + (4.0 * PI * PI) * (qr * qr + qi * qi) * gwg;
        }
        wave_lds_fence();
    }
#pragma unroll
    for (int k = 0; k < NPAR; ++k)
        if (k <= lane && lane < NPAR) {
            S.F[k][lane] = acc[k];
            S.F[lane][k] = acc[k];
        }
    wave_lds_fence();

    const double beta = st ? st[(size_t)run * SMCGW_STATE_SIZE + SMCGW_ST_BETA] : beta_dev ? *beta_dev : beta_host;
    finish_metric<NPAR>(S, pm.idx, D, beta, own, prec, fallback, chol, fisher, status, p, lane);
}

// The analytic test likelihoods take the exact Hessian of -log L as F: the
// identity (standard normal), diag(1 / sigma_l^2) (Gaussian likelihood), and
// for the unweighted sum of two isotropic Gaussians N(m1, s^2) + N(m2, s^2)
//   F = I / s^2 - r1 r2 (m1 - m2)(m1 - m2)^T / s^4,
// r_i the components' shares at the particle (the shares' mean of the
// components' Hessians less the shares' covariance of their gradients).
// Near a mode F is positive definite; across the saddle between the modes it
// is not, and the particle takes the fallback.
__global__ __launch_bounds__(64) void analytic_metric_kernel(TargetDesc tg, PrecDesc pd, int P,
                                                             const double* __restrict__ theta,
                                                             double beta_host, const double* __restrict__ beta_dev,
                                                             const double* __restrict__ fallback,
                                                             double* __restrict__ chol, double* __restrict__ fisher,
                                                             int32_t* __restrict__ status,
                                                             const double* __restrict__ st, int run_size) {
    __shared__ MetricSub sub[MET_SUBS];
    __shared__ int idx[MAXDIM];
    const int lane = threadIdx.x % SUB_LANES;
    MetricSub& S = sub[threadIdx.x / SUB_LANES];
    const int p = blockIdx.x * MET_SUBS + threadIdx.x / SUB_LANES;
    const int D = tg.dim;
    idx[lane] = lane;   // the same from every group
    if (p >= P) return;
    const int run = st ? p / run_size : 0;
    if (st && st[(size_t)run * SMCGW_STATE_SIZE + SMCGW_ST_DONE] != 0.0) return;
    if (st && fallback) fallback += (size_t)run * D * D;
    for (int e = lane; e < D * D; e += SUB_LANES) {
        const int k = e / D, l = e % D;
        double f = 0.0;
        if (tg.kind == SMCGW_TARGET_GAUSS) {
            f = k == l ? 1.0 : 0.0;
        } else if (tg.kind == SMCGW_TARGET_GAUSS_X_GAUSS) {
            const double sl = tg.params[D + k];
            f = k == l ? 1.0 / (sl * sl) : 0.0;
        } else {
            const double* x = theta + (size_t)p * D;
            const double* m1 = tg.params;
            const double* m2 = tg.params + D;
            const double sg = tg.params[2 * D], s2g = sg * sg;
            double s1 = 0.0, s2 = 0.0;
            for (int j = 0; j < D; ++j) {
                s1 += (x[j] - m1[j]) * (x[j] - m1[j]);
                s2 += (x[j] - m2[j]) * (x[j] - m2[j]);
            }
            const double r1 = 1.0 / (1.0 + exp(-0.5 * (s2 - s1) / s2g)), r2 = 1.0 - r1;
            f = (k == l ? 1.0 / s2g : 0.0) - r1 * r2 * (m1[k] - m2[k]) * (m1[l] - m2[l]) / (s2g * s2g);
        }
        S.F[k][l] = f;
    }
    wave_lds_fence();
    const double beta = st ? st[(size_t)run * SMCGW_STATE_SIZE + SMCGW_ST_BETA] : beta_dev ? *beta_dev : beta_host;
    const int own = max(D - 1 - lane, 0);
    finish_metric<MAXDIM>(S, idx, D, beta, own, pd.prec[own], fallback, chol, fisher, status, p, lane);
}

// Prior precision of each sampled coordinate: 12 / (hi - lo)^2 (uniform),
// the inverse variance of the log-uniform density, 1 / sigma^2 (Gaussian),
// 0 (flat).
static PrecDesc prior_precision(const PriorDesc& pr) {
    PrecDesc pd;
    for (int k = 0; k < MAXDIM; ++k) {
        double v = 0.0;
        if (k < pr.dim) {
            const double lo = pr.lo[k], hi = pr.hi[k];
            if (pr.kind[k] == SMCGW_PRIOR_UNIFORM) {
                v = 12.0 / ((hi - lo) * (hi - lo));
            } else if (pr.kind[k] == SMCGW_PRIOR_LOGUNIFORM) {
                const double lr = std::log(hi / lo);
                const double m1 = (hi - lo) / lr, m2 = (hi * hi - lo * lo) / (2.0 * lr);
                v = 1.0 / (m2 - m1 * m1);
            } else if (pr.kind[k] == SMCGW_PRIOR_GAUSSIAN) {
                v = 1.0 / (hi * hi);
            }
        }
        pd.prec[k] = v;
    }
    return pd;
}

}  // namespace smcgw

namespace smcgw {
// Local metric of n_runs * run_size particles at their runs' temperatures
// (state st), the run's own population factor as the fallback.
static int metric_target_ok(smcgw_ctx* c, int D) {
    if (!c->prior_set) return SMCGW_ERR_NOT_INIT;
    if (c->target.kind == SMCGW_TARGET_GW) {
        if (c->events.empty()) return SMCGW_ERR_NOT_INIT;
        return c->prior.dim == D && c->pmap.dim == D ? SMCGW_OK : SMCGW_ERR_INVALID;
    }
    if (c->target.dim <= 0) return SMCGW_ERR_NOT_INIT;
    return c->prior.dim == D && c->target.dim == D ? SMCGW_OK : SMCGW_ERR_INVALID;
}

static int launch_metric(smcgw_ctx* c, int P, const double* theta, double beta, const double* beta_dev,
                         const double* fallback, double* chol, double* fisher, int32_t* status, const double* st,
                         int run_size) {
    const PrecDesc pd = prior_precision(c->prior);
    TimedLaunch tl(c, SMCGW_KERNEL_METRIC);
    if (c->target.kind == SMCGW_TARGET_GW)
        hipLaunchKernelGGL(local_metric_kernel, dim3((P + MET_SUBS - 1) / MET_SUBS), dim3(64), 0, c->stream, c->d_events,
                           (int)c->events.size(), c->ev_of_p, c->pmap, pd, P, theta, beta, beta_dev, fallback, chol,
                           fisher, status, st, run_size);
    else
        hipLaunchKernelGGL(analytic_metric_kernel, dim3((P + MET_SUBS - 1) / MET_SUBS), dim3(64), 0, c->stream, c->target, pd, P, theta,
                           beta, beta_dev, fallback, chol, fisher, status, st, run_size);
    return hipGetLastError() == hipSuccess ? SMCGW_OK : SMCGW_ERR_HIP;
}

int queue_local_metric(smcgw_ctx* c, int P, int D, const double* theta, const double* st, int run_size,
                       const double* fallback_runs, double* chol, int32_t* status) {
    const int rc = metric_target_ok(c, D);
    if (rc) return rc;
    return launch_metric(c, P, theta, 0.0, nullptr, fallback_runs, chol, nullptr, status, st, run_size);
}
}  // namespace smcgw

using namespace smcgw;

extern "C" int smcgw_local_metric(smcgw_ctx* c, int P, int D, const double* theta, double beta,
                                  const double* beta_device, const double* fallback_chol, double* chol, double* fisher,
                                  int32_t* status) {
    if (!c || P < 0 || D <= 0 || D > MAXDIM || (!beta_device && !(beta >= 0.0 && beta <= 1.0)) ||
        (P > 0 && (!theta || !chol)))
        return SMCGW_ERR_INVALID;
    const int rc = metric_target_ok(c, D);
    if (rc) return rc;
    if (P == 0) return SMCGW_OK;
    if (hipSetDevice(c->device) != hipSuccess) return SMCGW_ERR_HIP;
    return launch_metric(c, P, theta, beta, beta_device, fallback_chol, chol, fisher, status, nullptr, P);
}
