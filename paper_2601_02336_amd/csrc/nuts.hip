// Persistent No-U-Turn kernel (arXiv:2601.02336, Sec. 4 and Sec. 5).
//
// One NUTS transition per particle: momentum r ~ N(0, M) with M^{-1} = L L^T,
// Hamiltonian H = -log p_t(x) + r^T M^{-1} r / 2 with p_t ~ L^beta pi (Sec. 3,
// Eq. 3), leapfrog steps (Eqs. 11-13) mapped back into the prior box by the
// reflective / periodic boundaries of Sec. 5, trajectory doubling in a random
// direction until the generalised U-turn criterion fires or the depth limit
// is reached (Hoffman & Gelman 2014; multinomial variant of Betancourt 2017,
// App. A): uniform progressive sampling inside each new subtree, biased
// progressive sampling when it is merged, divergence when H - H0 exceeds a
// threshold.
//
// Execution: a workgroup advances one particle's tree, or with a short event four
// particles' trees together, a leaf each per round; a particle's place takes the next one
// from an atomic queue when its transition ends.  A particle's blocks of bins are dealt
// out in WAVES residue classes, class r to one wavefront; wavefront 0 forms the epilogue
// and moves the tree (advance), the prologue of the next leaf is spread over the
// wavefronts while wavefront 0 books the last one.  The tree logic keeps one coordinate
// per lane, so four particles share its instructions, 16 lanes each.
//
// What bounds a leaf: on a full grid of 3 x 8033 bins the bin loop, 15000 of 23400
// cycles of one tree alone (advance 2500, prologue and book-keeping 4300, epilogue 1800;
// 10.6 us a leaf before the reads of each were put in flight together, the branches on
// single values taken out and the logarithms and divisions of the auxiliary wavefront
// merged, 10.3 us after), and with three trees on each compute unit the arithmetic of the
// bins again (45 to 47 M leaves/s of the 51 to 54 M evaluations/s of the batched likelihood).  On a
// folded event of ~310 edges the serial parts are nine tenths of a leaf's instructions:
// four particles to a workgroup share them (300 M leaves/s against 130 M with one).
// Random numbers come from Philox4x32-10 with counter (index, particle,
// iteration, purpose), so every decision can be replayed.
#include <algorithm>
#include <cstring>
#include <vector>

#include "binloop.h"
#include "coeffs.h"
#include "common.h"
#include "context.h"
#include "philox.h"

namespace smcgw {

struct NutsArgs {
    int P, D;
    double* theta;
    double* logl;
    double* grad;
    const double* chol;
    double step, beta, max_dh;
    int max_depth, uturn;
    uint64_t seed, iteration;
    const int32_t* md_per_p;
    int32_t* depth_out;
    int32_t* nlf_out;
    uint8_t* div_out;
    double* acc_out;
    const DevEvent* events;
    int n_events;
    const int32_t* ev_of_p;
    int* queue;
    const int32_t* order;   // start order of the particles (NULL: index order)
    int priority;           // raise wavefront priority with the tree depth
    int chol_pp;            // chol holds one [D][D] factor per particle
    const double* beta_dev; // beta from device memory (NULL: the value above)
    const double* state;    // independent runs' states (NULL: one run with the values above)
    int run_size;           // particles per run when state is set
    int stripe;             // neighbouring particles that go to one queue
};

// Wavefronts per SIMD the register budget is sized for (4: 128 VGPRs, 3: 168,
// 2: 256).
constexpr int NUTS_WAVES_PER_SIMD = 3;
constexpr int MAXD1 = SMCGW_MAX_DEPTH + 1;

// Per-detector terms of a leaf's epilogue (see leaf_finish).
enum { FD_LL = 0, FD_DLN, FD_GP, FD_T = FD_GP + 4, FD_RA, FD_DEC, FD_SIZE };

// Particles that a packed workgroup advances together, and the lanes of each: one per
// coordinate.  LDS holds twelve particles' states per compute unit, three workgroups of four.
constexpr int PACKED = 4;
constexpr int SUB_LANES = MAXDIM;
static_assert(PACKED * SUB_LANES == 64, "the particles of a workgroup share a wavefront");

// Rows of M^{-1} are this many doubles apart: the coordinate lanes read their rows
// 16 bytes at a time from different banks.
constexpr int MINV_STRIDE = MAXDIM + 2;

// Tree state of one particle's transition (LDS).
//
// Leaf pipeline: once the likelihood of leaf k is known, `advance` completes
// its momentum and moves to leaf k+1 on the assumption that the tree goes on
// (the position of the next leaf does not depend on the multinomial sampling
// or the U-turn checks).  `bookkeep` then takes those decisions for leaf k on
// wavefront 0 while the other wavefronts already run leaf k+1's prologue; if
// the tree stops, that prologue is discarded.  Every quantity is the one the
// plain sequential algorithm computes.
struct NutsState {
    double x[MAXDIM], r[MAXDIM];                         // the leaf in flight: position, half-step momentum
    double rho[MAXDIM], srho[MAXDIM];                    // momentum sums of the tree / subtree
    double gl_new[MAXDIM];                               // likelihood gradient of the leaf in flight
    double rec[4][MAXDIM];                               // finished leaf: x, r, g (grad log p_t), gl
    double pgp[MAXDIM];                                  // prior gradient at the leaf in flight
    double plp;                                          // log prior at the leaf in flight
    double ul[2][2];                                     // log u and log(1 - u) of the leaf uniforms, by leaf index parity
    double dtab_u[MAXD1];                                // log of the merge uniform of each doubling
    int dtab_dir[MAXD1];                                 // direction of each doubling
    double h0, logw, sub_logw, uacc, acc_sum, eps, prop_ll, sprop_ll, ll_new, rec_ll, rec_lp;
    int first, stop, j, n, nleaves, depth, nlf, div, dir, md, inflight;
    uint32_t leafc;
    // the particle's run: temperature, Philox key and iteration, particle index within the run
    double beta;
    uint64_t seed, iter;
    uint32_t pid;
};

// One particle of the workgroup.
struct NutsSubState {
    double Minv[MAXDIM * MINV_STRIDE];
    union {
        double L[MAXDIM * MAXDIM];               // the factor, until the transition has started
        struct {
            double ck_rho[MAXD1][MAXDIM], ck_v[MAXD1][MAXDIM];   // U-turn checkpoints: prefix sum, first velocity
        };
    };
    double vec[MAXDIM], red[2][MAXDIM];          // cross-lane exchange of wavefront 0
    double pred[MAXDIM];                         // cross-lane exchange of the auxiliary wavefront
    ExtAngles ang;                               // extrinsic transcendentals of the leaf in flight
    double cb[CB_SIZE];
    double mom[MOM_SIZE];                        // moments of the leaf
    double fin_det[MAXDET][FD_SIZE];             // epilogue terms of the leaf
    double th[NPAR];
    double left[5][MAXDIM], right[5][MAXDIM];    // x, r, g (grad log p_t), gl (grad logL), v = M^{-1} r
    double prop[2][MAXDIM], sprop[2][MAXDIM];    // x, gl
    double end_ll[2], end_lp[2];                 // logL, log p_t of left / right
    NutsState T;
    DevEvent ev;                                 // event of the particle
    int p;                                       // particle (-1: none)
    int e;                                       // event whose descriptor ev holds
    int run;                                     // run whose factor Minv holds (per-run factors)
};
static_assert(sizeof(DevEvent) % 8 == 0, "the event descriptor is copied in 8-byte words");

// The particles' states start 16 of the 64 banks apart: a broadcast read of each
// particle's own entry then takes no bank twice.
struct NutsSub : NutsSubState {
    double pad[8 + (256 - (sizeof(NutsSubState) + 64) % 256 + 64) % 256 / 8];
};
static_assert(sizeof(NutsSub) % 256 == 64, "bank offset of the particles' states");

// What the particles of a workgroup share.
struct NutsShared {
    double plo[MAXDIM], phi[MAXDIM];             // prior / boundary description
    double pnorm[MAXDIM];                        // log normalising constant of each coordinate's prior
    int pbnd[MAXDIM], pkind[MAXDIM];
    int pidx[MAXDIM];                            // sampled coordinate -> source parameter
    double pfixed[NPAR];
    // Wavefront 0's word on the places to the others: bit 16 s, place s's particle has a leaf to evaluate (after its
    // advance); and, after the bookkeeping, the places that go on (bits 0..), those whose transition has ended
    // (bits 8..) and the deepest doubling under way (bits 16..).
    unsigned long long evals;
    unsigned places;
    NutsArgs A;                                  // the arguments as the out-of-line tree steps read them
};

// The workgroup's LDS, for N particles (SUBS, or one in the lockstep sweeps) and
// the likelihood's wavefronts.  The out-of-line steps name it themselves: an
// address passed to them would be a generic one, slower to read through.
template <int N>
__device__ __forceinline__ NutsSub* lds_subs() {
    __shared__ NutsSub sub[N];
    return sub;
}

template <int N>
__device__ __forceinline__ NutsShared& lds_shared() {
    __shared__ NutsShared S;
    return S;
}

template <int N, int WAVES>
__device__ __forceinline__ double (*lds_moments(int g))[MOM_SIZE] {
    __shared__ double m[N][WAVES][MOM_SIZE];
    return m[g];
}

enum { CMD_EVAL = 0, CMD_DONE = 1 };

// log(e^a + e^b) = m + log(e^{a-m} + e^{b-m}) with m = max(a, b); the term of
// the larger argument is exp(0) = 1 exactly, so one exp suffices.
__device__ __forceinline__ double log_add_exp(double a, double b) {
    if (a == -INFINITY) return b;
    if (b == -INFINITY) return a;
    const double m = fmax(a, b);
    return m + log(1.0 + exp(fmin(a, b) - m));
}

// Cross-lane operations over a particle's coordinate lanes (lane = 0..15 below),
// done through LDS: each lane writes its value, then every lane reads all entries
// (zero beyond D) and combines them in the same fixed order, so all lanes of the
// particle obtain bitwise identical results.  LDS accesses of one wavefront
// complete in issue order, so no barrier is needed between the write and the
// reads.  A particle's lanes always take the same branches; different particles'
// may differ.
//
// Entries 12..15 are zero unless D > 12: a sum over 16 entries stops there (adding
// a zero changes nothing).

// Sum over the coordinate lanes of v.
__device__ __forceinline__ double dim_sum_at(double* red, int D, int lane, double v) {
    red[lane] = (lane < D) ? v : 0.0;
    __builtin_amdgcn_wave_barrier();
    double s = 0.0;
#pragma unroll
    for (int m = 0; m < 12; ++m) s += red[m];
    if (D > 12)
#pragma unroll
        for (int m = 12; m < MAXDIM; ++m) s += red[m];
    __builtin_amdgcn_wave_barrier();
    return s;
}

__device__ __forceinline__ double dim_sum(NutsSub& U, int D, int lane, double v) {
    return dim_sum_at(U.red[0], D, lane, v);
}

// Two sums at once.
__device__ __forceinline__ void dim_sum2(NutsSub& U, int D, int lane, double a, double b, double& sa, double& sb) {
    U.red[0][lane] = (lane < D) ? a : 0.0;
    U.red[1][lane] = (lane < D) ? b : 0.0;
    __builtin_amdgcn_wave_barrier();
    double x = 0.0, y = 0.0;
#pragma unroll
    for (int m = 0; m < 12; ++m) { x += U.red[0][m]; y += U.red[1][m]; }
    if (D > 12)
#pragma unroll
        for (int m = 12; m < MAXDIM; ++m) { x += U.red[0][m]; y += U.red[1][m]; }
    __builtin_amdgcn_wave_barrier();
    sa = x;
    sb = y;
}

// (M^{-1} v) for this lane's coordinate.
__device__ __forceinline__ double minv_apply(NutsSub& U, int D, int lane, double v) {
    U.vec[lane] = (lane < D) ? v : 0.0;
    __builtin_amdgcn_wave_barrier();
    const double* row = U.Minv + (lane < D ? lane : 0) * MINV_STRIDE;
    double acc = 0.0;
#pragma unroll
    for (int m = 0; m < 12; ++m) acc = fma(row[m], U.vec[m], acc);
    if (D > 12)
#pragma unroll
        for (int m = 12; m < MAXDIM; ++m) acc = fma(row[m], U.vec[m], acc);
    __builtin_amdgcn_wave_barrier();
    return lane < D ? acc : 0.0;
}

// Whether any lane of this lane's particle holds b.
__device__ __forceinline__ bool sub_any(bool b) {
    const unsigned long long m = __ballot(b);
    const int shift = (threadIdx.x & 63) & ~(SUB_LANES - 1);
    return ((m >> shift) & ((1ull << SUB_LANES) - 1)) != 0;
}

// v of lane k of this lane's particle.
__device__ __forceinline__ double sub_shfl(double v, int k) { return __shfl(v, k, SUB_LANES); }

// Normalised log prior of this lane's coordinate and its derivative.
__device__ __forceinline__ double log_prior_lane(const NutsShared& S, int k, double x, double& g) {
    g = 0.0;
    const double lo = S.plo[k], hi = S.phi[k];
    switch (S.pkind[k]) {
    case SMCGW_PRIOR_UNIFORM:
        return (x < lo || x > hi) ? -INFINITY : S.pnorm[k];
    case SMCGW_PRIOR_LOGUNIFORM:
        if (x < lo || x > hi) return -INFINITY;
        g = -1.0 / x;
        return -log(x) + S.pnorm[k];
    case SMCGW_PRIOR_GAUSSIAN: {
        const double r = (x - lo) / hi;
        g = -r / hi;
        return -0.5 * r * r + S.pnorm[k];
    }
    default:
        return 0.0;
    }
}

// The drift x += eps M^{-1} r of one leapfrog step inside the prior box
// (Sec. 4, Eq. 12; Sec. 5, Eqs. 15-18), one coordinate per lane, v = M^{-1} r on
// entry.  The drift runs at velocity v until the first
// reflective coordinate k reaches its wall (the earliest over the lanes,
// lowest k on ties); there the momentum is reflected in the metric,
//   r_k -> r_k - 2 v_k / (M^{-1})_kk,   v -> v - 2 v_k / (M^{-1})_kk M^{-1} e_k,
// which reverses v_k and keeps the kinetic energy, and the drift goes on for
// the rest of the step.  With a diagonal metric this is the fold of the
// coordinate and the flip of its momentum component; for any metric the step
// stays reversible and volume preserving.  Periodic coordinates wrap at the
// end.  A step that meets no wall costs one ballot.
__device__ __forceinline__ void drift_lane(const NutsShared& S, NutsSub& U, int D, int lane, double eps, double& x,
                                           double& r, double v) {
    const bool dl = lane < D;
    const int kk = dl ? lane : 0;
    const bool refl = dl && S.pbnd[kk] == SMCGW_BND_REFLECT;
    const double lo = S.plo[kk], hi = S.phi[kk];
    double rem = 1.0;   // fraction of the step left
    for (int it = 0; it < 64; ++it) {
        const double u = eps * v;
        double fr = 2.0, wall = 0.0;   // fraction of the step at which this coordinate meets its wall
        bool hit = refl && u != 0.0;
        if (hit) wall = u > 0.0 ? hi : lo;
        if (it == 0) {
            // rounded, max((wall - x) / u, 0) < 1 exactly where the wall lies nearer than the step's end (a quotient of
            // two doubles below one does not round up to it): most steps are told apart without the division
            const double away = u > 0.0 ? wall - x : x - wall;
            hit = hit && !(fabs(u) <= away && fabs(u) < INFINITY);
            if (!sub_any(hit)) {
                if (dl) x = fma(eps, v, x);
                break;
            }
        }
        if (hit) fr = fmax((wall - x) / u, 0.0);
        hit = fr < rem;
        if (!sub_any(hit)) {
            if (dl) x = fma(rem * eps, v, x);
            break;
        }
        U.red[0][lane] = hit ? fr : 2.0;
        __builtin_amdgcn_wave_barrier();
        double fmin = 2.0;
        int kmin = 0;
#pragma unroll
        for (int m = 0; m < MAXDIM; ++m) {
            const double f = U.red[0][m];
            if (f < fmin) { fmin = f; kmin = m; }
        }
        __builtin_amdgcn_wave_barrier();
        if (dl) x = lane == kmin ? wall : fma(fmin * eps, v, x);
        rem -= fmin;
        const double vk = sub_shfl(v, kmin);
        const double c = 2.0 * vk / U.Minv[kmin * MINV_STRIDE + kmin];
        if (lane == kmin) r -= c;
        if (dl) v = fma(-c, U.Minv[kk * MINV_STRIDE + kmin], v);
    }
    if (dl && S.pbnd[kk] == SMCGW_BND_PERIODIC) {
        const double w = hi - lo;
        for (int it = 0; it < 64 && (x < lo || x >= hi); ++it) x = (x >= hi) ? x - w : x + w;
    }
}

// Analytic likelihoods (one coordinate per lane of wavefront 0).
template <int TK>
__device__ __forceinline__ double analytic_loglike(NutsSub& S, const TargetDesc& t, int D, int lane, double x,
                                                   double& gl) {
    const bool dl = lane < D;
    if (TK == SMCGW_TARGET_GAUSS) {
        gl = dl ? -x : 0.0;
        return -0.5 * dim_sum(S, D, lane, x * x);
    } else if (TK == SMCGW_TARGET_GAUSS_X_GAUSS) {
        const double y = dl ? t.params[lane] : 0.0, s = dl ? t.params[D + lane] : 1.0;
        const double r = (y - x) / s;
        gl = dl ? r / s : 0.0;
        return dim_sum(S, D, lane, -0.5 * r * r - 0.5 * log(2.0 * PI * s * s));
    } else {
        const double m1 = dl ? t.params[lane] : 0.0, m2 = dl ? t.params[D + lane] : 0.0, sg = t.params[2 * D];
        double s1, s2;
        dim_sum2(S, D, lane, (x - m1) * (x - m1), (x - m2) * (x - m2), s1, s2);
        const double c = -0.5 * D * log(2.0 * PI * sg * sg);
        const double l1 = c - 0.5 * s1 / (sg * sg), l2 = c - 0.5 * s2 / (sg * sg);
        const double mx = fmax(l1, l2);
        const double w1 = exp(l1 - mx), w2 = exp(l2 - mx);
        gl = dl ? (w1 * (m1 - x) + w2 * (m2 - x)) / (sg * sg) / (w1 + w2) : 0.0;
        return mx + log(w1 + w2);
    }
}

// Direction and merge uniform of doubling j (Philox stream DOUBLING).
__device__ __forceinline__ void doubling_draw(const NutsState& T, int j, int& dir, double& uacc) {
    double ud0, ud1;
    rng_uniform2(T.seed, (uint32_t)j, T.pid, T.iter, RNG_DOUBLING, ud0, ud1);
    dir = (ud0 < 0.5) ? -1 : 1;
    uacc = ud1;
}

// Start a transition of particle U.p: momentum, H0, tree of one point.
template <int N>
__device__ __noinline__ void start_transition(int sub, int lane) {
    NutsShared& S = lds_shared<N>();
    NutsSub& U = lds_subs<N>()[sub];
    const NutsArgs& a = S.A;
    NutsState& T = U.T;
    const int D = a.D, p = U.p;
    const bool dl = lane < D;
    const int kk = dl ? lane : 0;
    const double x = dl ? a.theta[(size_t)p * D + lane] : 0.0;
    const double gl = dl ? a.grad[(size_t)p * D + lane] : 0.0;
    const double ll = a.logl[p];
    double gp;
    const double lpr = dim_sum(U, D, lane, dl ? log_prior_lane(S, kk, x, gp) : 0.0);
    if (!dl) gp = 0.0;
    const double beta = T.beta;
    const double lp = beta * ll + lpr;
    const double g = dl ? beta * gl + gp : 0.0;
    // r = L^{-T} z with z ~ N(0, I) from Box-Muller on Philox uniform pairs.
    double u0, u1;
    rng_uniform2(T.seed, (uint32_t)(lane >> 1), T.pid, T.iter, RNG_MOMENTUM, u0, u1);
    const double rad = sqrt(-2.0 * log(1.0 - u0));
    const double z = (lane & 1) ? rad * sin(2.0 * PI * u1) : rad * cos(2.0 * PI * u1);
    double accz = dl ? z : 0.0, r = 0.0;
    for (int i = D - 1; i >= 0; --i) {
        const double ri = sub_shfl(accz, i) / U.L[i * MAXDIM + i];
        if (lane == i) r = ri;
        if (lane < i) accz = fma(-U.L[i * MAXDIM + lane], ri, accz);
    }
    if (!dl) r = 0.0;
    const double v = minv_apply(U, D, lane, r);
    const double h0 = -lp + 0.5 * dim_sum(U, D, lane, r * v);
    // entries beyond D are zero
    U.left[0][lane] = x; U.left[1][lane] = r; U.left[2][lane] = g; U.left[3][lane] = gl; U.left[4][lane] = v;
    U.right[0][lane] = x; U.right[1][lane] = r; U.right[2][lane] = g; U.right[3][lane] = gl; U.right[4][lane] = v;
    U.prop[0][lane] = x; U.prop[1][lane] = gl;
    T.rho[lane] = r;
    T.srho[lane] = 0.0;
    if (lane < NPAR) U.th[lane] = S.pfixed[lane];   // advance replaces the sampled ones
    const int md = a.md_per_p ? min(a.md_per_p[p], SMCGW_MAX_DEPTH) : a.max_depth;
    // every doubling's draws at once, one per lane (the merge uniform as its
    // log: the merge test u < W_sub / W becomes log u < log W_sub - log W)
    if (lane < md) {
        int dj;
        double uj;
        doubling_draw(T, lane, dj, uj);
        T.dtab_dir[lane] = dj;
        T.dtab_u[lane] = log(uj);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int dir0 = md > 0 ? T.dtab_dir[0] : 1;
    const double ua0 = md > 0 ? T.dtab_u[0] : 0.0;
    if (lane == 0) {
        U.end_ll[0] = U.end_ll[1] = ll;
        U.end_lp[0] = U.end_lp[1] = lp;
        T.prop_ll = ll;
        T.h0 = h0;
        T.logw = 0.0;
        T.acc_sum = 0.0;
        T.first = 1;
        T.stop = 0;
        T.j = 0;
        T.n = 0;
        T.nleaves = 1;
        T.sub_logw = -INFINITY;
        T.depth = 0;
        T.nlf = 0;
        T.div = 0;
        T.leafc = 0;
        T.md = md;
        T.dir = dir0;
        T.uacc = ua0;
    }
}

// Complete the leaf in flight (momentum full step with its gradient) into the
// record for `bookkeep`, then take the leapfrog step to the next leaf: the
// next one in the current subtree, else the first leaf of the next doubling
// from the tree end on its side.  Returns CMD_DONE when no leaf follows (the
// depth limit, or no doubling at all).
template <int TK, int N>
__device__ __noinline__ int advance(int sub, int lane) {
    NutsShared& S = lds_shared<N>();
    NutsSub& U = lds_subs<N>()[sub];
    const NutsArgs& a = S.A;
    NutsState& T = U.T;
    const int D = a.D;
    const bool dl = lane < D;
    const int kk = dl ? lane : 0;
    // Every tree-state value the step may need is read up front, both tree ends
    // included, so the LDS round trips overlap instead of following the branches.
    const int first = T.first, n = T.n, nleaves = T.nleaves, j = T.j, md = T.md, dcur = T.dir;
    const double ll = T.ll_new, plp = T.plp, eps_prev = T.eps, beta = T.beta;
    const double gl = T.gl_new[kk], xf = T.x[kk], pg = T.pgp[kk], rh = T.r[kk];
    const double lx = U.left[0][kk], lr = U.left[1][kk], lg = U.left[2][kk];
    const double rx = U.right[0][kk], rr = U.right[1][kk], rg = U.right[2][kk];
    const int dnext = T.dtab_dir[min(j + 1, MAXD1 - 1)], nlf = T.nlf, pidx = S.pidx[lane];
    double xs, rs, gs;   // start point of the next leapfrog step
    int dir;
    if (first) {
        if (md < 1) return CMD_DONE;
        xs = dl ? lx : 0.0;
        rs = dl ? lr : 0.0;
        gs = dl ? lg : 0.0;
        dir = dcur;
    } else {
        const double x = dl ? xf : 0.0;
        const double lp = beta * ll + plp;
        const double g = dl ? beta * gl + pg : 0.0;
        const double r = dl ? fma(0.5 * eps_prev, g, rh) : 0.0;
        // entries of lanes beyond D are zero: written too, the store needs no branch
        T.rec[0][lane] = x; T.rec[1][lane] = r; T.rec[2][lane] = g; T.rec[3][lane] = dl ? gl : 0.0;
        T.rec_ll = ll;
        T.rec_lp = lp;
        if (n + 1 < nleaves) {
            xs = x; rs = r; gs = g;
            dir = dcur;
        } else if (j + 1 < md) {
            dir = dnext;
            if (dir == dcur) {
                xs = x; rs = r; gs = g;
            } else {
                xs = dl ? (dir > 0 ? rx : lx) : 0.0;
                rs = dl ? (dir > 0 ? rr : lr) : 0.0;
                gs = dl ? (dir > 0 ? rg : lg) : 0.0;
            }
        } else {
            return CMD_DONE;
        }
    }
    T.inflight = first ? 0 : nlf + 1;   // leaf index of the next leaf
    const double eps = dir * a.step;
    double r = dl ? fma(0.5 * eps, gs, rs) : 0.0;
    const double v = minv_apply(U, D, lane, r);
    double x = dl ? xs : 0.0;
    drift_lane(S, U, D, lane, eps, x, r, v);
    __builtin_amdgcn_wave_barrier();
    T.x[lane] = x;
    T.r[lane] = r;
    T.eps = eps;   // the same value from each lane
    if (TK == SMCGW_TARGET_GW && dl) U.th[pidx] = x;   // the fixed parameters stay from start_transition
    return CMD_EVAL;
}

// Work on the leaf in flight that `bookkeep` does not wait for (run on an
// otherwise idle wavefront): its amplitude entries of the coefficient block,
// the log prior and its gradient at its position (used by the next
// `advance`) and the uniform of its progressive sampling step (leaf index =
// leaves booked before it, the Philox LEAF counter).
template <int TK, int N>
__device__ __noinline__ void aux_in_flight(int sub, int lane) {
    NutsShared& S = lds_shared<N>();
    NutsSub& U = lds_subs<N>()[sub];
    NutsState& T = U.T;
    const int D = S.A.D;
    const bool dl = lane < D;
    const int idx = T.inflight;
    const double x = T.x[lane];
    double ul0, ul1;
    rng_uniform2(T.seed, (uint32_t)idx, T.pid, T.iter, RNG_LEAF, ul0, ul1);
    double lpk = 0.0, gp = 0.0;
    // The progressive sampling test u < w / (W + w) is taken as log u + log W < log(1 - u) + log w.
    if (TK == SMCGW_TARGET_GW) {
        // One logarithm and one division for everything: the coordinates' log priors on the lanes below D <= NPAR,
        // log u and log(1 - u) on two lanes behind them, the amplitude C_A u_scale and the derivatives of ln C_A on three.
        constexpr int L_U = 13, L_V = 14, L_AMP = 15, L_DMC = 13, L_DDL = 14;
        static_assert(NPAR <= L_U && L_AMP < SUB_LANES, "the lanes behind the coordinates");
        const double mc = U.th[P_MC], dlum = U.th[P_DL];
        const double lo = S.plo[lane], hi = S.phi[lane], norm = S.pnorm[lane];
        const int kind = dl ? S.pkind[lane] : -1;
        double arg = x;
        arg = lane == L_U ? ul0 : arg;
        arg = lane == L_V ? 1.0 - ul0 : arg;
        arg = lane == L_AMP ? mc * U.ev.t_sun : arg;
        const double lg = log(arg);
        double num = -1.0, den = x;
        den = lane == L_DMC ? mc : lane == L_DDL ? dlum : den;
        num = lane == L_DMC ? 5.0 / 6.0 : num;
        const double camp = CAMP_FACTOR * exp((5.0 / 6.0) * lg) * U.ev.c_light;
        num = lane == L_AMP ? camp : num;
        den = lane == L_AMP ? dlum * U.ev.mpc_m : den;
        const double quo = num / den;
        if (kind == SMCGW_PRIOR_GAUSSIAN) {
            const double r = (x - lo) / hi;
            gp = -r / hi;
            lpk = -0.5 * r * r + norm;
        } else if (kind == SMCGW_PRIOR_UNIFORM || kind == SMCGW_PRIOR_LOGUNIFORM) {
            const bool out = x < lo || x > hi, lu = kind == SMCGW_PRIOR_LOGUNIFORM;
            lpk = out ? -INFINITY : lu ? -lg + norm : norm;
            gp = lu && !out ? quo : 0.0;
        }
        if (lane >= L_DMC) U.cb[CB_DLNCA_MC + lane - L_DMC] = lane == L_AMP ? quo * U.ev.u_scale : quo;
        if (lane == L_U || lane == L_V) T.ul[idx & 1][lane - L_U] = lg;
    } else {
        const double lu = log(lane == 0 ? ul0 : 1.0 - ul0);   // lanes 0 and 1
        if (dl) lpk = log_prior_lane(S, lane, x, gp);
        if (lane < 2) T.ul[idx & 1][lane] = lu;
    }
    T.plp = dim_sum_at(U.pred, D, lane, lpk);
    T.pgp[lane] = gp;
}
static_assert(CB_DLNCA_DL == CB_DLNCA_MC + 1 && CB_AMP == CB_DLNCA_MC + 2, "written by three lanes");

// Decisions for the finished leaf: energy, divergence,
// progressive sampling, U-turn checks of the nodes it completes, the merge
// when its subtree is complete, and the set-up of the next doubling.  Sets
// T.stop when the transition ends here.
template <int N>
__device__ __noinline__ void bookkeep(int sub, int lane) {
    NutsShared& S = lds_shared<N>();
    NutsSub& U = lds_subs<N>()[sub];
    const NutsArgs& a = S.A;
    NutsState& T = U.T;
    if (T.first) {
        __builtin_amdgcn_wave_barrier();
        if (lane == 0) T.first = 0;
        return;
    }
    const int D = a.D;
    const bool dl = lane < D;
    // zero beyond D, like every per-coordinate array of the tree
    const double x = T.rec[0][lane], r = T.rec[1][lane], g = T.rec[2][lane], gl = T.rec[3][lane];
    const double ll = T.rec_ll, lp = T.rec_lp;
    double srho = T.srho[lane];
    const double rho_j = T.rho[lane];
    const double lu0[2] = {T.ul[0][0], T.ul[1][0]}, lu1[2] = {T.ul[0][1], T.ul[1][1]};
    uint32_t leafc = T.leafc;
    const int nleaves = T.nleaves, nlf = T.nlf, md = T.md;
    int depth = T.depth, dir = T.dir, div = T.div;
    double logw = T.logw, prop_ll = T.prop_ll, uacc = T.uacc, sprop_ll = T.sprop_ll, acc_sum = T.acc_sum;
    const double v = minv_apply(U, D, lane, r);   // velocity of this leaf: energy and every U-turn check
    const int j = T.j, n = T.n;
    const double h0 = T.h0;
    const double dh = -lp + 0.5 * dim_sum(U, D, lane, r * v) - h0;
    const bool finite = (dh == dh) && dh != INFINITY && dh != -INFINITY;
    double sub_logw = T.sub_logw;
    // Both exponentials of the leaf in one evaluation: lane 0 the log-add term e^{min - max} of the subtree
    // weight update, lane 1 the acceptance term e^{-dh}.
    const double lw = -dh;
    const double lmax = fmax(sub_logw, lw), lmin = fmin(sub_logw, lw);
    const double ee = exp(lane == 0 ? lmin - lmax : -dh);
    const double e_add = sub_shfl(ee, 0), e_acc = sub_shfl(ee, 1);
    acc_sum += finite ? fmin(1.0, e_acc) : 0.0;
    bool ok = true;
    if (!finite || dh > a.max_dh) {
        div = 1;
        ok = false;
    } else {
        // this leaf opens the nodes of levels 1 .. ls (n a multiple of 2^l)
        const int ls = n == 0 ? j : min(j, __builtin_ctz((unsigned)n));
        for (int l = 1; l <= ls; ++l) { U.ck_rho[l][lane] = srho; U.ck_v[l][lane] = v; }
        srho += r;
        // uniform drawn while this leaf was in flight: accept with probability w / (W + w)
        const double u0 = leafc & 1 ? lu0[1] : lu0[0], u1 = leafc & 1 ? lu1[1] : lu1[0];
        ++leafc;
        const double nlw = sub_logw == -INFINITY ? lw : lmax + log(1.0 + e_add);
        if (u0 + sub_logw < u1 + lw) {
            U.sprop[0][lane] = x;
            U.sprop[1][lane] = gl;
            sprop_ll = ll;
        }
        sub_logw = nlw;
        if (a.uturn && j > 0 && ((n + 1) & 1) == 0) {
            // nodes completed by this leaf: level l = 1 .. lc (lc = min(j, trailing
            // zeros of n + 1: one on average) covers leaves n+1-2^l .. n and needs
            // rho.v_first > 0 and rho.v_last > 0
            const int lc = min(j, __builtin_ctz((unsigned)(n + 1)));
            for (int l = 1; l <= lc; ++l) {
                const double nr = srho - U.ck_rho[l][lane];
                double sa, sb;
                dim_sum2(U, D, lane, nr * U.ck_v[l][lane], nr * v, sa, sb);
                if (!(sa > 0.0 && sb > 0.0)) ok = false;
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
    int jn = j, nn = n;
    bool stop = false;
    if (!ok) {
        stop = true;
    } else if (n + 1 == nleaves) {
        depth = j + 1;
        __builtin_amdgcn_wave_barrier();
        if (uacc < sub_logw - logw) {   // uacc holds the log of the merge uniform
            U.prop[0][lane] = U.sprop[0][lane];
            U.prop[1][lane] = U.sprop[1][lane];
            prop_ll = sprop_ll;
        }
        logw = log_add_exp(logw, sub_logw);
        const double rho = rho_j + srho;
        const int side = dir > 0 ? 1 : 0;
        double (*E)[MAXDIM] = side ? U.right : U.left;
        E[0][lane] = x; E[1][lane] = r; E[2][lane] = g; E[3][lane] = gl; E[4][lane] = v;
        T.rho[lane] = rho;
        U.end_ll[side] = ll;
        U.end_lp[side] = lp;
        __builtin_amdgcn_wave_barrier();
        if (a.uturn) {
            const double vl = U.left[4][lane], vr = U.right[4][lane];
            double sa, sb;
            dim_sum2(U, D, lane, rho * vl, rho * vr, sa, sb);
            stop = !(sa > 0.0 && sb > 0.0);
        }
        if (!stop && j + 1 >= md) stop = true;   // depth limit
        if (!stop) {
            // next doubling j + 1
            jn = j + 1;
            nn = 0;
            dir = T.dtab_dir[jn];
            uacc = T.dtab_u[jn];
            srho = 0.0;
            sub_logw = -INFINITY;
        }
    } else {
        nn = n + 1;
    }
    T.srho[lane] = srho;
    // the same values from each lane
    T.acc_sum = acc_sum; T.sub_logw = sub_logw; T.sprop_ll = sprop_ll; T.leafc = leafc;
    T.div = div; T.stop = stop ? 1 : 0; T.depth = depth; T.j = jn; T.n = nn; T.logw = logw; T.prop_ll = prop_ll;
    T.dir = dir; T.uacc = uacc;
    T.nleaves = 1 << jn;
    T.nlf = nlf + 1;
}

template <int N>
__device__ __noinline__ void write_outputs(int sub, int lane) {
    NutsShared& S = lds_shared<N>();
    NutsSub& U = lds_subs<N>()[sub];
    const NutsArgs& a = S.A;
    const NutsState& T = U.T;
    const int D = a.D, p = U.p;
    __builtin_amdgcn_wave_barrier();
    if (lane < D) {
        a.theta[(size_t)p * D + lane] = U.prop[0][lane];
        a.grad[(size_t)p * D + lane] = U.prop[1][lane];
    }
    if (lane == 0) {
        a.logl[p] = T.prop_ll;
        if (a.depth_out) a.depth_out[p] = T.depth;
        if (a.nlf_out) a.nlf_out[p] = T.nlf;
        if (a.div_out) a.div_out[p] = (uint8_t)T.div;
        if (a.acc_out) a.acc_out[p] = T.nlf > 0 ? T.acc_sum / T.nlf : 0.0;
    }
}

// Issue priority of the slot's wavefronts while doubling j runs: a tree that
// has reached 2^3, 2^4, 2^5 leaves outranks the shallower trees sharing its
// SIMDs, so the transitions that decide when the launch ends go first.  Trees
// past 2^5 leaves share the top level and are not ordered among themselves; where
// most trees are that deep (3 x 8033 bins, mean depth 5.7 to 7.4) the levels change
// nothing that can be measured.
__device__ __forceinline__ void tree_priority(int j) {
    if (j >= 5) __builtin_amdgcn_s_setprio(3);
    else if (j == 4) __builtin_amdgcn_s_setprio(2);
    else if (j == 3) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
}

// Prologue pieces of one leaf (kept out of line so their registers do not
// constrain the bin loop).
template <int N>
__device__ __noinline__ void leaf_prep_intrinsic(int sub, int lane) {
    NutsSub& U = lds_subs<N>()[sub];
    prep_intrinsic_n<1>(U.ev, U.th, U.cb, lane, lane == 0);
}

// Extrinsic prologue: the particle's lanes 0-3 take one sin / cos each (in
// parallel), then lane d (d < MAXDET) builds detector d with its ra
// derivatives and lane MAXDET + d the dec derivatives of the same detector
// (one tangent per lane keeps each lane's chain short).  The amplitude is
// computed on the auxiliary wavefront.
template <int N>
__device__ __noinline__ void leaf_prep_extrinsic(int sub, int lane) {
    NutsSub& U = lds_subs<N>()[sub];
    if (lane < ANG_COUNT) {
        double sn, cs;
        sincos(extrinsic_angle(U.ev, U.th, lane), &sn, &cs);
        U.ang.sc[lane][0] = sn;
        U.ang.sc[lane][1] = cs;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (lane < 2 * MAXDET) {
        const ExtAngles ang = U.ang;
        const int k = lane / MAXDET;
        prep_extrinsic_det_n<1>(U.ev, U.th, ang, U.cb, lane - k * MAXDET, k, k == 0);
    }
}

// Epilogue of one leaf: the classes' moments summed in class order, then logL and
// its gradient (the algebra of finish_particle) spread over the particle's lanes, without
// branches and with the reads of each step in flight together, so that the chain is four
// round trips to the LDS:
//   lanes 0..3        the phase part of d logL / d(Mc, q, chi1, chi2): a dot
//                     product of the basis moments with the prologue's Jacobian;
//   lanes 4..4+n_det  detector d's terms of logL, of d logL / d ln C_A, of the
//                     projection derivatives and of the arrival-time terms;
//   lanes 0..NPAR     one gradient component each, the sum of one or two of the detectors'
//                     terms in detector order; lane FIN_LL_LANE the log-likelihood.
constexpr int FIN_LL_LANE = NPAR;

// The detector term that lane `lane` sums (parameters in the order of P_*, then logL).
__device__ __forceinline__ int fin_term(int lane) {
    constexpr int t[FIN_LL_LANE + 1] = {FD_DLN, FD_LL, FD_LL, FD_LL, FD_DLN, FD_GP, FD_GP + 1, FD_RA, FD_DEC, FD_T,
                                        FD_LL, FD_LL};
    unsigned long long packed = 0;
    for (int k = 0; k <= FIN_LL_LANE; ++k) packed |= (unsigned long long)t[k] << (4 * k);
    return (int)(packed >> (4 * lane) & 15);
}

template <int NDET, int WAVES, int N>
__device__ __noinline__ void leaf_finish(int sub, int lane) {
    NutsShared& S = lds_shared<N>();
    NutsSub& U = lds_subs<N>()[sub];
    const double (*wm)[MOM_SIZE] = lds_moments<N, WAVES>(sub);
    NutsState& T = U.T;
    const DevEvent* ev = &U.ev;
    constexpr int NM = mom_g(NDET, NCOEF), PASSES = (NM + SUB_LANES - 1) / SUB_LANES;
    const double* c = U.cb;
    // the coefficients of both roles
    const int d = min(max(lane - 4, 0), NDET - 1);
    double jac[NCOEF], dpr[4], dpi[4];
#pragma unroll
    for (int b = 0; b < NCOEF; ++b) jac[b] = c[CB_DC + 4 * b + (lane & 3)];
#pragma unroll
    for (int k = 0; k < 4; ++k) { dpr[k] = c[CB_DPR + 4 * d + k]; dpi[k] = c[CB_DPI + 4 * d + k]; }
    const double amp = c[CB_AMP], prd = c[CB_PR + d], pid = c[CB_PI + d], h = ev->hnorm[d];
    const double tra = c[CB_DTAU + 2 * d], tdec = c[CB_DTAU + 2 * d + 1];
    const double lnca_mc = c[CB_DLNCA_MC], lnca_dl = c[CB_DLNCA_DL], dd = ev->dd;
    const int pidx = S.pidx[lane];
    // the classes beyond the event's blocks are empty (a lone particle's wavefronts write their zeros)
    const int classes = N > 1 ? ev->n_pad / TABLE_PAD : WAVES;
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
        const int e = min(lane + i * SUB_LANES, NM - 1);
        double s = wm[0][e];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) {
            const double t = wm[w][e];
            s += w < classes ? t : 0.0;
        }
        U.mom[e] = s;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const double* m = U.mom;
    double phase = 0.0;
#pragma unroll
    for (int b = 0; b < NCOEF; ++b) phase = fma(jac[b], m[mom_g(NDET, b)], phase);
    phase = TWO_PI * phase;
    const double g0 = m[mom_g(NDET, 0)];
    {
        const double pr = prd * amp, pi = pid * amp;
        const double zr = m[mom_zr(NDET, d)], zi = m[mom_zi(NDET, d)], t = m[mom_t(NDET, d)];
        const double re = pr * zr - pi * zi;
        const double p2 = pr * pr + pi * pi;
        double o[FD_SIZE];
        o[FD_LL] = re - 0.5 * p2 * h;
        o[FD_DLN] = re - p2 * h;
        const double ar = zr - h * pr, ai = -zi - h * pi;   // dlogL / d(Re P', Im P')
#pragma unroll
        for (int k = 0; k < 4; ++k) o[FD_GP + k] = amp * (ar * dpr[k] + ai * dpi[k]);
        o[FD_T] = t;
        o[FD_RA] = TWO_PI * t * tra;
        o[FD_DEC] = TWO_PI * t * tdec;
        if (lane >= 4 && lane < 4 + NDET)
#pragma unroll
            for (int f = 0; f < FD_SIZE; ++f) U.fin_det[d][f] = o[f];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int fa = fin_term(min(lane, FIN_LL_LANE)), fb = lane == P_DEC ? FD_GP + 3 : FD_GP + 2;
    double sa = 0.0, sb = 0.0;
#pragma unroll
    for (int k = 0; k < NDET; ++k) {
        sa += U.fin_det[k][fa];
        sb += U.fin_det[k][fb];
    }
    // factor and summand of the component: -0.0 leaves a product as it is
    double f = 1.0, add = -0.0;
    f = lane == P_MC ? lnca_mc : lane == P_DL ? lnca_dl : lane == P_TC ? TWO_PI : f;
    add = lane == P_MC ? phase : lane == P_RA || lane == P_DEC ? sb : lane == FIN_LL_LANE ? -0.5 * dd : add;
    double v = fma(sa, f, add);
    v = lane == P_Q || lane == P_CHI1 || lane == P_CHI2 ? phase : v;
    v = lane == P_PHIC ? -g0 : v;
    const double gl = sub_shfl(v, pidx);
    T.gl_new[lane] = gl;
    if (lane == FIN_LL_LANE) T.ll_new = v;
}
static_assert(P_Q == 1 && P_CHI1 == 2 && P_CHI2 == 3 && P_PHIC == 10 && FIN_LL_LANE < SUB_LANES, "lane roles");

// The Cholesky factor L of M^{-1} ([D][D], row-major) into LDS, zero-padded
// to MAXDIM; derive_metric then forms M^{-1} = L L^T from it (one wavefront, each
// lane a share of the entries).
__device__ __forceinline__ void load_factor(NutsSub& U, const double* chol, int D, int lane) {
    for (int i = lane; i < MAXDIM * MAXDIM; i += 64) {
        const int r = i / MAXDIM, c = i % MAXDIM;
        U.L[i] = (r < D && c < D) ? chol[r * D + c] : 0.0;
    }
}

template <int N>
__device__ __noinline__ void derive_metric(int sub, int D, int lane) {
    NutsSub& U = lds_subs<N>()[sub];
    for (int i = lane; i < MAXDIM * MAXDIM; i += 64) {
        const int r = i / MAXDIM, c = i % MAXDIM;
        double s = 0.0;
        for (int m = 0; m < D; ++m) s = fma(U.L[r * MAXDIM + m], U.L[c * MAXDIM + m], s);
        U.Minv[r * MINV_STRIDE + c] = s;
    }
}

// The prior description and the arguments (one lane).
__device__ __forceinline__ void share_arguments(NutsShared& S, const NutsArgs& a, const PriorDesc& pri,
                                                const ParamMap& pm) {
    S.A = a;
    if (a.beta_dev) S.A.beta = *a.beta_dev;
    // once per launch on one lane: kept rolled, so the logs are not copied out per coordinate
#pragma unroll 1
    for (int k = 0; k < MAXDIM; ++k) {
        S.plo[k] = pri.lo[k]; S.phi[k] = pri.hi[k]; S.pbnd[k] = pri.bnd[k]; S.pkind[k] = pri.kind[k];
        S.pidx[k] = pm.idx[k];
        const double lo = pri.lo[k], hi = pri.hi[k];
        S.pnorm[k] = k >= a.D ? 0.0
                   : pri.kind[k] == SMCGW_PRIOR_UNIFORM ? -log(hi - lo)
                   : pri.kind[k] == SMCGW_PRIOR_LOGUNIFORM ? -log(log(hi / lo))
                   : pri.kind[k] == SMCGW_PRIOR_GAUSSIAN ? -0.5 * log(2.0 * PI * hi * hi) : 0.0;
    }
    for (int k = 0; k < NPAR; ++k) S.pfixed[k] = pm.fixed[k];
}

// The particle's run into its tree state (one lane).
__device__ __forceinline__ void set_run(const NutsArgs& a, NutsState& T, int p, int run) {
    if (a.state) {
        const double* st = a.state + (size_t)run * SMCGW_STATE_SIZE;
        T.beta = st[SMCGW_ST_BETA];
        T.iter = (uint64_t)st[SMCGW_ST_ITER];
        T.seed = a.seed + (uint64_t)run;
        T.pid = (uint32_t)(p - run * a.run_size);
    } else {
        T.beta = a.beta;
        T.iter = a.iteration;
        T.seed = a.seed;
        T.pid = (uint32_t)p;
    }
}

// Particle queues of a launch without a work hint.  The particles are dealt
// in stripes of neighbouring indices, stripe g to queue g mod N_QUEUES,
// one queue per XCD: workgroups are dispatched to the XCDs in turn, so workgroup
// b starts on queue b mod N_QUEUES and, once that is drained, goes on to the
// others in turn.  Neighbouring particles, whose inputs and outputs share cache
// lines, then mostly pass through one XCD's L2 instead of leaving partly written
// lines in several.  The first particle of every place is fixed: place s of the
// w-th workgroup of a queue takes the queue's entry s W + w (W of its workgroups),
// so that every workgroup has its first particle before any has its second; the
// queue's counter starts behind those entries.  With a work hint there is one
// queue, the sorted order.  A queue is drained for good once a fetch runs past
// its end (its particle indices only grow), so a place is given up after at most
// N_QUEUES empty fetches.
constexpr int N_QUEUES = 8;

__device__ __forceinline__ int striped_particle(int queue, int k, int stripe) {
    return ((k / stripe) * N_QUEUES + queue) * stripe + k % stripe;
}

// Workgroups of a grid whose first queue is `queue`.
__device__ __forceinline__ int queue_workgroups(int grid, int queue) {
    return grid > queue ? (grid - queue + N_QUEUES - 1) / N_QUEUES : 0;
}

// The next particle for place s of this workgroup, or a.P when there is none
// (one lane).  first: the place's fixed particle; drained: the queues this
// workgroup has seen empty.
__device__ __forceinline__ int next_particle(const NutsArgs& a, int s, bool first, unsigned& drained) {
    const int b = blockIdx.x, grid = gridDim.x;
    if (a.order) {
        const int q = first ? s * grid + b
                            : __hip_atomic_fetch_add(a.queue, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return q < a.P ? a.order[q] : a.P;
    }
    const int home = b % N_QUEUES;
    if (first) {
        const int c = striped_particle(home, s * queue_workgroups(grid, home) + b / N_QUEUES, a.stripe);
        if (c < a.P) return c;
    }
    for (int t = 0; t < N_QUEUES; ++t) {
        const int x = (home + t) % N_QUEUES;
        if (drained & (1u << x)) continue;
        const int k = __hip_atomic_fetch_add(a.queue + x, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int c = striped_particle(x, k, a.stripe);
        if (c < a.P) return c;
        drained |= 1u << x;
    }
    return a.P;
}

template <int NDET, int PREC, int TK, int SUBS, int WAVES>
__global__ __launch_bounds__(WAVES * 64, (WAVES == 1 ? 1 : NUTS_WAVES_PER_SIMD)) void nuts_kernel(NutsArgs a, PriorDesc pri, ParamMap pm,
                                                                             TargetDesc tgt) {
    NutsShared& S = lds_shared<SUBS>();
    NutsSub* sub = lds_subs<SUBS>();
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int D = a.D;
    const int g = lane / SUB_LANES % SUBS, cl = lane % SUB_LANES;   // this lane's particle and coordinate
    const bool mine = SUBS * SUB_LANES == 64 || lane < SUBS * SUB_LANES;
    NutsSub& U = sub[g];

    if (tid == 0) share_arguments(S, a, pri, pm);
    if (tid < SUBS) { sub[tid].e = -1; sub[tid].run = -1; }
    __syncthreads();

    // one factor for the whole launch or per run stays in place from particle to particle
    const bool run_factor = !a.chol_pp;
    unsigned drained = 0;
    unsigned vacant = (1u << SUBS) - 1;   // places to fill (uniform)
    unsigned held = 0;                    // places with a particle (wavefront 0)
    bool first = true;                    // no place has been filled yet
    for (;;) {
        // Wavefront 0 fills the vacant places: the next particle, its run, event and
        // metric, and the start of its transition.  Meanwhile the others wait for the
        // places' first advance.
        if (wave == 0 && vacant) {
            if (lane == 0)
                for (int s = 0; s < SUBS; ++s)
                    if (vacant & (1u << s)) {
                        int p;
                        bool fixed = first;
                        do {   // a finished run's particles are left untouched
                            p = next_particle(a, s, fixed, drained);
                            fixed = false;
                        } while (p < a.P && a.state &&
                                 a.state[(size_t)(p / a.run_size) * SMCGW_STATE_SIZE + SMCGW_ST_DONE] != 0.0);
                        sub[s].p = p < a.P ? p : -1;
                        if (p < a.P) set_run(S.A, sub[s].T, p, a.state ? p / a.run_size : 0);
                    }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            for (int s = 0; s < SUBS; ++s) {
                if (!(vacant & (1u << s))) continue;
                const int p = __builtin_amdgcn_readfirstlane(sub[s].p);
                held = p < 0 ? held & ~(1u << s) : held | 1u << s;
                if (p < 0) continue;
                const int run = a.state ? p / a.run_size : 0;
                if (TK == SMCGW_TARGET_GW) {   // the event's descriptor: the leaf's serial phases read it from LDS
                    const int e = __builtin_amdgcn_readfirstlane(event_index(a.ev_of_p, p, a.n_events));
                    if (e != __builtin_amdgcn_readfirstlane(sub[s].e)) {
                        const unsigned long long* src = (const unsigned long long*)(a.events + e);
                        unsigned long long* dst = (unsigned long long*)&sub[s].ev;
                        for (int i = lane; i < (int)(sizeof(DevEvent) / 8); i += 64) dst[i] = src[i];
                        if (lane == 0) sub[s].e = e;
                    }
                }
                load_factor(sub[s], a.chol + (size_t)(a.chol_pp ? p : run) * D * D, D, lane);
                if (!run_factor || run != __builtin_amdgcn_readfirstlane(sub[s].run)) {
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    derive_metric<SUBS>(s, D, lane);
                    if (lane == 0) sub[s].run = run;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (mine && (vacant & held & (1u << g))) start_transition<SUBS>(g, cl);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        first = false;

        // Wavefronts of the leaf prologue: intrinsic and extrinsic parts on
        // wavefronts 1 and 2 while wavefront 0 books the previous leaf (both on
        // wavefront 1 when the workgroup has two).
        constexpr int W_INTR = WAVES > 1 ? 1 : 0;
        constexpr int W_EXTR = WAVES > 2 ? 2 : W_INTR;
        constexpr int W_AUX = WAVES > 3 ? 3 : 0;
        const bool live = wave == 0 && mine && (held & (1u << g));
        unsigned long long evals = 0;
        if (wave == 0) {
            int cmd = CMD_DONE;
            if (live) cmd = advance<TK, SUBS>(g, cl);
            evals = __ballot(cl == 0 && cmd == CMD_EVAL);
            if (lane == 0) S.evals = evals;
        }
        __syncthreads();
        if (WAVES > 1) {
            const bool eval = mine && (S.evals >> (g * SUB_LANES) & 1);
            if (wave == W_AUX && W_AUX > 0 && eval) aux_in_flight<TK, SUBS>(g, cl);
            if (TK == SMCGW_TARGET_GW) {
                if (wave == W_INTR && eval && cl < 4) leaf_prep_intrinsic<SUBS>(g, cl);
                if (wave == W_EXTR && eval && cl < 2 * MAXDET) leaf_prep_extrinsic<SUBS>(g, cl);
            }
        }
        if (wave == 0) {
            const bool eval = evals >> (g * SUB_LANES) & 1;
            bool stop = true;
            if (live) {
                bookkeep<SUBS>(g, cl);
                stop = U.T.stop;
            }
            if (W_AUX == 0 && mine && eval) aux_in_flight<TK, SUBS>(g, cl);
            const unsigned long long go = __ballot(live && eval && !stop);
            unsigned word = 0;
            int jmax = 0;
#pragma unroll
            for (int s = 0; s < SUBS; ++s) {
                if (!(held & (1u << s))) continue;
                if (go >> (s * SUB_LANES) & 1) {
                    word |= 1u << s;
                    if (a.priority) jmax = max(jmax, __builtin_amdgcn_readfirstlane(sub[s].T.j));
                } else
                    word |= 256u << s;
            }
            if (lane == 0) S.places = word | (unsigned)jmax << 16;
        }
        __syncthreads();
        const unsigned word = __builtin_amdgcn_readfirstlane(S.places);
        const unsigned running = word & 255;
        vacant = word >> 8 & 255;
        if (!(running | vacant)) break;   // every place has been given up
        if (a.priority) tree_priority(word >> 16);
        if (wave == 0 && mine && (vacant & (1u << g))) write_outputs<SUBS>(g, cl);
        if (TK == SMCGW_TARGET_GW) {
            for (int s = 0; s < SUBS; ++s) {
                if (!(running & (1u << s))) continue;
                // particle s's class r goes to wavefront r + s: an event of fewer blocks than classes (one, of a
                // folded event) leaves the higher classes empty, and the particles' first ones on different wavefronts
                const int r = (wave + SUBS * WAVES - s) % WAVES;
                const DevEvent* ev = &sub[s].ev;
                const TableView t = PREC == SMCGW_MIXED ? mixed_tables<NDET>(ev) : fp64_tables<NDET>(ev);
                if (SUBS > 1 && r >= t.npad / TABLE_PAD) continue;
                const BinCoef k = load_coef(sub[s].cb);
                if (PREC == SMCGW_MIXED)
                    bins_mixed_wave<NDET>(t, k, r, WAVES, t.npad / TABLE_PAD, lds_moments<SUBS, WAVES>(s)[r]);
                else
                    // with the library's sin and cos: a deep tree's leaves follow their last bits
                    bins_fp64_wave<NDET, true, true>(t, k, r, WAVES, t.npad / TABLE_PAD, lds_moments<SUBS, WAVES>(s)[r]);
            }
            __syncthreads();
            if (wave == 0 && mine && (running & (1u << g))) leaf_finish<NDET, WAVES, SUBS>(g, cl);
        } else if (wave == 0 && mine && (running & (1u << g))) {
            double gl;
            const double ll = analytic_loglike<TK>(U, tgt, D, cl, cl < D ? U.T.x[cl] : 0.0, gl);
            if (cl < D) U.T.gl_new[cl] = gl;
            if (cl == 0) U.T.ll_new = ll;
        }
    }
}

// Start order from a work hint: particles sorted by descending bucket
// floor(log2(hint)) + 1 (0 for hint <= 0), stable in the particle index.
// One workgroup; thread t owns the contiguous index chunk [t*ch, (t+1)*ch).
// Four wavefronts (one per SIMD) fit in the registers of a single NUTS slot,
// so the kernel starts as soon as one slot of a co-running launch frees.
constexpr int ORDER_THREADS = 256;
constexpr int ORDER_BUCKETS = 16;

__device__ __forceinline__ int hint_bucket(int32_t h) { return h <= 0 ? 0 : min(ORDER_BUCKETS - 1, 32 - __clz(h)); }

__global__ __launch_bounds__(ORDER_THREADS) void order_kernel(const int32_t* __restrict__ hint, int P,
                                                              int32_t* __restrict__ order) {
    __shared__ int wsum[ORDER_THREADS / 64][ORDER_BUCKETS];
    __shared__ int base[ORDER_THREADS / 64][ORDER_BUCKETS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ch = (P + ORDER_THREADS - 1) / ORDER_THREADS;
    const int lo = min(P, tid * ch), hi = min(P, lo + ch);
    int cnt[ORDER_BUCKETS];
#pragma unroll
    for (int k = 0; k < ORDER_BUCKETS; ++k) cnt[k] = 0;
    for (int i = lo; i < hi; ++i) {
        const int b = hint_bucket(hint[i]);
#pragma unroll
        for (int k = 0; k < ORDER_BUCKETS; ++k) cnt[k] += (b == k);
    }
    // exclusive offsets of this thread inside each bucket: lanes, then wavefronts
    int off[ORDER_BUCKETS];
#pragma unroll
    for (int k = 0; k < ORDER_BUCKETS; ++k) {
        int inc = cnt[k];
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(inc, o);
            if (lane >= o) inc += t;
        }
        off[k] = inc - cnt[k];
        if (lane == 63) wsum[wave][k] = inc;
    }
    __syncthreads();
    if (tid == 0) {   // bucket starts in descending bucket order, then wavefront order inside a bucket
        int start = 0;
        for (int k = ORDER_BUCKETS - 1; k >= 0; --k) {
            for (int w = 0; w < ORDER_THREADS / 64; ++w) {
                base[w][k] = start;
                start += wsum[w][k];
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ORDER_BUCKETS; ++k) off[k] += base[wave][k];
    for (int i = lo; i < hi; ++i) {
        const int b = hint_bucket(hint[i]);
        int pos = 0;
#pragma unroll
        for (int k = 0; k < ORDER_BUCKETS; ++k) {
            if (b == k) { pos = off[k]; ++off[k]; }
        }
        order[pos] = i;
    }
}

// Queue counters behind the places' fixed first particles.
__global__ void start_queues_kernel(int* q, int grid, int subs, int ordered) {
    const int x = threadIdx.x;
    if (x < N_QUEUES) q[x] = subs * (ordered ? grid : queue_workgroups(grid, x));
}

// ------------------------------------------------------------------ lockstep sweeps
// The plain comparison form of the transition: the same tree, random streams
// and decisions as nuts_kernel, but advanced one leapfrog step per particle per
// sweep.  A sweep is one launch of nuts_sweep_kernel (one wavefront per
// particle: the tree step that books the leaf just evaluated and moves to the
// next one) and one batched likelihood launch over the particles still
// building their tree; the tree state waits in global memory between sweeps.

// A particle's tree between sweeps.
struct SweepState {
    NutsState T;
    double left[5][MAXDIM], right[5][MAXDIM];
    double prop[2][MAXDIM], sprop[2][MAXDIM];
    double ck_rho[MAXD1][MAXDIM], ck_v[MAXD1][MAXDIM];
    double end_ll[2], end_lp[2];
    int phase;
    int pad;
};
static_assert(sizeof(NutsState) % 8 == 0 && sizeof(SweepState) % 8 == 0, "copied in 8-byte words");
enum { SW_START = 0, SW_RUN = 1, SW_DONE = 2 };

__device__ __forceinline__ void copy_words(void* dst, const void* src, size_t bytes, int lane) {
    unsigned long long* d = (unsigned long long*)dst;
    const unsigned long long* s = (const unsigned long long*)src;
    for (size_t i = lane; i < bytes / 8; i += 64) d[i] = s[i];
}

// Tree state between LDS and the particle's record.
__device__ __forceinline__ void sweep_save(SweepState& G, const NutsSub& S, int lane) {
    copy_words(&G.T, &S.T, sizeof(NutsState), lane);
    copy_words(G.left, S.left, sizeof(S.left), lane);
    copy_words(G.right, S.right, sizeof(S.right), lane);
    copy_words(G.prop, S.prop, sizeof(S.prop), lane);
    copy_words(G.sprop, S.sprop, sizeof(S.sprop), lane);
    copy_words(G.ck_rho, S.ck_rho, sizeof(S.ck_rho), lane);
    copy_words(G.ck_v, S.ck_v, sizeof(S.ck_v), lane);
    copy_words(G.end_ll, S.end_ll, sizeof(S.end_ll), lane);
    copy_words(G.end_lp, S.end_lp, sizeof(S.end_lp), lane);
}

__device__ __forceinline__ void sweep_load(const SweepState& G, NutsSub& S, int lane) {
    copy_words(&S.T, &G.T, sizeof(NutsState), lane);
    copy_words(S.left, G.left, sizeof(S.left), lane);
    copy_words(S.right, G.right, sizeof(S.right), lane);
    copy_words(S.prop, G.prop, sizeof(S.prop), lane);
    copy_words(S.sprop, G.sprop, sizeof(S.sprop), lane);
    copy_words(S.ck_rho, G.ck_rho, sizeof(S.ck_rho), lane);
    copy_words(S.ck_v, G.ck_v, sizeof(S.ck_v), lane);
    copy_words(S.end_ll, G.end_ll, sizeof(S.end_ll), lane);
    copy_words(S.end_lp, G.end_lp, sizeof(S.end_lp), lane);
}

// Every particle starts its transition; the next-position rows hold the
// current points until the first sweep replaces them.
__global__ __launch_bounds__(256) void sweep_init_kernel(SweepState* __restrict__ st, uint8_t* __restrict__ active,
                                                         const double* __restrict__ theta, double* __restrict__ x_next,
                                                         int P, int D) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P) return;
    st[p].phase = SW_START;
    active[p] = 1;
    for (int k = 0; k < D; ++k) x_next[(size_t)p * D + k] = theta[(size_t)p * D + k];
}

// One tree step of particle p = blockIdx.x: the transition's start on the
// first sweep, else the booking of the leaf whose likelihood ll_in / gl_in
// the batched likelihood has just computed; then either the next leaf's
// position (x_next, active = 1) or the transition's outputs (active = 0).
// The tree steps are out-of-line functions shared with nuts_kernel, and a
// function's register budget is the loosest of its callers': the occupancy
// bound here matches nuts_kernel's so the shared steps keep its budget.
__global__ __launch_bounds__(64, NUTS_WAVES_PER_SIMD) void nuts_sweep_kernel(NutsArgs a, PriorDesc pri, ParamMap pm,
                                                        SweepState* __restrict__ st,
                                                        const double* __restrict__ ll_in,
                                                        const double* __restrict__ gl_in,
                                                        double* __restrict__ x_next, uint8_t* __restrict__ active) {
    NutsShared& S = lds_shared<1>();
    NutsSub& U = lds_subs<1>()[0];
    const int p = blockIdx.x;
    const int lane = threadIdx.x;
    const int D = a.D;
    SweepState& G = st[p];
    const int phase = __builtin_amdgcn_readfirstlane(G.phase);
    if (phase == SW_DONE) return;
    const int run = a.state ? p / a.run_size : 0;
    if (a.state && a.state[(size_t)run * SMCGW_STATE_SIZE + SMCGW_ST_DONE] != 0.0) {
        if (lane == 0) { G.phase = SW_DONE; active[p] = 0; }   // a finished run's particles are left untouched
        return;
    }
    const double* chol = a.chol_pp ? a.chol + (size_t)p * D * D : a.state ? a.chol + (size_t)run * D * D : a.chol;
    load_factor(U, chol, D, lane);
    copy_words(&U.ev, a.events + event_index(a.ev_of_p, p, a.n_events), sizeof(DevEvent), lane);
    if (lane == 0) {
        share_arguments(S, a, pri, pm);
        U.p = p;
    }
    __syncthreads();
    derive_metric<1>(0, D, lane);
    if (phase == SW_START) {
        if (lane == 0) set_run(S.A, U.T, p, run);
        __syncthreads();
        if (lane < SUB_LANES) start_transition<1>(0, lane);
    } else {
        __syncthreads();   // the checkpoints take the factor's place
        sweep_load(G, U, lane);
        __syncthreads();
        if (lane < D) U.T.gl_new[lane] = gl_in[(size_t)p * D + lane];
        if (lane == 0) U.T.ll_new = ll_in[p];
    }
    __syncthreads();
    int cmd = CMD_DONE;
    if (lane < SUB_LANES) {
        cmd = advance<SMCGW_TARGET_GW, 1>(0, lane);
        bookkeep<1>(0, lane);
    }
    __syncthreads();
    cmd = __builtin_amdgcn_readfirstlane(cmd);
    if (cmd == CMD_DONE || __builtin_amdgcn_readfirstlane(U.T.stop)) {
        if (lane < SUB_LANES) write_outputs<1>(0, lane);
        if (lane == 0) { G.phase = SW_DONE; active[p] = 0; }
        return;
    }
    if (lane < SUB_LANES) aux_in_flight<SMCGW_TARGET_GW, 1>(0, lane);
    __syncthreads();
    if (lane < D) x_next[(size_t)p * D + lane] = U.T.x[lane];
    sweep_save(G, U, lane);
    if (lane == 0) { G.phase = SW_RUN; active[p] = 1; }
}

// Particles still building their tree (one workgroup).
__global__ __launch_bounds__(256) void sweep_count_kernel(const uint8_t* __restrict__ active, int P,
                                                          int* __restrict__ count) {
    __shared__ int part[256];
    int n = 0;
    for (int i = threadIdx.x; i < P; i += blockDim.x) n += active[i];
    part[threadIdx.x] = n;
    __syncthreads();
    if (threadIdx.x == 0) {
        int s = 0;
        for (int t = 0; t < 256; ++t) s += part[t];
        *count = s;
    }
}

}  // namespace smcgw

using namespace smcgw;

namespace {

template <class K>
int launch_persistent(smcgw_ctx* c, K kernel, int subs, int block, const NutsArgs& a, const PriorDesc& pri,
                      const ParamMap& pm, const TargetDesc& t) {
    auto it = c->resident.find((const void*)kernel);
    if (it == c->resident.end()) {
        int dev_cus = 0, per_cu = 0;
        if (hipDeviceGetAttribute(&dev_cus, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess)
            return SMCGW_ERR_HIP;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block, 0) != hipSuccess || per_cu < 1)
            per_cu = 1;
        it = c->resident.emplace((const void*)kernel, std::make_pair(dev_cus, per_cu)).first;
    }
    int per_cu = it->second.second;
    if (c->nuts_slots_per_cu > 0) per_cu = std::min(per_cu, c->nuts_slots_per_cu);
    const int grid = std::max(1, std::min(a.P, it->second.first * per_cu));
    NutsArgs b = a;
    // stripes only where particles wait: dealt out one by one, each queue has its share of fewer
    b.stripe = (long)grid * subs < a.P ? 16 : 1;
    hipLaunchKernelGGL(start_queues_kernel, dim3(1), dim3(64), 0, c->stream, a.queue, grid, subs, a.order ? 1 : 0);
    {
        TimedLaunch tl(c, SMCGW_KERNEL_NUTS);
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(block), 0, c->stream, b, pri, pm, t);
    }
    return hipGetLastError() == hipSuccess ? SMCGW_OK : SMCGW_ERR_HIP;
}

template <int NDET, int SUBS, int W>
int launch_gw_w(smcgw_ctx* c, int precision, const NutsArgs& a, const PriorDesc& pri, const ParamMap& pm,
                const TargetDesc& t) {
    if (precision == SMCGW_MIXED)
        return launch_persistent(c, nuts_kernel<NDET, SMCGW_MIXED, SMCGW_TARGET_GW, SUBS, W>, SUBS, W * 64, a, pri, pm,
                                 t);
    return launch_persistent(c, nuts_kernel<NDET, SMCGW_PLAIN_FP64, SMCGW_TARGET_GW, SUBS, W>, SUBS, W * 64, a, pri, pm,
                             t);
}

// The forms of a transition of P particles on events of at most `blocks` blocks of bins: one
// particle to a workgroup of four wavefronts, four (packed), or one to two wavefronts.  Packing pays where a
// leaf's serial work outweighs its bins and there are particles enough to fill the places: on
// a folded event of one block (milliseconds, one particle per workgroup / packed) 700
// particles take 6.2 / 6.6, 1000 6.2 / 6.6, 1536 6.8 / 6.6, 2048 7.9 / 7.2, 6144 14.5 / 9.6;
// without bins (a Gaussian in 16 dimensions) 256 take 0.18 / 0.20, 2048 0.36 / 0.26.  With two blocks of three detectors, trees of up to 15
// and of up to 255 leaves, four wavefronts / packed / two wavefronts, us: 1536 particles 240 / 270 / 232 and 2061 /
// 2263 / 2404; 2048 279 / 292 / 239 and 2104 / 2390 / 2821; 3000 352 / 268 / 310 and 2274 / 2836 / 2903; in FP64,
// where the bins weigh more, 1536 341 / 400 / 312 and 3202 / 3585 / 3603; 2048 401 / 448 / 339 and 3283 / 3991 / 4486;
// 4096 665 / 490 / 531 and 4142 / 5286 / 4645.  So MIXED packs from 2560 particles, and FP64 of three and four
// detectors, where a packed leaf waits too long for its neighbours' bins, takes two wavefronts from 1536, twice the
// trees in flight: the better of the other two on short trees.  With one and two detectors in FP64 the bins weigh
// less and packing is the better again from 2560 (900 bins of two, trees of up to 15 leaves: 4096 particles 530 / 396 /
// 472).  With four blocks the packed particles wait for each other's bins, most of all the long trees at the end, ms:
// 2048 take 10.9 / 11.8, and 6144 21.8 / 20.7.  The classes are the same either way, so the bits are.
enum NutsForm { FORM_SINGLE, FORM_PACKED, FORM_NARROW };
constexpr int PACK_FROM = 1280;
constexpr int PACK_FROM_2 = 2560;     // two blocks
constexpr int NARROW_FROM_2 = 1536;   // two blocks in FP64: up to PACK_FROM_2 with one or two detectors

NutsForm nuts_form(int P, int blocks, int precision, int n_det) {
    if (blocks <= 1) return P > PACK_FROM ? FORM_PACKED : FORM_SINGLE;
    if (blocks > 2) return FORM_SINGLE;
    if (precision == SMCGW_PLAIN_FP64 && (n_det > 2 || P <= PACK_FROM_2))
        return P > NARROW_FROM_2 ? FORM_NARROW : FORM_SINGLE;
    return P > PACK_FROM_2 ? FORM_PACKED : FORM_SINGLE;
}

template <int NDET>
int launch_gw(smcgw_ctx* c, int precision, const NutsArgs& a, const PriorDesc& pri, const ParamMap& pm,
              const TargetDesc& t) {
    int blocks = 0;
    for (const DevEvent& e : c->events) blocks = std::max(blocks, e.n_pad / TABLE_PAD);
    switch (c->nuts_waves) {
    case 2: return launch_gw_w<NDET, 1, 2>(c, precision, a, pri, pm, t);
    case 6: return launch_gw_w<NDET, 1, 6>(c, precision, a, pri, pm, t);
    case 8: return launch_gw_w<NDET, 1, 8>(c, precision, a, pri, pm, t);
    default: break;
    }
    const NutsForm form = nuts_form(a.P, blocks, precision, NDET);
    if (form == FORM_PACKED) return launch_gw_w<NDET, PACKED, 4>(c, precision, a, pri, pm, t);
    if (form == FORM_NARROW && !c->nuts_waves) return launch_gw_w<NDET, 1, 2>(c, precision, a, pri, pm, t);
    return launch_gw_w<NDET, 1, 4>(c, precision, a, pri, pm, t);
}

template <int TK>
int launch_analytic(smcgw_ctx* c, const NutsArgs& a, const PriorDesc& pri, const ParamMap& pm, const TargetDesc& t) {
    if (nuts_form(a.P, 0, SMCGW_PLAIN_FP64, 1) == FORM_PACKED)
        return launch_persistent(c, nuts_kernel<1, SMCGW_PLAIN_FP64, TK, PACKED, 1>, PACKED, 64, a, pri, pm, t);
    return launch_persistent(c, nuts_kernel<1, SMCGW_PLAIN_FP64, TK, 1, 1>, 1, 64, a, pri, pm, t);
}

}  // namespace

// The work-queue counter and the start-order buffer for P particles.
int smcgw::nuts_reserve(smcgw_ctx* c, int P, bool hint) {
    note_capture(c);
    if (!c->d_queue && hipMalloc(&c->d_queue, 256) != hipSuccess) return SMCGW_ERR_OOM;
    if (hint && P > c->order_cap) {
        give_up(c, c->d_order);
        c->d_order = nullptr;
        c->order_cap = 0;
        if (hipMalloc(&c->d_order, (size_t)P * sizeof(int32_t)) != hipSuccess) return SMCGW_ERR_OOM;
        c->order_cap = P;
    }
    return SMCGW_OK;
}

extern "C" int smcgw_nuts_step(smcgw_ctx* c, int P, int D, double* theta, double* logl, double* grad,
                               const double* chol, const smcgw_nuts_params* prm,
                               const int32_t* max_depth_per_particle, const int32_t* work_hint, int precision,
                               int32_t* depth, int32_t* n_leapfrog, uint8_t* divergent, double* accept_stat) {
    if (!c || !prm || P < 0 || D <= 0 || D > MAXDIM || (P > 0 && (!theta || !logl || !grad || !chol)))
        return SMCGW_ERR_INVALID;
    if (precision != SMCGW_PLAIN_FP64 && precision != SMCGW_MIXED) return SMCGW_ERR_INVALID;
    if (prm->max_depth < 0 || prm->max_depth > SMCGW_MAX_DEPTH || !(prm->step > 0.0) ||
        (!prm->beta_device && !(prm->beta >= 0.0)) ||
        !(prm->max_delta_h > 0.0) || (prm->chol_per_particle != 0 && prm->chol_per_particle != 1) ||
        prm->reserved != 0 || prm->reserved2 != 0)
        return SMCGW_ERR_INVALID;
    if (prm->state_device && (prm->run_size < 1 || P % prm->run_size != 0 || P / prm->run_size > SMCGW_MAX_RUNS))
        return SMCGW_ERR_INVALID;
    if (!c->prior_set || c->prior.dim != D) return SMCGW_ERR_NOT_INIT;
    const int kind = c->target.kind;
    if (kind == SMCGW_TARGET_GW) {
        if (c->events.empty() || c->pmap.dim != D) return SMCGW_ERR_NOT_INIT;
    } else if (c->target.dim != D) {
        return SMCGW_ERR_NOT_INIT;
    }
    if (P == 0) return SMCGW_OK;
    if (hipSetDevice(c->device) != hipSuccess) return SMCGW_ERR_HIP;
    if (nuts_reserve(c, P, work_hint != nullptr) != SMCGW_OK) return SMCGW_ERR_OOM;
    if (work_hint) {
        hipLaunchKernelGGL(order_kernel, dim3(1), dim3(ORDER_THREADS), 0, c->stream, work_hint, P, c->d_order);
        if (hipGetLastError() != hipSuccess) return SMCGW_ERR_HIP;
    }
    NutsArgs a;
    a.P = P;
    a.D = D;
    a.theta = theta;
    a.logl = logl;
    a.grad = grad;
    a.chol = chol;
    a.step = prm->step;
    a.beta = prm->beta;
    a.max_dh = prm->max_delta_h;
    a.max_depth = prm->max_depth;
    a.uturn = prm->uturn ? 1 : 0;
    a.seed = prm->seed;
    a.iteration = prm->iteration;
    a.md_per_p = max_depth_per_particle;
    a.depth_out = depth;
    a.nlf_out = n_leapfrog;
    a.div_out = divergent;
    a.acc_out = accept_stat;
    a.events = c->d_events;
    a.n_events = (int)c->events.size();
    a.ev_of_p = c->ev_of_p;
    a.queue = (int*)c->d_queue;
    a.order = work_hint ? c->d_order : nullptr;
    a.priority = c->nuts_priority;
    a.chol_pp = prm->chol_per_particle;
    a.beta_dev = prm->beta_device;
    a.state = prm->state_device;
    a.run_size = prm->state_device ? prm->run_size : P;
    const TargetDesc t = c->target;
    switch (kind) {
    case SMCGW_TARGET_GW:
        switch (c->n_det) {
        case 1: return launch_gw<1>(c, precision, a, c->prior, c->pmap, t);
        case 2: return launch_gw<2>(c, precision, a, c->prior, c->pmap, t);
        case 3: return launch_gw<3>(c, precision, a, c->prior, c->pmap, t);
        case 4: return launch_gw<4>(c, precision, a, c->prior, c->pmap, t);
        default: return SMCGW_ERR_SHAPE;
        }
    case SMCGW_TARGET_GAUSS:
        return launch_analytic<SMCGW_TARGET_GAUSS>(c, a, c->prior, c->pmap, t);
    case SMCGW_TARGET_GAUSS_X_GAUSS:
        return launch_analytic<SMCGW_TARGET_GAUSS_X_GAUSS>(c, a, c->prior, c->pmap, t);
    case SMCGW_TARGET_BIMODAL:
        return launch_analytic<SMCGW_TARGET_BIMODAL>(c, a, c->prior, c->pmap, t);
    default:
        return SMCGW_ERR_INVALID;
    }
}

extern "C" int smcgw_autotune_nuts(smcgw_ctx* c, int P, int D, const double* theta, const double* logl,
                                   const double* grad, const double* chol, const smcgw_nuts_params* prm, int precision,
                                   int trials, int* best_waves, double* times_ms) {
    if (!c || !prm || P < 1 || D <= 0 || D > MAXDIM || !theta || !logl || !grad || !chol || trials < 1 || trials > 16)
        return SMCGW_ERR_INVALID;
    if (hipSetDevice(c->device) != hipSuccess) return SMCGW_ERR_HIP;
    const size_t nx = (size_t)P * D * sizeof(double), nl = (size_t)P * sizeof(double);
    double *x = nullptr, *l = nullptr, *g = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    int rc = SMCGW_OK;
    if (hipMalloc(&x, nx) != hipSuccess || hipMalloc(&l, nl) != hipSuccess || hipMalloc(&g, nx) != hipSuccess ||
        hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)
        rc = SMCGW_ERR_OOM;
    const int widths[4] = {2, 4, 6, 8};
    double med[4] = {0.0, 0.0, 0.0, 0.0};
    const int saved = c->nuts_waves;
    for (int w = 0; w < 4 && rc == SMCGW_OK; ++w) {
        c->nuts_waves = widths[w];
        float t[16];
        for (int k = 0; k < trials && rc == SMCGW_OK; ++k) {
            if (hipMemcpyAsync(x, theta, nx, hipMemcpyDeviceToDevice, c->stream) != hipSuccess ||
                hipMemcpyAsync(l, logl, nl, hipMemcpyDeviceToDevice, c->stream) != hipSuccess ||
                hipMemcpyAsync(g, grad, nx, hipMemcpyDeviceToDevice, c->stream) != hipSuccess ||
                hipEventRecord(e0, c->stream) != hipSuccess) {
                rc = SMCGW_ERR_HIP;
                break;
            }
            rc = smcgw_nuts_step(c, P, D, x, l, g, chol, prm, nullptr, nullptr, precision, nullptr, nullptr, nullptr,
                                 nullptr);
            if (rc != SMCGW_OK) break;
            if (hipEventRecord(e1, c->stream) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                hipEventElapsedTime(&t[k], e0, e1) != hipSuccess)
                rc = SMCGW_ERR_HIP;
        }
        if (rc == SMCGW_OK) {
            std::sort(t, t + trials);
            med[w] = t[trials / 2];
        }
    }
    int best = saved;
    if (rc == SMCGW_OK) {
        int bi = 0;
        for (int w = 1; w < 4; ++w)
            if (med[w] < med[bi]) bi = w;
        best = widths[bi];
        if (best_waves) *best_waves = best;
        if (times_ms)
            for (int w = 0; w < 4; ++w) times_ms[w] = med[w];
    }
    c->nuts_waves = best;
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    (void)hipFree(x);
    (void)hipFree(l);
    (void)hipFree(g);
    return rc;
}

namespace {

// Scratch of the sweep form: tree states [P], next positions [P][D], their
// logL [P] and gradients [P][D], active flags [P] and the active count.
struct SweepScratch {
    SweepState* st;
    double *x_next, *ll, *gl;
    uint8_t* active;
    int* count;
};

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

int sweep_reserve(smcgw_ctx* c, int P, int D, SweepScratch& s) {
    const size_t b_st = align256((size_t)P * sizeof(SweepState));
    const size_t b_x = align256((size_t)P * D * sizeof(double));
    const size_t b_ll = align256((size_t)P * sizeof(double));
    const size_t b_act = align256((size_t)P);
    const size_t need = b_st + 2 * b_x + b_ll + b_act + 256;
    if (need > c->sweep_bytes) {
        c->sweep_free();
        if (hipMalloc(&c->d_sweep, need) != hipSuccess) return SMCGW_ERR_OOM;
        c->sweep_bytes = need;
    }
    char* base = (char*)c->d_sweep;
    s.st = (SweepState*)base;
    s.x_next = (double*)(base + b_st);
    s.ll = (double*)(base + b_st + b_x);
    s.gl = (double*)(base + b_st + b_x + b_ll);
    s.active = (uint8_t*)(base + b_st + 2 * b_x + b_ll);
    s.count = (int*)(base + b_st + 2 * b_x + b_ll + b_act);
    return SMCGW_OK;
}

// One group of sweeps and the active count, on the context's stream.
int queue_sweep_group(smcgw_ctx* c, const NutsArgs& a, const SweepScratch& s, int sweeps) {
    for (int k = 0; k < sweeps; ++k) {
        {
            TimedLaunch tl(c, SMCGW_KERNEL_NUTS);
            hipLaunchKernelGGL(nuts_sweep_kernel, dim3(a.P), dim3(64), 0, c->stream, a, c->prior, c->pmap, s.st,
                               (const double*)s.ll, (const double*)s.gl, s.x_next, s.active);
        }
        if (hipGetLastError() != hipSuccess) return SMCGW_ERR_HIP;
        const int rc = queue_loglike_tangent(c, a.P, c->ev_of_p, s.x_next, s.active, s.ll, s.gl);
        if (rc) return rc;
    }
    hipLaunchKernelGGL(sweep_count_kernel, dim3(1), dim3(256), 0, c->stream, (const uint8_t*)s.active, a.P, s.count);
    return hipGetLastError() == hipSuccess ? SMCGW_OK : SMCGW_ERR_HIP;
}

}  // namespace

extern "C" int smcgw_nuts_step_sweeps(smcgw_ctx* c, int P, int D, double* theta, double* logl, double* grad,
                                      const double* chol, const smcgw_nuts_params* prm,
                                      const int32_t* max_depth_per_particle, int32_t* depth, int32_t* n_leapfrog,
                                      uint8_t* divergent, double* accept_stat, int sweeps_per_group,
                                      int* n_sweeps_host) {
    if (!c || !prm || P < 0 || D <= 0 || D > MAXDIM || (P > 0 && (!theta || !logl || !grad || !chol)) ||
        sweeps_per_group < 1 || sweeps_per_group > 64)
        return SMCGW_ERR_INVALID;
    if (prm->max_depth < 0 || prm->max_depth > SMCGW_MAX_DEPTH || !(prm->step > 0.0) ||
        (!prm->beta_device && !prm->state_device && !(prm->beta >= 0.0)) || !(prm->max_delta_h > 0.0) ||
        (prm->chol_per_particle != 0 && prm->chol_per_particle != 1) || prm->reserved != 0 || prm->reserved2 != 0)
        return SMCGW_ERR_INVALID;
    if (prm->state_device && (prm->run_size < 1 || P % prm->run_size != 0 || P / prm->run_size > SMCGW_MAX_RUNS))
        return SMCGW_ERR_INVALID;
    if (!c->prior_set || c->prior.dim != D || c->target.kind != SMCGW_TARGET_GW || c->events.empty() ||
        c->pmap.dim != D)
        return SMCGW_ERR_NOT_INIT;
    if (!tangent_supported(c)) return SMCGW_ERR_INVALID;
    if (n_sweeps_host) *n_sweeps_host = 0;
    if (P == 0) return SMCGW_OK;
    if (hipSetDevice(c->device) != hipSuccess) return SMCGW_ERR_HIP;
    SweepScratch s;
    int rc = tangent_reserve(c, P);
    if (rc == SMCGW_OK) rc = sweep_reserve(c, P, D, s);
    int* hp = (int*)pinned(c);
    if (rc) return rc;
    if (!hp) return SMCGW_ERR_OOM;
    NutsArgs a{};
    a.P = P;
    a.D = D;
    a.theta = theta;
    a.logl = logl;
    a.grad = grad;
    a.chol = chol;
    a.step = prm->step;
    a.beta = prm->beta;
    a.max_dh = prm->max_delta_h;
    a.max_depth = prm->max_depth;
    a.uturn = prm->uturn ? 1 : 0;
    a.seed = prm->seed;
    a.iteration = prm->iteration;
    a.md_per_p = max_depth_per_particle;
    a.depth_out = depth;
    a.nlf_out = n_leapfrog;
    a.div_out = divergent;
    a.acc_out = accept_stat;
    a.events = c->d_events;
    a.n_events = (int)c->events.size();
    a.ev_of_p = c->ev_of_p;
    a.chol_pp = prm->chol_per_particle;
    a.beta_dev = prm->beta_device;
    a.state = prm->state_device;
    a.run_size = prm->state_device ? prm->run_size : P;
    hipLaunchKernelGGL(sweep_init_kernel, dim3((P + 255) / 256), dim3(256), 0, c->stream, s.st, s.active,
                       (const double*)theta, s.x_next, P, D);
    if (hipGetLastError() != hipSuccess) return SMCGW_ERR_HIP;
    // the group graph is captured once for these arguments and replayed
    std::vector<unsigned char> key(sizeof(NutsArgs) + sizeof(PriorDesc) + sizeof(ParamMap) + 3 * sizeof(int));
    unsigned char* kp = key.data();
    std::memcpy(kp, &a, sizeof(a));
    std::memcpy(kp + sizeof(a), &c->prior, sizeof(PriorDesc));
    std::memcpy(kp + sizeof(a) + sizeof(PriorDesc), &c->pmap, sizeof(ParamMap));
    const int extra[3] = {sweeps_per_group, c->n_det, (int)(c->timing_mask != 0)};
    std::memcpy(kp + sizeof(a) + sizeof(PriorDesc) + sizeof(ParamMap), extra, sizeof(extra));
    if (key != c->sweep_key || !c->sweep_exec) {
        if (c->sweep_exec) (void)hipGraphExecDestroy(c->sweep_exec);
        if (c->sweep_graph) (void)hipGraphDestroy(c->sweep_graph);
        c->sweep_exec = nullptr;
        c->sweep_graph = nullptr;
        c->sweep_key.clear();
        hipStream_t cap = nullptr;
        if (hipStreamCreateWithFlags(&cap, hipStreamNonBlocking) != hipSuccess) return SMCGW_ERR_HIP;
        const hipStream_t saved = c->stream;
        const unsigned saved_mask = c->timing_mask;
        c->stream = cap;
        c->timing_mask = 0;   // no timing events inside the graph
        bool ok = hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal) == hipSuccess;
        hipGraph_t g = nullptr;
        if (ok) {
            rc = queue_sweep_group(c, a, s, sweeps_per_group);
            ok = hipStreamEndCapture(cap, &g) == hipSuccess && rc == SMCGW_OK;
        }
        c->stream = saved;
        c->timing_mask = saved_mask;
        (void)hipStreamDestroy(cap);
        if (ok) ok = hipGraphInstantiate(&c->sweep_exec, g, nullptr, nullptr, 0) == hipSuccess;
        if (!ok) {
            if (g) (void)hipGraphDestroy(g);
            c->sweep_exec = nullptr;
            return rc ? rc : SMCGW_ERR_HIP;
        }
        c->sweep_graph = g;
        c->sweep_key = key;
    }
    // every transition ends within 2^max_depth sweeps (one leaf per sweep, the start included)
    const int md = max_depth_per_particle ? SMCGW_MAX_DEPTH : prm->max_depth;
    const long limit = (1L << md) + 1;
    long sweeps = 0;
    for (;;) {
        if (hipGraphLaunch(c->sweep_exec, c->stream) != hipSuccess) return SMCGW_ERR_HIP;
        sweeps += sweeps_per_group;
        if (hipMemcpyAsync(hp, s.count, sizeof(int), hipMemcpyDeviceToHost, c->stream) != hipSuccess ||
            hipStreamSynchronize(c->stream) != hipSuccess)
            return SMCGW_ERR_HIP;
        if (*hp == 0) break;
        if (sweeps > limit + sweeps_per_group) return SMCGW_ERR_HIP;
    }
    if (n_sweeps_host) *n_sweeps_host = (int)sweeps;
    return SMCGW_OK;
}
