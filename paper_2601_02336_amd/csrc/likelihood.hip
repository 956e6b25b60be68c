// Batched GW log-likelihood and hand-written adjoint gradient.
//
// logL = -1/2 <d-h|d-h>, <a|b> = 4 Re sum_j a_j* b_j / S_j df (arXiv:2601.02336,
// Sec. 2, Eq. 2), expanded as
//   logL = -<d|d>/2 + sum_d [ Re(P'_d Z_d) - |P'_d|^2 H_d / 2 ],
//   Z_d  = sum_j u_dj e^{-2 pi i Phi_dj},   u_dj = 4 df conj(d_dj) f_j^-7/6 / S_dj,
// with P'_d = C_A P_d the per-particle amplitude and projection and Phi_dj the
// phase in cycles.  The adjoint of Z_d with respect to Phi_dj is
//   dlogL/dPhi_dj = 2 pi q_dj,  q_dj = Im(P'_d u_dj e^{-2 pi i Phi_dj}),
// so the gradient needs only the bin moments
//   G_b = sum_j psibar_j B_b(f_j),  psibar_j = sum_d q_dj,   T_d = sum_j q_dj f_j,
// accumulated in the same pass as Z_d; the epilogue chains them through the
// prologue's Jacobians.
//
// Kernels:
//   bins (one wavefront per particle): the workgroup builds the coefficient
//        blocks of its particles in LDS (eight lanes per particle, FP64 dual
//        numbers with one tangent per lane), then each wavefront walks the bins
//        of its particles (lanes stride the frequency bins, the shared per-bin
//        tables are read coalesced, each lane keeps its own partial sums) and one
//        lane per particle forms logL and the gradient from the moments.
//   point, segment, finish, finish_point (few particles): a particle's bins spread over
//        wavefronts.
//   prep: the coefficient blocks alone, in global memory, for the plain
//        comparison form and the waveform.
//   sort_events: start order of a batch over events of different lengths.
#include <algorithm>
#include <functional>
#include <vector>

#include "binloop.h"
#include "coeffs.h"
#include "common.h"
#include "context.h"

namespace smcgw {

constexpr int LL_WAVES = 4;   // wavefronts per workgroup
constexpr int LDS_BYTES = 160 * 1024;   // of a compute unit

// Eight lanes per particle, as the persistent NUTS kernel splits a leaf's
// prologue: lanes 0-3 carry one intrinsic tangent each (Mc, q, chi1, chi2)
// while lanes 4-7 take the sines and cosines of the four extrinsic angles;
// then lane 4k + d (k = 0, 1) builds detector d with its ra (k = 0) or dec
// (k = 1) tangent, and lane 0 the amplitude.  One particle's chain is a
// quarter of the one-lane prologue's.  Without the gradient there are no tangents:
// lane 0 has the intrinsic part and lanes 0-3 a detector each.  Called by every thread
// of the workgroup (it holds a barrier); ang is the particle's exchange of the angles.
constexpr int PREP_LANES = 8;
constexpr int PREP_PER_BLOCK = 256 / PREP_LANES;
static_assert(2 * MAXDET == PREP_LANES && ANG_COUNT == PREP_LANES - 4, "prologue lane split");

template <bool GRAD>
__device__ __forceinline__ void prologue_lanes(const DevEvent& ev, const ParamMap& pm, const double* __restrict__ x,
                                               double* c, double (*ang_sh)[2], int j, bool live) {
    double th[NPAR];
    if (live) {
        expand_params(pm, x, th);
        if (j < 4) {
            if (GRAD) prep_intrinsic_n<1>(ev, th, c, j, j == 0);
            else if (j == 0) prep_intrinsic_n<0>(ev, th, c, 0, true);
        } else {
            double sn, cs;
            sincos(extrinsic_angle(ev, th, j - 4), &sn, &cs);
            ang_sh[j - 4][0] = sn;
            ang_sh[j - 4][1] = cs;
        }
    }
    __syncthreads();
    if (live) {
        ExtAngles ang;
#pragma unroll
        for (int k = 0; k < ANG_COUNT; ++k) { ang.sc[k][0] = ang_sh[k][0]; ang.sc[k][1] = ang_sh[k][1]; }
        const int k = j / MAXDET, d = j % MAXDET;
        if (GRAD) prep_extrinsic_det_n<1>(ev, th, ang, c, d, k, k == 0);
        else if (k == 0) prep_extrinsic_det_n<0>(ev, th, ang, c, d, 0, true);
        if (j == 0) {
            if (GRAD) prep_extrinsic_common(ev, th, c);
            else c[CB_AMP] = extrinsic_amplitude(ev, th);
        }
    }
}

__global__ __launch_bounds__(256) void prep_kernel(const DevEvent* __restrict__ evs, int n_events,
                                                   const int32_t* __restrict__ ev_of_p, ParamMap pm, int P,
                                                   const double* __restrict__ theta, double* __restrict__ cb) {
    __shared__ double ang_sh[PREP_PER_BLOCK][ANG_COUNT][2];
    const int g = threadIdx.x / PREP_LANES;
    const int p = blockIdx.x * PREP_PER_BLOCK + g;
    const int q = p < P ? p : 0;
    prologue_lanes<true>(evs[event_index(ev_of_p, q, n_events)], pm, theta + (size_t)q * pm.dim,
                         cb + (size_t)q * CB_SIZE, ang_sh[g], threadIdx.x % PREP_LANES, p < P);
}

// logL and gradient of particle p from its coefficient block and moments (one lane).
template <bool GRAD>
__device__ __forceinline__ void write_result(const DevEvent& ev, const ParamMap& pm, const double* cb,
                                             const double* mom, int p, double* __restrict__ logl,
                                             double* __restrict__ grad) {
    if (GRAD) {
        double g[NPAR];
        logl[p] = finish_particle(ev, cb, mom, g);
        for (int q = 0; q < pm.dim; ++q) grad[(size_t)p * pm.dim + q] = g[pm.idx[q]];
    } else {
        logl[p] = finish_value(ev, cb, mom);
    }
}

// Particle i of the start order (NULL: index order).  The order lies in scratch that overlapping calls share: an entry
// of another call's, larger batch must not lead out of this one's arrays.
__device__ __forceinline__ int ordered_particle(const int32_t* __restrict__ order, int i, int P) {
    return order ? (int)min((unsigned)order[i], (unsigned)P - 1u) : i;
}

// Particles [LL_WAVES per_wave blockIdx.x, ...) of the start order (order NULL:
// index order), per_wave <= 8 for each wavefront.  Bound by the VALU issue rate
// of the bin loop; the coefficient blocks and moments stay in LDS, so a call is
// one launch (a prologue launch of its own cost 6 to 17 us a call: 4096 particles
// of 3 x 8033 bins took 83.3 us with it and take 77.6 without, 6000 of a folded
// event 25.0 and 18.0).  The workgroup's first lanes form the results of all its
// particles together, where a lane of every wavefront took its instructions four
// times (6000 of a folded event 17.2 -> 16.0 us, 16384 of eight events 974 -> 955).
// GRAD = false leaves the tangents and the gradient's moments out (20000 values of
// 1969 bins 50.1 -> 46.7 us without the tangents); logL is the same bit for bit.
//
// MULTI: events of several segments, whose wavefronts keep columns of lane sums behind the particles in LDS; with
// three detectors four workgroups just fit a compute unit, as many as its registers hold.  Without them a particle's
// block is spread over the banks.
struct LoglikeParticle {
    double cb[CB_SIZE];
    union {
        double ang[ANG_COUNT][2];   // prologue
        double mom[MOM_SIZE];       // bins
    };
};
template <bool MULTI> struct LoglikeShared : LoglikeParticle {};
template <> struct LoglikeShared<false> : LoglikeParticle { double pad[MOM_SIZE]; };
template <bool MULTI>
size_t loglike_lds(int per_wave, int n_moments) {
    return LL_WAVES * (per_wave * sizeof(LoglikeShared<MULTI>) + (MULTI ? 64 * n_moments * sizeof(double) : 0));
}
static_assert(4 * LL_WAVES * (sizeof(LoglikeShared<true>) + 64 * moments(3, true) * sizeof(double)) <= LDS_BYTES, "four fit");

template <int NDET, int PREC, bool GRAD, bool MULTI>
__device__ __forceinline__ void loglike_workgroup(const DevEvent* __restrict__ evs, int n_events,
                                                  const int32_t* __restrict__ ev_of_p,
                                                  const int32_t* __restrict__ order, const ParamMap& pm, int P,
                                                  int per_wave, const double* __restrict__ theta,
                                                  double* __restrict__ logl, double* __restrict__ grad) {
    extern __shared__ double lds[];
    LoglikeShared<MULTI>* sh = (LoglikeShared<MULTI>*)lds;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int first = blockIdx.x * LL_WAVES * per_wave;
    {
        // prologue: the workgroup's particles on consecutive groups of eight lanes
        const int g = threadIdx.x / PREP_LANES;
        const bool live = g < LL_WAVES * per_wave && first + g < P;
        const int i = live ? first + g : 0, p = ordered_particle(order, i, P);
        LoglikeParticle& s = sh[live ? g : 0];
        prologue_lanes<GRAD>(evs[event_index(ev_of_p, p, n_events)], pm, theta + (size_t)p * pm.dim, s.cb, s.ang,
                             threadIdx.x % PREP_LANES, live);
    }
    __syncthreads();
    // wavefront w takes the particles w per_wave, ... of the workgroup
    const int g0 = wave * per_wave;
    const int n = min(per_wave, P - first - g0);
    double* col = (double*)(sh + LL_WAVES * per_wave) + wave * 64 * moments(NDET, GRAD);
    for (int g = g0; g < g0 + n; ++g) {
        const int p = ordered_particle(order, first + g, P);
        const int e = __builtin_amdgcn_readfirstlane(event_index(ev_of_p, p, n_events));
        const BinCoef k = load_coef(sh[g].cb);
        const TableView t = PREC == SMCGW_MIXED ? mixed_tables<NDET>(evs + e) : fp64_tables<NDET>(evs + e);
        // (values alone: without the test in the loop the compiler moves the loads behind their block's arithmetic, 1024
        // particles of 4 x 8033 bins 26.5 -> 32.7 us)
        constexpr BinLoop LOOP = MULTI && PREC == SMCGW_MIXED && GRAD && NDET <= 3 ? LOOP_TIGHT
                               : MULTI || !GRAD ? LOOP_SEGMENTS : LOOP_ALL;
        if (PREC == SMCGW_MIXED)
            event_moments<NDET, GRAD, LOOP, BinPair<NDET, float2>, MixedAcc<NDET, GRAD>>(t, k, sh[g].mom, col);
        else
            event_moments<NDET, GRAD, LOOP, BinPair<NDET, double2>, Fp64Acc<NDET, GRAD>>(t, k, sh[g].mom, col);
    }
    __syncthreads();
    // results: a lane per particle of the workgroup
    if ((int)threadIdx.x < min(LL_WAVES * per_wave, P - first)) {
        const LoglikeParticle& s = sh[threadIdx.x];
        const int p = ordered_particle(order, first + threadIdx.x, P);
        write_result<GRAD>(evs[event_index(ev_of_p, p, n_events)], pm, s.cb, s.mom, p, logl, grad);
    }
}

// Wavefronts per SIMD the register budget is sized for: four (128 registers)
// where the loop's sums fit, so that a launch of one particle per wavefront
// keeps 4096 particles on the chip at once, else three.
__host__ __device__ constexpr int ll_residents(int n_det, bool grad, int precision) {
    return precision == SMCGW_MIXED ? (n_det < 4 ? 4 : 3) : n_det <= 2 || !grad ? 4 : 3;
}

template <int NDET, bool GRAD, bool MULTI>
__global__ __launch_bounds__(64 * LL_WAVES, ll_residents(NDET, GRAD, SMCGW_MIXED)) void bins_mixed_kernel(
    const DevEvent* __restrict__ evs, int n_events, const int32_t* __restrict__ ev_of_p,
    const int32_t* __restrict__ order, ParamMap pm, int P, int per_wave, const double* __restrict__ theta,
    double* __restrict__ logl, double* __restrict__ grad) {
    loglike_workgroup<NDET, SMCGW_MIXED, GRAD, MULTI>(evs, n_events, ev_of_p, order, pm, P, per_wave, theta, logl,
                                             grad);
}

template <int NDET, bool GRAD, bool MULTI>
__global__ __launch_bounds__(64 * LL_WAVES, ll_residents(NDET, GRAD, SMCGW_PLAIN_FP64)) void bins_fp64_kernel(
    const DevEvent* __restrict__ evs, int n_events, const int32_t* __restrict__ ev_of_p,
    const int32_t* __restrict__ order, ParamMap pm, int P, int per_wave, const double* __restrict__ theta,
    double* __restrict__ logl, double* __restrict__ grad) {
    loglike_workgroup<NDET, SMCGW_PLAIN_FP64, GRAD, MULTI>(evs, n_events, ev_of_p, order, pm, P, per_wave, theta, logl,
                                             grad);
}

// ------------------------------------------------------------ few particles
// A launch of one wavefront per particle leaves most of the chip idle when
// there are few particles: one particle of 3 x 8033 bins kept one SIMD busy for
// 20 us, 37 of a 259585-bin event 37 of 1024 SIMDs for 630.  Two ways to spread
// a particle, both to the same bits:
//   segment_kernel: a wavefront per segment (those 37 particles: 636 -> 54 us);
//   point_kernel:   a workgroup of 16 wavefronts per segment, for so few that even
//       the segments leave compute units idle (one particle of 8033 bins:
//       29.9 -> 15.8 us, of 259585 bins: 630 -> 31).  A lane adds its FP64 terms
//       one after the other over the segment's blocks, so the work is split by
//       kind: first every wavefront takes one block's bins (FP32 terms, their
//       partial sums over the block, psibar of every bin, all into LDS), then one
//       wavefront per moment adds its lanes' terms in block order.
// Events of one segment finish there.  Of more, a segment_kernel workgroup leaves the moments of its group of
// segments and finish_kernel adds the groups; point_kernel leaves the lanes' sums of its segment and
// finish_point_kernel does both.
constexpr int PT_WAVES = 16;
constexpr int PT_BLOCKS = PT_WAVES;   // blocks in LDS at once; a segment is one or two such rounds
constexpr int PT_THREADS = 64 * PT_WAVES;

template <int NDET>
struct PointPartials {      // one block's terms
    float z[3 * NDET][64];  // zr, zi, tq of every lane, in mom_* order
};

// Prologue on three wavefronts of the workgroup; the caller's barrier follows.
__device__ __forceinline__ void point_prologue(const DevEvent& ev, const ParamMap& pm, const double* __restrict__ x,
                                               double* cb, double (*ang_sh)[2], int wave, int lane) {
    if (wave > 2 || lane >= PREP_LANES) return;
    double th[NPAR];
    expand_params(pm, x, th);
    if (wave == 0 && lane < 4) prep_intrinsic_n<1>(ev, th, cb, lane, lane == 0);
    if (wave == 1) {
        if (lane < ANG_COUNT) {
            double sn, cs;
            sincos(extrinsic_angle(ev, th, lane), &sn, &cs);
            ang_sh[lane][0] = sn;
            ang_sh[lane][1] = cs;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        ExtAngles ang;
#pragma unroll
        for (int k = 0; k < ANG_COUNT; ++k) { ang.sc[k][0] = ang_sh[k][0]; ang.sc[k][1] = ang_sh[k][1]; }
        const int k = lane / MAXDET;
        prep_extrinsic_det_n<1>(ev, th, ang, cb, lane % MAXDET, k, k == 0);
    }
    if (wave == 2 && lane == 0) prep_extrinsic_common(ev, th, cb);
}

// Terms of block blk (its chunks below t.chunks): psibar of every bin to psi and
// its f^1/3 to u, the block's partial sums to part.
template <int NDET, bool GRAD>
__device__ __forceinline__ void point_terms(const TableView& t, const BinCoef& k, int blk, float* psi, double* u,
                                            PointPartials<NDET>& part) {
    const unsigned lane = threadIdx.x & 63;
    MixedAcc<NDET, GRAD> A;
#pragma unroll
    for (int d = 0; d < NDET; ++d) { A.pr[d] = uniform_f((float)k.pr[d]); A.pim[d] = uniform_f((float)k.pi[d]); }
    A.clear();
    const int n = min(BLK_CHUNKS, t.chunks - blk * BLK_CHUNKS);
    constexpr int DEPTH = NDET < 3 ? 4 : 3;   // chunks in flight, by the registers there are
    BinPair<NDET, float2> x[DEPTH];
#pragma unroll
    for (int c = 0; c < DEPTH; ++c) load_chunk(x[c], t, blk * TABLE_PAD + CHUNK_BINS * min(c, n - 1), lane);
#pragma unroll
    for (int c = 0; c < BLK_CHUNKS; ++c)
        if (c < n) {
            double Ba[NBASIS], Bb[NBASIS];
            const float a = A.terms(k, x[c % DEPTH].b[0], c == 0, Ba);
            const float b = A.terms(k, x[c % DEPTH].b[1], false, Bb);
            if (c + DEPTH < BLK_CHUNKS)
                load_chunk(x[c % DEPTH], t, blk * TABLE_PAD + CHUNK_BINS * min(c + DEPTH, n - 1), lane);
            if (GRAD) {
                *(float2*)(psi + CHUNK_BINS * c + 2 * lane) = make_float2(a, b);
                *(double2*)(u + CHUNK_BINS * c + 2 * lane) = make_double2(Ba[B_P13], Bb[B_P13]);
            }
        }
#pragma unroll
    for (int d = 0; d < NDET; ++d) {
        part.z[mom_zr(NDET, d)][lane] = A.zr[d];
        part.z[mom_zi(NDET, d)][lane] = A.zi[d];
        if (GRAD) part.z[mom_t(NDET, d)][lane] = A.tq[d];
    }
}

// One bin's term onto the lane sum s of basis moment B (0: the constant), with
// the basis row as basis_rows forms it from w, ln f and u = f^1/3.
template <int B>
__device__ __forceinline__ double point_add(double s, float psib, double w, double l, double u) {
    const double pb = (double)psib;
    if (B == 0) return s + pb;
    const double w2 = w * w, w3 = w2 * w;
    const double row = B == 1 + B_M53 ? w3 * w2 : B == 1 + B_M1 ? w3 : B == 1 + B_M23 ? w2 : B == 1 + B_M13 ? w
                     : B == 1 + B_LN ? l : B == 1 + B_P13 ? u : B == 1 + B_P13LN ? u * l : u * u;
    return fma(pb, row, s);
}

// Calls f.run<B>() for the wave-uniform B = wave < NCOEF.
template <class F>
__device__ __forceinline__ void for_basis(int wave, F& f) {
    switch (wave) {
    case 0: f.template run<0>(); break;
    case 1: f.template run<1>(); break;
    case 2: f.template run<2>(); break;
    case 3: f.template run<3>(); break;
    case 4: f.template run<4>(); break;
    case 5: f.template run<5>(); break;
    case 6: f.template run<6>(); break;
    case 7: f.template run<7>(); break;
    case 8: f.template run<8>(); break;
    default: break;
    }
}
static_assert(NCOEF == 9, "for_basis lists the basis moments");

// Lane sums of a basis moment over n chunks from chunk c0 in the bin loop's
// order: psibar and f^1/3 from LDS, at most one table row from the cache (the
// terms have just read it; a second row would halve the chunks in flight).
struct PointBasisSum {
    const TableView& t;
    const float* psi;
    const double* u;
    int c0, n;
    double s;
    template <int B>
    __device__ __forceinline__ void run() {
        const unsigned lane = threadIdx.x & 63;
        constexpr bool W = B >= 1 && B <= 1 + B_M13, L = B == 1 + B_LN || B == 1 + B_P13LN, U = B >= 1 + B_P13;
        constexpr int DEPTH = 8;   // chunks in flight
        double2 x[DEPTH];
        auto load = [&](double2& v, int c) {
            if (W || L) v = buf_f64x2(t.fwl, lane * 16u, ((W ? ROW_W : ROW_LN) * t.npad + (c0 + c) * CHUNK_BINS) * 8);
        };
        auto add = [&](const double2& v, int c) {
            const float2 p = *(const float2*)(psi + c * CHUNK_BINS + 2 * lane);
            double2 q = make_double2(0.0, 0.0);
            if (U) q = *(const double2*)(u + c * CHUNK_BINS + 2 * lane);
            s = point_add<B>(s, p.x, v.x, v.x, q.x);
            s = point_add<B>(s, p.y, v.y, v.y, q.y);
        };
        const int last = n - 1;
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) load(x[d], min(d, last));
        int c = 0;
        for (; c + DEPTH <= n; c += DEPTH) {
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                add(x[d], c + d);
                load(x[d], min(c + d + DEPTH, last));
            }
        }
#pragma unroll
        for (int d = 0; d < DEPTH; ++d)
            if (c + d < n) add(x[d], c + d);
    }
};
static_assert(B_M53 == 0 && B_M13 == 3 && B_P13 == 5 && B_P23 == 7, "the rows a moment needs go by its place");

struct PointShared {
    double cb[CB_SIZE], mom[MOM_SIZE], ang[ANG_COUNT][2];
    double row[mom_g(MAXDET, NCOEF)][64];   // lane sums of every moment
};

// Where the few-particle kernels leave what the finishing kernels need, for calls on
// events of more than one segment: per particle a coefficient block, and moment blocks of its max_group groups of
// segments (segment_kernel) or the lanes' sums of its max_seg segments (point_kernel).
struct SegmentScratch {
    double *cb, *sums;
    int max_seg, max_group;
};

// The point kernel's static LDS of NDET detectors: with four, 2.8 % below a compute unit's.
template <int NDET>
constexpr size_t point_lds() {
    return sizeof(PointShared) + PT_BLOCKS * (sizeof(PointPartials<NDET>) + TABLE_PAD * (sizeof(float) + sizeof(double)));
}
static_assert(point_lds<MAXDET>() <= LDS_BYTES, "LDS of the point kernel");

// Segment blockIdx.x of particle blockIdx.y.
template <int NDET, bool GRAD>
__global__ __launch_bounds__(PT_THREADS) void point_kernel(const DevEvent* __restrict__ evs, int n_events,
                                                           const int32_t* __restrict__ ev_of_p, ParamMap pm,
                                                           SegmentScratch scr, const double* __restrict__ theta,
                                                           double* __restrict__ logl, double* __restrict__ grad) {
    __shared__ PointShared S;
    __shared__ PointPartials<NDET> part[PT_BLOCKS];
    __shared__ float psi[PT_BLOCKS * TABLE_PAD];
    __shared__ double u[GRAD ? PT_BLOCKS * TABLE_PAD : 1];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int seg = blockIdx.x, p = blockIdx.y;
    const DevEvent& ev = evs[__builtin_amdgcn_readfirstlane(event_index(ev_of_p, p, n_events))];
    const TableView t = mixed_tables<NDET>(&ev);
    if (seg >= segments(t.npad)) return;   // a shorter event of the batch
    point_prologue(ev, pm, theta + (size_t)p * pm.dim, S.cb, S.ang, wave, lane);
    const int seg0 = seg * segment_blocks(t.npad), seg1 = min(t.npad / TABLE_PAD, seg0 + segment_blocks(t.npad));
    constexpr int W0 = GRAD ? NCOEF : 0, ROWS = GRAD ? 3 * NDET : 2 * NDET;   // partials' rows, their first wavefront
    constexpr int RPW = (ROWS + PT_WAVES - W0 - 1) / (PT_WAVES - W0);
    double sum = 0.0, zsum[RPW];
#pragma unroll
    for (int q = 0; q < RPW; ++q) zsum[q] = 0.0;
    for (int b0 = seg0; b0 < seg1; b0 += PT_BLOCKS) {
        const int nblk = min(seg1 - b0, PT_BLOCKS);
        __syncthreads();   // the prologue, or the last round's readers
        if (wave < nblk)
            point_terms<NDET, GRAD>(t, load_coef(S.cb), b0 + wave, psi + wave * TABLE_PAD,
                                    u + (GRAD ? wave * TABLE_PAD : 0), part[wave]);
        __syncthreads();
        if (GRAD && wave < NCOEF) {
            PointBasisSum b{t, psi, u, b0 * BLK_CHUNKS, min(t.chunks - b0 * BLK_CHUNKS, nblk * BLK_CHUNKS), sum};
            for_basis(wave, b);
            sum = b.s;
        } else {
#pragma unroll
            for (int q = 0; q < RPW; ++q) {
                const int r = min(wave - W0 + q * (PT_WAVES - W0), ROWS - 1);
#pragma unroll
                for (int b = 0; b < PT_BLOCKS; ++b)
                    if (b < nblk) zsum[q] += part[b].z[r][lane];
            }
        }
    }
    if (GRAD && wave < NCOEF) {
        S.row[mom_g(NDET, wave)][lane] = sum;
    } else {
#pragma unroll
        for (int q = 0; q < RPW; ++q) {
            const int r = wave - W0 + q * (PT_WAVES - W0);
            if (r < ROWS) S.row[r][lane] = zsum[q];
        }
    }
    __syncthreads();
    constexpr int K = moments(NDET, GRAD);
    if (scr.max_seg > 1) {
        double* out = scr.sums + ((size_t)p * scr.max_seg + seg) * K * 64;
        for (int e = threadIdx.x; e < K * 64; e += PT_THREADS) out[e] = (&S.row[0][0])[e];
        if (seg == 0 && (int)threadIdx.x < CB_SIZE) scr.cb[(size_t)p * CB_SIZE + threadIdx.x] = S.cb[threadIdx.x];
        return;
    }
    if (wave != 0) return;
    double v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = S.row[k][lane];
    store_totals<NDET, GRAD>(v, S.mom);
    wave_lds_fence();
    if (lane == 0) write_result<GRAD>(ev, pm, S.cb, S.mom, p, logl, grad);
}

// Group blockIdx.x of the segments of particle blockIdx.y, a segment per wavefront; the
// first wavefront then adds the lanes' sums in segment order and totals them.
static_assert(LL_WAVES == SEG_GROUP, "a workgroup takes a group");
template <int NDET, int PREC, bool GRAD>
__global__ __launch_bounds__(64 * LL_WAVES, 3) void segment_kernel(
    const DevEvent* __restrict__ evs, int n_events, const int32_t* __restrict__ ev_of_p, ParamMap pm,
    SegmentScratch scr, const double* __restrict__ theta) {
    constexpr int K = moments(NDET, GRAD);
    __shared__ double cb[CB_SIZE], ang[ANG_COUNT][2];
    __shared__ double col[SEG_GROUP][K][64];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int p = blockIdx.y, seg = blockIdx.x * SEG_GROUP + wave;
    const DevEvent& ev = evs[__builtin_amdgcn_readfirstlane(event_index(ev_of_p, p, n_events))];
    const TableView t = PREC == SMCGW_MIXED ? mixed_tables<NDET>(&ev) : fp64_tables<NDET>(&ev);
    const int nseg = segments(t.npad), n = min(SEG_GROUP, nseg - (int)blockIdx.x * SEG_GROUP);
    if (n <= 0) return;
    point_prologue(ev, pm, theta + (size_t)p * pm.dim, cb, ang, wave, lane);
    __syncthreads();
    if (blockIdx.x == 0)
        for (int e = threadIdx.x; e < CB_SIZE; e += 64 * LL_WAVES) scr.cb[(size_t)p * CB_SIZE + e] = cb[e];
    double v[K];
    if (wave < n) {
        const int b0 = seg * segment_blocks(t.npad), b1 = min(t.npad / TABLE_PAD, b0 + segment_blocks(t.npad));
        const BinCoef k = load_coef(cb);
        if constexpr (PREC == SMCGW_MIXED) {
            MixedAcc<NDET, GRAD> A;
            A.start(k);
            bin_loop<BinPair<NDET, float2>, LOOP_ALL>(A, k, t, b0, 1, b1, 0, [] {});
            lane_sums<NDET, GRAD>(A, v);
        } else {
            Fp64Acc<NDET, GRAD> A;
            A.start(k);
            bin_loop<BinPair<NDET, double2>, LOOP_ALL>(A, k, t, b0, 1, b1, 0, [] {});
            lane_sums<NDET, GRAD>(A, v);
        }
        if (wave != 0)
#pragma unroll
            for (int q = 0; q < K; ++q) col[wave][q][lane] = v[q];
    }
    __syncthreads();
    if (wave != 0) return;
#pragma unroll
    for (int w = 1; w < SEG_GROUP; ++w)
        if (w < n)
#pragma unroll
            for (int q = 0; q < K; ++q) v[q] += col[w][q][lane];
    store_totals<NDET, GRAD>(v, scr.sums + ((size_t)p * scr.max_group + blockIdx.x) * MOM_SIZE);
}

// Results of the particles whose groups segment_kernel left in scratch:
// a wavefront per particle adds the groups in order, one lane finishes.
template <bool GRAD>
__global__ __launch_bounds__(64) void finish_kernel(const DevEvent* __restrict__ evs, int n_events,
                                                    const int32_t* __restrict__ ev_of_p, ParamMap pm,
                                                    SegmentScratch scr, double* __restrict__ logl,
                                                    double* __restrict__ grad) {
    __shared__ double cb[CB_SIZE], mom[MOM_SIZE];
    const int lane = threadIdx.x, p = blockIdx.x;
    const DevEvent& ev = evs[__builtin_amdgcn_readfirstlane(event_index(ev_of_p, p, n_events))];
    for (int e = lane; e < CB_SIZE; e += 64) cb[e] = scr.cb[(size_t)p * CB_SIZE + e];
    const double* m = scr.sums + (size_t)p * scr.max_group * MOM_SIZE;
    if (lane < moments(ev.n_det, GRAD)) {
        double s = m[lane];
        const int n = segment_groups(ev.n_pad);
#pragma unroll 8
        for (int k = 1; k < n; ++k) s += m[(size_t)k * MOM_SIZE + lane];
        mom[lane] = s;
    }
    wave_lds_fence();
    if (lane == 0) write_result<GRAD>(ev, pm, cb, mom, p, logl, grad);
}

// The same from the lanes' sums of point_kernel: a workgroup per particle, its wavefronts
// taking the groups of segments in turn.
constexpr int PF_WAVES = 4;
constexpr int POINT_WORKGROUPS = 256;   // of a point call: compute units
constexpr int PF_GROUPS = (POINT_WORKGROUPS + SEG_GROUP - 1) / SEG_GROUP;
template <int NDET, bool GRAD>
__global__ __launch_bounds__(64 * PF_WAVES) void finish_point_kernel(const DevEvent* __restrict__ evs, int n_events,
                                                                     const int32_t* __restrict__ ev_of_p, ParamMap pm,
                                                                     SegmentScratch scr, double* __restrict__ logl,
                                                                     double* __restrict__ grad) {
    constexpr int K = moments(NDET, GRAD);
    __shared__ double cb[CB_SIZE], mom[PF_GROUPS][MOM_SIZE];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, p = blockIdx.x;
    const DevEvent& ev = evs[__builtin_amdgcn_readfirstlane(event_index(ev_of_p, p, n_events))];
    const int nseg = segments(ev.n_pad), groups = segment_groups(ev.n_pad);
    if ((int)threadIdx.x < CB_SIZE) cb[threadIdx.x] = scr.cb[(size_t)p * CB_SIZE + threadIdx.x];
    for (int g = wave; g < groups; g += PF_WAVES) {
        const double* s = scr.sums + ((size_t)p * scr.max_seg + g * SEG_GROUP) * K * 64 + lane;
        const int n = min(SEG_GROUP, nseg - g * SEG_GROUP);
        double x[SEG_GROUP][K];   // in flight together; a missing segment reads the group's first and is not added
#pragma unroll
        for (int w = 0; w < SEG_GROUP; ++w)
#pragma unroll
            for (int q = 0; q < K; ++q) x[w][q] = s[((w < n ? w : 0) * K + q) * 64];
#pragma unroll
        for (int w = 1; w < SEG_GROUP; ++w)
#pragma unroll
            for (int q = 0; q < K; ++q) x[0][q] = w < n ? x[0][q] + x[w][q] : x[0][q];
        store_totals<NDET, GRAD>(x[0], mom[g]);
    }
    __syncthreads();
    if (wave != 0) return;
    if (lane < K) {
        double s = mom[0][lane];
        for (int g = 1; g < groups; ++g) s += mom[g][lane];
        mom[0][lane] = s;
    }
    wave_lds_fence();
    if (lane == 0) write_result<GRAD>(ev, pm, cb, mom[0], p, logl, grad);
}

// Start order of a batch whose events differ in length: particles by falling
// table length (rank[e] of event e, 0 the longest), index order inside a rank.
// A wavefront walks one particle's bins alone, so a workgroup lasts as long as
// its longest event: equal lengths side by side leave no wavefront waiting, and
// with the longest first the short ones fill the end of the launch (16384
// particles over eight events of 4017 to 64897 bins: 1523 us a call in index
// order, 955 sorted, the sort included).  A workgroup orders up to SORT_CHUNK particles,
// its wavefront w the contiguous index range w; larger batches take a workgroup for
// each chunk, after a launch that counts every chunk's ranks.  Bound by the
// instructions issued on a compute unit: one workgroup would take 8 us for 2000 particles,
// 23 for 20000 and 90 for 100000, the chunks 8, 13 and 14.
//
// Where it is worth that (index order / sorted, us; events in turn, rising, at random): 16 events of 1 to 16
// blocks, 1025 particles 31.7 / 36.1, 30.2 / 35.3, 30.0 / 35.0; 1300: 42.3 / 37.5, 34.1 / 37.5, 40.9 / 37.6;
// 6000: 105 / 77, 72 / 77, 94 / 77.  Not with lengths within a factor of two (8 and 16 blocks, 3000 particles:
// 52.6 / 55.1, 50.8 / 56.2, 58.7 / 55.3; 16 and 17: 63.8 / 68.0, 61.8 / 69.3, 64.3 / 68.3) and not on short events
// (1 to 8 blocks, 3000 particles: 30.8 / 33.7, 28.0 / 35.0, 33.8 / 34.7; 1 and 2 blocks, 6000: 17.8 / 26.8).  A
// caller's own longest-first order costs the launch for nothing (4 to 7 us).
constexpr int SORT_FROM = 1280;
constexpr int SORT_BLOCKS = 16;
bool sort_pays(int P, int longest, int shortest) {
    return P > SORT_FROM && longest >= SORT_BLOCKS * TABLE_PAD && longest > 2 * shortest;
}

struct EventRanks { int bits; uint8_t rank[SMCGW_MAX_EVENTS]; };   // ranks below 2^bits
constexpr int SORT_THREADS = 1024;
constexpr int SORT_WAVES = SORT_THREADS / 64;
constexpr int SORT_AHEAD = 8;   // event indices of a lane in flight
constexpr int SORT_CHUNK = 4096;
constexpr int sort_chunks(int P) { return (P - 1) / SORT_CHUNK + 1; }
// entries of the order array: the order, then every chunk's counts where there are several
constexpr size_t sort_entries(int P) { return P + (sort_chunks(P) > 1 ? (size_t)sort_chunks(P) * SMCGW_MAX_EVENTS : 0); }

struct SortShared {
    int pos[SMCGW_MAX_EVENTS][SORT_WAVES];   // counts, then running positions, of every (rank, wavefront)
    int part[SORT_WAVES];
    int before[SMCGW_MAX_EVENTS], others[SMCGW_MAX_EVENTS];   // a rank's entries in the earlier chunks, in all other chunks
    uint8_t rank[SMCGW_MAX_EVENTS];
};

// Calls f(particle, whether there is one, its rank, the lanes of its rank) for this wavefront's particles, 64 at a time.
template <class F>
__device__ __forceinline__ void sort_each(const SortShared& S, const int32_t* __restrict__ ev_of_p, int n_events,
                                          const EventRanks& er, int P, F&& f) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c0 = blockIdx.x * SORT_CHUNK, n = min(SORT_CHUNK, P - c0);
    const int per = ((n + SORT_WAVES - 1) / SORT_WAVES + 63) & ~63;
    const int i0 = c0 + min(n, wave * per), i1 = c0 + min(n, wave * per + per);
    for (int b = i0; b < i1; b += 64 * SORT_AHEAD) {
        int e[SORT_AHEAD];
#pragma unroll
        for (int k = 0; k < SORT_AHEAD; ++k) e[k] = event_index(ev_of_p, min(b + 64 * k + lane, P - 1), n_events);
#pragma unroll
        for (int k = 0; k < SORT_AHEAD; ++k)
            if (b + 64 * k < i1) {
                const int i = b + 64 * k + lane, r = S.rank[e[k]];
                const bool in = i < i1;
                unsigned long long same = __ballot(in);
                for (int q = 0; q < er.bits; ++q) {
                    const unsigned long long one = __ballot(r >> q & 1);
                    same &= r >> q & 1 ? one : ~one;
                }
                f(i, in, r, same);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
    }
}

// The chunk's counts of every (rank, wavefront) into pos.
__device__ __forceinline__ void sort_count(SortShared& S, const int32_t* __restrict__ ev_of_p, int n_events,
                                           const EventRanks& er, int P) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    static_assert(SMCGW_MAX_EVENTS * SORT_WAVES == SORT_THREADS, "one entry per thread");
    (&S.pos[0][0])[tid] = 0;
    if (tid < SMCGW_MAX_EVENTS) S.rank[tid] = er.rank[tid];
    __syncthreads();
    sort_each(S, ev_of_p, n_events, er, P, [&](int, bool in, int r, unsigned long long same) {
        if (in && __builtin_ctzll(same) == lane) S.pos[r][wave] += __popcll(same);   // this wavefront's entries alone
    });
    __syncthreads();
}

__global__ __launch_bounds__(SORT_THREADS) void count_events_kernel(const int32_t* __restrict__ ev_of_p, int n_events,
                                                                    EventRanks er, int P, int32_t* __restrict__ counts) {
    __shared__ SortShared S;
    sort_count(S, ev_of_p, n_events, er, P);
    const int r = threadIdx.x;
    if (r >= SMCGW_MAX_EVENTS) return;
    int n = 0;
    for (int w = 0; w < SORT_WAVES; ++w) n += S.pos[r][w];
    counts[blockIdx.x * SMCGW_MAX_EVENTS + r] = n;
}

__global__ __launch_bounds__(SORT_THREADS) void sort_events_kernel(const int32_t* __restrict__ ev_of_p, int n_events,
                                                                   EventRanks er, int P,
                                                                   const int32_t* __restrict__ counts,
                                                                   int32_t* __restrict__ order) {
    __shared__ SortShared S;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    sort_count(S, ev_of_p, n_events, er, P);
    if (tid < SMCGW_MAX_EVENTS) {
        int before = 0, others = 0;
        for (int b = 0; b < (int)gridDim.x; ++b) {
            const int n = gridDim.x > 1 && b != (int)blockIdx.x ? counts[b * SMCGW_MAX_EVENTS + tid] : 0;
            others += n;
            if (b < (int)blockIdx.x) before += n;
        }
        S.before[tid] = before;
        S.others[tid] = others;
    }
    // exclusive scan over (rank, wavefront) in the chunk
    const int c = (&S.pos[0][0])[tid];
    int inc = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(inc, o);
        if (lane >= o) inc += t;
    }
    if (lane == 63) S.part[wave] = inc;
    __syncthreads();
    const int r = tid / SORT_WAVES;
    int at0 = S.before[r] + inc - c;
    for (int w = 0; w < wave; ++w) at0 += S.part[w];
    for (int q = 0; q < r; ++q) at0 += S.others[q];
    (&S.pos[0][0])[tid] = at0;
    __syncthreads();
    sort_each(S, ev_of_p, n_events, er, P, [&](int i, bool in, int rk, unsigned long long same) {
        const int at = S.pos[rk][wave];   // this wavefront's entries alone
        const int ahead = __popcll(same & ((1ull << lane) - 1));
        if (in) order[min(at + ahead, P - 1)] = i;
        __builtin_amdgcn_wave_barrier();
        if (in && ahead == 0) S.pos[rk][wave] = at + __popcll(same);
    });
}

// Projected strain of one parameter point (FP64), h_reim [n_det][N][2].
__global__ __launch_bounds__(256) void waveform_kernel(const DevEvent* __restrict__ evs, int e,
                                                       const double* __restrict__ c, double* __restrict__ h, int n,
                                                       int n_det) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const DevEvent& ev = evs[e];
    const double f = ev.fwl[(size_t)ROW_F * ev.n_pad + j];
    double B[NBASIS];
    basis_rows(f, ev.fwl[(size_t)ROW_W * ev.n_pad + j], ev.fwl[(size_t)ROW_LN * ev.n_pad + j], B);
    double ph = c[CB_C];
    for (int b = 0; b < NBASIS; ++b) ph = fma(c[CB_C + 1 + b], B[b], ph);
    const double a = pow(f, -7.0 / 6.0) / ev.u_scale * c[CB_AMP];
    for (int d = 0; d < n_det; ++d) {
        const double phd = fma(f, c[CB_TAU + d], ph);
        const double x = phd - rint(phd);
        double sn, cs;
        sincospi(2.0 * x, &sn, &cs);
        const double pr = c[CB_PR + d] * a, pi = c[CB_PI + d] * a;
        h[2 * ((size_t)d * n + j)] = pr * cs + pi * sn;
        h[2 * ((size_t)d * n + j) + 1] = pi * cs - pr * sn;
    }
}

// ------------------------------------------------------------- fixed scratch
// Start order of smcgw_loglike_grad_noalloc, for at most SMCGW_NOALLOC_MAX_P
// particles.  Every GPU the library runs on holds its own copy until the
// process ends.  Host code must not pass the array's name to a kernel (it is a
// host-side stand-in there): the device address of each GPU's copy is looked up
// once per device at context set-up and kept in noalloc_base.
static __device__ __align__(256) int32_t scratch[sort_entries(SMCGW_NOALLOC_MAX_P)];

constexpr int NOALLOC_DEVICES = 64;
static int32_t* noalloc_base[NOALLOC_DEVICES] = {};

// Resolves this device's scratch address (the device must be current).
int noalloc_init(int device) {
    if (device < 0 || device >= NOALLOC_DEVICES) return SMCGW_ERR_INVALID;
    if (noalloc_base[device]) return SMCGW_OK;
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return SMCGW_ERR_HIP;
    noalloc_base[device] = (int32_t*)ptr;
    return SMCGW_OK;
}

// ------------------------------------------------------------- launchers
hipError_t launch_prep(const DevEvent* d_events, int n_events, const int32_t* ev_of_p, const ParamMap& pm, int P,
                       const double* theta, double* cb, hipStream_t s) {
    if (P <= 0) return hipSuccess;
    hipLaunchKernelGGL(prep_kernel, dim3((P + PREP_PER_BLOCK - 1) / PREP_PER_BLOCK), dim3(256), 0, s, d_events,
                       n_events, ev_of_p, pm, P, theta, cb);
    return hipGetLastError();
}

// Particles per wavefront of the batched likelihood.  One keeps the most
// wavefronts in flight, and as long as the SIMDs hold them all (`residents` each, 4096 particles or 3072) that is what
// counts:
// on a folded event of 310 edges 700 particles take 10.7 us with one per
// wavefront, 12.4 with two, 16.3 with four; 3000 of 1969 bins 22.0, 27.5 and 32.9.  Once the chip is full, more of them
// share a prologue (eight lanes each, so a wavefront's instructions serve up to
// eight particles): 6000 particles take 23.4, 18.0 and 21.8 us, 20000 take 61.6,
// 44.7 and 39.9.  Kernels of three wavefronts per SIMD are full at 3072: 4096 of 100 bins and four detectors take
// 16.5 us with one (two rounds of workgroups), 12.2 with two.  On events of five to eight blocks the prologue weighs
// less and the grain of the launch more: with two per wavefront 5000 particles of 4017 bins take 59.5 us (53.1 with
// one), 100000 take 959 (995).  On longer ones the prologue is a few per cent of a wavefront's work and one per
// wavefront stays.
int per_wave_of(int P, int longest, int residents) {
    if (longest > 8 * TABLE_PAD) return 1;
    if (longest > 4 * TABLE_PAD) return P >= 16384 ? 2 : 1;
    return P >= 16384 ? 4 : P > 1024 * residents ? 2 : 1;
}

template <int NDET, bool GRAD, bool MULTI>
hipError_t launch_loglike_multi(const LoglikeCall& a, int precision, hipStream_t s) {
    const int per_wave = per_wave_of(a.P, a.longest, ll_residents(NDET, GRAD, precision));
    const int n = LL_WAVES * per_wave;
    const dim3 grid((a.P + n - 1) / n), block(64 * LL_WAVES);
    const size_t lds = loglike_lds<MULTI>(per_wave, moments(NDET, GRAD));
    if (precision == SMCGW_MIXED)
        hipLaunchKernelGGL((bins_mixed_kernel<NDET, GRAD, MULTI>), grid, block, lds, s, a.events, a.n_events,
                           a.ev_of_p, a.order, a.pm, a.P, per_wave, a.theta, a.logl, a.grad);
    else
        hipLaunchKernelGGL((bins_fp64_kernel<NDET, GRAD, MULTI>), grid, block, lds, s, a.events, a.n_events,
                           a.ev_of_p, a.order, a.pm, a.P, per_wave, a.theta, a.logl, a.grad);
    return hipGetLastError();
}

template <int NDET, bool GRAD>
hipError_t launch_loglike_ndet(const LoglikeCall& a, int precision, hipStream_t s) {
    return a.max_seg > 1 ? launch_loglike_multi<NDET, GRAD, true>(a, precision, s)
                         : launch_loglike_multi<NDET, GRAD, false>(a, precision, s);
}

hipError_t launch_loglike(const LoglikeCall& a, int n_det, int precision, hipStream_t s) {
    if (a.P <= 0) return hipSuccess;
    switch (n_det) {
    case 1: return a.grad ? launch_loglike_ndet<1, true>(a, precision, s) : launch_loglike_ndet<1, false>(a, precision, s);
    case 2: return a.grad ? launch_loglike_ndet<2, true>(a, precision, s) : launch_loglike_ndet<2, false>(a, precision, s);
    case 3: return a.grad ? launch_loglike_ndet<3, true>(a, precision, s) : launch_loglike_ndet<3, false>(a, precision, s);
    case 4: return a.grad ? launch_loglike_ndet<4, true>(a, precision, s) : launch_loglike_ndet<4, false>(a, precision, s);
    default: return hipErrorInvalidValue;
    }
}

// The few-particle paths, and where they end.  POINT: MIXED calls on events of
// POINT_MIN_BLOCKS blocks and more, while every segment gets a compute unit of
// its own (256 particles of 8033 bins: 18.7 us, 33.3 with a wavefront each; 400,
// in two rounds of workgroups: 38 against 31).
// SEGMENTS: events of more than one segment, as long as a wavefront per particle leaves SIMDs idle and the
// segments' wavefronts are evenly loaded.  A workgroup walks four segments; where the last ones are short or missing,
// its wavefronts wait for the longest, so what counts is the share of the workgroups' blocks that hold bins (`fill`).
// Segments against one wavefront per particle, 3 detectors, us: share 0.28 (18 blocks) 128 particles 21 / 32, 256
// 31 / 32, 600 40 / 32; 0.38 (24) 256 0.78 of the time, 512 0.95, 600 1.13; 0.53 (34) 512 0.88, 600 1.00, 1024 1.19;
// 0.77 (49) 700 0.84, 800 1.03, 1024 1.05; 1 (64) 1024 0.87, 1500 0.80, 1800 1.00, 2047 1.02; 1 (508) 1536 856 / 1106,
// 2047 1120 / 1150 (plain 2657 / 2593).
constexpr int POINT_MIN_BLOCKS = 8;
constexpr int GROUP_MAX = 65536;        // groups of segments of a call (192 B each)
static int segment_max_particles(int npad) {
    const int blocks = npad / TABLE_PAD;
    const int wgs = (segments(npad) + LL_WAVES - 1) / LL_WAVES;
    const double fill = (double)blocks / (wgs * LL_WAVES * segment_blocks(npad));
    return fill < 0.375 ? 256 : fill < 0.75 ? 512 : fill < 0.875 ? 704 : 1536;
}
enum LoglikePath { PATH_BATCH, PATH_POINT, PATH_SEGMENTS };

static LoglikePath loglike_path(int P, int longest, int nseg, int precision) {
    if ((long)P * nseg > GROUP_MAX) return PATH_BATCH;
    if (precision == SMCGW_MIXED && longest >= POINT_MIN_BLOCKS * TABLE_PAD && P * nseg <= POINT_WORKGROUPS)
        return PATH_POINT;
    return nseg > 1 && P <= segment_max_particles(longest) ? PATH_SEGMENTS : PATH_BATCH;
}

// Bytes of the few-particle scratch: coefficient blocks, then groups' moments or segments' lane sums.
static size_t segment_scratch_bytes(LoglikePath path, int P, int nseg, int n_det) {
    const size_t each = path == PATH_POINT ? (size_t)nseg * 64 * moments(n_det, true)
                                           : (size_t)((nseg + SEG_GROUP - 1) / SEG_GROUP) * MOM_SIZE;
    return P * (CB_SIZE + each) * sizeof(double);
}

template <int NDET, bool GRAD>
hipError_t launch_few_ndet(const LoglikeCall& a, LoglikePath path, int precision, void* scratch, hipStream_t s) {
    const int nseg = a.max_seg;
    const int groups = (nseg + SEG_GROUP - 1) / SEG_GROUP;
    SegmentScratch scr{(double*)scratch, (double*)scratch + (size_t)a.P * CB_SIZE, nseg, groups};
    const dim3 segs(groups, a.P), block(64 * LL_WAVES);
    if (path == PATH_POINT)
        hipLaunchKernelGGL((point_kernel<NDET, GRAD>), dim3(nseg, a.P), dim3(PT_THREADS), 0, s, a.events, a.n_events,
                           a.ev_of_p, a.pm, scr, a.theta, a.logl, a.grad);
    else if (precision == SMCGW_MIXED)
        hipLaunchKernelGGL((segment_kernel<NDET, SMCGW_MIXED, GRAD>), segs, block, 0, s, a.events, a.n_events,
                           a.ev_of_p, a.pm, scr, a.theta);
    else
        hipLaunchKernelGGL((segment_kernel<NDET, SMCGW_PLAIN_FP64, GRAD>), segs, block, 0, s, a.events, a.n_events,
                           a.ev_of_p, a.pm, scr, a.theta);
    if (nseg > 1 && path == PATH_POINT)
        hipLaunchKernelGGL((finish_point_kernel<NDET, GRAD>), dim3(a.P), dim3(64 * PF_WAVES), 0, s, a.events, a.n_events,
                           a.ev_of_p, a.pm, scr, a.logl, a.grad);
    else if (nseg > 1)
        hipLaunchKernelGGL(finish_kernel<GRAD>, dim3(a.P), dim3(64), 0, s, a.events, a.n_events, a.ev_of_p, a.pm, scr,
                           a.logl, a.grad);
    return hipGetLastError();
}

hipError_t launch_few(const LoglikeCall& a, LoglikePath path, int n_det, int precision, void* scratch,
                      hipStream_t s) {
    const bool g = a.grad != nullptr;
    switch (n_det) {
    case 1: return g ? launch_few_ndet<1, true>(a, path, precision, scratch, s) : launch_few_ndet<1, false>(a, path, precision, scratch, s);
    case 2: return g ? launch_few_ndet<2, true>(a, path, precision, scratch, s) : launch_few_ndet<2, false>(a, path, precision, scratch, s);
    case 3: return g ? launch_few_ndet<3, true>(a, path, precision, scratch, s) : launch_few_ndet<3, false>(a, path, precision, scratch, s);
    case 4: return g ? launch_few_ndet<4, true>(a, path, precision, scratch, s) : launch_few_ndet<4, false>(a, path, precision, scratch, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_waveform(const DevEvent* d_events, int event_id, const double* cb, double* h_reim, int n_bins,
                           int n_det, hipStream_t s) {
    hipLaunchKernelGGL(waveform_kernel, dim3((n_bins + 255) / 256), dim3(256), 0, s, d_events, event_id, cb, h_reim,
                       n_bins, n_det);
    return hipGetLastError();
}

}  // namespace smcgw

using namespace smcgw;

namespace smcgw {
// int32 entries of the start order a call takes, its scratch (0: index order).
size_t loglike_order_entries(const smcgw_ctx* c, int P, const int32_t* ev_of_p) {
    if (!ev_of_p) return 0;
    int longest = 0, shortest = INT32_MAX;
    for (const DevEvent& e : c->events) {
        longest = std::max(longest, e.n_pad);
        shortest = std::min(shortest, e.n_pad);
    }
    return sort_pays(P, longest, shortest) ? sort_entries(P) : 0;
}

// The longest table and the most segments among the events a call can meet.
static void event_extent(const smcgw_ctx* c, const int32_t* ev_of_p, int& longest, int& max_seg) {
    longest = c->events[0].n_pad;
    max_seg = segments(longest);
    if (ev_of_p)
        for (const DevEvent& e : c->events) {
            longest = std::max(longest, e.n_pad);
            max_seg = std::max(max_seg, segments(e.n_pad));
        }
}

// Scratch the call would use on the few-particle paths (0: none).
size_t loglike_scratch_bytes(const smcgw_ctx* c, int P, const int32_t* ev_of_p, int precision) {
    int longest, nseg;
    event_extent(c, ev_of_p, longest, nseg);
    const LoglikePath path = loglike_path(P, longest, nseg, precision);
    return path != PATH_BATCH && nseg > 1 ? segment_scratch_bytes(path, P, nseg, c->n_det) : 0;
}

// The batched likelihood on the context's stream; order: loglike_order_entries of
// scratch for the start order (NULL: index order), few: loglike_scratch_bytes of scratch for the
// few-particle paths (NULL: they are taken only where they need none).  Every
// path gives the same bits.
int queue_loglike(smcgw_ctx* c, int P, const int32_t* ev_of_p, const double* theta, double* logl, double* grad,
                  int precision, int32_t* order, void* few) {
    LoglikeCall a{c->d_events, (int)c->events.size(), ev_of_p, nullptr, c->pmap, P, 0, 0, theta, logl, grad};
    event_extent(c, ev_of_p, a.longest, a.max_seg);
    const LoglikePath path = loglike_path(P, a.longest, a.max_seg, precision);
    if (path != PATH_BATCH && (few || a.max_seg == 1)) {
        TimedLaunch t(c, SMCGW_KERNEL_BINS);
        return launch_few(a, path, c->n_det, precision, few, c->stream) == hipSuccess ? SMCGW_OK : SMCGW_ERR_HIP;
    }
    if (order && loglike_order_entries(c, P, ev_of_p)) {
        std::vector<int> len;
        for (const DevEvent& e : c->events) len.push_back(e.n_pad);
        std::sort(len.begin(), len.end(), std::greater<int>());
        len.erase(std::unique(len.begin(), len.end()), len.end());
        EventRanks er{};
        for (size_t e = 0; e < c->events.size(); ++e)
            er.rank[e] = (uint8_t)(std::find(len.begin(), len.end(), c->events[e].n_pad) - len.begin());
        while (1 << er.bits < (int)len.size()) ++er.bits;
        const dim3 grid(sort_chunks(P)), block(SORT_THREADS);
        TimedLaunch t(c, SMCGW_KERNEL_PREP);
        if (grid.x > 1)
            hipLaunchKernelGGL(count_events_kernel, grid, block, 0, c->stream, ev_of_p, a.n_events, er, P, order + P);
        hipLaunchKernelGGL(sort_events_kernel, grid, block, 0, c->stream, ev_of_p, a.n_events, er, P,
                           (const int32_t*)(order + P), order);
        if (hipGetLastError() != hipSuccess) return SMCGW_ERR_HIP;
        a.order = order;
    }
    TimedLaunch t(c, SMCGW_KERNEL_BINS);
    return launch_loglike(a, c->n_det, precision, c->stream) == hipSuccess ? SMCGW_OK : SMCGW_ERR_HIP;
}
}  // namespace smcgw

// The batched likelihood of smcgw_loglike_grad with its start order in the
// fixed scratch array: no allocation, no event, no host synchronisation.
extern "C" int smcgw_loglike_grad_noalloc(smcgw_ctx* c, int P, const int32_t* event_of_particle, const double* theta,
                                          double* logl, double* grad, int precision) {
    if (!c || P < 0 || (P > 0 && (!theta || !logl))) return SMCGW_ERR_INVALID;
    if (precision != SMCGW_PLAIN_FP64 && precision != SMCGW_MIXED) return SMCGW_ERR_INVALID;
    if (P > SMCGW_NOALLOC_MAX_P) return SMCGW_ERR_SHAPE;
    if (c->events.empty()) return SMCGW_ERR_NOT_INIT;
    if (P == 0) return SMCGW_OK;
    if (c->device < 0 || c->device >= NOALLOC_DEVICES || !noalloc_base[c->device]) return SMCGW_ERR_NOT_INIT;
    if (hipSetDevice(c->device) != hipSuccess) return SMCGW_ERR_HIP;
    return queue_loglike(c, P, event_of_particle, theta, logl, grad, precision, noalloc_base[c->device], nullptr);
}
