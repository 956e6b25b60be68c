// Internal declarations shared by the library's HIP translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "smcgw.h"

namespace smcgw {

constexpr int NPAR = 11;            // source parameters
constexpr int MAXDET = SMCGW_MAX_DET;
constexpr int MAXDIM = SMCGW_MAX_DIM;
constexpr int NBASIS = 8;           // per-bin phase basis rows kept in the tables
constexpr int NCOEF = NBASIS + 1;   // + the constant term
constexpr int TABLE_PAD = 512;      // tables are zero-padded to a multiple of this many bins
constexpr double PI = 3.14159265358979323846;
constexpr double TWO_PI = 6.28318530717958647692;

// Source-parameter indices.
enum { P_MC = 0, P_Q, P_CHI1, P_CHI2, P_DL, P_IOTA, P_PSI, P_RA, P_DEC, P_TC, P_PHIC };

// Phase basis: the TaylorF2 phase in cycles is
//   Phi(f) = c_0 + sum_b c_b B_b(f) + f (t_c + dt_det)
// with B = {f^-5/3, f^-1, f^-2/3, f^-1/3, ln f, f^1/3, f^1/3 ln f, f^2/3}.  The
// tables keep three FP64 rows per bin, f, w = f^-1/3 and ln f; every basis
// value is a product of them (basis_rows).
enum { B_M53 = 0, B_M1, B_M23, B_M13, B_LN, B_P13, B_P13LN, B_P23 };
enum { ROW_F = 0, ROW_W = 1, ROW_LN = 2, NROWS = 3 };

__device__ __forceinline__ void basis_rows(double f, double w, double lnf, double B[8]) {
    const double w2 = w * w;
    const double w3 = w2 * w;
    const double u = f * w2;   // f^1/3
    B[B_M53] = w3 * w2;
    B[B_M1] = w3;
    B[B_M23] = w2;
    B[B_M13] = w;
    B[B_LN] = lnf;
    B[B_P13] = u;
    B[B_P13LN] = u * lnf;
    B[B_P23] = u * u;
}

// Cross-lane moves through the VALU's data-parallel-primitive (DPP) lanes:
// no LDS round trip, unlike a shuffle.  A double moves as two 32-bit halves.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)b, CTRL, 0xf, 0xf, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// This lane's index, computed anew at every call: lane masks and addresses made
// from it are not carried in registers through the loops around the call (in the
// bin loops that costs spills).
__device__ __forceinline__ int lane_here() {
    unsigned zero = 0;
    __asm__ volatile("" : "+s"(zero));
    return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero));
}

// Sum over the 64 lanes of a wavefront in a fixed order: pairs and quads
// (quad permutations), rows of 16 (row rotations by 4 and 8), then the rows
// through the row-15 and row-31 broadcasts.  The total is valid in lane 63
// only (TOTAL_LANE).
constexpr int TOTAL_LANE = 63;
__device__ __forceinline__ double wave_total(double v) {
    v += dpp_move<0xb1>(v);    // quad_perm [1,0,3,2]
    v += dpp_move<0x4e>(v);    // quad_perm [2,3,0,1]
    v += dpp_move<0x124>(v);   // row_ror:4
    v += dpp_move<0x128>(v);   // row_ror:8
    v += dpp_move<0x142>(v);   // row_bcast:15
    v += dpp_move<0x143>(v);   // row_bcast:31
    return v;
}

// Wavefront totals of K per-lane values, entry k written to (or added to) out[k stride]
// (any address space) by lanes 0..7.  Three halving steps over lane bits 0-2 scatter the
// values: at each step a lane keeps one half of its list (by its lane bit) and
// adds the partner lane's copy of that half, the partner being the lane with the
// opposite bit and the same lower bits (xor 1, xor 2, a rotation by 4 inside
// the row of 16).  A lane then holds ceil(K/8) partial sums, which full sums
// over bits 3-5 (a rotation by 8 inside the row, then xor 16 and xor 32)
// complete.  A list of odd length pads its upper half with a zero.  The order
// of the additions is fixed, so the totals do not depend on anything but the
// inputs.  A halving step costs 7 instructions per kept value (selects of the
// sent and kept halves, two DPP moves, an add), so the reduction takes about
// 7 (K/2 + K/4 + K/8) + 9 K/8 instructions instead of 18 K for K separate
// wavefront sums.
template <int K>
__device__ __forceinline__ void wave_totals_to(const double (&v)[K], double* out, int stride = 1, bool add = false) {
    constexpr int M1 = (K + 1) / 2, M2 = (M1 + 1) / 2, M3 = (M2 + 1) / 2;
    const int lane = lane_here();
    const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4;
    double c1[M1], c2[M2], c3[M3];
#pragma unroll
    for (int k = 0; k < M1; ++k) {
        const double hi = k + M1 < K ? v[k + M1] : 0.0;
        const double send = b0 ? v[k] : hi;
        c1[k] = (b0 ? hi : v[k]) + dpp_move<0xb1>(send);   // quad_perm [1,0,3,2]
    }
#pragma unroll
    for (int k = 0; k < M2; ++k) {
        const double hi = k + M2 < M1 ? c1[k + M2] : 0.0;
        const double send = b1 ? c1[k] : hi;
        c2[k] = (b1 ? hi : c1[k]) + dpp_move<0x4e>(send);   // quad_perm [2,3,0,1]
    }
#pragma unroll
    for (int k = 0; k < M3; ++k) {
        const double hi = k + M3 < M2 ? c2[k + M3] : 0.0;
        const double send = b2 ? c2[k] : hi;
        c3[k] = (b2 ? hi : c2[k]) + dpp_move<0x124>(send);   // row_ror:4
    }
#pragma unroll
    for (int k = 0; k < M3; ++k) {
        double t = c3[k] + dpp_move<0x128>(c3[k]);   // row_ror:8
        t += __shfl_xor(t, 16, 64);
        t += __shfl_xor(t, 32, 64);
        c3[k] = t;
    }
    // entry k of the lane's list is entry (its bits' offsets) + k of the whole
    // one: one base per lane, no lookup per entry
    if (lane < 8) {
        const int p2 = b2 ? M3 : 0, p1 = p2 + (b1 ? M2 : 0), p0 = p1 + (b0 ? M1 : 0);
#pragma unroll
        for (int k = 0; k < M3; ++k)
            if (p2 + k < M2 && p1 + k < M1 && p0 + k < K) {
                double* o = out + (p0 + k) * stride;
                *o = add ? *o + c3[k] : c3[k];
            }
    }
}

// Total of one value over the lanes, valid in every lane, added in the order
// wave_totals_to<K> adds entry k of its list.  That order depends on the entry
// only where the quads of a row of 16 are paired: entries that end up on lanes
// with bit 2 clear pair quads (0, 3) and (1, 2), the others (0, 1) and (2, 3).
template <int K>
__device__ __forceinline__ double wave_total_as(double v, int k) {
    constexpr int M1 = (K + 1) / 2, M2 = (M1 + 1) / 2, M3 = (M2 + 1) / 2;
    const int p1 = k % M1, p2 = p1 % M2;
    v += dpp_move<0xb1>(v);   // quad_perm [1,0,3,2]
    v += dpp_move<0x4e>(v);   // quad_perm [2,3,0,1]
    v += p2 < M3 ? dpp_move<0x140>(v) : dpp_move<0x141>(v);   // row_mirror / row_half_mirror
    v += dpp_move<0x128>(v);  // row_ror:8
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    return v;
}

__device__ __forceinline__ double wave_max_total(double v) {
    v = fmax(v, dpp_move<0xb1>(v));
    v = fmax(v, dpp_move<0x4e>(v));
    v = fmax(v, dpp_move<0x124>(v));
    v = fmax(v, dpp_move<0x128>(v));
    v = fmax(v, dpp_move<0x142>(v));
    v = fmax(v, dpp_move<0x143>(v));
    return v;
}

// Device view of one event's bin tables (frequency-major, padded to n_pad).
struct DevEvent {
    int n_bins, n_pad, n_det, pn_order;
    double f_low, df;
    const double* fwl;       // [NROWS][n_pad]: f, f^-1/3, ln f
    const float2* u32;       // [n_det][n_pad]  4 df conj(d) f^-7/6 / (S u_scale), FP32
    const double2* u64;      // [n_det][n_pad]  same in FP64
    double hnorm[MAXDET];    // sum_j 4 df f^-7/3 / S / u_scale^2
    double dd;               // sum_d <d|d>_d
    double u_scale;          // power of two keeping the FP32 table near unit magnitude
    double t_sun, mpc_m, c_light, gmst;
    double ln_pi_tsun;       // ln(pi G Msun / c^3)
    double pos[MAXDET][3];   // detector positions [m]
    double resp[MAXDET][3][3];
    const double* wmom;      // [n_det][NGEO][NGEO]: sum_j 4 df f^-7/3 / S / u_scale^2 g_a g_b (local metric)
    const double* wa2;       // [n_det][n_pad]: 4 df f^-7/3 / S / u_scale^2 per bin (plain form; NULL for a
                             // relative-binning event)
};

// Functions of f whose combination is the phase of detector d in cycles:
// g_0 = 1, g_{1+b} = basis row b, g_{NCOEF} = f (the delay term).
constexpr int NGEO = NCOEF + 1;

// Sampled-coordinate map into the 11 source parameters.
struct ParamMap {
    int dim;
    int idx[MAXDIM];
    double fixed[NPAR];
};

// Per-particle coefficient block written by the prologue kernel (FP64).
// The first CB_BINS entries are all the bin loop reads.
enum {
    CB_C = 0,                            // NCOEF phase coefficients (cycles): const, then basis rows
    CB_TAU = CB_C + NCOEF,               // MAXDET: t_c + delay of each detector
    CB_PR = CB_TAU + MAXDET,             // MAXDET: Re P_d (times CB_AMP in use)
    CB_PI = CB_PR + MAXDET,              // MAXDET: Im P_d
    CB_BINS = CB_PI + MAXDET,
    CB_DC = CB_BINS,                     // [NCOEF][4]: d c_b / d(Mc, q, chi1, chi2)
    CB_DTAU = CB_DC + 4 * NCOEF,         // [MAXDET][2]: d tau_d / d(ra, dec)
    CB_DPR = CB_DTAU + 2 * MAXDET,       // [MAXDET][4]: d Re P_d / d(iota, psi, ra, dec)
    CB_DPI = CB_DPR + 4 * MAXDET,        // [MAXDET][4]: d Im P_d / d(iota, psi, ra, dec)
    CB_DLNCA_MC = CB_DPI + 4 * MAXDET,   // d ln C_A / d Mc
    CB_DLNCA_DL = CB_DLNCA_MC + 1,       // d ln C_A / d d_L
    CB_AMP = CB_DLNCA_DL + 1,            // C_A u_scale: the projection P'_d = CB_AMP P_d
    CB_SIZE = 104
};
static_assert(CB_AMP < CB_SIZE, "coefficient block overflow");

// Per-particle bin moments written by the bin loop (FP64), for n detectors, in
// the order in which store_moments reduces them:
//   Re Z_d, Im Z_d (d < n; Z_d = sum_j u_dj e^{-2 pi i Phi_dj}), T_d = sum_j q_dj f_j,
//   then NCOEF basis sums G_b = sum_j psibar_j B_b(f_j), the constant first.
__host__ __device__ constexpr int mom_zr(int, int d) { return d; }
__host__ __device__ constexpr int mom_zi(int n, int d) { return n + d; }
__host__ __device__ constexpr int mom_t(int n, int d) { return 2 * n + d; }
__host__ __device__ constexpr int mom_g(int n, int b) { return 3 * n + b; }
constexpr int MOM_SIZE = 24;
__host__ __device__ constexpr int moments(int n_det, bool grad) { return grad ? mom_g(n_det, NCOEF) : 2 * n_det; }
static_assert(mom_g(MAXDET, NCOEF) <= MOM_SIZE, "moment block overflow");

// Event index of particle p (out-of-range indices are clamped to a valid event).
__device__ __forceinline__ int event_index(const int32_t* ev_of_p, int p, int n_events) {
    if (!ev_of_p) return 0;
    const int e = ev_of_p[p];
    return e < 0 ? 0 : (e >= n_events ? n_events - 1 : e);
}

// ------------------------------------------------------------- host launchers
// (each .hip file exposes host functions; kernels stay in their own unit)
hipError_t launch_metric_moments(const double* d_psd, int n_det, int n_bins, double f_low, double df, double u_scale,
                                 double* wmom, hipStream_t s);
hipError_t launch_rb_tables(const double* fwl_full, const double2* u64_full, int n, int npad_full, int n_det,
                            const double* cb0, const int32_t* edges, int ne, double2* v, double2* a0, double2* a1,
                            int npad, double* fwl, float2* u32, double2* u64, hipStream_t s);
hipError_t launch_build_tables(const double* d_data, const double* d_psd, int n_det, int n_bins, int n_pad,
                               double f_low, double df, double u_scale, double* fwl, float2* u32, double2* u64,
                               double* wa2, double* sums, hipStream_t s);
hipError_t launch_prep(const DevEvent* d_events, int n_events, const int32_t* ev_of_p, const ParamMap& pm, int P,
                       const double* theta, double* cb, hipStream_t s);
// One batched likelihood launch: logl [P] and grad [P][pm.dim] (NULL: values
// only) of theta [P][pm.dim]; order [P] (NULL: index order) is the start order,
// longest and max_seg the largest n_pad and segment count among the events.
struct LoglikeCall {
    const DevEvent* events;
    int n_events;
    const int32_t* ev_of_p;
    const int32_t* order;
    ParamMap pm;
    int P, longest, max_seg;
    const double* theta;
    double *logl, *grad;
};
hipError_t launch_loglike(const LoglikeCall& a, int n_det, int precision, hipStream_t s);
hipError_t launch_waveform(const DevEvent* d_events, int event_id, const double* cb, double* h_reim, int n_bins,
                           int n_det, hipStream_t s);
int noalloc_init(int device);   // the fixed scratch of smcgw_loglike_grad_noalloc on this device

__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Lower Cholesky factor of an N x N matrix on lanes 0 .. N-1, lane i holding row i in A
// (its lower part), diag[i] its diagonal entry (LDS, N doubles).  Column k of the factor
// goes to Rt[k][0..N-1] (LDS, entries above the diagonal undefined).  Whether every
// pivot was positive; the same in all lanes.  An entry is the matrix entry minus the
// products of the finished columns, k ascending, as in the textbook's row-by-row form,
// but the products are subtracted as the columns come, for all entries at once; every
// lane follows the diagonal, so a pivot needs no exchange.
template <int N>
__device__ __forceinline__ bool cholesky_rows(double (&A)[N], double (*Rt)[MAXDIM], double* diag, int lane) {
    double dg[N];
#pragma unroll
    for (int j = 0; j < N; ++j)
        if (j == lane) diag[lane] = A[j];
    wave_lds_fence();
#pragma unroll
    for (int j = 0; j < N; ++j) dg[j] = diag[j];
    bool ok = true;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        ok = ok && dg[k] > 0.0;
        const double lkk = sqrt(dg[k]);
        const double l = lane == k ? lkk : A[k] / lkk;
        Rt[k][lane] = l;
        wave_lds_fence();
#pragma unroll
        for (int j = k + 1; j < N; ++j) {
            const double lj = Rt[k][j];
            dg[j] = fma(-lj, lj, dg[j]);
            A[j] = fma(-l, lj, A[j]);
        }
    }
    return ok;
}

}  // namespace smcgw
