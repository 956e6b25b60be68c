// Per-wavefront bin loop of the likelihood and its FP64 epilogue, shared by
// the batched likelihood kernels and the persistent NUTS kernel.
//
// A wavefront walks blocks of TABLE_PAD bins starting at block `blk0` with
// stride `blk_step`.  A block is read in chunks of 128 bins, lane l taking
// bins 2l and 2l + 1 of each chunk (TABLE_PAD/64 bins per lane per block); the
// per-bin tables are read coalesced and shared by every particle.  The
// wavefront's moments (see likelihood.hip), summed in FP64 over the blocks it
// visited, are written to a moment block by lanes 0..7.
#pragma once

#include "common.h"
#include "trig.h"

namespace smcgw {

// Wave-uniform per-particle values the bin loop needs (from the coefficient block).
struct BinCoef {
    double c[NCOEF];
    double tau[MAXDET];
    double pr[MAXDET], pi[MAXDET];
};

__device__ __forceinline__ double uniform_d(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)b);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

__device__ __forceinline__ float uniform_f(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}

// sin(2 pi x), cos(2 pi x) for 0 <= x < 1 on the hardware transcendental unit
// (v_sin_f32 / v_cos_f32 take their argument in revolutions).
__device__ __forceinline__ void sincos_rev_hw(float x, float& s, float& c) {
    s = __builtin_amdgcn_sinf(x);
    c = __builtin_amdgcn_cosf(x);
}

// Coefficients of one particle from a coefficient block in any address space.
__device__ __forceinline__ BinCoef load_coef(const double* cb) {
    BinCoef k;
#pragma unroll
    for (int b = 0; b < NCOEF; ++b) k.c[b] = uniform_d(cb[CB_C + b]);
#pragma unroll
    for (int d = 0; d < MAXDET; ++d) {
        k.tau[d] = uniform_d(cb[CB_TAU + d]);
        k.pr[d] = uniform_d(cb[CB_PR + d] * cb[CB_AMP]);
        k.pi[d] = uniform_d(cb[CB_PI + d] * cb[CB_AMP]);
    }
    return k;
}

// Per-lane inputs of one bin: f, f^-1/3, ln f and the detectors' whitened data.
template <int NDET, class U>
struct BinIn {
    double f, w, l;
    U u[NDET];
};

// The bin tables as raw buffer resources.  A chunk's loads then take the
// chunk's wave-uniform byte offset in a scalar register and a loop-invariant
// per-lane byte offset, so they cost no vector instructions for addresses.
// Resource word 3 of a raw (stride-0) buffer on this GPU family: 32-bit data
// format, no swizzle.
constexpr int BUF_RSRC_WORD3 = 0x00020000;

struct TableView {
    __amdgpu_buffer_rsrc_t fwl, u;
    int npad;
    int chunks;   // chunks that hold a bin
};

// The pointer and size are made wave-uniform first: a resource must sit in
// scalar registers, and a descriptor read from LDS is not known to be uniform.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t raw_rsrc(const void* p, size_t bytes) {
    const unsigned long long a = (unsigned long long)p;
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)a);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(a >> 32));
    const int n = __builtin_amdgcn_readfirstlane((int)min(bytes, (size_t)0x7fffffff));
    void* q = (void*)(((unsigned long long)hi << 32) | lo);
    return __builtin_amdgcn_make_buffer_rsrc(q, (short)0, n, BUF_RSRC_WORD3);
}

__device__ __forceinline__ double buf_f64(__amdgpu_buffer_rsrc_t r, unsigned lane_bytes, int uniform_bytes) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, lane_bytes, uniform_bytes, 0));
}

// A chunk is 128 consecutive bins; lane l takes bins 2l and 2l + 1, so every
// row of a chunk is read with one 16-byte load per lane.  Wider loads move
// twice the bytes per memory instruction: the bin loop is bound by the memory
// instructions in flight (one wavefront alone) or by the request rate of the
// cache hierarchy (a full device), not by the bytes themselves.
constexpr int CHUNK_BINS = 128;
constexpr int BLK_CHUNKS = TABLE_PAD / CHUNK_BINS;   // chunks per block

template <int NDET, class U>
struct BinPair {
    BinIn<NDET, U> b[2];
};

__device__ __forceinline__ double2 buf_f64x2(__amdgpu_buffer_rsrc_t r, unsigned lane_bytes, int uniform_bytes) {
    return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(r, lane_bytes, uniform_bytes, 0));
}

// One chunk starting at bin `base` (wave-uniform) + ch CHUNK_BINS (ch known to the compiler:
// the loads' own offsets hold it, so a block's chunks share their scalar addresses).
template <int NDET>
__device__ __forceinline__ void load_chunk(BinPair<NDET, float2>& x, const TableView& t, int base, unsigned lane,
                                           unsigned ch = 0) {
    const int np8 = t.npad * 8;
    const unsigned at = lane * 16u + ch * (CHUNK_BINS * 8u);
    const double2 f = buf_f64x2(t.fwl, at, ROW_F * np8 + base * 8);
    const double2 w = buf_f64x2(t.fwl, at, ROW_W * np8 + base * 8);
    const double2 l = buf_f64x2(t.fwl, at, ROW_LN * np8 + base * 8);
    x.b[0].f = f.x; x.b[1].f = f.y;
    x.b[0].w = w.x; x.b[1].w = w.y;
    x.b[0].l = l.x; x.b[1].l = l.y;
#pragma unroll
    for (int d = 0; d < NDET; ++d) {
        const float4 u = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(t.u, at, d * np8 + base * 8, 0));
        x.b[0].u[d] = make_float2(u.x, u.y);
        x.b[1].u[d] = make_float2(u.z, u.w);
    }
}

template <int NDET>
__device__ __forceinline__ void load_chunk(BinPair<NDET, double2>& x, const TableView& t, int base, unsigned lane,
                                           unsigned ch = 0) {
    const int np8 = t.npad * 8;
    const unsigned at = lane * 16u + ch * (CHUNK_BINS * 8u), at2 = lane * 32u + ch * (CHUNK_BINS * 16u);
    const double2 f = buf_f64x2(t.fwl, at, ROW_F * np8 + base * 8);
    const double2 w = buf_f64x2(t.fwl, at, ROW_W * np8 + base * 8);
    const double2 l = buf_f64x2(t.fwl, at, ROW_LN * np8 + base * 8);
    x.b[0].f = f.x; x.b[1].f = f.y;
    x.b[0].w = w.x; x.b[1].w = w.y;
    x.b[0].l = l.x; x.b[1].l = l.y;
#pragma unroll
    for (int d = 0; d < NDET; ++d) {
        x.b[0].u[d] = buf_f64x2(t.u, at2, 2 * (d * np8 + base * 8));
        x.b[1].u[d] = buf_f64x2(t.u, at2 + 16u, 2 * (d * np8 + base * 8));
    }
}

// A wavefront visits the blocks blk0, blk0 + blk_step, ... below blk_end of the
// padded table; each block is BLK_CHUNKS chunks.  The chunks run through two register
// buffers in turn: while one buffer is computed the other one's table entries
// are in flight.  Every prefetch is unconditional (the one past the last chunk
// re-reads the last chunk), so the buffers need no register copies.  The first
// bin of a block starts the per-lane partial sums and the block ends with
// their flush.  A lane adds its bins in chunk order, each chunk's pair in bin
// order.
//
// The table's last block ends with the chunk that holds the last bin: a chunk
// of padding alone (u = 0) adds only zeros, so it is not visited.  Of a
// folded event's ~310 edges that skips one chunk in four, of the 8033-bin
// grid's 64 chunks one.
//
// LOOP_SEGMENTS, LOOP_TIGHT: after every `seg` blocks, except the last one's, end_segment() is called:
// it takes A's sums and clears them.  The test for it inside the loop costs 0.5 to 1.5 % of long events' batches;
// LOOP_TIGHT has a segment's blocks in a loop of their own, with a block's scalar addresses made once, which costs
// nothing where the compiler keeps the loads as early as they are written: MIXED with the gradient of up to three
// detectors (3 x 259585 bins, 2048 particles 1141 -> 1118 us, 4096 2203 -> 2180; four detectors 1.0 % slower, values of
// three 1.4 times).
enum BinLoop { LOOP_ALL, LOOP_SEGMENTS, LOOP_TIGHT };
template <class In, BinLoop LOOP, class Acc, class F>
__device__ __forceinline__ void bin_loop(Acc& A, const BinCoef& k, const TableView& t, int blk0, int blk_step,
                                         int blk_end, int seg, F&& end_segment) {
    static_assert(BLK_CHUNKS % 2 == 0, "a block holds a whole number of buffer pairs");
    const unsigned lane = lane_here();
    const int nb = blk0 < blk_end ? (blk_end - blk0 + blk_step - 1) / blk_step : 0;   // this wave's blocks
    if (nb == 0) return;
    const int lastblk = blk0 + (nb - 1) * blk_step;
    const int rem = lastblk == t.npad / TABLE_PAD - 1 ? t.chunks - lastblk * BLK_CHUNKS : BLK_CHUNKS;   // its chunks in the last one
    const int full = rem == BLK_CHUNKS ? nb : nb - 1;
    const int last = (nb - 1) * BLK_CHUNKS + rem - 1;                           // this wave's last chunk
    auto base_of = [&](int c) {
        return (blk0 + (c / BLK_CHUNKS) * blk_step) * TABLE_PAD + CHUNK_BINS * (c % BLK_CHUNKS);
    };
    In a, b;
    load_chunk(a, t, base_of(0), lane);
    if constexpr (LOOP == LOOP_TIGHT) {
        const int step = blk_step * TABLE_PAD, end = base_of(last);
        int at = blk0 * TABLE_PAD;
        for (int blk = 0; blk < full;) {
            const int stop = min(full, blk + seg);
            for (; blk < stop; ++blk) {
                const int next = min(at + step, end);
#pragma unroll
                for (int pr = 0; pr < BLK_CHUNKS / 2; ++pr) {
                    load_chunk(b, t, at, lane, 2 * pr + 1);
                    A.bin(k, a.b[0], pr == 0);
                    A.bin(k, a.b[1], false);
                    if (pr + 1 < BLK_CHUNKS / 2) load_chunk(a, t, at, lane, 2 * pr + 2);
                    else load_chunk(a, t, next, lane);
                    A.bin(k, b.b[0], false);
                    A.bin(k, b.b[1], false);
                }
                A.flush();
                at = next;
            }
            if (blk < nb && blk % seg == 0) end_segment();
        }
    } else {
        for (int blk = 0; blk < full; ++blk) {
#pragma unroll
            for (int pr = 0; pr < BLK_CHUNKS / 2; ++pr) {
                const int c = blk * BLK_CHUNKS + 2 * pr;
                load_chunk(b, t, base_of(c + 1), lane);
                A.bin(k, a.b[0], pr == 0);
                A.bin(k, a.b[1], false);
                load_chunk(a, t, base_of(min(c + 2, last)), lane);
                A.bin(k, b.b[0], false);
                A.bin(k, b.b[1], false);
            }
            A.flush();
            if (LOOP == LOOP_SEGMENTS && (blk + 1) % seg == 0 && blk + 1 < nb) end_segment();
        }
    }
    if (full < nb) {
        A.clear();
        for (int c = full * BLK_CHUNKS; c <= last; c += 2) {
            load_chunk(b, t, base_of(min(c + 1, last)), lane);
            A.bin(k, a.b[0], false);
            A.bin(k, a.b[1], false);
            if (c == last) break;
            load_chunk(a, t, base_of(min(c + 2, last)), lane);
            A.bin(k, b.b[0], false);
            A.bin(k, b.b[1], false);
        }
        A.flush();
    }
}

// Totals over the lanes of a wavefront's per-lane sums (mom_* order) into, or onto, a moment
// block.  Without the gradient (Z alone) each is summed over the lanes in the order of its
// place in the full list, so that the value is the same with and without the gradient.
template <int NDET, bool GRAD>
__device__ __forceinline__ void store_totals(const double (&v)[moments(NDET, GRAD)], double* out, bool add = false) {
    if constexpr (GRAD) {
        wave_totals_to<moments(NDET, true)>(v, out, 1, add);
    } else {
        const int lane = lane_here();
#pragma unroll
        for (int k = 0; k < 2 * NDET; ++k) {
            const double t = wave_total_as<moments(NDET, true)>(v[k], k);
            if (lane == 0) out[k] = add ? out[k] + t : t;
        }
    }
}

// The per-lane sums of an accumulator in mom_* order.
template <int NDET, bool GRAD, class Acc>
__device__ __forceinline__ void lane_sums(const Acc& A, double (&v)[moments(NDET, GRAD)]) {
#pragma unroll
    for (int d = 0; d < NDET; ++d) {
        v[mom_zr(NDET, d)] = A.Zr[d];
        v[mom_zi(NDET, d)] = A.Zi[d];
        if (GRAD) v[mom_t(NDET, d)] = A.T[d];
    }
    if (GRAD)
#pragma unroll
        for (int b = 0; b < NCOEF; ++b) v[mom_g(NDET, b)] = A.G[b];
}

// MIXED: FP64 phase and argument reduction, FP32 sin/cos, complex products and
// per-lane partial sums (flushed into FP64 once per block), FP64 basis moments.
// GRAD = false keeps only Z (the value needs no more).
template <int NDET, bool GRAD = true>
struct MixedAcc {
    float pr[NDET], pim[NDET];
    double Zr[NDET], Zi[NDET], T[NDET], G[NCOEF];
    float zr[NDET], zi[NDET], tq[NDET];

    __device__ __forceinline__ void start(const BinCoef& k) {
#pragma unroll
        for (int d = 0; d < NDET; ++d) { pr[d] = uniform_f((float)k.pr[d]); pim[d] = uniform_f((float)k.pi[d]); }
        zero();
    }

    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int d = 0; d < NDET; ++d) { Zr[d] = 0.0; Zi[d] = 0.0; T[d] = 0.0; }
#pragma unroll
        for (int b = 0; b < NCOEF; ++b) G[b] = 0.0;
    }

    // One bin's FP32 terms into the partial sums; returns psibar_j.  B: the bin's basis rows.
    __device__ __forceinline__ float terms(const BinCoef& k, const BinIn<NDET, float2>& x, bool first,
                                           double (&B)[NBASIS]) {
        basis_rows(x.f, x.w, x.l, B);
        double ph = k.c[0];
#pragma unroll
        for (int b = 0; b < NBASIS; ++b) ph = fma(k.c[1 + b], B[b], ph);
        const float ff = (float)x.f;
        float psib = 0.f;
#pragma unroll
        for (int d = 0; d < NDET; ++d) {
            // fractional part of the phase in one FP64 instruction (exact); as a float
            // it is within 2^-25 revolutions of the exact value
            const double phd = fma(x.f, k.tau[d], ph);
            const float xr = (float)__builtin_amdgcn_fract(phd);
            float sn, cs;
            sincos_rev_hw(xr, sn, cs);
            const float sr = fmaf(x.u[d].x, cs, x.u[d].y * sn);    // u e^{-2 pi i x}
            const float si = fmaf(x.u[d].y, cs, -x.u[d].x * sn);
            zr[d] = first ? sr : zr[d] + sr;
            zi[d] = first ? si : zi[d] + si;
            if (GRAD) {
                const float q = fmaf(pr[d], si, pim[d] * sr);
                psib = (d == 0) ? q : psib + q;
                tq[d] = first ? q * ff : fmaf(q, ff, tq[d]);
            }
        }
        return psib;
    }

    __device__ __forceinline__ void bin(const BinCoef& k, const BinIn<NDET, float2>& x, bool first) {
        double B[NBASIS];
        const float psib = terms(k, x, first, B);
        if (!GRAD) return;
        const double pb = (double)psib;
        G[0] += pb;
#pragma unroll
        for (int b = 0; b < NBASIS; ++b) G[1 + b] = fma(pb, B[b], G[1 + b]);
    }

    // Block start with zeros instead of the first bin (the same sums).
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int d = 0; d < NDET; ++d) { zr[d] = 0.f; zi[d] = 0.f; tq[d] = 0.f; }
    }

    // Block end: the block's FP32 partials into the FP64 sums (the next block's
    // first bin restarts them).
    __device__ __forceinline__ void flush() {
#pragma unroll
        for (int d = 0; d < NDET; ++d) {
            Zr[d] += zr[d]; Zi[d] += zi[d];
            if (GRAD) T[d] += tq[d];
        }
    }
};

template <int NDET>
__device__ __forceinline__ TableView mixed_tables(const DevEvent* __restrict__ ev) {
    const int npad = __builtin_amdgcn_readfirstlane(ev->n_pad);
    return TableView{raw_rsrc(ev->fwl, (size_t)NROWS * npad * sizeof(double)),
                     raw_rsrc(ev->u32, (size_t)NDET * npad * sizeof(float2)), npad,
                     (__builtin_amdgcn_readfirstlane(ev->n_bins) + CHUNK_BINS - 1) / CHUNK_BINS};
}

// The moments of the blocks blk0, blk0 + blk_step, ... from one wavefront.
template <int NDET, bool GRAD = true>
__device__ __forceinline__ void bins_mixed_wave(const TableView& t, const BinCoef& k, int blk0, int blk_step,
                                                int blk_end, double* mom) {
    MixedAcc<NDET, GRAD> A;
    A.start(k);
    bin_loop<BinPair<NDET, float2>, LOOP_ALL>(A, k, t, blk0, blk_step, blk_end, 0, [] {});
    double v[moments(NDET, GRAD)];
    lane_sums<NDET, GRAD>(A, v);
    store_totals<NDET, GRAD>(v, mom);
}

// PLAIN_FP64: the same algebra in FP64 throughout.  LIBM: sin and cos from sincospi.
template <int NDET, bool GRAD = true, bool LIBM = false>
struct Fp64Acc {
    double Zr[NDET], Zi[NDET], T[NDET], G[NCOEF];

    __device__ __forceinline__ void start(const BinCoef&) { zero(); }

    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int d = 0; d < NDET; ++d) { Zr[d] = 0.0; Zi[d] = 0.0; T[d] = 0.0; }
#pragma unroll
        for (int b = 0; b < NCOEF; ++b) G[b] = 0.0;
    }

    __device__ __forceinline__ void bin(const BinCoef& k, const BinIn<NDET, double2>& x, bool) {
        double B[NBASIS];
        basis_rows(x.f, x.w, x.l, B);
        double ph = k.c[0];
#pragma unroll
        for (int b = 0; b < NBASIS; ++b) ph = fma(k.c[1 + b], B[b], ph);
        double psib;
#pragma unroll
        for (int d = 0; d < NDET; ++d) {
            const double phd = fma(x.f, k.tau[d], ph);
            double sn, cs;
            if (LIBM) sincospi(2.0 * (phd - rint(phd)), &sn, &cs);
            else sincos_rev(phd, sn, cs);
            const double sr = fma(x.u[d].x, cs, x.u[d].y * sn);
            const double si = fma(x.u[d].y, cs, -x.u[d].x * sn);
            Zr[d] += sr;
            Zi[d] += si;
            if (GRAD) {
                const double q = fma(k.pr[d], si, k.pi[d] * sr);
                psib = (d == 0) ? q : psib + q;
                T[d] = fma(q, x.f, T[d]);
            }
        }
        if (!GRAD) return;
        G[0] += psib;
#pragma unroll
        for (int b = 0; b < NBASIS; ++b) G[1 + b] = fma(psib, B[b], G[1 + b]);
    }

    __device__ __forceinline__ void clear() {}
    __device__ __forceinline__ void flush() {}
};

template <int NDET>
__device__ __forceinline__ TableView fp64_tables(const DevEvent* __restrict__ ev) {
    const int npad = __builtin_amdgcn_readfirstlane(ev->n_pad);
    return TableView{raw_rsrc(ev->fwl, (size_t)NROWS * npad * sizeof(double)),
                     raw_rsrc(ev->u64, (size_t)NDET * npad * sizeof(double2)), npad,
                     (__builtin_amdgcn_readfirstlane(ev->n_bins) + CHUNK_BINS - 1) / CHUNK_BINS};
}

template <int NDET, bool GRAD = true, bool LIBM = false>
__device__ __forceinline__ void bins_fp64_wave(const TableView& t, const BinCoef& k, int blk0, int blk_step,
                                               int blk_end, double* mom) {
    Fp64Acc<NDET, GRAD, LIBM> A;
    A.start(k);
    bin_loop<BinPair<NDET, double2>, LOOP_ALL>(A, k, t, blk0, blk_step, blk_end, 0, [] {});
    double v[moments(NDET, GRAD)];
    lane_sums<NDET, GRAD>(A, v);
    store_totals<NDET, GRAD>(v, mom);
}

// A particle's moments are summed in segments of blocks of bins, and the segments in groups
// of SEG_GROUP: each lane adds its segments' sums in order, a group's sums are totalled over
// the lanes, then the groups are added in order.  So they come
// out the same, bit for bit, whether one wavefront walks them all or each segment has a
// wavefront of its own (a particle's value may not depend on the size of its
// batch).  Events of up to 8192 bins are one segment.  In a wavefront that walks them all a segment's end costs 18 of
// the 9000 (or 18000) vector instructions of its bins, the resets of its sums, and a group's end a reduction of 150
// (one at every segment's end costs the 128 s batch 0.6 % more).
constexpr int SEG_GROUP = 4;
__host__ __device__ constexpr int segment_blocks(int npad) { return npad <= 64 * TABLE_PAD ? 16 : 32; }
__host__ __device__ constexpr int segments(int npad) {
    return (npad / TABLE_PAD + segment_blocks(npad) - 1) / segment_blocks(npad);
}
__host__ __device__ constexpr int segment_groups(int npad) { return (segments(npad) + SEG_GROUP - 1) / SEG_GROUP; }

// All segments from one wavefront into mom (LDS).  LOOP_ALL: events of one segment; else col holds LDS columns of the
// lanes' sums, [moments][64] doubles.
template <int NDET, bool GRAD, BinLoop LOOP, class In, class Acc>
__device__ __forceinline__ void event_moments(const TableView& t, const BinCoef& k, double* mom, double* col) {
    constexpr int K = moments(NDET, GRAD);
    Acc A;
    A.start(k);
    int done = 0;   // segments
    auto finish = [&] {
        double v[K];
        lane_sums<NDET, GRAD>(A, v);
        if (LOOP != LOOP_ALL && done % SEG_GROUP != 0) {
            const double* c = col + lane_here();
#pragma unroll
            for (int q = 0; q < K; ++q) v[q] = c[64 * q] + v[q];
        }
        store_totals<NDET, GRAD>(v, mom, LOOP != LOOP_ALL && done >= SEG_GROUP);
    };
    auto end = [&] {
        if (done % SEG_GROUP == SEG_GROUP - 1) {
            finish();
        } else {
            double v[K];
            lane_sums<NDET, GRAD>(A, v);
            double* c = col + lane_here();
            if (done % SEG_GROUP == 0) {
#pragma unroll
                for (int q = 0; q < K; ++q) c[64 * q] = v[q];
            } else {
                // an LDS addition, one instruction and no answer to wait for; a lane's own entries, so in order
#pragma unroll
                for (int q = 0; q < K; ++q)
                    (void)__hip_atomic_fetch_add(c + 64 * q, v[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
        ++done;
        A.zero();
    };
    bin_loop<In, LOOP>(A, k, t, 0, 1, t.npad / TABLE_PAD, segment_blocks(t.npad), end);
    finish();
    wave_lds_fence();
}

// logL from the Z moments alone (the sum of finish_particle, term by term).
__device__ __forceinline__ double finish_value(const DevEvent& ev, const double* c, const double* m) {
    double ll = -0.5 * ev.dd;
    const double amp = c[CB_AMP];
    for (int d = 0; d < ev.n_det; ++d) {
        const double pr = c[CB_PR + d] * amp, pi = c[CB_PI + d] * amp;
        const double re = pr * m[mom_zr(ev.n_det, d)] - pi * m[mom_zi(ev.n_det, d)];
        const double p2 = pr * pr + pi * pi;
        ll += re - 0.5 * p2 * ev.hnorm[d];
    }
    return ll;
}

// logL and its gradient with respect to the 11 source parameters from the
// moments and the prologue's Jacobians (FP64, one lane).
__device__ __forceinline__ double finish_particle(const DevEvent& ev, const double* c, const double* m,
                                                  double g[NPAR]) {
    double ll = -0.5 * ev.dd;
    double dlnca = 0.0, sum_t = 0.0;
    const double amp = c[CB_AMP];          // P'_d = amp P_d
    double gp[4] = {0.0, 0.0, 0.0, 0.0};   // iota, psi, ra, dec through P'_d
    for (int k = 0; k < NPAR; ++k) g[k] = 0.0;
    for (int d = 0; d < ev.n_det; ++d) {
        const double pr = c[CB_PR + d] * amp, pi = c[CB_PI + d] * amp;
        const double zr = m[mom_zr(ev.n_det, d)], zi = m[mom_zi(ev.n_det, d)], h = ev.hnorm[d];
        const double re = pr * zr - pi * zi;
        const double p2 = pr * pr + pi * pi;
        ll += re - 0.5 * p2 * h;
        dlnca += re - p2 * h;
        const double ar = zr - h * pr, ai = -zi - h * pi;   // dlogL / d(Re P', Im P')
#pragma unroll
        for (int k = 0; k < 4; ++k) gp[k] += amp * (ar * c[CB_DPR + 4 * d + k] + ai * c[CB_DPI + 4 * d + k]);
        const double t = m[mom_t(ev.n_det, d)];
        sum_t += t;
        g[P_RA] += TWO_PI * t * c[CB_DTAU + 2 * d];
        g[P_DEC] += TWO_PI * t * c[CB_DTAU + 2 * d + 1];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        double s = 0.0;
        for (int b = 0; b < NCOEF; ++b) s += c[CB_DC + 4 * b + k] * m[mom_g(ev.n_det, b)];
        g[k] = TWO_PI * s;   // Mc, q, chi1, chi2 through the phase
    }
    g[P_MC] += dlnca * c[CB_DLNCA_MC];
    g[P_DL] = dlnca * c[CB_DLNCA_DL];
    g[P_IOTA] = gp[0];
    g[P_PSI] = gp[1];
    g[P_RA] += gp[2];
    g[P_DEC] += gp[3];
    g[P_TC] = TWO_PI * sum_t;
    g[P_PHIC] = -m[mom_g(ev.n_det, 0)];
    return ll;
}

}  // namespace smcgw
