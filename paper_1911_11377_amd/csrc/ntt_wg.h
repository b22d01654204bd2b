// Whole limb transforms inside one workgroup for 2^12 <= N <= 2^14: the limb crosses HBM once.
//
// The transform is the same N1 x 256 decomposition as in ntt_v2.h, with the same butterflies and twiddles (the words are reduced at
// other places in part; the residues that come out are the same), but both passes run in one workgroup of N/16 threads and the intermediate between them
// lives in LDS instead of HBM: every thread keeps 16 words in registers, and the N1 x 256 matrix sits in LDS in the
// padded row layout of the row pass (row r, column q at r*V2_GS + (q/16)*17 + q%16: 34 KiB at N = 2^12, 136 KiB at
// N = 2^14).  Each 256-thread quarter of the workgroup does the column pass of one 4096-word column tile, exchanging
// through the tile's own columns of that matrix in place; after one workgroup barrier every row is finished by its own
// 16 lanes exactly as in ntt_v2_rows.  Twiddles are fetched per round (they are shared by every limb of the modulus and
// stay in L2) instead of being held across items: a thread's registers hold one round's set at a time, which keeps the
// 1024-thread size within its 128 registers (with both rounds' twiddles requested early 21 forward and 34 inverse registers
// spilled).  Passes over 4096 limbs one after the other, forward / inverse: N = 2^12 57 / 60 us, 2^13 136 / 126, 2^14 278 / 303, which is 4.7 / 4.4,
// 3.9 / 4.3 and 3.9 / 3.5 TB/s (a device copy moves 4.85); 4608 limbs of 2^14 words in bench.py's sweep 3.1 / 3.4 TB/s.  Before reductions were
// thinned out: 56 / 59 us at 2^12 (two passes through HBM: 87 / 91), 139 / 126 at 2^13 (both rounds' twiddles early: 147 / 144), 300 / 297 at 2^14
// (324 / 308).  8 limbs of 2^13 words: 8.9 / 9.0 us.  At N = 2^12 the row pass reduces four more of 16 words than elsewhere, because one round only
// follows it (INV_ROW2_12): 4096 limbs inverse 60.4 us without them, 60.6 with.
#pragma once
#include "ntt_v2.h"

__device__ __forceinline__ unsigned wg_pad(unsigned row, unsigned col) { return row * V2_GS + (col >> 4) * 17u + (col & 15u); }

// Forward transform of block `base - 2^S` of a ring of M * 2^S words (base = 1: the whole ring): x in the column layout (word
// (geo.r + G*e, geo.c0 + geo.c)), at most ENTRY256 / 256 p in magnitude; the results end in LDS as X says (p < 2^51 and not ROW_LAZY:
// balanced-reduced), word (row g, position q) at wg_pad(g, q).  Every row is finished by its own 16 lanes (a row-group sync suffices to read it).
// `request` is called once the first row round is done: the place for memory requests whose latency the rest covers.
template <int LOGM, bool P51, int ENTRY256, int X, class F>
__device__ __forceinline__ void wg_fwd_block(double (&x)[16], const double *tw, unsigned base, double *lds, double p, double pinv, F request) {
    constexpr int Q = LOGM - 12;
    typedef ColsGeom<Q> Geo;
    typedef ColsMasks<Q, P51, ENTRY256> Mk;
    typedef RowMasks<P51, X> Rm;
    constexpr unsigned MR = (1u << LOGM) >> 8;
    const unsigned tid = threadIdx.x, row = tid >> 4, lo4 = tid & 15;
    const Geo geo(tid & 255u, tid >> 8);
    double *grp = lds + row * V2_GS;
    {
        double tw1[15];
#pragma unroll
        for (int s = 0; s < 4; s++)
#pragma unroll
            for (int b = 0; b < (1 << s); b++) tw1[(1 << s) - 1 + b] = tw[(base << s) + b];
        fwd_round<Mk::F1>(x, tw1, p, pinv);
    }
    double tw1[15], tw2[15];
    if (Q > 0) {
#pragma unroll
        for (int s = 0; s < 4; s++)
#pragma unroll
            for (int b = 0; b < (1 << s); b++) {
                if (s >= 4 - Q) {
                    const int u = s - (4 - Q);
                    tw2[(1 << s) - 1 + b] = tw[((16u * base + geo.a) << u) + (b & ((1 << u) - 1))];
                } else {
                    tw2[(1 << s) - 1 + b] = 0.0;
                }
            }
#pragma unroll
        for (int e = 0; e < 16; e++) lds[wg_pad(geo.r + Geo::G * e, geo.c0 + geo.c)] = x[e];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 16; i++) x[i] = lds[wg_pad(Geo::G * geo.a + (i % Geo::G), geo.c0 + geo.l16 + 16 * (i / Geo::G))];
        fwd_stages<Geo::S0, Mk::F2>(x, tw2, p, pinv);
#pragma unroll
        for (int i = 0; i < 16; i++) lds[wg_pad(Geo::G * geo.a + (i % Geo::G), geo.c0 + geo.l16 + 16 * (i / Geo::G))] = x[i];
    } else {
#pragma unroll
        for (int e = 0; e < 16; e++) lds[wg_pad(e, geo.c0 + geo.c)] = x[e];
    }
    const unsigned base1 = base * MR + row;
#pragma unroll
    for (int s = 0; s < 4; s++)
#pragma unroll
        for (int b = 0; b < (1 << s); b++) tw1[(1 << s) - 1 + b] = tw[(base1 << s) + b];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 16; e++) x[e] = grp[e * 17 + lo4];
    fwd_round<Rm::F1>(x, tw1, p, pinv);
#pragma unroll
    for (int s = 0; s < 4; s++)
#pragma unroll
        for (int b = 0; b < (1 << s); b++) tw2[(1 << s) - 1 + b] = tw[((16u * base1 + lo4) << s) + b];
#pragma unroll
    for (int e = 0; e < 16; e++) grp[e * 17 + lo4] = x[e];
    request();
    ROW_GROUP_SYNC();
#pragma unroll
    for (int e = 0; e < 16; e++) x[e] = grp[lo4 * 17 + e];
    fwd_round<Rm::F2>(x, tw2, p, pinv);
#pragma unroll
    for (int e = 0; e < 16; e++) grp[lo4 * 17 + e] = X == ROW_LAZY || (X != ROW_REDUCED && !P51) ? x[e] : reduce_balanced(x[e], p, pinv);
    ROW_GROUP_SYNC();
}

// Operands of a product whose third tensor component enters its key switch through the inverse transform
struct TensorSrc {
    const u64d *a, *b;  // [items][terms][2][level][N]
    int level, terms;
};

// Inverse transform of one limb: word (geo.r + G*e, geo.c0 + geo.c) of the result in x[e], before the final addend and the
// canonical form.  SRC 0: the words of src; 1: read through the automorphism X -> X^g of item `it` (a rotation's polynomial);
// 2: the third tensor component sum_t a1_t * b1_t of limb li of item `it`, formed on the way (never written).
// Ends without a barrier: the caller puts one before the matrix is used again.
template <int LOGN, bool P51, int SRC>
__device__ __forceinline__ void wg_inv_limb(double (&x)[16], const u64d *src, const double *tw, double *lds, double p, double pinv, WMul ninv, WMul wlast,
                                            unsigned li, unsigned it, const GaloisTab *gal, const TensorSrc *ten) {
    BODY_TAG(P51);
    constexpr int Q = LOGN - 12;
    typedef ColsGeom<Q> Geo;
    constexpr unsigned N = 1u << LOGN, N1 = N >> 8;
    constexpr InvRound ROW2 = Q ? INV_ROW2 : INV_ROW2_12, AFTER_ROW2 = Q ? INV_COL2 : INV_COL1;
    INV_JOIN(P51, INV_ROW1, ROW2);
    INV_JOIN(P51, ROW2, AFTER_ROW2);
    INV_JOIN(P51, INV_COL2, INV_COL1);
    const unsigned tid = threadIdx.x, row = tid >> 4, lo4 = tid & 15, pr = row_pair_index(row, lo4, 0);
    const Geo geo(tid & 255u, tid >> 8);
    double *grp = lds + row * V2_GS;
    const WMul unused = WMul{0.0, 0.0};
    // ---- row pass, from HBM into the LDS matrix
    {
        double tw1[15], tw2[15];
        const unsigned base1 = N1 + row;
        if (SRC == 2) {
            const size_t st = (size_t)ten->level * N / 2, it0 = (size_t)it * ten->terms * 2 * st;  // pairs between components
            const ulonglong2 *pa = (const ulonglong2 *)ten->a + it0 + st + (size_t)li * (N / 2);
            const ulonglong2 *pb = (const ulonglong2 *)ten->b + it0 + st + (size_t)li * (N / 2);
#pragma unroll
            for (int h = 0; h < 2; h++) {  // four pairs at a time: bounds the registers in flight
                double d2[8];
                for (int tm = 0; tm < ten->terms; tm++) {
                    ulonglong2 a1[4], b1[4];
#pragma unroll
                    for (int s = 0; s < 4; s++) {
                        a1[s] = (pa + 2 * st * tm + 16 * (4 * h + s))[pr];
                        b1[s] = (pb + 2 * st * tm + 16 * (4 * h + s))[pr];
                    }
                    NTT_SCHED_FENCE();
#pragma unroll
                    for (int s = 0; s < 4; s++) {  // one product 1.25p, a sum is reduced
                        const double v0 = mulmod(u2d(a1[s].x), u2d(b1[s].x), p, pinv), v1 = mulmod(u2d(a1[s].y), u2d(b1[s].y), p, pinv);
                        d2[2 * s] = tm ? reduce_balanced(d2[2 * s] + v0, p, pinv) : v0;
                        d2[2 * s + 1] = tm ? reduce_balanced(d2[2 * s + 1] + v1, p, pinv) : v1;
                    }
                }
#pragma unroll
                for (int s = 0; s < 4; s++) {
                    double *rr = grp + row_pair_lds(lo4, 4 * h + s);
                    rr[0] = d2[2 * s];
                    rr[1] = d2[2 * s + 1];
                }
            }
            LOAD_FENCE();
        } else {
            ulonglong2 raw[8];
#pragma unroll
            for (int s = 0; s < 8; s++) {
                if (SRC == 1) raw[s] = galois_pair_load(src, row * 256u + 32u * s + 2u * lo4, gal->g[it], LOGN);
                else raw[s] = ((const ulonglong2 *)src + 16 * s)[pr];
            }
            if (SRC == 0) {
#pragma unroll
                for (int s = 0; s < 4; s++)
#pragma unroll
                    for (int b = 0; b < (1 << s); b++) tw2[(1 << s) - 1 + b] = tw[((16u * base1 + lo4) << s) + b];
            }
            NTT_SCHED_FENCE();
#pragma unroll
            for (int s = 0; s < 8; s++) {
                double *rr = grp + row_pair_lds(lo4, s);
                rr[0] = u2d(raw[s].x);
                rr[1] = u2d(raw[s].y);
            }
            if (SRC != 0) LOAD_FENCE();
        }
        if (SRC != 0) {  // the source needs the registers: the first round's twiddles come after it
#pragma unroll
            for (int s = 0; s < 4; s++)
#pragma unroll
                for (int b = 0; b < (1 << s); b++) tw2[(1 << s) - 1 + b] = tw[((16u * base1 + lo4) << s) + b];
        }
        ROW_GROUP_SYNC();
#pragma unroll
        for (int e = 0; e < 16; e++) x[e] = grp[lo4 * 17 + e];
        inv_stages<0, INV_ROW1, P51>(x, tw2, p, pinv, unused, unused);
#pragma unroll
        for (int e = 0; e < 16; e++) PIN_VALUE(x[e]);  // the first round is done with its twiddles before the second's arrive
#pragma unroll
        for (int s = 0; s < 4; s++)
#pragma unroll
            for (int b = 0; b < (1 << s); b++) tw1[(1 << s) - 1 + b] = tw[(base1 << s) + b];
#pragma unroll
        for (int e = 0; e < 16; e++) grp[lo4 * 17 + e] = x[e];
        ROW_GROUP_SYNC();
#pragma unroll
        for (int e = 0; e < 16; e++) x[e] = grp[e * 17 + lo4];
        inv_stages<0, ROW2, P51>(x, tw1, p, pinv, unused, unused);
#pragma unroll
        for (int e = 0; e < 16; e++) PIN_VALUE(x[e]);
#pragma unroll
        for (int e = 0; e < 16; e++) grp[e * 17 + lo4] = x[e];
    }
    // ---- column pass, from the LDS matrix to HBM
    {
        double tw1[15], tw2u[15];
        load_cols_twiddles<Q>(tw, geo.a, tw1, tw2u);
        __syncthreads();
        if (Q > 0) {
#pragma unroll
            for (int i = 0; i < 16; i++) x[i] = lds[wg_pad(Geo::G * geo.a + (i % Geo::G), geo.c0 + geo.l16 + 16 * (i / Geo::G))];
            inv_stages<Geo::S0, INV_COL2, P51>(x, tw2u, p, pinv, ninv, wlast);
#pragma unroll
            for (int i = 0; i < 16; i++) lds[wg_pad(Geo::G * geo.a + (i % Geo::G), geo.c0 + geo.l16 + 16 * (i / Geo::G))] = x[i];
            __syncthreads();
        }
#pragma unroll
        for (int e = 0; e < 16; e++) x[e] = lds[wg_pad(geo.r + Geo::G * e, geo.c0 + geo.c)];
        inv_stages<0, INV_COL1, P51>(x, tw1, p, pinv, ninv, wlast);
    }
}

// SRC: inverse see wg_inv_limb, forward SRC_WORDS or SRC_REAL
template <bool INV, int LOGN, bool P51, bool F64, bool NT, int SRC = 0>
__device__ __forceinline__ void ntt_wg_body(const NttV2Args &A, double *lds, int t, unsigned li, const GaloisTab *gal = nullptr,
                                            const TensorSrc *ten = nullptr) {
    BODY_TAG(P51);
    constexpr int Q = LOGN - 12;
    typedef ColsGeom<Q> Geo;
    constexpr unsigned N = 1u << LOGN;
    const double p = A.modc[t].p, pinv = A.modc[t].pinv;
    const double *tw = A.tw + (size_t)t * N;
    const unsigned tid = threadIdx.x;
    const Geo geo(tid & 255u, tid >> 8);          // column pass: this quarter's column tile
    const unsigned row = tid >> 4, lo4 = tid & 15;  // row pass: one row per 16 lanes
    const unsigned voff = geo.r * 256u + geo.c0 + geo.c, pr = row_pair_index(row, lo4, 0);
    double *grp = lds + row * V2_GS;
    WMul ninv = WMul{0.0, 0.0}, wlast = WMul{0.0, 0.0};
    double cadd = 0.0;
    if (INV) {
        ninv = A.tw_ninv[t];
        wlast = A.tw_last[t];
        if (F64 && A.use_fin_val) { ninv = A.fin_val.ninv; wlast = A.fin_val.wlast; cadd = A.fin_val.cadd; }
        else if (A.fin) { ninv = A.fin[li].ninv; wlast = A.fin[li].wlast; cadd = A.fin[li].cadd; }
    }
    const unsigned i0 = blockIdx.y * (unsigned)A.items_per_z;
    const unsigned i1 = (i0 + A.items_per_z < (unsigned)A.items) ? i0 + A.items_per_z : (unsigned)A.items;
    for (unsigned it = i0; it < i1; it++) {
        const u64d *src = A.src + (size_t)it * A.map.src_item_stride + (size_t)li * N;
        u64d *dst = A.dst + (size_t)it * A.map.dst_item_stride + (size_t)li * N;
        double x[16];
        if (!INV) {
            u64d raw[16];
            if (SRC == SRC_REAL) {  // every other word: the real parts
                const u64d *cw = A.src + 2 * (size_t)it * A.map.src_item_stride;
#pragma unroll
                for (int e = 0; e < 16; e++) raw[e] = *(scalar_base(cw + Geo::G * 512u * e) + 2u * voff);
            } else {
#pragma unroll
                for (int e = 0; e < 16; e++) raw[e] = stream_load<NT>(scalar_base(src + Geo::G * 256u * e) + voff);
            }
            NTT_SCHED_FENCE();
            double largest = 0.0;
#pragma unroll
            for (int e = 0; e < 16; e++) x[e] = SRC == SRC_REAL ? real_word(__longlong_as_double((long long)raw[e]), A.factor, p, pinv, largest) : u2d(raw[e]);
            if (SRC == SRC_REAL && !(largest < 4.0e18)) *A.overflow = 1;
            // Limbs of N >= 2^13 that stay in the caches (streamed from 256 MB on) lose by the shorter plan with canon_near: 200 items of 9 limbs at
            // N = 2^14 123.2 us reduced, 125.4 near, at 2^13 69.8 and 70.6, 400 120.5 and 123.0; streamed or smaller ones gain (1000 at 2^14 650.7 and 647.5, 400 at
            // 2^12 48.0 and 47.3).  Reduced with a plan for 1p as well (these words are canonical) N = 2^14 spills: 128.9.
            constexpr bool NEAR = NT || LOGN == 12 || SRC == SRC_REAL;
            wg_fwd_block<LOGN, P51, NEAR ? 256 : P51 ? 308 : 692, NEAR ? ROW_NEAR : ROW_REDUCED>(x, tw, 1u, lds, p, pinv, []() {});
            // canonical words out in word pairs: 16 bytes per lane, 256 contiguous bytes per row and store
#pragma unroll
            for (int s = 0; s < 8; s++) {
                const double *rr = grp + row_pair_lds(lo4, s);
                const double v0 = P51 || !NEAR ? canon_small(rr[0], p) : canon_near<P51>(rr[0], p, pinv), v1 = P51 || !NEAR ? canon_small(rr[1], p) : canon_near<P51>(rr[1], p, pinv);
                stream_store<NT>((ulonglong2 *)dst + 16 * s + pr, make_ulonglong2(d2u(v0), d2u(v1)));
            }
        } else {
            wg_inv_limb<LOGN, P51, SRC>(x, src, tw, lds, p, pinv, ninv, wlast, li, it, gal, ten);
#pragma unroll
            for (int e = 0; e < 16; e++) {
                const double v = canon_near<P51>(x[e] + cadd, p, pinv);  // 1.5p and less than p
                stream_store<NT>(scalar_base(dst + Geo::G * 256u * e) + voff, F64 ? (u64d)__double_as_longlong(v) : d2u(v));
            }
        }
        __syncthreads();  // the matrix is free for the next item
    }
}

// grid: x = limb slot within an item, y = chunk of items; block = N/16 threads
template <bool INV, int LOGN, bool NT = false, bool F64 = false>
__global__ __launch_bounds__((1 << LOGN) / 16) void ntt_wg_kernel(NttV2Args A) {
    __shared__ double lds[((1 << LOGN) >> 8) * V2_GS];
    unsigned item_unused, li;
    const int t = resolve_limb(A.map, blockIdx.x, item_unused, li);
    if (t < 0) return;
    if (is_p51(A.p51, t))
        ntt_wg_body<INV, LOGN, true, F64, NT>(A, lds, t, li);
    else
        ntt_wg_body<INV, LOGN, false, F64, NT>(A, lds, t, li);
}

// an encoding's real coefficients, same grid
template <int LOGN, bool NT>
__global__ __launch_bounds__((1 << LOGN) / 16) void ntt_wg_fwd_real_kernel(NttV2Args A) {
    __shared__ double lds[((1 << LOGN) >> 8) * V2_GS];
    unsigned item_unused, li;
    const int t = resolve_limb(A.map, blockIdx.x, item_unused, li);
    if (t < 0) return;
    if (is_p51(A.p51, t)) ntt_wg_body<false, LOGN, true, false, NT, SRC_REAL>(A, lds, t, li);
    else ntt_wg_body<false, LOGN, false, false, NT, SRC_REAL>(A, lds, t, li);
}

// conversion inputs of a key switch (doubles), same grid: a rotation's polynomial, a product's third tensor component
template <int LOGN>
__global__ __launch_bounds__((1 << LOGN) / 16) void ntt_wg_inv_gal_kernel(NttV2Args A, GaloisTab G) {
    __shared__ double lds[((1 << LOGN) >> 8) * V2_GS];
    unsigned item_unused, li;
    const int t = resolve_limb(A.map, blockIdx.x, item_unused, li);
    if (t < 0) return;
    if (is_p51(A.p51, t)) ntt_wg_body<true, LOGN, true, true, false, 1>(A, lds, t, li, &G);
    else ntt_wg_body<true, LOGN, false, true, false, 1>(A, lds, t, li, &G);
}
template <int LOGN>
__global__ __launch_bounds__((1 << LOGN) / 16) void tensor_wg_kernel(NttV2Args A, TensorSrc T) {
    __shared__ double lds[((1 << LOGN) >> 8) * V2_GS];
    unsigned item_unused, li;
    const int t = resolve_limb(A.map, blockIdx.x, item_unused, li);
    if (t < 0) return;
    if (is_p51(A.p51, t)) ntt_wg_body<true, LOGN, true, true, false, 2>(A, lds, t, li, nullptr, &T);
    else ntt_wg_body<true, LOGN, false, true, false, 2>(A, lds, t, li, nullptr, &T);
}
