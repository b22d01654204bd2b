// Key switching at N = 2^12 and 2^13 without the lifted limbs in memory: ModUp's conversion, the whole forward transform of a
// lifted limb and the inner product with the switching key in ONE workgroup.
//
// modup_cols_kernel + rows_inner_kernel (ks_fused.h) carry beta * E limbs per polynomial through memory between the column
// and the row pass of their transform, the largest traffic of a product.  A block of 2^12 words does not need to: a workgroup
// owns (extended limb x, block, item), walks the digits, converts the digit's words (coefficient form, read by all extended
// limbs of the item), transforms them in LDS and adds their products with the key words to the accumulators in its
// registers.  N = 2^13 is cut into two blocks as in ks_wg.h.  Two workgroups of four waves per compute unit (256 registers:
// accumulators, key words and the words in transform; the product form spills 20 around its own digit's operands); what bounds it is
// the vector ALU (about 95 instructions per word and digit) and two barriers per digit.  Products at 8 primes, 256 items, with the on-chip
// tail of ks_wg.h: N = 2^12 621 -> 427 us, 2^13 1160 -> 920 us (this kernel 354 and 734).
#pragma once
#include "ks_wg.h"

struct InnerWgArgs {
    RowsInnerArgs R;   // dtA, kt unused
    const double *y;   // [items][level][N] conversion inputs, coefficient form, canonical, as doubles
    const WMul *cc;    // ModUp constants [beta_top][alpha][alpha][T]
    int items, items_x;
};

// LDS of a workgroup: the matrix of wg_fwd_block, the first row round's twiddles [M/256][16] and the second's [15][M/16].  All
// digits of a workgroup use the same twiddles, and fetching them per digit exposes their latency three times.
template <int LOGM>
struct InnerWgLds {
    static constexpr unsigned T = (1u << LOGM) / 16, MAT = ((1u << LOGM) >> 8) * V2_GS, TW1 = MAT, TW2 = TW1 + T, TOTAL = TW2 + 15 * T;
};

// wg_fwd_block with the twiddles at hand: twc the column round's (a block of 2^12 words has one), the row rounds' in LDS.  One
// barrier inside; the caller puts one between a digit's last use of the matrix and the next digit.
template <int LOGM, bool P51, int ENTRY256, class F>
__device__ __forceinline__ void inner_fwd_block(double (&x)[16], const double (&twc)[15], double *lds, double p, double pinv, F request) {
    static_assert(LOGM == 12, "one column round");
    typedef ColsGeom<0> Geo;
    typedef ColsMasks<0, P51, ENTRY256> Mk;
    typedef RowMasks<P51, ROW_FACTOR> Rm;
    typedef InnerWgLds<LOGM> Lay;
    const unsigned tid = threadIdx.x, row = tid >> 4, lo4 = tid & 15;
    const Geo geo(tid & 255u, tid >> 8);
    double *grp = lds + row * V2_GS;
    fwd_round<Mk::F1>(x, twc, p, pinv);
#pragma unroll
    for (int e = 0; e < 16; e++) lds[wg_pad(e, geo.c0 + geo.c)] = x[e];
    __syncthreads();
    request();
#pragma unroll
    for (int e = 0; e < 16; e++) x[e] = grp[e * 17 + lo4];
    {
        double t1[15];
#pragma unroll
        for (int i = 0; i < 15; i++) t1[i] = lds[Lay::TW1 + row * 16 + i];
        fwd_round<Rm::F1>(x, t1, p, pinv);
    }
#pragma unroll
    for (int e = 0; e < 16; e++) grp[e * 17 + lo4] = x[e];
    ROW_GROUP_SYNC();
#pragma unroll
    for (int e = 0; e < 16; e++) x[e] = grp[lo4 * 17 + e];
    {
        double t2[15];
#pragma unroll
        for (int i = 0; i < 15; i++) t2[i] = lds[Lay::TW2 + i * Lay::T + tid];
        fwd_round<Rm::F2>(x, t2, p, pinv);
    }
#pragma unroll
    for (int e = 0; e < 16; e++) grp[lo4 * 17 + e] = P51 ? reduce_balanced(x[e], p, pinv) : x[e];
    ROW_GROUP_SYNC();
}

template <int LOGM, int S, int NSRC, bool P51, bool GAL>
__device__ __forceinline__ void inner_wg_body(const InnerWgArgs &A, const KeyTab &K, double *lds, int t, unsigned x, unsigned item, unsigned blk,
                                              const GaloisTab *gal) {
    BODY_TAG(P51);
    typedef ColsGeom<LOGM - 12> Geo;
    constexpr unsigned M = 1u << LOGM, N = M << S;
    typedef InnerWgLds<LOGM> Lay;
    const RowsInnerArgs &R = A.R;
    const double p = R.modc[t].p, pinv = R.modc[t].pinv;
    const double *tw = R.tw + (size_t)t * N;
    const unsigned tid = threadIdx.x, prow = tid >> 4, lo4 = tid & 15, base = (1u << S) + blk;
    const u64d *key = K.key[K.slot[item]];
    const size_t tile0 = (size_t)blk * M;
    double a0[16], a1[16];
#pragma unroll
    for (int i = 0; i < 16; i++) a0[i] = a1[i] = 0.0;
    const int j_own = (int)x < R.level ? (int)x / R.alpha : -1;
    const bool tensor_mode = !GAL && R.ta != nullptr && j_own >= 0;
    int pending = 1;
    inner_own_digit<P51, GAL>(R, key, item, t, x, j_own, tensor_mode, tile0, prow, lo4, p, pinv, a0, a1, pending, gal);
    // twiddles of the first S stages on the way to this block, see conv_final_body
    double w[S + 1], wp[S + 1];
#pragma unroll
    for (int q = 0; q < S; q++) {
        const double v = tw[(1u << q) + (blk >> (S - q))];
        w[q] = ((blk >> (S - 1 - q)) & 1u) ? -v : v;
        wp[q] = w[q] * pinv;
    }
    const Geo geo(tid & 255u, tid >> 8);
    const unsigned voff = geo.r * 256u + geo.c0 + geo.c, pr = row_pair_index(prow, lo4, 0);
    double twc[15];
#pragma unroll
    for (int s = 0; s < 4; s++)
#pragma unroll
        for (int b = 0; b < (1 << s); b++) twc[(1 << s) - 1 + b] = table_load(tw, (base << s) + b);
    {
        const unsigned base1 = base * (M >> 8) + prow;
#pragma unroll
        for (int s = 0; s < 4; s++)
#pragma unroll
            for (int b = 0; b < (1 << s); b++) lds[Lay::TW2 + ((1 << s) - 1 + b) * Lay::T + tid] = tw[((16u * base1 + lo4) << s) + b];
        if (lo4 < 15) {
            // entry i = (1 << s) - 1 + b of the row's first round
            const unsigned s = (lo4 >= 7) ? 3 : (lo4 >= 3) ? 2 : (lo4 >= 1) ? 1 : 0, b = lo4 - ((1u << s) - 1);
            lds[Lay::TW1 + prow * 16 + lo4] = tw[(base1 << s) + b];
        }
    }
    for (int j = 0; j < R.beta; j++) {
        if (j == j_own) continue;
        const int lo = j * R.alpha, nd = R.level - lo < R.alpha ? R.level - lo : R.alpha;
        double xx[16];
        {
            const double *y = A.y + ((size_t)item * R.level + lo) * N;
            WMul Wc[NSRC];
            const size_t crow = ((size_t)lo + (nd - 1)) * R.alpha;
#pragma unroll
            for (int a = 0; a < NSRC; a++) Wc[a] = a < nd ? A.cc[(crow + a) * R.T + t] : WMul{0.0, 0.0};
            constexpr int CH = NSRC > 1 ? (8 >> S) : (16 >> S);  // words formed together: bounds the source words in flight
#pragma unroll
            for (int e0 = 0; e0 < 16; e0 += CH) {
                double src[CH][1 << S][NSRC];
#pragma unroll
                for (int e = 0; e < CH; e++)
#pragma unroll
                    for (int q = 0; q < (1 << S); q++)
#pragma unroll
                        for (int a = 0; a < NSRC; a++)  // a missing source (digit cut short by the level) re-reads the first one: its constant is zero
                            src[e][q][a] = scalar_base(y + ((size_t)(a < nd ? a : 0) * N + (size_t)q * M + Geo::G * 256u * (e0 + e)))[voff];
                SCHED_FENCE();
#pragma unroll
                for (int e = 0; e < CH; e++) {
                    double u[1 << S];
#pragma unroll
                    for (int q = 0; q < (1 << S); q++) u[q] = conv_word<NSRC, P51>(src[e][q], Wc, 0.0, p, pinv);
#pragma unroll
                    for (int q1 = 0; q1 < S; q1++)
#pragma unroll
                        for (int q = 0; q < (1 << (S - 1 - q1)); q++) u[q] += mulmod_w(u[q + (1 << (S - 1 - q1))], w[q1], wp[q1], p);
                    xx[e0 + e] = (P51 && S >= 2) ? reduce_balanced(u[0], p, pinv) : u[0];
                }
#pragma unroll
                for (int e = 0; e < CH; e++) PIN_VALUE(xx[e0 + e]);
            }
        }
        const ulonglong2 *k0 = (const ulonglong2 *)(key + (((size_t)j * 2 + 0) * R.T + t) * N + tile0);
        const ulonglong2 *k1 = (const ulonglong2 *)(key + (((size_t)j * 2 + 1) * R.T + t) * N + tile0);
        ulonglong2 kr0[8], kr1[8];
        __syncthreads();  // everybody is done with the matrix (before the first digit: the twiddles are in place)
        inner_fwd_block<LOGM, P51, block_entry<P51, NSRC, false, S>()>(xx, twc, lds, p, pinv, [&]() {
#pragma unroll
            for (int s = 0; s < 8; s++) {
                kr0[s] = (k0 + 16 * s)[pr];
                kr1[s] = (k1 + 16 * s)[pr];
            }
        });
        const double *grp = lds + prow * V2_GS;
#pragma unroll
        for (int s = 0; s < 8; s++) {
            const double *vrow = grp + row_pair_lds(lo4, s);
            key_term<P51>(kr0[s].x, kr1[s].x, vrow[0], p, pinv, a0[2 * s], a1[2 * s]);
            key_term<P51>(kr0[s].y, kr1[s].y, vrow[1], p, pinv, a0[2 * s + 1], a1[2 * s + 1]);
        }
        if (++pending == KEY_TERMS<P51>) {
#pragma unroll
            for (int i = 0; i < 16; i++) {
                a0[i] = reduce_balanced(a0[i], p, pinv);
                a1[i] = reduce_balanced(a1[i], p, pinv);
            }
            pending = 0;
        }
    }
    inner_store<P51, GAL, false>(R, item, t, x, tensor_mode, tile0, prow, lo4, p, pinv, a0, a1, gal);
}

// Consecutive workgroups go to the 8 XCDs in turn: an item's blocks sit on one XCD (they read the same sources), the items of an
// extended limb are dealt over the XCDs (each keeps the limb's key words, 2 * beta * N of them, in its L2).
__device__ __forceinline__ bool inner_wg_place(const InnerWgArgs &A, int S, unsigned &item, unsigned &blk) {
    const unsigned X = (unsigned)A.items_x, g = blockIdx.x / (X << S), r = blockIdx.x % (X << S);
    blk = WG_UNIFORM(r / X);
    item = WG_UNIFORM(g * X + r % X);
    return item < (unsigned)A.items;
}

// grid: x = see inner_wg_place, y = extended limb; block = M/16 threads
template <int LOGM, int S, int NSRC>
__global__ __launch_bounds__((1 << LOGM) / 16, 2) void inner_wg_kernel(InnerWgArgs A, KeyTab K) {
    __shared__ double lds[InnerWgLds<LOGM>::TOTAL];
    unsigned item, blk;
    if (!inner_wg_place(A, S, item, blk)) return;
    const unsigned x = blockIdx.y;
    const int t = (int)x < A.R.level ? (int)x : A.R.n_q + (int)x - A.R.level;
    if (is_p51(A.R.p51, t)) inner_wg_body<LOGM, S, NSRC, true, false>(A, K, lds, t, x, item, blk, nullptr);
    else inner_wg_body<LOGM, S, NSRC, false, false>(A, K, lds, t, x, item, blk, nullptr);
}

// the same for rotations: source polynomial and addend read through the items' automorphisms
template <int LOGM, int S, int NSRC>
__global__ __launch_bounds__((1 << LOGM) / 16, 2) void inner_wg_gal_kernel(InnerWgArgs A, KeyTab K, GaloisTab G) {
    __shared__ double lds[InnerWgLds<LOGM>::TOTAL];
    unsigned item, blk;
    if (!inner_wg_place(A, S, item, blk)) return;
    const unsigned x = blockIdx.y;
    const int t = (int)x < A.R.level ? (int)x : A.R.n_q + (int)x - A.R.level;
    if (is_p51(A.R.p51, t)) inner_wg_body<LOGM, S, NSRC, true, true>(A, K, lds, t, x, item, blk, &G);
    else inner_wg_body<LOGM, S, NSRC, false, true>(A, K, lds, t, x, item, blk, &G);
}
