// DivRound without an intermediate in memory (2^12 <= N <= 2^16, one dropped prime, and a product's tail): conversion, forward transform, last
// step of a kept limb in ONE workgroup.
//
// The register-tiled pair modup_cols_kernel / rows_final_kernel (ks_fused.h) writes every converted limb after the column
// pass of its transform and reads it back for the row pass: for a rescale that is two of the four limb transfers a kept
// limb costs, and both kernels run at the speed of a device copy.  Here a workgroup owns M = 2^LOGM words of one kept
// limb: it reads the dropped limb's words (coefficient form, shared by all kept limbs of a row and served by the L2 of the
// XCD the row's workgroups run on), converts them, takes them through the whole transform with the M x 256 decomposition of
// ntt_wg.h in LDS, and finishes its words of the kept limb.  What crosses HBM is the kept limb in and out, and the source.
//
// A ring larger than M is cut into 2^S blocks: the first S stages of the forward transform send block b of the result only
// to linear combinations of the 2^S words n + q*M, so a workgroup forms its own block's word from 2^S source words with
// 2^S - 1 products (the other blocks' workgroups repeat the conversion, which for one dropped prime is a subtraction, p < 2^50, or a reduction) and
// transforms M words from there: stage s of the block uses the twiddles (2^S + b) * 2^s + i of the whole transform's table.
//
// Measured, whole rescales as two kernels after the inverse row pass and as this one: N = 2^14, 256 ciphertexts of 8 primes 476 and 323 us;
// 2^15, 448 of 16 primes 3333 and 2460; 2^16, 64 of 24 primes 1433 and 1261; 2^13, 512 of 8 primes 499 and 303.  At N = 2^15 the kernel
// executes 110 vector instructions per word (vector ALU 0.64 busy) and moves 4.7 TB/s, where a device copy moves 4.85: the kept
// limbs in and out, and every dropped limb about 12 times of the 30 that its kept limbs and blocks read it.
// With four waves per SIMD a thread has 128 registers; a single spilled register set costs more than everything else here (0.16 us per
// 2^14 words with 44 registers spilled, 0.08 without), hence the notes to the compiler (ntt_v2.h).  Variants that lost (both sides with
// flat accesses, 0.078): 32 words per thread at two waves per SIMD with the kept limb requested before the transform (0.081 - 0.099), the
// kept limb requested after the transform (0.083 - 0.095).
#pragma once
#include "ks_fused.h"
#include "ntt_wg.h"

struct ConvFinalArgs {
    RowsFinalArgs F;        // kept limbs, addend, output (tmpA, pre, rows_per_x unused); F.rows rows of F.nc kept limbs
    const double *y;        // sources in coefficient form, canonical, stored as doubles: row r, source m at y + r*y_row_stride + m*N
    unsigned long long y_row_stride;
    DivRoundDev D;
    const double *hc2;      // FIN 4: the rescale's h mod c
    int T;
    int rows_x, rows_g;     // workgroup order, see conv_final_place
};

// Workgroup order.  Consecutive workgroup ids go to the 8 XCDs in turn, and every XCD has its own L2 (4 MB).  Rows are dealt to
// the XCDs round-robin; an XCD takes its rows in groups of rows_g (at most 8) and walks the kept limbs over a group, so
// that the group's sources (rows_g limbs) and the current limb's twiddle table stay in its L2.  A few rows that do not divide
// evenly over the XCDs form one group of rows_x = rows instead (rows_g = 1): consecutive workgroups take them in turn.
__device__ __forceinline__ bool conv_final_place(const ConvFinalArgs &A, int S, unsigned &row, unsigned &blk, int &limb) {
    const unsigned X = (unsigned)A.rows_x, G = (unsigned)A.rows_g, nc = (unsigned)A.F.nc;
    unsigned k = blockIdx.x / X;
    blk = WG_UNIFORM(k & ((1u << S) - 1u));
    k >>= S;
    const unsigned r = k % G;
    k /= G;
    limb = (int)WG_UNIFORM(k % nc);
    row = WG_UNIFORM((k / nc * G + r) * X + blockIdx.x % X);
    return row < (unsigned)A.F.rows;
}

// sum_a y_a * conv_a - h, at most p + SUM of chain_bound / 0.75p per product (four products and h of a 50-bit prime could pass 2^53
// as a ProductChain: they are summed one by one)
template <int NPROD, bool P51>
__device__ __forceinline__ double conv_sum(const double *y, const WMul *Wc, double hsub, double p, double pinv) {
    if (P51 || NPROD < 2 || NPROD > 3) {
        double v = -hsub;
#pragma unroll
        for (int a = 0; a < NPROD; a++) v += mulmod_w(y[a], Wc[a].w, Wc[a].wp, p);
        return v;
    }
    ProductChain c = chain_first(chain_origin(p), y[0], Wc[0].w);
#pragma unroll
    for (int a = 1; a < NPROD; a++) chain_add(c, y[a], Wc[a].w);
    return chain_value(c, p, pinv) - hsub;
}

// One converted coefficient: sum_a y_a * conv_a - h, balanced-reduced but for one source and p < 2^50: y - h lies between -2^50 and
// 2^51 then, 2 units of 2^50 (in which the bounds of words modulo any p < 2^50 may be read).  A single source has conv = 1 (the empty product).
template <int NSRC, bool P51>
__device__ __forceinline__ double conv_word(const double (&y)[NSRC], const WMul (&Wc)[NSRC], double hsub, double p, double pinv) {
    if (NSRC == 1) return P51 ? reduce_balanced(y[0] - hsub, p, pinv) : y[0] - hsub;  // below 2^51 + p
    return reduce_balanced(conv_sum<NSRC, P51>(y, Wc, hsub, p, pinv), p, pinv);
}
// bound of a word after the first S stages that join 2^S words of at most b
template <bool P51>
constexpr double join_bound(double b, int S) {
    for (int t = 0; t < S; t++) b += 0.5 + 1.5 * b / LazyRange<P51>::LIM;
    return b;
}
// the same in 1/256 for a block of conv_word's or (TAIL) tail_word's; p < 2^51: reduced words, and reduced again after two stages
template <bool P51, int NSRC, bool TAIL, int S>
constexpr int block_entry() {
    const double b = P51 || (NSRC > 1 && !TAIL) ? LAZY_REDUCED : TAIL ? 2.75 : 2.0;
    return (int)(256.0 * (P51 && S >= 2 ? LAZY_REDUCED : join_bound<P51>(b, S)) + 0.999);
}

// The same for ModDown followed by rescale as one conversion (see modup_cols_kernel MODE 3): y[0] is the rescale's conversion
// input y_B, y[1 ..] ModDown's; the value is (sum_a y_a * conv_a - hA) * P^-1 + y_B - hB.
template <int NSRC, bool P51>
__device__ __forceinline__ double tail_word(const double (&y)[NSRC], const WMul (&Wc)[NSRC], double hA, WMul Pinv, double hB, double p, double pinv) {
    // one special prime: its constant is 1; below 2^51 + p
    const double v = NSRC == 2 ? y[1] - hA : conv_sum<NSRC - 1, P51>(&y[1], &Wc[1], hA, p, pinv);
    if (P51) return reduce_balanced(mulmod_w(reduce_balanced(v, p, pinv), Pinv.w, Pinv.wp, p) + y[0] - hB, p, pinv);
    // p < 2^50: y_B is below 2^51, and v (2 units of 2^50 with one special prime, below 2^53 with more, which are reduced) gives a
    // product of at most 0.75p: 2.75
    return mulmod_w(NSRC == 2 ? v : reduce_balanced(v, p, pinv), Pinv.w, Pinv.wp, p) + y[0] - hB;
}

// FIN 0: out = (x - r) * Binv;  1: out = x - r * Binv (x holds x * Binv + addend);  2: out = (x * xmv - r) * Binv (+ addend);
// 3: out = (x - r) * Binv + sigma_g(addend) on even rows (rotations from a shared ModUp, see RowsFinalGal);  4: FIN 0 for ModDown
// followed by rescale in one conversion (sources from tail_sources_kernel; D describes the ModDown, F.Binv the rescale)
template <int LOGM, int S, int NSRC, int FIN, bool P51, bool NTS>
__device__ __forceinline__ void conv_final_body(const ConvFinalArgs &A, double *lds, int i, unsigned row, unsigned blk, WMul xmv,
                                                const RowsFinalGal *gal) {
    typedef ColsGeom<LOGM - 12> Geo;
    constexpr unsigned M = 1u << LOGM, N = M << S;
    BODY_TAG(P51);
    const RowsFinalArgs &F = A.F;
    const double p = F.modc[i].p, pinv = F.modc[i].pinv;
    const double *tw = F.tw + (size_t)i * N;
    const unsigned tid = threadIdx.x, prow = tid >> 4, lo4 = tid & 15, base = (1u << S) + blk;
    double x[16];
    {
        const Geo geo(tid & 255u, tid >> 8);
        // uniform base addresses plus one offset per thread: no 64-bit address arithmetic per load
        const double *y = A.y + (size_t)row * A.y_row_stride;
        const unsigned voff = geo.r * 256u + geo.c0 + geo.c;
        WMul Wc[NSRC];
#pragma unroll
        for (int a = 0; a < NSRC; a++) Wc[a] = A.D.conv[(size_t)(FIN == 4 ? (a ? a - 1 : 0) : a) * A.T + i];
        const double hsub = A.D.hc[i];
        const WMul Pinv = FIN == 4 ? A.D.Binv[i] : WMul{0.0, 0.0};
        const double hB = FIN == 4 ? A.hc2[i] : 0.0;
        // twiddles of the first S stages on the way to this block (negative: the block lies in the lower branch's difference)
        double w[S + 1], wp[S + 1];
#pragma unroll
        for (int t = 0; t < S; t++) {
            const double v = tw[(1u << t) + (blk >> (S - t))];
            w[t] = ((blk >> (S - 1 - t)) & 1u) ? -v : v;
            wp[t] = w[t] * pinv;
        }
        constexpr int CH = (NSRC > 1 ? 8 : 16) >> S;  // words formed together: bounds the source words in flight
#pragma unroll
        for (int e0 = 0; e0 < 16; e0 += CH) {
            double src[CH][1 << S][NSRC];
#pragma unroll
            for (int e = 0; e < CH; e++)
#pragma unroll
                for (int q = 0; q < (1 << S); q++)
#pragma unroll
                    for (int a = 0; a < NSRC; a++) src[e][q][a] = scalar_base(y + ((size_t)a * N + (size_t)q * M + Geo::G * 256u * (e0 + e)))[voff];
            SCHED_FENCE();
#pragma unroll
            for (int e = 0; e < CH; e++) {
                double u[1 << S];
#pragma unroll
                for (int q = 0; q < (1 << S); q++)
                    u[q] = FIN == 4 ? tail_word<NSRC, P51>(src[e][q], Wc, hsub, Pinv, hB, p, pinv) : conv_word<NSRC, P51>(src[e][q], Wc, hsub, p, pinv);
                // stage t joins the words 2^(S-1-t) * M apart
#pragma unroll
                for (int t = 0; t < S; t++)
#pragma unroll
                    for (int q = 0; q < (1 << (S - 1 - t)); q++) u[q] += mulmod_w(u[q + (1 << (S - 1 - t))], w[t], wp[t], p);
                x[e0 + e] = (P51 && S >= 2) ? reduce_balanced(u[0], p, pinv) : u[0];
            }
#pragma unroll
            for (int e = 0; e < CH; e++) PIN_VALUE(x[e0 + e]);
        }
    }
    const size_t off = (size_t)i * N + (size_t)blk * M;
    const ulonglong2 *xin = (const ulonglong2 *)(F.x + (size_t)row * F.x_row_stride + off);
    ulonglong2 *out = (ulonglong2 *)(F.out + (size_t)row * F.out_row_stride + off);
    const unsigned pr = row_pair_index(prow, lo4, 0);
    ulonglong2 xr[8];
    wg_fwd_block<LOGM, P51, block_entry<P51, NSRC, FIN == 4, S>(), ROW_LAZY>(x, tw, base, lds, p, pinv, [&]() {
        stream_if(F.stream == STREAM_ALL, [&](auto nt) {
#pragma unroll
            for (int s = 0; s < 8; s++) xr[s] = stream_load<nt>(xin + 16 * s + pr);
        });
    });
    const WMul W = F.Binv[i];
    const bool add = F.addend != nullptr && (FIN == 2 || (FIN == 3 && (row & 1u) == 0));
    const double *grp = lds + prow * V2_GS;
    auto finish = [&](int s, bool with, ulonglong2 ar) {
        const double *rr = grp + row_pair_lds(lo4, s);
        double x0 = u2d(xr[s].x), x1 = u2d(xr[s].y);
        if (FIN == 2) {  // |x * xmv| <= 0.75p; r is below ROWX, x - r within the range of a product
            x0 = mulmod_w(x0, xmv.w, xmv.wp, p);
            x1 = mulmod_w(x1, xmv.w, xmv.wp, p);
        }
        double v0 = FIN == 1 ? x0 - mulmod_w(rr[0], W.w, W.wp, p) : mulmod_w(x0 - rr[0], W.w, W.wp, p);
        double v1 = FIN == 1 ? x1 - mulmod_w(rr[1], W.w, W.wp, p) : mulmod_w(x1 - rr[1], W.w, W.wp, p);
        if (with) {
            v0 += u2d(ar.x);
            v1 += u2d(ar.y);
        }
        // a product below 1.5p and an addend, or a word and a product of a word of at most ROWX: 2.5p
        stream_store<NTS>(out + 16 * s + pr, make_ulonglong2(d2u(canon_near<P51>(v0, p, pinv)), d2u(canon_near<P51>(v1, p, pinv))));
    };
    if (FIN < 2 || FIN == 4 || !add) {
#pragma unroll
        for (int s = 0; s < 8; s++) finish(s, false, make_ulonglong2(0ull, 0ull));
        return;
    }
    ulonglong2 ar[8];
    if (FIN == 3) {
        const unsigned pair = row / 2u, item = pair / (unsigned)gal->R, g = gal->g[pair % (unsigned)gal->R];
        const u64d *limb = F.addend + (size_t)item * F.add_item_stride + (size_t)i * N;
#pragma unroll
        for (int s = 0; s < 8; s++) ar[s] = galois_pair_load(limb, blk * M + prow * 256u + 32u * s + 2u * lo4, g, LOGM + S);
    } else {
        const ulonglong2 *ad = (const ulonglong2 *)(F.addend + (size_t)(row / 2) * F.add_item_stride + (size_t)(row % 2) * F.add_comp_stride + off);
#pragma unroll
        for (int s = 0; s < 8; s++) ar[s] = (ad + 16 * s)[pr];
    }
#pragma unroll
    for (int s = 0; s < 8; s++) finish(s, true, ar[s]);
}

// grid: x = rows_x * 2^S * rows_g * nc * (row groups), see conv_final_place; block = M/16 threads
template <int LOGM, int S, int NSRC, int FIN, bool NTS = false>
__global__ __launch_bounds__((1 << LOGM) / 16, 4) void conv_final_kernel(ConvFinalArgs A) {
    __shared__ double lds[((1 << LOGM) >> 8) * V2_GS];
    unsigned row, blk;
    int i;
    if (!conv_final_place(A, S, row, blk, i)) return;
    if (is_p51(A.F.p51, i)) conv_final_body<LOGM, S, NSRC, FIN, true, NTS>(A, lds, i, row, blk, WMul{0.0, 0.0}, nullptr);
    else conv_final_body<LOGM, S, NSRC, FIN, false, NTS>(A, lds, i, row, blk, WMul{0.0, 0.0}, nullptr);
}

// the kept limb multiplied by a per-call scalar first (rescale of a scalar multiple)
template <int LOGM, int S, bool NTS>
__global__ __launch_bounds__((1 << LOGM) / 16, 4) void conv_final_scalar_kernel(ConvFinalArgs A, ScalarTab Sc) {
    __shared__ double lds[((1 << LOGM) >> 8) * V2_GS];
    unsigned row, blk;
    int i;
    if (!conv_final_place(A, S, row, blk, i)) return;
    if (is_p51(A.F.p51, i)) conv_final_body<LOGM, S, 1, 2, true, NTS>(A, lds, i, row, blk, Sc.c[i], nullptr);
    else conv_final_body<LOGM, S, 1, 2, false, NTS>(A, lds, i, row, blk, Sc.c[i], nullptr);
}

// rotations from a shared ModUp
template <int LOGM, int S, int NSRC, bool NTS = false>
__global__ __launch_bounds__((1 << LOGM) / 16, 4) void conv_final_gal_kernel(ConvFinalArgs A, RowsFinalGal G) {
    __shared__ double lds[((1 << LOGM) >> 8) * V2_GS];
    unsigned row, blk;
    int i;
    if (!conv_final_place(A, S, row, blk, i)) return;
    if (is_p51(A.F.p51, i)) conv_final_body<LOGM, S, NSRC, 3, true, NTS>(A, lds, i, row, blk, WMul{0.0, 0.0}, &G);
    else conv_final_body<LOGM, S, NSRC, 3, false, NTS>(A, lds, i, row, blk, WMul{0.0, 0.0}, &G);
}

// ------------------------------------------------------------------ sources of ModDown followed by rescale
// The limb a product's rescale drops and the special limbs of one row (neighbours in the extended layout), taken through their
// inverse transforms by one workgroup, in place: ModDown's conversion inputs y_m, and in place of the dropped limb the
// rescale's y_B = (s + h_B) mod q_last, s = u - (sum_m y_m * conv_m - h_A) * P^-1 the ModDown result of that limb, whose
// evaluation form u comes in with P^-1 and the addend already applied (z of the inner product).  512 rows of two limbs at N = 2^14: 0.11 ms
// for this kernel and 0.36 for the kept limbs, against 0.07 (inverse row pass) + 0.21 (conversion) + 0.30 (last pass).
struct TailSourcesArgs {
    u64d *bl;                          // row r, limb m at bl + r*row_stride + m*N; results as doubles
    unsigned long long row_stride;
    const ModConst *modc;
    const double *tw_inv;
    const FinConst *fin;               // [k + 1] last-stage constants
    DivRoundDev D;                     // the ModDown; its kept limb b_idx0 is the dropped one
    double hb2;
    int T, last, n_q, k;
    P51Mask p51;
};

template <int LOGN>
__global__ __launch_bounds__((1 << LOGN) / 16) void tail_sources_kernel(TailSourcesArgs A) {
    __shared__ double lds[((1 << LOGN) >> 8) * V2_GS];
    typedef ColsGeom<LOGN - 12> Geo;
    constexpr unsigned N = 1u << LOGN;
    const unsigned tid = threadIdx.x;
    const Geo geo(tid & 255u, tid >> 8);
    const unsigned voff = geo.r * 256u + geo.c0 + geo.c;
    u64d *bl = A.bl + (size_t)blockIdx.x * A.row_stride;
    for (int mm = 1; mm <= A.k + 1; mm++) {
        const int m = mm <= A.k ? mm : 0;  // the dropped limb comes last
        const int t = m ? A.n_q + m - 1 : A.last;
        const double p = A.modc[t].p, pinv = A.modc[t].pinv;
        const FinConst F = A.fin[m];
        u64d *limb = bl + (size_t)m * N;
        double x[16];
        if (is_p51(A.p51, t)) wg_inv_limb<LOGN, true, 0>(x, limb, A.tw_inv + (size_t)t * N, lds, p, pinv, F.ninv, F.wlast, 0, 0, nullptr, nullptr);
        else wg_inv_limb<LOGN, false, 0>(x, limb, A.tw_inv + (size_t)t * N, lds, p, pinv, F.ninv, F.wlast, 0, 0, nullptr, nullptr);
        if (m) {
#pragma unroll
            for (int e = 0; e < 16; e++) scalar_base((double *)limb + Geo::G * 256u * e)[voff] = canon(x[e] + F.cadd, p, pinv);
        } else {
            const double hA = A.D.hc[t];
            const WMul Pinv = A.D.Binv[t];
            double v[16];
#pragma unroll
            for (int e = 0; e < 16; e++) v[e] = -hA;
            for (int a = 0; a < A.k; a++) {  // this thread wrote these words itself
                const WMul W = A.D.conv[(size_t)a * A.T + t];
                const u64d *y = bl + (size_t)(a + 1) * N;
                // Words requested together, as many as the registers hold beside the waves that were there: all of them at N = 2^12 (one by one: 12.4 us for 32 rows,
                // 11.4 like this; 27.1 and 24.8 for 1024), four above (eight at 2^14 spill, 512 rows 119 us, four 107, one by one 108; 16 at
                // 2^13 are one workgroup per compute unit instead of two, 512 rows 46.3 -> 49.5, four 43.6).
                constexpr int CH = LOGN == 12 ? 16 : 4;
#pragma unroll
                for (int e0 = 0; e0 < 16; e0 += CH) {
                    double yw[CH];
#pragma unroll
                    for (int e = 0; e < CH; e++) yw[e] = scalar_base((const double *)y + Geo::G * 256u * (e0 + e))[voff];
                    SCHED_FENCE();
#pragma unroll
                    for (int e = 0; e < CH; e++) v[e0 + e] += mulmod_w(yw[e], W.w, W.wp, p);  // <= p + 3 * 0.75p
                }
            }
#pragma unroll
            for (int e = 0; e < 16; e++) {
                const double s = canon(x[e] + F.cadd, p, pinv) - mulmod_w(reduce_balanced(v[e], p, pinv), Pinv.w, Pinv.wp, p);  // (-0.75p, 1.75p)
                scalar_base((double *)limb + Geo::G * 256u * e)[voff] = canon(s + A.hb2, p, pinv);
            }
        }
        __syncthreads();  // the matrix is free for the next limb
    }
}
