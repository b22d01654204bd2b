// Fused key-switch / DivRound kernels for 2^12 <= N <= 2^16, built on the register-tiled
// transform passes of ntt_v2.h.  They remove the HBM round trips between a transform and the
// limb-wise step next to it:
//
//   tensor_rows_kernel : tensor product of a tile + the inverse row pass of its third component;
//   modup_cols_kernel  : inverse column pass of the source tiles, fast basis conversion (ModUp of
//                        a digit, or the conversion step of DivRound) and the column pass of the
//                        forward transform of every converted limb -- neither the conversion
//                        inputs nor the converted limbs are ever stored in coefficient form;
//   rows_inner_kernel  : row pass of the forward transform of every digit's extended limb,
//                        multiplied by the switching key and accumulated over the digits in
//                        registers -- the transformed limbs are never stored;
//   rows_final_kernel  : row pass fused with DivRound's last step
//                        out = (x - NTT(r - h)) * Bbar^-1 (+ addend).
//
// The conversion inputs y (y_i = d_i * qhat_i^-1 mod q_i, canonical) come out of the inverse
// transform itself: its last stage multiplies by 1/N anyway, so the extra constant rides along
// (FinConst).
#pragma once
#include "ntt_v2.h"

#ifdef CKKSMI_EMULATE
#define SCHED_FENCE() ((void)0)
#else
#define SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)
#endif

// ------------------------------------------------------------------ third tensor component + its inverse row pass
// The composite multiply feeds d2 = a1*b1 straight into key switching, whose first step is the inverse transform of
// d2.  This kernel forms d2 of one 4096-word tile (summed over the terms of a sum of products) and takes it through the
// inverse ROW pass while it is on chip; the column pass follows in the ModUp kernel.  Nothing else of the tensor is
// written anywhere: the fused inner product forms d0, d1 and d2 again from the operands where it needs them
// (rows_inner_kernel, tensor mode), which costs it one more limb read and saves this kernel six limb transfers.
struct TensorRowsArgs {
    const u64d *a, *b;   // [items][terms][2][level][N]
    u64d *ymid;          // [items][level][N]: inverse row pass of d2 (reduced doubles)
    const ModConst *modc;
    const double *tw_inv;
    int logN, level;
    int terms;
    int stream;          // STREAM_* of the result
    int stream_src;      // the operands are streamed: 64 items of 24 primes at N = 2^16 386 us, 435 without
    P51Mask p51;
};

template <bool P51>
__device__ __forceinline__ void tensor_rows_body(const TensorRowsArgs &A, double *lds, unsigned item, int i) {
    BODY_TAG(P51);
    const unsigned N = 1u << A.logN, N1 = N >> 8;
    const ModConst mc = A.modc[i];
    const double p = mc.p, pinv = mc.pinv;
    const unsigned tid = threadIdx.x, hi4 = tid >> 4, lo4 = tid & 15;
    const size_t tile0 = (size_t)blockIdx.x * 4096, st = (size_t)A.level * N;
    double tw1[15], tw2[15];
    load_twiddles(A.tw_inv + (size_t)i * N, N1 + blockIdx.x * 16 + hi4, lo4, tw1, tw2);
    // second components of the operands
    const ulonglong2 *a1 = (const ulonglong2 *)(A.a + ((size_t)item * A.terms * 2 * A.level + A.level + i) * N + tile0);
    const ulonglong2 *b1 = (const ulonglong2 *)(A.b + ((size_t)item * A.terms * 2 * A.level + A.level + i) * N + tile0);
    double *grp = lds + hi4 * V2_GS;
    // word pairs in the row-pair layout (every row stays with its 16 lanes: no workgroup barrier)
    ulonglong2 A1[8], B1[8];
    stream_if(A.stream_src, [&](auto nt) {
#pragma unroll
        for (int s = 0; s < 8; s++) {
            A1[s] = stream_load<nt>(a1 + row_pair_index(hi4, lo4, s));
            B1[s] = stream_load<nt>(b1 + row_pair_index(hi4, lo4, s));
        }
    });
    SCHED_FENCE();
    double d2[16];
#pragma unroll
    for (int s = 0; s < 8; s++) {
        d2[2 * s] = mulmod(u2d(A1[s].x), u2d(B1[s].x), p, pinv);
        d2[2 * s + 1] = mulmod(u2d(A1[s].y), u2d(B1[s].y), p, pinv);
    }
    for (int t = 1; t < A.terms; t++) {  // further terms of a sum of products
        const size_t to = (size_t)t * st;  // 2*level*N words = st pairs
#pragma unroll
        for (int s = 0; s < 8; s++) {
            A1[s] = a1[to + row_pair_index(hi4, lo4, s)];
            B1[s] = b1[to + row_pair_index(hi4, lo4, s)];
        }
        SCHED_FENCE();
#pragma unroll
        for (int s = 0; s < 8; s++) {  // one product 1.25p, a sum is reduced
            d2[2 * s] = reduce_balanced(d2[2 * s] + mulmod(u2d(A1[s].x), u2d(B1[s].x), p, pinv), p, pinv);
            d2[2 * s + 1] = reduce_balanced(d2[2 * s + 1] + mulmod(u2d(A1[s].y), u2d(B1[s].y), p, pinv), p, pinv);
        }
    }
#pragma unroll
    for (int s = 0; s < 8; s++) {
        double *rr = grp + row_pair_lds(lo4, s);
        rr[0] = d2[2 * s];
        rr[1] = d2[2 * s + 1];
    }
    ROW_GROUP_SYNC();
    // inverse row pass of d2 exactly as in ntt_v2_rows
    const WMul unused = WMul{0.0, 0.0};
    double x[16];
#pragma unroll
    for (int e = 0; e < 16; e++) x[e] = grp[lo4 * 17 + e];
    inv_stages<0, INV_ROW1, P51>(x, tw2, p, pinv, unused, unused);
    INV_JOIN(P51, INV_ROW1, INV_ROW2);
#pragma unroll
    for (int e = 0; e < 16; e++) grp[lo4 * 17 + e] = x[e];
    ROW_GROUP_SYNC();
#pragma unroll
    for (int e = 0; e < 16; e++) x[e] = grp[e * 17 + lo4];
    inv_stages<0, INV_ROW2, P51>(x, tw1, p, pinv, unused, unused);
    u64d *ym = A.ymid + ((size_t)item * A.level + i) * N + tile0;
    stream_if(A.stream != STREAM_NONE, [&](auto nt) {
#pragma unroll
        for (int e = 0; e < 16; e++) stream_store<nt>(&ym[hi4 * 256 + lo4 + 16 * e], mid_store(x[e]));
    });
}

// grid: x = tile (N/4096), y = limb, z = item
__global__ __launch_bounds__(V2_THREADS, 2) void tensor_rows_kernel(TensorRowsArgs A) {
    __shared__ double lds[16 * V2_GS];
    const int i = (int)blockIdx.y;
    if (is_p51(A.p51, i))
        tensor_rows_body<true>(A, lds, blockIdx.z, i);
    else
        tensor_rows_body<false>(A, lds, blockIdx.z, i);
}

// ------------------------------------------------------------------ conversion + column pass, targets looped in the workgroup
// Fast basis conversion and the column pass of the forward transform of its results, organised around the SOURCE tile:
// a workgroup reads the source tiles once (as the output of the inverse row pass, and runs their inverse column pass
// itself), keeps them in registers as doubles and produces the
// column-pass tile of every target limb of its chunk from them.  What remains per target is arithmetic and stores
// (which do not stall a wave), so the loads no longer alternate with the butterflies.  Per target the 255 column-pass
// twiddles of its modulus go through LDS (one coalesced 2 KB read per workgroup, fetched one target ahead).
// MODE 0 (ModUp): grid y = item * beta + digit, sources = the digit's limbs of y, targets = the other limbs of the
// extended basis.  MODE 1 (DivRound conversion, ModDown or rescale): grid y = row, sources = the D.nb dropped limbs
// (row r at y + r*y_row_stride), targets = the nc kept limbs, h subtracted.  MODE 2: MODE 1 in the exact form of DivRound:
// the overshoot v = floor(sum_m y_m * (1/b_m)) of every coefficient (double precision, products and sums in source
// order, each rounded) is found once from the sources and v * (Bbar mod c) leaves every target.
// MODE 3: ModDown FOLLOWED BY rescale, in the strict sequence's own bits, as one conversion.  Source 0 is the limb
// u = x_last * P^-1 + d_last (last = nc, the limb the rescale drops) and sources 1.. are the special limbs (D describes the
// ModDown over them, with b_idx[0] = last put in front).  Per coefficient the workgroup first forms the ModDown result of
// the dropped limb in coefficient form, s = u - (ModDown's conversion to limb `last`) * P^-1, and from it the rescale's
// conversion input y_B = (s + h_B) mod q_last; every target then receives the combination given at modup_cols_target.
struct ModupColsArgs {
    const u64d *y;                // MODE 0: [items][level][N] conversion inputs y_i, coefficient form, canonical
    unsigned long long y_row_stride;  // MODE 1
    u64d *dst;                    // MODE 0: [items][beta][E][N]; MODE 1: [rows][nc][N]
    const ModConst *modc;
    const double *tw;             // forward twiddles [T][N]
    const WMul *cc;               // ModUp constants [beta_top][alpha][alpha][T]
    DivRoundDev D;                // MODE 1 constants
    int logN, level, E, n_q, alpha, beta, T, nc;
    int targets_per_wg;
    int stream;                   // STREAM_*
    P51Mask p51;
    // y holds the output of the inverse ROW pass (reduced doubles); the inverse column pass with its folded
    // constants runs in the workgroup's prologue and the conversion inputs never go through memory
    const double *tw_inv;         // inverse twiddles [T][N]
    const FinConst *fin;          // last-stage constants of source limb s (MODE 0: limb index; MODE 1: s-th dropped limb)
    // MODE 3: constants of the rescale that follows the ModDown described by D
    const double *hc2;            // [T] the rescale's h mod c
    double hb2;                   // the rescale's h mod q_last
    // per-call constants of the single source of a rescale whose input is multiplied by a scalar on the way
    int use_fin_val;
    FinConst fin_val;
};

// Inverse column pass of one source tile in registers: x in the round-2 register layout on entry, the canonical
// coefficient-form words (as doubles) in the round-1 layout on return.
template <bool P51, int Q>
__device__ __forceinline__ void inv_cols_in_regs(double (&x)[16], const double *twl, double *lds, const ColsGeom<Q> &geo, double p, double pinv,
                                                 const FinConst &F) {
    typedef ColsGeom<Q> Geo;
    const WMul unused = WMul{0.0, 0.0};
    {
        double tw2[15];
#pragma unroll
        for (int s = 0; s < 4; s++)
#pragma unroll
            for (int b = 0; b < (1 << s); b++) {
                if (s >= 4 - Q) {
                    const int u = s - (4 - Q);
                    tw2[(1 << s) - 1 + b] = twl[(16u << u) + (geo.a << u) + (b & ((1 << u) - 1))];
                } else {
                    tw2[(1 << s) - 1 + b] = 0.0;
                }
            }
        INV_JOIN(P51, INV_ROW2, INV_COL2);
        inv_stages<Geo::S0, INV_COL2, P51>(x, tw2, p, pinv, unused, unused);
        INV_JOIN(P51, INV_COL2, INV_COL1);
    }
#pragma unroll
    for (int i = 0; i < 16; i++) lds[geo.l2(i)] = x[i];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 16; e++) x[e] = lds[geo.l1(e)];
    {
        double tw1[15];
#pragma unroll
        for (int i = 0; i < 15; i++) tw1[i] = twl[1 + i];
        inv_stages<0, INV_COL1, P51>(x, tw1, p, pinv, F.ninv, F.wlast);
    }
#pragma unroll
    for (int e = 0; e < 16; e++) x[e] = canon_near<P51>(x[e] + F.cadd, p, pinv);  // 1.5p and less than p
}

// VARIANT 1 (exact DivRound): vpack holds the overshoot of the thread's 16 coefficients, 3 bits each; Bm = Bbar mod p.
// VARIANT 2 (ModDown and rescale in one conversion): source 0 is the rescale's conversion input y_B, sources 1.. are
// ModDown's; Wc[0] = P^-1 mod p, hsub = ModDown's h mod p, Bm = the rescale's h mod p:
//     value = (sum_a y_a*conv_a - hA) * P^-1 + y_B - hB     (the two conversion results the last pass would subtract,
//                                                            brought to one: the transforms are linear)
// SUB: h is subtracted (every mode but ModUp)
// SRC0_LDS: the words of source 0 are in ybl instead of yd[0]
template <bool P51, int NSRC, int Q, int VARIANT, bool SUB, bool SRC0_LDS>
__device__ __forceinline__ void modup_cols_target(const double (&yd)[NSRC][16], WMul (&Wc)[NSRC], const double *twl, double *lds, u64d *dst,
                                                  const ColsGeom<Q> &geo, double p, double pinv, double *twl_next, double tw_next, double hsub,
                                                  unsigned long long vpack, double Bm, bool stream, const double *ybl) {
    typedef ColsGeom<Q> Geo;
    constexpr int NPROD = VARIANT == 2 ? NSRC - 1 : NSRC;
    // four products and h could pass 2^53 (without h, in ModUp from four sources, they could not: not measured there)
    // one source of a plain conversion: its constant is 1, the word itself (2 units of 2^50, conv_word in ks_wg.h, or one of 2^51) enters the transform
    constexpr bool COPY = VARIANT == 0 && NSRC == 1;
    constexpr bool CHAIN = !P51 && NPROD >= 2 && !(VARIANT == 0 && NSRC == 4);
    // bounds, in units of p: the sum of products, and what enters the first stage (with h <= p, the reduced overshoot term, or, one
    // conversion for two divisions, a prepared product of the sum, y_B below 2p and h)
    constexpr double SUM = CHAIN ? chain_bound(NPROD) : 0.75 * NPROD;
    constexpr double IN = COPY ? (P51 ? 1.0 : 2.0) : VARIANT == 0 ? SUM + (SUB ? 1.0 : 0.0) : VARIANT == 1 ? SUM + LAZY_REDUCED : (P51 ? 0.64 : 0.5 + (SUM + 1.0) / 8.0) + 3.0;
    constexpr int ENTRY = (int)(256.0 * IN + 0.999);
    static_assert(IN <= LazyRange<P51>::LIM, "the sum leaves the exact range");
    typedef ColsMasks<Q, P51, ENTRY> Mk;
    // A copied word is bounded in units of 2^50 and p may be far smaller.  After a stage that reduces, all words are bounded in p itself, as the
    // canonical form behind the row pass (ROW_NEAR) needs it.
    static_assert(!COPY || P51 || Mk::PLAN != 0, "a copied word that no stage reduces");
    BODY_TAG(P51);
    if (VARIANT == 2) {  // the products by these constants would be moved above the branch all the same: 350 registers spilled
#pragma unroll
        for (int a = 0; a < NSRC; a++) PIN_UNIFORM(Wc[a].w);
    }
    const double M = CHAIN ? chain_origin(p) : 0.0;
    double x[16];
    if (SRC0_LDS) {  // all of them requested at once
#pragma unroll
        for (int e = 0; e < 16; e++) x[e] = ybl[e * 256 + threadIdx.x];
        SCHED_FENCE();
    }
#pragma unroll
    for (int e = 0; e < 16; e++) {
        double v = -hsub;
        if (VARIANT == 1) v = -reduce_balanced(hsub + (double)(unsigned)((vpack >> (3 * e)) & 7u) * Bm, p, pinv);  // v <= 3: below 4p, exact
        ProductChain c{0.0, 0.0};
#pragma unroll
        for (int a = NSRC - NPROD; a < NSRC; a++) {
            const double ya = (SRC0_LDS && a == 0) ? x[e] : yd[a][e];
            if (COPY) v = SUB ? ya - hsub : ya;
            else if (!CHAIN) v += mulmod_w(ya, Wc[a].w, Wc[a].wp, p);
            else if (a == NSRC - NPROD) c = chain_first(M, ya, Wc[a].w);
            else chain_add(c, ya, Wc[a].w);
        }
        if (CHAIN) v = SUB ? v + chain_value(c, p, pinv) : chain_value(c, p, pinv);
        x[e] = v;
        if (VARIANT == 2) {  // y_B is below the dropped prime, which has as many bits as p: below 2p
            x[e] = mulmod_w(P51 ? reduce_balanced(v, p, pinv) : v, Wc[0].w, Wc[0].wp, p) + ybl[e * 256 + threadIdx.x] - Bm;
        }
    }
    {
        double tw1[15];
#pragma unroll
        for (int i = 0; i < 15; i++) tw1[i] = twl[1 + i];
        fwd_round<Mk::F1>(x, tw1, p, pinv);
    }
#pragma unroll
    for (int e = 0; e < 16; e++) lds[geo.l1(e)] = x[e];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; i++) x[i] = lds[geo.l2(i)];
    {
        double tw2[15];
#pragma unroll
        for (int s = 0; s < 4; s++)
#pragma unroll
            for (int b = 0; b < (1 << s); b++) {
                if (s >= 4 - Q) {
                    const int u = s - (4 - Q);
                    tw2[(1 << s) - 1 + b] = twl[(16u << u) + (geo.a << u) + (b & ((1 << u) - 1))];
                } else {
                    tw2[(1 << s) - 1 + b] = 0.0;
                }
            }
        fwd_stages<Geo::S0, Mk::F2>(x, tw2, p, pinv);
    }
    twl_next[threadIdx.x] = tw_next;
    stream_if(stream, [&](auto nt) {
#pragma unroll
        for (int i = 0; i < 16; i++) stream_store<nt>(scalar_base(dst + geo.c0 + Geo::d2(i)) + geo.t2(), mid_store(x[i]));
    });
}

// grid: x = column tile (N/4096), y = item * beta + digit, z = chunk of targets_per_wg target limbs
// Four source tiles do not fit the registers of two waves per SIMD.  MODE 3 keeps y_B, which enters every target as a plain
// addend, in the second exchange buffer and pays a second barrier per target (0.80 ms; all four in registers at one wave
// per SIMD: 1.0 ms).  MODE 2 multiplies all four sources per target: it runs one wave per SIMD with all of them in
// registers (0.97 ms; one of them in LDS at two waves: 1.21 ms; with spills at two: 1.4 ms).
// One source tile leaves room for a third wave per SIMD, with one exchange buffer and two barriers per target (256 items of 8 primes at N = 2^14,
// one prime per digit: 650 us with two waves and two buffers, 571 like this; with three source tiles the third wave spills, 2270 against 2240).
template <int NSRC, int MODE>
constexpr int modup_cols_waves() { return NSRC >= 4 && MODE == 2 ? 1 : NSRC == 1 && MODE <= 1 ? 3 : 2; }
template <int Q, int NSRC, int MODE>
__global__ __launch_bounds__(V2_THREADS, (modup_cols_waves<NSRC, MODE>())) void modup_cols_kernel(ModupColsArgs A) {
    // the twiddles rotate through three sets; the second buffer alternates with the first, or holds a source (below)
    constexpr bool WAVES3 = modup_cols_waves<NSRC, MODE>() == 3;
    __shared__ double lds[WAVES3 ? 1 : 2][4096];
    __shared__ double twl[3][256];
    const unsigned N = 1u << A.logN;
    unsigned item = 0, j = 0;
    int lo = 0, nsrc, n_targets;
    const u64d *ysrc;
    static_assert(MODE != 2 || NSRC <= 4, "overshoot below 4: 3 bits each, h + v*Bbar below 4p");
    if (MODE == 0) {
        item = blockIdx.y / (unsigned)A.beta;
        j = blockIdx.y % (unsigned)A.beta;
        lo = (int)j * A.alpha;
        nsrc = (A.level - lo < A.alpha) ? A.level - lo : A.alpha;
        n_targets = A.E - nsrc;  // every limb of the extended basis outside the digit
        ysrc = A.y + ((size_t)item * A.level + lo) * N;
    } else {
        nsrc = A.D.nb;
        n_targets = A.nc;
        ysrc = A.y + (size_t)blockIdx.y * A.y_row_stride;
    }
    const int k0 = (int)blockIdx.z * A.targets_per_wg;
    const int k1 = k0 + A.targets_per_wg < n_targets ? k0 + A.targets_per_wg : n_targets;
    if (k0 >= k1) return;
    const ColsGeom<Q> geo(threadIdx.x, blockIdx.x);
    // the source words, once: a missing source (digit cut short by the level) re-reads the first limb, its constants are zero
    double yd[NSRC][16];
    {
        // every source tile is requested first, then taken through its inverse column pass one after the other
        u64d raw[NSRC][16];
#pragma unroll
        for (int a = 0; a < NSRC; a++) {
            const u64d *ya = ysrc + (size_t)(a < nsrc ? a : 0) * N;
#pragma unroll
            for (int i = 0; i < 16; i++) raw[a][i] = ya[geo.g2(i)];
        }
#pragma unroll
        for (int a = 0; a < NSRC; a++) {
            if (a < nsrc) {  // uniform
                const int ls = MODE == 0 ? lo + a : a;                 // index of the source among the transformed limbs
                const int ts = MODE == 0 ? lo + a : A.D.b_idx[a];      // its modulus
                const double ps = A.modc[ts].p, psinv = A.modc[ts].pinv;
                const FinConst F = A.use_fin_val ? A.fin_val : A.fin[ls];
                __syncthreads();  // the previous source is done with twl[2] and lds[0]
                twl[2][threadIdx.x] = A.tw_inv[(size_t)ts * N + threadIdx.x];
                __syncthreads();
                double x[16];
#pragma unroll
                for (int i = 0; i < 16; i++) x[i] = mid_load(raw[a][i]);
                if (is_p51(A.p51, ts))
                    inv_cols_in_regs<true, Q>(x, twl[2], lds[0], geo, ps, psinv, F);
                else
                    inv_cols_in_regs<false, Q>(x, twl[2], lds[0], geo, ps, psinv, F);
#pragma unroll
                for (int e = 0; e < 16; e++) yd[a][e] = x[e];
            } else {
#pragma unroll
                for (int e = 0; e < 16; e++) yd[a][e] = 0.0;
            }
        }
        __syncthreads();  // lds[0] and twl are about to be reused by the targets
    }
    unsigned long long vpack = 0;
    if (MODE == 2) {
#pragma unroll
        for (int e = 0; e < 16; e++) {
            double sum = yd[0][e] * A.D.invb_f[0];
#pragma unroll
            for (int a = 1; a < NSRC; a++)
                if (a < nsrc) sum = sum + yd[a][e] * A.D.invb_f[a];
            vpack |= (unsigned long long)floor(sum) << (3 * e);
        }
    }
    if (MODE == 3) {
        // the dropped limb's ModDown result in coefficient form, then the rescale's conversion input, in place of source 0
        const int tl = A.nc;
        const double pl = A.modc[tl].p, plinv = A.modc[tl].pinv;
        const WMul Pinv = A.D.Binv[tl];
        const double hA = A.D.hc[tl];
        WMul Wl[NSRC];
#pragma unroll
        for (int a = 1; a < NSRC; a++) Wl[a] = a < nsrc ? A.D.conv[(size_t)(a - 1) * A.T + tl] : WMul{0.0, 0.0};
#pragma unroll
        for (int e = 0; e < 16; e++) {
            double v = -hA;
#pragma unroll
            for (int a = 1; a < NSRC; a++) v += mulmod_w(yd[a][e], Wl[a].w, Wl[a].wp, pl);
            v = reduce_balanced(v, pl, plinv);
            const double sl = yd[0][e] - mulmod_w(v, Pinv.w, Pinv.wp, pl);  // (-0.75p, 1.75p)
            // y_B lives in the second exchange buffer from here on (this mode uses one buffer and two barriers per target):
            // four source tiles do not fit the registers of two waves per SIMD
            lds[WAVES3 ? 0 : 1][e * 256 + threadIdx.x] = canon(sl + A.hb2, pl, plinv);
        }
    }
    // three source tiles: the first one lives in the second exchange buffer (one buffer, two barriers per target): without
    // it the kernel spills at two waves per SIMD (ModUp at the benchmark shape: 2.35 against 2.58 ms)
    constexpr bool SRC0_LDS = (MODE <= 1 && NSRC == 3);
    if (SRC0_LDS) {
#pragma unroll
        for (int e = 0; e < 16; e++) lds[WAVES3 ? 0 : 1][e * 256 + threadIdx.x] = yd[0][e];
    }
    const size_t crow = ((size_t)j * A.alpha + (nsrc - 1)) * A.alpha;
    // MODE 0: extended-basis index of target k (the digit's own limbs are skipped) and its modulus index;
    // MODE 1: target k is kept limb k
    auto ext_of = [&](int k) { return MODE == 0 ? (k < lo ? k : k + nsrc) : k; };
    auto mod_of = [&](int x) { return MODE == 0 ? (x < A.level ? x : A.n_q + x - A.level) : x; };
    twl[0][threadIdx.x] = A.tw[(size_t)mod_of(ext_of(k0)) * N + threadIdx.x];
    twl[1][threadIdx.x] = A.tw[(size_t)mod_of(ext_of(k0 + 1 < k1 ? k0 + 1 : k0)) * N + threadIdx.x];
    __syncthreads();
    for (int k = k0; k < k1; k++) {
        const int x = ext_of(k), t = mod_of(x);
        const double *tcur = twl[(k - k0) % 3];
        // The twiddles of target k + 2 are requested here and go to LDS just before this target's stores, into the set of target k - 1
        // (everybody has passed this target's barrier by then).  Memory operations complete in order, so waiting for this word waits
        // for the stores of target k - 1, which have had all of this target's arithmetic to drain; a request that is waited for behind
        // stores makes the wave stand until they are written (ModUp of 64 items of 24 primes at N = 2^16 2180 us with such a request, 2070 like
        // this, which includes all of a source's words fetched from LDS at once and stores with scalar bases).
        const double tw_next = A.tw[(size_t)mod_of(ext_of(k + 2 < k1 ? k + 2 : k1 - 1)) * N + threadIdx.x];
        double *tnext = twl[(k - k0 + 2) % 3];
        const double p = table_load(&A.modc[t].p, 0), pinv = table_load(&A.modc[t].pinv, 0);
        WMul Wc[NSRC];
        double hsub = 0.0, Bm = 0.0;
        u64d *dst;
        if (MODE == 0) {
#pragma unroll
            for (int a = 0; a < NSRC; a++) Wc[a] = a < nsrc ? table_load(&A.cc[(crow + a) * A.T + t]) : WMul{0.0, 0.0};
            dst = A.dst + (((size_t)item * A.beta + j) * A.E + x) * N;
        } else {
#pragma unroll
            for (int a = 0; a < NSRC; a++)
                Wc[a] = a < nsrc ? table_load(&A.D.conv[(size_t)(MODE == 3 ? (a ? a - 1 : 0) : a) * A.T + t]) : WMul{0.0, 0.0};
            hsub = table_load(A.D.hc, t);
            if (MODE == 2) Bm = table_load(A.D.Bmod, t);
            if (MODE == 3) {
                Wc[0] = table_load(&A.D.Binv[t]);
                Bm = table_load(A.hc2, t);
            }
            dst = A.dst + ((size_t)blockIdx.y * A.nc + t) * N;
        }
        constexpr bool ONE_BUF = MODE == 3 || SRC0_LDS || WAVES3;  // the second buffer holds y_B / the first source tile, or there is none
        double *xbuf = ONE_BUF ? lds[0] : lds[(k - k0) & 1], *ybuf = lds[WAVES3 ? 0 : 1];
        constexpr int VAR = MODE >= 2 ? MODE - 1 : 0;
        if (is_p51(A.p51, t))
            modup_cols_target<true, NSRC, Q, VAR, MODE != 0, SRC0_LDS>(yd, Wc, tcur, xbuf, dst, geo, p, pinv, tnext, tw_next, hsub, vpack, Bm, A.stream != STREAM_NONE, ybuf);
        else
            modup_cols_target<false, NSRC, Q, VAR, MODE != 0, SRC0_LDS>(yd, Wc, tcur, xbuf, dst, geo, p, pinv, tnext, tw_next, hsub, vpack, Bm, A.stream != STREAM_NONE, ybuf);
        if (ONE_BUF) __syncthreads();  // single exchange buffer: everybody has read it before the next target writes
    }
}

// ------------------------------------------------------------------ row pass helper
// round-2 twiddles of a thread (registers) and the round-1 twiddles of the tile's 16 rows (LDS, [16][16])
__device__ __forceinline__ void load_row_twiddles(const double *tw, unsigned N1, unsigned tile, unsigned hi4, unsigned lo4, double *tw1_lds,
                                                  double (&tw2)[15]) {
    const unsigned base1 = N1 + tile * 16 + hi4;
#pragma unroll
    for (int s = 0; s < 4; s++)
#pragma unroll
        for (int b = 0; b < (1 << s); b++) tw2[(1 << s) - 1 + b] = tw[((16u * base1 + lo4) << s) + b];
    if (lo4 < 15) {
        // entry i = (1<<s)-1+b  ->  tw[(base1 << s) + b]
        const unsigned i = lo4, s = (i >= 7) ? 3 : (i >= 3) ? 2 : (i >= 1) ? 1 : 0, b = i - ((1u << s) - 1);
        tw1_lds[hi4 * 16 + i] = tw[(base1 << s) + b];
    }
    __syncthreads();
}

// Finish the forward transform of one 16-row tile (column pass already done) and leave the results, balanced-reduced or (ROW_LAZY)
// at most LazyRange::ROWX, in LDS in the padded layout: word (row g, position q) at g*V2_GS + (q/16)*17 + q%16.
// Every row is handled by its own 16 lanes: ends with a row-group sync, and the caller puts one before the next call.
// SBASE: the words are requested from a scalar base.  The last pass without an addend is faster with it (14 products of 5 primes at N = 2^14 13.7 -> 13.1 us, 2 of 8 at
// 2^16 15.5 -> 14.9), the one for scalar multiples and the row pass of an encryption are slower (29.6 -> 30.5, 20.8 -> 21.2).
template <bool P51, int X, bool SBASE = false>
__device__ __forceinline__ void rows_fwd_to_lds(const u64d *tile, double *lds, const double *tw1_lds, const double (&tw2)[15], double p,
                                                double pinv, unsigned hi4, unsigned lo4, bool stream) {
    typedef RowMasks<P51, X> Mk;
    double *grp = lds + hi4 * V2_GS;
    double x[16];
    stream_if(stream, [&](auto nt) {
#pragma unroll
        for (int e = 0; e < 16; e++) {
            if constexpr (SBASE) x[e] = mid_load(stream_load<nt>(scalar_base(tile) + (hi4 * 256 + lo4 + 16 * e)));
            else x[e] = mid_load(stream_load<nt>(&tile[hi4 * 256 + lo4 + 16 * e]));
        }
    });
    {
        // round-1 twiddles are the same for the 16 lanes of a row: kept in LDS, not in registers
        double tw1[15];
#pragma unroll
        for (int i = 0; i < 15; i++) tw1[i] = tw1_lds[hi4 * 16 + i];
        fwd_round<Mk::F1>(x, tw1, p, pinv);
    }
#pragma unroll
    for (int e = 0; e < 16; e++) grp[e * 17 + lo4] = x[e];
    ROW_GROUP_SYNC();
#pragma unroll
    for (int e = 0; e < 16; e++) x[e] = grp[lo4 * 17 + e];
    fwd_round<Mk::F2>(x, tw2, p, pinv);
#pragma unroll
    for (int e = 0; e < 16; e++) grp[lo4 * 17 + e] = X == ROW_LAZY ? x[e] : reduce_balanced(x[e], p, pinv);
    ROW_GROUP_SYNC();
}

// ------------------------------------------------------------------ row pass + inner product
struct RowsInnerArgs {
    const u64d *dtA;     // [items][beta][E][N] column-pass output of the converted limbs
    const u64d *d_eval;  // evaluation-form source polynomial, item i at d_eval + i*d_eval_item_stride, [level][N]
    unsigned long long d_eval_item_stride;
    u64d *acc;           // [items][2][E][N]
    const ModConst *modc;
    const double *tw;    // forward twiddles
    int logN, level, E, n_q, alpha, beta, T;
    unsigned kt;         // min(N/4096, 8): see the grid mapping in rows_inner_body
    int stream;          // STREAM_*
    P51Mask p51;
    // fold_tail: the ciphertext limbs leave this kernel as z = acc * P^-1 + d (d = the addend of the same row: the product's
    // component, or sigma(c0) for the first row of a rotation), which is what the ModDown (and rescale) that follows reads.
    // 1: both components have an addend, 2: the first one only
    int fold_tail;
    const WMul *Pinv;    // [T] P^-1 mod q_i
    const u64d *addend;  // item i, component c, limb l at addend + i*add_item_stride + c*add_comp_stride + l*N
    unsigned long long add_item_stride, add_comp_stride;
    // Tensor mode (ta != nullptr; the composite multiply): the source polynomial is d2 = sum_t a1_t*b1_t of the operands
    // ta, tb: [items][terms][2][level][N], formed here for the limb's own digit, and the accumulators of the ciphertext limbs
    // start at P*d0 and P*d1 (d0 = sum a0*b0, d1 = sum a0*b1 + a1*b0), so that they leave as
    // z = (acc + P*d) * P^-1 = acc * P^-1 + d, or as acc + P*d itself (keep_acc: what the merged division divides).
    const u64d *ta, *tb;
    int terms, keep_acc;
    const WMul *Pmod;    // [T] P mod q_i
};

// One word's terms of both accumulators: key words (canonical) times the transformed word v.
// p < 2^51: |v| <= p/2 + 1 is the prepared factor (v/p computed once for both), a term is below 0.875p and four of them on a
// reduced sum stay below 4p = 2^53.
// p < 2^50: |v| <= LazyRange::FACTOR p: the quotient is taken from the product, which is off by less than 2 * 2.2 / 8, and what the
// product drops is below 2.2p / 8: a term is below 1.33p, five of them on a reduced sum below 7.2p.
template <bool P51> constexpr int KEY_TERMS = P51 ? 4 : 5;
template <bool P51>
__device__ __forceinline__ void key_term(u64d k0, u64d k1, double v, double p, double pinv, double &a0, double &a1) {
    if (P51) {
        const double vp = v * pinv;
        a0 += mulmod_w(u2d(k0), v, vp, p);
        a1 += mulmod_w(u2d(k1), v, vp, p);
    } else {
        a0 += mulmod(u2d(k0), v, p, pinv);
        a1 += mulmod(u2d(k1), v, p, pinv);
    }
}

// The term of the digit that contains limb x (its operand is the source polynomial itself, no transform) of a thread's 16
// words: pairs row_pair_index(hi4, lo4, s) from word tile0 of the limb; accumulator 2*s + b belongs to word b of pair s.
// In tensor mode also P * (d0, d1).  pending: terms in the accumulators since their last reduction.
template <bool P51, bool GAL>
__device__ __forceinline__ void inner_own_digit(const RowsInnerArgs &A, const u64d *key, unsigned item, int t, unsigned x, int j_own, bool tensor_mode,
                                                size_t tile0, unsigned hi4, unsigned lo4, double p, double pinv, double (&a0)[16], double (&a1)[16],
                                                int &pending, const GaloisTab *gal) {
    const unsigned N = 1u << A.logN;
    if (tensor_mode) {
        // d0, d1, d2 of the thread's 16 words from the operands: one term and p < 2^50 as they come (0.875p, 1.75p, 0.875p), otherwise summed
        // over the terms and balanced-reduced
        const size_t st = (size_t)A.level * N / 2;  // pairs between the two components of a ciphertext
        const ulonglong2 *pa = (const ulonglong2 *)(A.ta + ((size_t)item * A.terms * 2 * A.level + x) * N + tile0);
        const ulonglong2 *pb = (const ulonglong2 *)(A.tb + ((size_t)item * A.terms * 2 * A.level + x) * N + tile0);
        const ulonglong2 *k0 = (const ulonglong2 *)(key + (((size_t)j_own * 2 + 0) * A.T + t) * N + tile0);
        const ulonglong2 *k1 = (const ulonglong2 *)(key + (((size_t)j_own * 2 + 1) * A.T + t) * N + tile0);
        const WMul Pm = A.Pmod[t];
#pragma unroll
        for (int h = 0; h < 2; h++) {  // four pairs at a time: bounds the registers in flight
            // the own digit's key words travel with the first term's operands
            ulonglong2 kr0[4], kr1[4];
#pragma unroll
            for (int s = 0; s < 4; s++) {
                kr0[s] = k0[row_pair_index(hi4, lo4, 4 * h + s)];
                kr1[s] = k1[row_pair_index(hi4, lo4, 4 * h + s)];
            }
            double l0[8], l1[8], l2[8];
            auto term = [&](int tm, auto add) {
                const size_t to = (size_t)tm * 2 * st;
                ulonglong2 A0[4], A1[4], B0[4], B1[4];
#pragma unroll
                for (int s = 0; s < 4; s++) {
                    const unsigned e = row_pair_index(hi4, lo4, 4 * h + s);
                    A0[s] = pa[to + e]; A1[s] = pa[to + st + e]; B0[s] = pb[to + e]; B1[s] = pb[to + st + e];
                }
                SCHED_FENCE();
#pragma unroll
                for (int s = 0; s < 4; s++) {
#pragma unroll
                    for (int b = 0; b < 2; b++) {
                        const int i = 2 * s + b;
                        const double x0 = u2d(b ? A0[s].y : A0[s].x), x1 = u2d(b ? A1[s].y : A1[s].x);
                        const double y0 = u2d(b ? B0[s].y : B0[s].x), y1 = u2d(b ? B1[s].y : B1[s].x);
                        const double t0 = mulmod(x0, y0, p, pinv), t1 = mulmod(x0, y1, p, pinv) + mulmod(x1, y0, p, pinv), t2 = mulmod(x1, y1, p, pinv);
                        // |t| <= 1.75p (2.5p for p < 2^51) on top of a reduced sum, or of one term as it comes: below 2^53
                        l0[i] = add ? reduce_balanced(l0[i] + t0, p, pinv) : P51 ? reduce_balanced(t0, p, pinv) : t0;
                        l1[i] = add ? reduce_balanced(l1[i] + t1, p, pinv) : P51 ? reduce_balanced(t1, p, pinv) : t1;
                        l2[i] = add ? reduce_balanced(l2[i] + t2, p, pinv) : P51 ? reduce_balanced(t2, p, pinv) : t2;
                    }
                }
            };
            term(0, StreamFlag<false>());
            for (int tm = 1; tm < A.terms; tm++) term(tm, StreamFlag<true>());
#pragma unroll
            for (int s = 0; s < 4; s++) {
                // two terms of at most the bound of key_term each: P*d (0.72p) and the own digit's product
                a0[8 * h + 2 * s] = mulmod_w(l0[2 * s], Pm.w, Pm.wp, p);
                a1[8 * h + 2 * s] = mulmod_w(l1[2 * s], Pm.w, Pm.wp, p);
                a0[8 * h + 2 * s + 1] = mulmod_w(l0[2 * s + 1], Pm.w, Pm.wp, p);
                a1[8 * h + 2 * s + 1] = mulmod_w(l1[2 * s + 1], Pm.w, Pm.wp, p);
                key_term<P51>(kr0[s].x, kr1[s].x, l2[2 * s], p, pinv, a0[8 * h + 2 * s], a1[8 * h + 2 * s]);
                key_term<P51>(kr0[s].y, kr1[s].y, l2[2 * s + 1], p, pinv, a0[8 * h + 2 * s + 1], a1[8 * h + 2 * s + 1]);
            }
        }
        pending = 2;
    } else if (j_own >= 0) {
        const u64d *k0 = key + (((size_t)j_own * 2 + 0) * A.T + t) * N + tile0;
        const u64d *k1 = key + (((size_t)j_own * 2 + 1) * A.T + t) * N + tile0;
        const u64d *limb = A.d_eval + (size_t)item * A.d_eval_item_stride + (size_t)x * N, *src = limb + tile0;
        ulonglong2 kr0[8], kr1[8], xo[8];
#pragma unroll
        for (int s = 0; s < 8; s++) {
            if (GAL) xo[s] = galois_pair_load(limb, (unsigned)tile0 + hi4 * 256u + 32u * s + 2u * lo4, gal->g[item], A.logN);
            else xo[s] = ((const ulonglong2 *)src)[row_pair_index(hi4, lo4, s)];
            kr0[s] = ((const ulonglong2 *)k0)[row_pair_index(hi4, lo4, s)];
            kr1[s] = ((const ulonglong2 *)k1)[row_pair_index(hi4, lo4, s)];
        }
        SCHED_FENCE();
#pragma unroll
        for (int s = 0; s < 8; s++) {
            double v0 = u2d(xo[s].x), v1 = u2d(xo[s].y);
            if (P51) {
                v0 = reduce_balanced(v0, p, pinv);
                v1 = reduce_balanced(v1, p, pinv);
            }
            key_term<P51>(kr0[s].x, kr1[s].x, v0, p, pinv, a0[2 * s], a1[2 * s]);
            key_term<P51>(kr0[s].y, kr1[s].y, v1, p, pinv, a0[2 * s + 1], a1[2 * s + 1]);
        }
    }
}

// The accumulators leave as z (folded tail), as acc + P*d, or as they are
template <bool P51, bool GAL, bool NTS>
__device__ __forceinline__ void inner_store(const RowsInnerArgs &A, unsigned item, int t, unsigned x, bool tensor_mode, size_t tile0, unsigned hi4,
                                            unsigned lo4, double p, double pinv, const double (&a0)[16], const double (&a1)[16], const GaloisTab *gal) {
    const unsigned N = 1u << A.logN;
    u64d *o0 = A.acc + (((size_t)item * 2 + 0) * A.E + x) * N + tile0;
    u64d *o1 = A.acc + (((size_t)item * 2 + 1) * A.E + x) * N + tile0;
    if (tensor_mode && !A.keep_acc) {
        // z = (acc + P*d) * P^-1; accumulators are below 2^53: the prepared product is exact for them as they are, and below 1.5p
        const WMul Pi = A.Pinv[t];
#pragma unroll
        for (int s = 0; s < 8; s++) {
            const double z00 = mulmod_w(a0[2 * s], Pi.w, Pi.wp, p), z01 = mulmod_w(a0[2 * s + 1], Pi.w, Pi.wp, p);
            const double z10 = mulmod_w(a1[2 * s], Pi.w, Pi.wp, p), z11 = mulmod_w(a1[2 * s + 1], Pi.w, Pi.wp, p);
            stream_store<NTS>((ulonglong2 *)o0 + row_pair_index(hi4, lo4, s), make_ulonglong2(d2u(canon_near<P51>(z00, p, pinv)), d2u(canon_near<P51>(z01, p, pinv))));
            stream_store<NTS>((ulonglong2 *)o1 + row_pair_index(hi4, lo4, s), make_ulonglong2(d2u(canon_near<P51>(z10, p, pinv)), d2u(canon_near<P51>(z11, p, pinv))));
        }
        return;
    }
    if (!tensor_mode && A.fold_tail && (int)x < A.level) {
        const WMul Pi = A.Pinv[t];
        const u64d *l0 = A.addend + (size_t)item * A.add_item_stride + (size_t)x * N, *d0 = l0 + tile0;
        const bool both = !GAL && A.fold_tail == 1;  // only the first component of a rotation has an addend
        const u64d *l1 = both ? l0 + A.add_comp_stride : l0, *d1 = l1 + tile0;
        const double has1 = both ? 1.0 : 0.0;
        ulonglong2 dw0[8], dw1[8];
#pragma unroll
        for (int s = 0; s < 8; s++) {
            if (GAL) {  // (a load that only some calls make had every one before it waited for: 131 rotations at N = 2^14, 8 primes 428 us, 417 like this)
                dw0[s] = galois_pair_load(l0, (unsigned)tile0 + hi4 * 256u + 32u * s + 2u * lo4, gal->g[item], A.logN);
                dw1[s] = make_ulonglong2(0ull, 0ull);
            } else {
                dw0[s] = ((const ulonglong2 *)d0)[row_pair_index(hi4, lo4, s)];
                dw1[s] = ((const ulonglong2 *)d1)[row_pair_index(hi4, lo4, s)];
            }
        }
#pragma unroll
        for (int s = 0; s < 8; s++) {
            // the same plus a canonical word: below 2.5p
            const double z00 = mulmod_w(a0[2 * s], Pi.w, Pi.wp, p) + u2d(dw0[s].x), z01 = mulmod_w(a0[2 * s + 1], Pi.w, Pi.wp, p) + u2d(dw0[s].y);
            const double z10 = mulmod_w(a1[2 * s], Pi.w, Pi.wp, p) + has1 * u2d(dw1[s].x), z11 = mulmod_w(a1[2 * s + 1], Pi.w, Pi.wp, p) + has1 * u2d(dw1[s].y);
            stream_store<NTS>((ulonglong2 *)o0 + row_pair_index(hi4, lo4, s), make_ulonglong2(d2u(canon_near<P51>(z00, p, pinv)), d2u(canon_near<P51>(z01, p, pinv))));
            stream_store<NTS>((ulonglong2 *)o1 + row_pair_index(hi4, lo4, s), make_ulonglong2(d2u(canon_near<P51>(z10, p, pinv)), d2u(canon_near<P51>(z11, p, pinv))));
        }
        return;
    }
#pragma unroll
    for (int s = 0; s < 8; s++) {
        stream_store<NTS>((ulonglong2 *)o0 + row_pair_index(hi4, lo4, s), make_ulonglong2(d2u(canon(a0[2 * s], p, pinv)), d2u(canon(a0[2 * s + 1], p, pinv))));
        stream_store<NTS>((ulonglong2 *)o1 + row_pair_index(hi4, lo4, s), make_ulonglong2(d2u(canon(a1[2 * s], p, pinv)), d2u(canon(a1[2 * s + 1], p, pinv))));
    }
}

// GAL (a rotation): the source polynomial d_eval and the addend are read through the automorphism X -> X^g of their item
// (gal->g[item]), so that no rotated copy of the ciphertext is ever written
template <bool P51, bool GAL, int STREAM>
__device__ __forceinline__ void rows_inner_body(const RowsInnerArgs &A, const KeyTab &K, double *lds, double *tw1_lds, double *tw2_lds, int t,
                                                unsigned x, const GaloisTab *gal = nullptr) {
    BODY_TAG(P51);
    typedef RowMasks<P51, ROW_FACTOR> Mk;
    const unsigned N = 1u << A.logN, N1 = N >> 8;
    const double p = A.modc[t].p, pinv = A.modc[t].pinv;
    const unsigned tid = threadIdx.x, hi4 = tid >> 4, lo4 = tid & 15;
    // Workgroups are handed to the 8 XCDs round-robin by linear id, and every XCD has its own L2.  blockIdx.x packs
    // (row tile mod KT, item) with KT = min(tiles, 8) in the low position, so that all items' workgroups for one key
    // tile (same extended limb, same row tile) land on the same XCD and the key tile is fetched from HBM once.
    const unsigned KT = A.kt;
    const unsigned item = blockIdx.x / KT, tile = blockIdx.x % KT + KT * blockIdx.y;
    {
        // both rounds' twiddles live in LDS here (round 2: [15][256], conflict-free): the registers are needed for the
        // accumulators and the operands in flight
        double tw2[15];
        load_row_twiddles(A.tw + (size_t)t * N, N1, tile, hi4, lo4, tw1_lds, tw2);
#pragma unroll
        for (int i = 0; i < 15; i++) tw2_lds[i * 256 + tid] = tw2[i];
    }
    const u64d *key = K.key[K.slot[item]];
    const size_t tile0 = (size_t)tile * 4096;
    double *grp = lds + hi4 * V2_GS;
    double a0[16], a1[16];
#pragma unroll
    for (int i = 0; i < 16; i++) a0[i] = a1[i] = 0.0;
    // Multiply-accumulate layout (row_pair_index): a thread owns 8 word pairs of the row its 16 lanes transform, so that key
    // words, the own digit's words and the results move 16 bytes per lane and the whole digit loop needs no workgroup barrier;
    // accumulator 2*s + b belongs to the word at column 32*s + 2*lo4 + b of row hi4.
    // The digit that contains this limb needs no transform: its operand is the source polynomial itself.
    const int j_own = (int)x < A.level ? (int)x / A.alpha : -1;
    const bool tensor_mode = !GAL && A.ta != nullptr && j_own >= 0;
    int pending = 1;  // terms in the accumulators since their last reduction (the own digit's term counts)
    inner_own_digit<P51, GAL>(A, key, item, t, x, j_own, tensor_mode, tile0, hi4, lo4, p, pinv, a0, a1, pending, gal);
    // The other digits, software-pipelined so that no memory latency sits in front of arithmetic: the limb words of a
    // digit are requested while the previous digit is multiplied, its key words while the limb goes through the row
    // pass.  xr holds the column-pass output of the converted limb in the register layout of the row pass.
    // (The requests stand in straight-line code, also past the last digit, where they re-read key words: behind a branch that may not be
    // taken the compiler has to wait for all of them where it wants the key words, which exposes the latency of every digit's limb.)
    int j = (j_own == 0) ? 1 : 0;
    const unsigned vr = hi4 * 256 + lo4, pr = row_pair_index(hi4, lo4, 0);
    u64d xr[16];
    if (j < A.beta) {
        const u64d *src = A.dtA + (((size_t)item * A.beta + j) * A.E + x) * N + tile0;
#pragma unroll
        for (int i = 0; i < 16; i++) xr[i] = stream_load<STREAM == STREAM_ALL>(scalar_base(src) + (vr + 16 * i));
    }
    while (j < A.beta) {
        const u64d *k0 = key + (((size_t)j * 2 + 0) * A.T + t) * N + tile0;
        const u64d *k1 = key + (((size_t)j * 2 + 1) * A.T + t) * N + tile0;
        ulonglong2 kr0[8], kr1[8];
#pragma unroll
        for (int s = 0; s < 8; s++) {
            kr0[s] = pair_load<false>(k0, pr + 16 * s);
            kr1[s] = pair_load<false>(k1, pr + 16 * s);
        }
        SCHED_FENCE();
        {
            double xx[16];
#pragma unroll
            for (int e = 0; e < 16; e++) xx[e] = mid_load(xr[e]);
            {
                double tw1[15];
#pragma unroll
                for (int i = 0; i < 15; i++) tw1[i] = tw1_lds[hi4 * 16 + i];
                fwd_round<Mk::F1>(xx, tw1, p, pinv);
            }
#pragma unroll
            for (int e = 0; e < 16; e++) grp[e * 17 + lo4] = xx[e];
            ROW_GROUP_SYNC();
#pragma unroll
            for (int e = 0; e < 16; e++) xx[e] = grp[lo4 * 17 + e];
            {
                double tw2[15];
#pragma unroll
                for (int i = 0; i < 15; i++) tw2[i] = tw2_lds[i * 256 + tid];
                fwd_round<Mk::F2>(xx, tw2, p, pinv);
            }
#pragma unroll
            for (int e = 0; e < 16; e++) grp[lo4 * 17 + e] = P51 ? reduce_balanced(xx[e], p, pinv) : xx[e];
        }
        ROW_GROUP_SYNC();
        int jn = j + 1;
        if (jn == j_own) jn++;
        const u64d *src = jn < A.beta ? A.dtA + (((size_t)item * A.beta + jn) * A.E + x) * N + tile0 : k0;
        const unsigned vn = jn < A.beta ? vr : 0u;  // (past the last digit all lanes re-read the same few words: two digits 21.9 -> 21.5 us)
#pragma unroll
        for (int i = 0; i < 16; i++) xr[i] = stream_load<STREAM == STREAM_ALL>(scalar_base(src) + (vn + 16 * i));
        SCHED_FENCE();
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
        ROW_GROUP_SYNC();  // the row's lanes have read its words before the next digit overwrites them
        j = jn;
    }
    inner_store<P51, GAL, STREAM != STREAM_NONE>(A, item, t, x, tensor_mode, tile0, hi4, lo4, p, pinv, a0, a1, gal);
}

// grid: x = (row tile mod kt) + kt * item, y = row tile / kt, z = extended limb
template <int STREAM>
__global__ __launch_bounds__(V2_THREADS, 2) void rows_inner_kernel(RowsInnerArgs A, KeyTab K) {
    __shared__ double lds[16 * V2_GS];
    __shared__ double tw1_lds[16 * 16];
    __shared__ double tw2_lds[15 * 256];
    const unsigned x = blockIdx.z;
    const int t = (int)x < A.level ? (int)x : A.n_q + (int)x - A.level;
    if (is_p51(A.p51, t))
        rows_inner_body<true, false, STREAM>(A, K, lds, tw1_lds, tw2_lds, t, x);
    else
        rows_inner_body<false, false, STREAM>(A, K, lds, tw1_lds, tw2_lds, t, x);
}

// the same for rotations: source polynomial and addend read through the items' automorphisms (no tensor mode here)
template <int STREAM>
__global__ __launch_bounds__(V2_THREADS, 2) void rows_inner_gal_kernel(RowsInnerArgs A, KeyTab K, GaloisTab G) {
    __shared__ double lds[16 * V2_GS];
    __shared__ double tw1_lds[16 * 16];
    __shared__ double tw2_lds[15 * 256];
    const unsigned x = blockIdx.z;
    const int t = (int)x < A.level ? (int)x : A.n_q + (int)x - A.level;
    if (is_p51(A.p51, t))
        rows_inner_body<true, true, STREAM>(A, K, lds, tw1_lds, tw2_lds, t, x, &G);
    else
        rows_inner_body<false, true, STREAM>(A, K, lds, tw1_lds, tw2_lds, t, x, &G);
}

// ------------------------------------------------------------------ row pass + DivRound final step
struct RowsFinalArgs {
    const u64d *tmpA;    // [rows][nc][N] column-pass output of (r_i - h)
    const u64d *x;       // kept limbs, evaluation form: row r, limb i at x + r*x_row_stride + i*N
    unsigned long long x_row_stride;
    const u64d *addend;  // optional: row r limb i at addend + (r/2)*add_item_stride + (r%2)*add_comp_stride + i*N (odd rows: with pre or a scalar)
    unsigned long long add_item_stride, add_comp_stride;
    u64d *out;           // row r, limb i at out + r*out_row_stride + (i - out_limb0)*N
    unsigned long long out_row_stride;
    int out_limb0;
    const ModConst *modc;
    const double *tw;
    const WMul *Binv;    // [T]
    const WMul *pre;     // optional [T]: the addend enters BEFORE the division, out = (x + pre_i*addend - r) * Binv
    int zsub;            // 1: x already holds x*Binv + addend: out = x - r * Binv
    int logN, nc;
    int limb0;             // first limb handled (grid z counts from it)
    int stream;            // STREAM_*
    int rows, rows_per_x;  // a workgroup loops over rows_per_x rows (same limb, same tile: twiddles reused)
    P51Mask p51;
};

// Rotations from a shared ModUp: rows come in pairs (item, rotation r), R rotations per item; the first row of a pair adds
// sigma_r(c0 of its item), read through the automorphism from the input ciphertext itself (A.addend = c0 of item 0,
// A.add_item_stride = words between the items' ciphertexts)
struct RowsFinalGal { int R; unsigned g[CKKSMI_MAX_KEYS]; };

template <bool P51, bool NTS, bool ADD, bool KEPT_NT, bool GAL = false>
__device__ __forceinline__ void rows_final_body(const RowsFinalArgs &A, double *lds, double *tw1_lds, int i, bool xm_val = false,
                                                WMul xmv = WMul{0.0, 0.0}, const RowsFinalGal *gal = nullptr) {
    // KEPT_NT: the kept limb's words are streamed with the results, from 16 MB on, where the call's own kernels wrote them: without an addend (three waves per
    // SIMD: a product's tail at N = 2^16, 24 primes, 4 ciphertexts 69.2 -> 62.0 us, 63.6 without; 150 of 9 at N = 2^14 184 -> 173, 182 without) and for
    // rotations from a shared ModUp (128 rotations of 11 primes at N = 2^14 257 -> 228, 246 without).  Words of the caller may be in the caches: rescales of
    // 30 kept limbs at N = 2^16 31.8 us, 34.5 streamed, of 72 39.9 and 42.2 (other buffers each time 34.5 both and 42.4, 42.3).  So may those of
    // scalar multiples, at two waves besides: 4 rows of 17 kept limbs 28.2 -> 31.4, 80 of 1 29.4 -> 32.6, 400 of 1 122 -> 128.
    const unsigned N = 1u << A.logN, N1 = N >> 8;
    const double p = A.modc[i].p, pinv = A.modc[i].pinv;
    const unsigned tid = threadIdx.x, hi4 = tid >> 4, lo4 = tid & 15;
    const unsigned tile = blockIdx.y;
    double tw2[15];
    load_row_twiddles(A.tw + (size_t)i * N, N1, tile, hi4, lo4, tw1_lds, tw2);
    const size_t tile0 = (size_t)tile * 4096;
    const WMul W = A.Binv[i];
    const bool pre = ADD && A.pre != nullptr, xm = xm_val;
    const WMul Pm = pre ? A.pre[i] : xmv;
    const unsigned r0 = blockIdx.x * (unsigned)A.rows_per_x;
    const unsigned r1 = (r0 + A.rows_per_x < (unsigned)A.rows) ? r0 + A.rows_per_x : (unsigned)A.rows;
    for (unsigned row = r0; row < r1; row++) {
        const u64d *xin = A.x + (size_t)row * A.x_row_stride + (size_t)i * N + tile0;
        u64d *out = A.out + (size_t)row * A.out_row_stride + (size_t)(i - A.out_limb0) * N + tile0;
        const bool add = ADD && A.addend && (pre || xm || (row & 1u) == 0);
        const u64d *ad = add ? A.addend + (size_t)(row / 2) * A.add_item_stride + (size_t)(row % 2) * A.add_comp_stride + (size_t)i * N + tile0 : xin;
        // operands of the last step are requested before the transform so that their latency overlaps it
        // pointwise part in the row-pair layout: 16 bytes per lane and memory instruction, no workgroup barrier
        ulonglong2 xr[8], ar[ADD ? 8 : 1];
#pragma unroll
        for (int s = 0; s < 8; s++) {
            xr[s] = pair_load<KEPT_NT>(xin, row_pair_index(hi4, lo4, s));
            if (ADD && !GAL) ar[s] = ((const ulonglong2 *)ad)[row_pair_index(hi4, lo4, s)];
        }
        if (GAL && add) {
            const unsigned pair = row / 2u, item = pair / (unsigned)gal->R, r = pair % (unsigned)gal->R;
#pragma unroll
            for (int s = 0; s < 8; s++)
                ar[s] = galois_pair_load(A.addend + (size_t)item * A.add_item_stride + (size_t)i * N,
                                         (unsigned)tile0 + hi4 * 256u + 32u * s + 2u * lo4, gal->g[r], A.logN);
        }
        SCHED_FENCE();
        rows_fwd_to_lds<P51, ROW_LAZY, !ADD>(A.tmpA + ((size_t)row * A.nc + i) * N + tile0, lds, tw1_lds, tw2, p, pinv, hi4, lo4, A.stream == STREAM_ALL);
#pragma unroll
        for (int s = 0; s < 8; s++) {
            const double *rr = lds + hi4 * V2_GS + row_pair_lds(lo4, s);
            double x0 = u2d(xr[s].x), x1 = u2d(xr[s].y);
            if (ADD && pre) {  // |x + pre*addend - r| < p + 0.75p + ROWX: below 2^53
                x0 += mulmod_w(u2d(ar[s].x), Pm.w, Pm.wp, p);
                x1 += mulmod_w(u2d(ar[s].y), Pm.w, Pm.wp, p);
            }
            if (xm) {  // |x*xmv - r| < 0.75p + ROWX (without an addend `ar` is a copy of x: not used)
                x0 = mulmod_w(x0, Pm.w, Pm.wp, p);
                x1 = mulmod_w(x1, Pm.w, Pm.wp, p);
            }
            double v0, v1;
            if (A.zsub) {
                v0 = x0 - mulmod_w(rr[0], W.w, W.wp, p);
                v1 = x1 - mulmod_w(rr[1], W.w, W.wp, p);
            } else {
                v0 = mulmod_w(x0 - rr[0], W.w, W.wp, p);
                v1 = mulmod_w(x1 - rr[1], W.w, W.wp, p);
            }
            if (ADD && add && !pre) {
                v0 += u2d(ar[s].x);
                v1 += u2d(ar[s].y);
            }
            // a product below 1.5p and an addend, or (zsub: no addend) a word and a product of a word of at most ROWX: 2.5p
            pair_store<NTS>(out, row_pair_index(hi4, lo4, s), make_ulonglong2(d2u(canon_near<P51>(v0, p, pinv)), d2u(canon_near<P51>(v1, p, pinv))));
        }
        ROW_GROUP_SYNC();
    }
}

// grid: x = chunk of rows (item, component), y = row tile (N/4096), z = kept limb.  ADD: with an addend; without one (a product's
// tail, plain divisions) the words in flight leave room for a third wave per SIMD; with that and the kept limb's words streamed
// 128 rows of 23 kept limbs at N = 2^16 take 906 us against 931: 5.1 TB/s, where a copy of large pieces moves 6.2
template <bool NTS, bool ADD, bool KEPT_NT>
__global__ __launch_bounds__(V2_THREADS, ADD ? 2 : 3) void rows_final_kernel(RowsFinalArgs A) {
    __shared__ double lds[16 * V2_GS];
    __shared__ double tw1_lds[16 * 16];
    const int i = A.limb0 + (int)blockIdx.z;
    if (is_p51(A.p51, i))
        rows_final_body<true, NTS, ADD, KEPT_NT>(A, lds, tw1_lds, i);
    else
        rows_final_body<false, NTS, ADD, KEPT_NT>(A, lds, tw1_lds, i);
}

// the same for rotations from a shared ModUp: the addend sigma_r(c0) is read through the automorphism
template <bool NTS>
__global__ __launch_bounds__(V2_THREADS) void rows_final_gal_kernel(RowsFinalArgs A, RowsFinalGal G) {
    __shared__ double lds[16 * V2_GS];
    __shared__ double tw1_lds[16 * 16];
    const int i = A.limb0 + (int)blockIdx.z;
    if (is_p51(A.p51, i))
        rows_final_body<true, NTS, true, NTS, true>(A, lds, tw1_lds, i, false, WMul{0.0, 0.0}, &G);
    else
        rows_final_body<false, NTS, true, NTS, true>(A, lds, tw1_lds, i, false, WMul{0.0, 0.0}, &G);
}

// the same with the kept limb multiplied by a per-call scalar first: out = (c*x - r) * Binv (+ addend): rescale of c*x
template <bool NTS>
__global__ __launch_bounds__(V2_THREADS) void rows_final_scalar_kernel(RowsFinalArgs A, ScalarTab S) {
    __shared__ double lds[16 * V2_GS];
    __shared__ double tw1_lds[16 * 16];
    const int i = A.limb0 + (int)blockIdx.z;
    const WMul xmv = S.c[i];
    if (is_p51(A.p51, i))
        rows_final_body<true, NTS, true, false>(A, lds, tw1_lds, i, true, xmv);
    else
        rows_final_body<false, NTS, true, false>(A, lds, tw1_lds, i, true, xmv);
}
