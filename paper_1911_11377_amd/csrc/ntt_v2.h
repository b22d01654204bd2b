// Register-tiled limb transforms for N = N1 x 256, N1 = 16 .. 256 (2^12 <= N <= 2^16), gfx950.
//
// A transform of N = 2^logN points is split into a strided pass over columns (the first
// k = logN-8 stages, N1 = 2^k-point sub-transforms down the columns of the N1 x 256 matrix)
// and a contiguous pass over rows of 256 words (the last 8 stages).  In both, a workgroup of
// 256 threads works on a tile of 4096 words: every thread keeps 16 words in registers and does
// up to four butterfly stages on them without touching memory ("round"); one exchange through
// LDS regroups the words for the second round.
//
//   row pass   : tile = 16 rows.  A row is a 16x16 matrix M[a][b] (position 16a+b); round 1
//                (spans >= 16) works along a, round 2 (spans < 16) along b.
//   column pass: tile = N1 rows x C columns, C = 4096/N1.  With G = N1/16 = 2^Q: round 1 does the
//                first four stages on the rows {r + G*e}; round 2 does the remaining Q stages on
//                groups of G consecutive rows, a thread holding 16/G columns of one group.
//
// Twiddles: stage s of the whole transform multiplies block i by psi^brev(2^s + i).  For a thread
// they reduce to at most 15 values per round that depend only on the tile position and the lane,
// so they are loaded into registers once per workgroup and reused for every item the workgroup
// loops over (same modulus, same tile): twiddle traffic is amortised over the batch.
//
// Between the two passes the words are stored as lazily reduced doubles (mid_store / mid_load), not as canonical
// integers: that intermediate never leaves the library.
//
// Lazy ranges (units of p, see device_arith.h): a twiddle product of y is bounded by (1/2 + 1.5*|y|/2^53) p, so a butterfly
// stage maps a bound B to B + 1/2 + 1.5*B*p/2^53 forward and to 2B (the sum) or 1/2 + 3*B*p/2^53 (the product) inverse; values
// must stay below 2^53, i.e. 8p for p < 2^50 and 4p for p < 2^51 (template parameter P51).  A reduction costs three
// instructions of the eight of a butterfly, so the words that are reduced, and where, are found at compile time (fwd_plan,
// inv_plan below): forward only the addends u of u +- w*v at one or two of eight stages, inverse only the registers whose
// sum would pass the limit.  That is 3 (forward) and 6 (inverse) instructions per word of a 16-stage transform at p < 2^50,
// against 9 and 15 with all words reduced at the end of every round.  With the quotient taken from the product itself (mulmod)
// a twiddle costs no register and no instruction beside its word.  Together, against reductions of whole rounds and w/p
// recomputed per block: 64 products at N = 2^16, 24 primes 7569 -> 7216 us, 256 at 2^14, 8 primes 2213 -> 2103, 64 fresh
// ciphertexts 3474 -> 2790 (their row pass at two waves per SIMD instead of one).
#pragma once
#include "device_arith.h"

#define V2_THREADS 256
#ifdef CKKSMI_EMULATE
#define NTT_SCHED_FENCE() ((void)0)
#else
#define NTT_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)
#endif
// Two instantiations of a body behind one uniform branch start with different (empty) asm statements: the compiler otherwise
// merges their identical beginnings into the block before the branch and spills what it computed there.
#ifdef CKKSMI_EMULATE
#define BODY_TAG(V) ((void)0)
#else
#define BODY_TAG(V)                              \
    do {                                         \
        if (V) asm volatile("; body, 51 bits");  \
        else asm volatile("; body, 50 bits");    \
    } while (0)
#endif

// What the compiler has to be told to stay within a kernel's registers (all empty on the CPU stand-in):
//   PIN_VALUE(x)    x is computed before the next pinned point and not sunk below later loads;
//   scalar_base(p)  a workgroup-uniform address of global memory stays in scalar registers: the accesses p[thread offset] are
//                   global ones with a scalar base and one 32-bit offset per thread.  The global address space is part of
//                   what is returned: a generic pointer that comes out of an asm statement makes flat accesses, which take
//                   no scalar base (one 64-bit vector addition each) and are counted as LDS accesses too, so that all of them
//                   arrive before the first is used.  8 limbs of 2^13 words forward 9.5 us with flat, 9.1 with global
//                   accesses; rescale of 256 ciphertexts at N = 2^14, 8 primes 335 and 321 us, N = 2^15, 16 primes, 448
//                   ciphertexts 2503 and 2469 us;
//   WG_UNIFORM(v)   a workgroup-uniform value goes to a scalar register;
//   PIN_UNIFORM(x)  the same as PIN_VALUE for a workgroup-uniform value in scalar registers;
//   LOAD_FENCE()    memory accesses stay on their side.
#ifdef CKKSMI_EMULATE
#define PIN_VALUE(x) ((void)0)
#define PIN_UNIFORM(x) ((void)0)
#define LOAD_FENCE() ((void)0)
#define WG_UNIFORM(v) (v)
template <class T> __device__ __forceinline__ T *scalar_base(T *p) { return p; }
#else
#define PIN_VALUE(x) asm volatile("" : "+v"(x))
#define PIN_UNIFORM(x) asm volatile("" : "+s"(x))
#define LOAD_FENCE() asm volatile("" ::: "memory")
#define WG_UNIFORM(v) ((unsigned)__builtin_amdgcn_readfirstlane((int)(v)))
template <class T> __device__ __forceinline__ __attribute__((address_space(1))) T *scalar_base(T *p) {
    auto g = (__attribute__((address_space(1))) T *)p;
    asm volatile("" : "+s"(g));
    return g;
}
#endif

// A workgroup-uniform entry of a read-only table through the scalar cache: it arrives in scalar registers.  (A kernel that also
// stores gets its uniform loads in vector registers otherwise.)
#ifdef CKKSMI_EMULATE
static inline double table_load(const double *t, unsigned i) { return t[i]; }
#else
typedef const __attribute__((address_space(4))) double *ConstTable;
__device__ __forceinline__ double table_load(const double *t, unsigned i) { return ((ConstTable)(unsigned long long)t)[i]; }
#endif
__device__ __forceinline__ WMul table_load(const WMul *t) { return WMul{table_load((const double *)t, 0), table_load((const double *)t, 1)}; }

// Streamed accesses (non-temporal): words that the caches could not keep until they are wanted again.  How much of a launch is
// streamed is decided on the host from the bytes it moves (stream_level, ckksmi_device.hip): STREAM_STORES results only,
// STREAM_ALL operands too.  It is a template parameter of the kernel, or where that would double many instances a loop of
// accesses behind one uniform branch:
//     stream_if(A.stream != STREAM_NONE, [&](auto nt) { for (...) stream_store<nt>(p, v); });
enum { STREAM_NONE, STREAM_STORES, STREAM_ALL };
template <bool V> struct StreamFlag { constexpr operator bool() const { return V; } };
#ifdef CKKSMI_EMULATE
#define STREAM_TAG(T) ((void)0)
template <bool NT, class P> static inline auto stream_load(P p) { return *p; }
template <bool NT, class P, class V> static inline void stream_store(P p, V v) { *p = v; }
#else
// (the compiler merges accesses of both branches that differ in the hint only, into plain ones: the notes keep them apart)
#define STREAM_TAG(T) asm volatile("; " T ::: "memory")
typedef unsigned long long u64pair __attribute__((ext_vector_type(2)));
template <bool NT, class P> __device__ __forceinline__ auto stream_load(P p) {
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}
template <bool NT> __device__ __forceinline__ ulonglong2 stream_load(const ulonglong2 *p) {
    const u64pair v = stream_load<NT>((const u64pair *)p);
    return make_ulonglong2(v.x, v.y);
}
template <bool NT, class P, class V> __device__ __forceinline__ void stream_store(P p, V v) {
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}
template <bool NT> __device__ __forceinline__ void stream_store(ulonglong2 *p, ulonglong2 v) { stream_store<NT>((u64pair *)p, u64pair{v.x, v.y}); }
#endif
// the i-th word pair from a workgroup-uniform address
#ifdef CKKSMI_EMULATE
template <bool NT> static inline ulonglong2 pair_load(const u64d *base, unsigned i) { return ((const ulonglong2 *)base)[i]; }
template <bool NT> static inline void pair_store(u64d *base, unsigned i, ulonglong2 v) { ((ulonglong2 *)base)[i] = v; }
#else
template <bool NT> __device__ __forceinline__ ulonglong2 pair_load(const u64d *base, unsigned i) {
    const u64pair v = stream_load<NT>(scalar_base((const u64pair *)base) + i);
    return make_ulonglong2(v.x, v.y);
}
template <bool NT> __device__ __forceinline__ void pair_store(u64d *base, unsigned i, ulonglong2 v) {
    stream_store<NT>(scalar_base((u64pair *)base) + i, u64pair{v.x, v.y});
}
#endif
template <class F> __device__ __forceinline__ void stream_if(bool on, F f) {
    if (on) {
        STREAM_TAG("streamed");
        f(StreamFlag<true>());
        STREAM_TAG("streamed, end");
    } else {
        STREAM_TAG("cached");
        f(StreamFlag<false>());
        STREAM_TAG("cached, end");
    }
}

#define V2_GS 272  // doubles per padded 16x17 group in LDS (row pass)

// Row pass: the 16 lanes that work on one row of 256 words exchange their words through that row's own LDS group and
// nothing else, and 16 consecutive lanes always sit in one wavefront.  A wavefront's LDS instructions execute in program
// order, so these exchanges need no workgroup barrier: the fences only keep the compiler from moving LDS accesses across
// the exchange point.  (The CPU stand-in runs one thread at a time and needs a real barrier there.)
#ifdef CKKSMI_EMULATE
#define ROW_GROUP_SYNC() __syncthreads()
#else
#define ROW_GROUP_SYNC()                                        \
    do {                                                        \
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  \
        __builtin_amdgcn_wave_barrier();                        \
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");  \
    } while (0)
#endif

// Pointwise layout of the row-pass kernels: thread (hi4 = tid / 16, lo4 = tid % 16) owns the word pairs at columns
// 32*s + 2*lo4, +1 (s < 8) of row hi4 of the tile: 16 bytes per lane and memory instruction, 256 contiguous bytes per
// row and instruction, and every word of a row stays with the 16 lanes that transform that row.
__device__ __forceinline__ unsigned row_pair_index(unsigned hi4, unsigned lo4, int s) { return hi4 * 128u + 16u * s + lo4; }  // in 16-byte units from the tile
// the same pair in the row's LDS group (padded 16 x 17 doubles; word q of the row at (q / 16) * 17 + q % 16)
__device__ __forceinline__ unsigned row_pair_lds(unsigned lo4, int s) { return (2u * s + (lo4 >> 3)) * 17u + 2u * (lo4 & 7u); }

struct NttV2Args {
    const u64d *src;
    u64d *dst;
    const ModConst *modc;
    const double *tw;     // [T][N] twiddles of the direction, balanced representatives
    const WMul *tw_ninv;  // [T] inverse only: 1/N
    const WMul *tw_last;  // [T] inverse only: psi^-brev(1)/N
    const FinConst *fin;  // optional, inverse column pass: per limb slot, replaces the 1/N constants of the last stage
    int use_fin_val;      // ... or, where the coefficients leave as doubles, one set passed by value (per-call constants)
    FinConst fin_val;
    int logN;
    int items, items_per_z;
    P51Mask p51;
    LimbMap map;
    // source of real coefficients (real_word): their scale, and the word that is raised where one is too large
    double factor;
    int *overflow;
};

// Coefficient rint(v * factor) of an encoding as a residue: |m| < 2^62 is an integer that the double holds exactly, and p > 2N >= 2^13 keeps the
// quotient below 2^49 and its error below 1/8 before rounding, so that the remainder (0.63p) is exact.  largest: of the magnitudes so far (a NaN stays out
// of a maximum: it is turned into an infinity).
__device__ __forceinline__ double real_word(double v, double factor, double p, double pinv, double &largest) {
    const double m = rint(v * factor);
    largest = fmax(largest, m == m ? fabs(m) : HUGE_VAL);
    return reduce_balanced(m, p, pinv);
}
enum { SRC_WORDS, SRC_SMALL, SRC_REAL };  // sources of a forward transform

// Bounds (units of p) where a value changes hands
template <bool P51>
struct LazyRange {
    static constexpr double LIM = P51 ? 4.0 : 8.0;    // 2^53 / p
    static constexpr double MIDF = P51 ? 2.5 : 3.5;   // forward, between column and row pass
    static constexpr double ROWX = P51 ? 2.0 : 6.2;   // forward, results that a pointwise step takes as they are
    static constexpr double FACTOR = P51 ? 0.51 : 2.2;  // forward, results that are multiplied by words of a switching key
    static constexpr double INV0 = 1.25, INV1 = 2.0, MIDI = P51 ? 2.0 : 4.0;  // inverse: entry, between rounds, between row and column pass
};
#define LAZY_REDUCED 0.51  // |x| <= p/2 + 1

// bound after n forward stages from `entry` when the addends are reduced at the stages of `mask`; above the limit: -1
constexpr double fwd_bound(bool p51, double entry, int n, int mask) {
    const double lim = p51 ? 4.0 : 8.0;
    double b = entry;
    for (int s = 0; s < n; s++) {
        if (b > lim) return -1.0;
        b = ((mask >> s) & 1 ? LAZY_REDUCED : b) + 0.5 + 1.5 * b / lim;
    }
    return b > lim ? -1.0 : b;
}
// fewest reductions that end at or below `exit`
constexpr int fwd_plan(bool p51, double entry, int n, double exit) {
    int best = -1, best_count = n + 1;
    for (int m = 0; m < (1 << n); m++) {
        int count = 0;
        for (int s = 0; s < n; s++) count += (m >> s) & 1;
        const double b = fwd_bound(p51, entry, n, m);
        if (b >= 0.0 && b <= exit && count < best_count) {
            best = m;
            best_count = count;
        }
    }
    return best;
}

// Inverse stages 3 .. S0 of a 16-point round: registers reduced before the k-th executed stage (bit = register), and at the end
struct InvPlan {
    unsigned before[4], after;
};
constexpr InvPlan inv_plan(bool p51, double entry, int S0, double exit, bool final) {
    const double lim = p51 ? 4.0 : 8.0;
    InvPlan P{{0, 0, 0, 0}, 0};
    double b[16] = {};
    for (int i = 0; i < 16; i++) b[i] = entry;
    for (int k = 0; k < 4 - S0; k++) {
        const int s = 3 - k, span = 8 >> s;
        for (int lo = 0; lo < 16; lo++) {
            if (lo & span) continue;
            const int hi = lo + span;
            for (int r = 0; r < 2 && b[lo] + b[hi] > lim; r++) {  // the larger one first
                const int i = b[lo] >= b[hi] ? lo : hi;
                b[i] = LAZY_REDUCED;
                P.before[k] |= 1u << i;
            }
            const double sum = b[lo] + b[hi], prod = 0.5 + 1.5 * sum / lim;
            b[lo] = final && s == 0 ? prod : sum;
            b[hi] = prod;
        }
    }
    for (int i = 0; i < 16; i++)
        if (b[i] > exit) P.after |= 1u << i;
    return P;
}

// decimation-in-time stages S0..3 of a 16-point round (spans 8 >> s over the register index);
// MASK bit s: the addends of stage s are reduced first
template <int S0, int MASK>
__device__ __forceinline__ void fwd_stages(double (&x)[16], const double (&tw)[15], double p, double pinv) {
#pragma unroll
    for (int s = S0; s < 4; s++) {
        const int span = 8 >> s;
#pragma unroll
        for (int b = 0; b < (1 << s); b++) {
#pragma unroll
            for (int j = 0; j < span; j++) {
                const int lo = b * 2 * span + j, hi = lo + span;
                // the quotient from the product itself: no w/p to keep or to compute
                const double v = mulmod(x[hi], tw[(1 << s) - 1 + b], p, pinv);
                const double u = (MASK & (1 << s)) ? reduce_balanced(x[lo], p, pinv) : x[lo];
                x[lo] = u + v;
                x[hi] = u - v;
            }
        }
    }
}
template <int MASK>
__device__ __forceinline__ void fwd_round(double (&x)[16], const double (&tw)[15], double p, double pinv) {
    fwd_stages<0, MASK>(x, tw, p, pinv);
}

// the same stages undone, 3 down to S0 (spans 1,2,..), with the reductions of inv_plan; B: where the round stands, which gives the
// bounds of its words; FINAL folds 1/N into the very last stage (s = 0) of the whole transform.  The rounds follow one another as
// they are listed.  In a workgroup that holds all 2^12 words of a ring INV_COL2 is left out (the column pass has one round), and
// the row pass ends with INV_ROW2_12 instead, within what INV_COL1 takes.
enum InvRound { INV_ROW1, INV_ROW2, INV_COL2, INV_COL1, INV_ROW2_12 };
template <bool P51>
constexpr double inv_entry(InvRound B) {
    typedef LazyRange<P51> R;
    return B == INV_ROW1 ? R::INV0 : B == INV_COL2 ? R::MIDI : R::INV1;
}
template <bool P51>
constexpr double inv_exit(InvRound B) {
    typedef LazyRange<P51> R;
    return B == INV_ROW2 ? R::MIDI : B == INV_COL1 ? R::LIM : R::INV1;
}
// stands where the words of round A become those of round B
#define INV_JOIN(P51, A, B) static_assert(inv_exit<P51>(A) <= inv_entry<P51>(B), "the second round takes less than the first one leaves")
template <int S0, InvRound B, bool P51>
__device__ __forceinline__ void inv_stages(double (&x)[16], const double (&tw)[15], double p, double pinv, WMul ninv, WMul wlast) {
    constexpr bool FINAL = B == INV_COL1;
    constexpr InvPlan PL = inv_plan(P51, inv_entry<P51>(B), S0, inv_exit<P51>(B), FINAL);
#pragma unroll
    for (int k = 0; k < 4 - S0; k++) {
        const int s = 3 - k, span = 8 >> s;
#pragma unroll
        for (int b = 0; b < (1 << s); b++) {
#pragma unroll
            for (int j = 0; j < span; j++) {
                const int lo = b * 2 * span + j, hi = lo + span;
                const double u = (PL.before[k] >> lo) & 1u ? reduce_balanced(x[lo], p, pinv) : x[lo];
                const double v = (PL.before[k] >> hi) & 1u ? reduce_balanced(x[hi], p, pinv) : x[hi];
                if (FINAL && s == 0) {
                    x[lo] = mulmod_w(u + v, ninv.w, ninv.wp, p);
                    x[hi] = mulmod_w(u - v, wlast.w, wlast.wp, p);
                } else {
                    x[lo] = u + v;
                    x[hi] = mulmod(u - v, tw[(1 << s) - 1 + b], p, pinv);
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 16; i++)
        if ((PL.after >> i) & 1u) x[i] = reduce_balanced(x[i], p, pinv);
}

// ------------------------------------------------------------------ row pass twiddles
// base1 = N1 + row; round 1 uses tw[(base1 << s) + b], round 2 (lane = the thread's a) tw[((16*base1 + lane) << s) + b]
__device__ __forceinline__ void load_twiddles(const double *tw, unsigned base1, unsigned lane, double (&tw1)[15], double (&tw2)[15]) {
#pragma unroll
    for (int s = 0; s < 4; s++)
#pragma unroll
        for (int b = 0; b < (1 << s); b++) {
            tw1[(1 << s) - 1 + b] = tw[(base1 << s) + b];
            tw2[(1 << s) - 1 + b] = tw[((16u * base1 + lane) << s) + b];
        }
}

// ------------------------------------------------------------------ column pass geometry
// Q = log2(N1/16).  Round 1: register e <-> row r + G*e, column c0 + c   (r = tid / C, c = tid % C).
// Round 2: register pp*G + g <-> row G*a + g, column c0 + l16 + 16*pp     (a = tid >> 4, l16 = tid & 15).
template <int Q>
struct ColsGeom {
    static constexpr unsigned G = 1u << Q, C = 256u >> Q, P = 16u >> Q;
    static constexpr int S0 = 4 - Q;  // first register stage of round 2
    unsigned r, c, a, l16, c0;
    __device__ __forceinline__ ColsGeom(unsigned tid, unsigned tile) : r(tid / C), c(tid % C), a(tid >> 4), l16(tid & 15), c0(tile * C) {}
    __device__ __forceinline__ size_t g1(int e) const { return (size_t)(r + G * e) * 256 + c0 + c; }                       // global, round-1 register e
    __device__ __forceinline__ size_t g2(int i) const { return (size_t)(G * a + (i % G)) * 256 + c0 + l16 + 16 * (i / G); }  // global, round-2 register i
    // the same in parts, g1(e) = c0 + d1(e) + t1() and g2(i) = c0 + d2(i) + t2(): uniform, constant, and the thread's own
    static constexpr unsigned d1(int e) { return G * e * 256u; }
    static constexpr unsigned d2(int i) { return (i % G) * 256u + 16u * (i / G); }
    __device__ __forceinline__ unsigned t1() const { return r * 256u + c; }
    __device__ __forceinline__ unsigned t2() const { return G * a * 256u + l16; }
    __device__ __forceinline__ unsigned l1(int e) const { return (r + G * e) * C + c; }                                    // LDS [N1][C]
    __device__ __forceinline__ unsigned l2(int i) const { return (G * a + (i % G)) * C + l16 + 16 * (i / G); }
};

// round 1: the first four stages, block b of stage s uses tw[2^s + b] (same for every thread);
// round 2: register stage s = S0 + u is transform stage 4 + u, block = a*2^u + (b mod 2^u)
template <int Q>
__device__ __forceinline__ void load_cols_twiddles(const double *tw, unsigned a, double (&tw1)[15], double (&tw2)[15]) {
#pragma unroll
    for (int s = 0; s < 4; s++)
#pragma unroll
        for (int b = 0; b < (1 << s); b++) {
            tw1[(1 << s) - 1 + b] = tw[(1u << s) + b];
            if (s >= 4 - Q) {
                const int u = s - (4 - Q);
                tw2[(1 << s) - 1 + b] = tw[(16u << u) + (a << u) + (b & ((1 << u) - 1))];
            } else {
                tw2[(1 << s) - 1 + b] = 0.0;
            }
        }
}

// forward reduction masks of the column pass: round 1, and round 2 (Q stages, register stages from 4 - Q on).  ENTRY256: bound of
// the input in 1/256 p
template <int Q, bool P51, int ENTRY256>
struct ColsMasks {
    static constexpr int PLAN = fwd_plan(P51, ENTRY256 / 256.0, 4 + Q, LazyRange<P51>::MIDF);
    static_assert(PLAN >= 0, "no reduction schedule");
    static constexpr int F1 = PLAN & 15, F2 = (PLAN >> 4) << (4 - Q);
};
// ... and of the row pass, from MIDF.  What becomes of the results:
//   ROW_REDUCED  they are reduced or made canonical whatever they are;
//   ROW_LAZY     a pointwise step takes them as they are (ROWX);
//   ROW_NEAR     p < 2^50: canon_near takes them (the words that enter have to be bounded in p itself);  ROW_FACTOR: a key word's product takes
//                them (FACTOR).  Both cost one reduction of half of the words more than ROW_REDUCED and save that of all of them.  p < 2^51: as
//                ROW_REDUCED.
enum { ROW_REDUCED, ROW_LAZY, ROW_NEAR, ROW_FACTOR };
template <bool P51, int X>
struct RowMasks {
    typedef LazyRange<P51> R;
    static constexpr int PLAN = fwd_plan(P51, R::MIDF, 8, X == ROW_LAZY ? R::ROWX : P51 || X == ROW_REDUCED ? R::LIM : X == ROW_NEAR ? 2.9 : R::FACTOR);
    static_assert(PLAN >= 0, "no reduction schedule");
    static constexpr int F1 = PLAN & 15, F2 = PLAN >> 4;
};

// SRC (forward only): SRC_SMALL a polynomial with small signed coefficients, one int64 per coefficient and the same
// for every limb (item i at (const long long *)A.src + i * src_item_stride): its residues are the values themselves; SRC_REAL the real parts of
// complex words (item i at (const double2 *)A.src + i * src_item_stride), see real_word
// F64 (inverse only): the canonical coefficients leave as doubles (the input of a conversion, never visible outside)
// NT: operands and results are streamed
template <bool INV, int Q, bool P51, int SRC, bool F64, bool NT>
__device__ __forceinline__ void ntt_v2_cols(const NttV2Args &A, double *lds, int t, unsigned li) {
    typedef ColsGeom<Q> Geo;
    typedef ColsMasks<Q, P51, 256> Mk;
    const unsigned N = 1u << A.logN;
    const double p = A.modc[t].p, pinv = A.modc[t].pinv;
    const double *tw = A.tw + (size_t)t * N;
    const Geo geo(threadIdx.x, blockIdx.x);
    double tw1[15], tw2[15];
    load_cols_twiddles<Q>(tw, geo.a, tw1, tw2);
    WMul ninv = WMul{0.0, 0.0}, wlast = WMul{0.0, 0.0};
    double cadd = 0.0;
    if (INV) {
        ninv = A.tw_ninv[t];
        wlast = A.tw_last[t];
        if (F64 && A.use_fin_val) { ninv = A.fin_val.ninv; wlast = A.fin_val.wlast; cadd = A.fin_val.cadd; }
        else if (A.fin) { ninv = A.fin[li].ninv; wlast = A.fin[li].wlast; cadd = A.fin[li].cadd; }
    }
    const unsigned i0 = blockIdx.z * (unsigned)A.items_per_z;
    const unsigned i1 = (i0 + A.items_per_z < (unsigned)A.items) ? i0 + A.items_per_z : (unsigned)A.items;
    for (unsigned it = i0; it < i1; it++) {
        const u64d *src = A.src + (size_t)it * A.map.src_item_stride + (size_t)li * N;
        u64d *dst = A.dst + (size_t)it * A.map.dst_item_stride + (size_t)li * N;
        double x[16];
        if (!INV) {
            // Real coefficients: all of them requested before the first is used, whose test would keep the requests apart (64 encodings of 24
            // primes at N = 2^16 282 -> 215 us).  The others are requested and used in the compiler's order: held back like that, the pass took 1.02 - 1.04 x the
            // time for small polynomials up to 64 rows of 8 primes at N = 2^14, and for words (100 items of 16 primes at N = 2^15, 4 at 2^16).
            u64d raw[SRC == SRC_REAL ? 16 : 1];
            if (SRC == SRC_REAL) {
#pragma unroll
                for (int e = 0; e < 16; e++) raw[SRC == SRC_REAL ? e : 0] = ((const u64d *)A.src + 2 * (size_t)it * A.map.src_item_stride)[2 * geo.g1(e)];
                NTT_SCHED_FENCE();
            }
            double largest = 0.0;
#pragma unroll
            for (int e = 0; e < 16; e++) {
                // SRC_SMALL, magnitudes below 2^51: shifted to a non-negative integer, which becomes a double without a conversion of 64 bits;
                // the reduction brings it into the range of the first round
                if (SRC == SRC_REAL) {
                    x[e] = real_word(__longlong_as_double((long long)raw[SRC == SRC_REAL ? e : 0]), A.factor, p, pinv, largest);
                } else if (SRC == SRC_SMALL) {
                    const long long v = ((const long long *)A.src + (size_t)it * A.map.src_item_stride)[geo.g1(e)];
                    x[e] = reduce_balanced(u2d((unsigned long long)(v + (1ll << 51))) - 2251799813685248.0, p, pinv);
                }
                else x[e] = u2d(stream_load<NT>(&src[geo.g1(e)]));
            }
            if (SRC == SRC_REAL && !(largest < 4.0e18)) *A.overflow = 1;
            fwd_round<Mk::F1>(x, tw1, p, pinv);
#pragma unroll
            for (int e = 0; e < 16; e++) lds[geo.l1(e)] = x[e];
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 16; i++) x[i] = lds[geo.l2(i)];
            fwd_stages<Geo::S0, Mk::F2>(x, tw2, p, pinv);
#pragma unroll
            for (int i = 0; i < 16; i++) stream_store<NT>(&dst[geo.g2(i)], mid_store(x[i]));
        } else {
#pragma unroll
            for (int i = 0; i < 16; i++) x[i] = mid_load(stream_load<NT>(&src[geo.g2(i)]));
            INV_JOIN(P51, INV_ROW2, INV_COL2);
            inv_stages<Geo::S0, INV_COL2, P51>(x, tw2, p, pinv, ninv, wlast);
            INV_JOIN(P51, INV_COL2, INV_COL1);
#pragma unroll
            for (int i = 0; i < 16; i++) lds[geo.l2(i)] = x[i];
            __syncthreads();
#pragma unroll
            for (int e = 0; e < 16; e++) x[e] = lds[geo.l1(e)];
            inv_stages<0, INV_COL1, P51>(x, tw1, p, pinv, ninv, wlast);
#pragma unroll
            for (int e = 0; e < 16; e++) {
                const double v = canon_near<P51>(x[e] + cadd, p, pinv);  // 1.5p and less than p
                stream_store<NT>(&dst[geo.g1(e)], F64 ? (u64d)__double_as_longlong(v) : d2u(v));
            }
        }
        __syncthreads();
    }
}

// GAL (inverse only): the input is read through the automorphism X -> X^g of its item (G->g[item]): a rotation's
// polynomial enters its key switch without a pass of its own
template <bool INV, bool P51, bool NT, bool GAL = false>
__device__ __forceinline__ void ntt_v2_rows(const NttV2Args &A, double *lds, int t, unsigned li, const GaloisTab *G = nullptr) {
    const unsigned N = 1u << A.logN, N1 = N >> 8;
    const double p = A.modc[t].p, pinv = A.modc[t].pinv;
    const double *tw = A.tw + (size_t)t * N;
    const unsigned tid = threadIdx.x, hi4 = tid >> 4, lo4 = tid & 15;
    double tw1[15], tw2[15];
    const WMul unused = WMul{0.0, 0.0};
    load_twiddles(tw, N1 + blockIdx.x * 16 + hi4, lo4, tw1, tw2);
    const unsigned i0 = blockIdx.z * (unsigned)A.items_per_z;
    const unsigned i1 = (i0 + A.items_per_z < (unsigned)A.items) ? i0 + A.items_per_z : (unsigned)A.items;
    typedef RowMasks<P51, ROW_NEAR> Mk;
    const size_t tile0 = (size_t)blockIdx.x * 4096;
    double *grp = lds + hi4 * V2_GS;
    for (unsigned it = i0; it < i1; it++) {
        const u64d *src = A.src + (size_t)it * A.map.src_item_stride + (size_t)li * N;
        u64d *dst = A.dst + (size_t)it * A.map.dst_item_stride + (size_t)li * N;
        double x[16];
        if (!INV) {
#pragma unroll
            for (int e = 0; e < 16; e++) x[e] = mid_load(stream_load<NT>(&src[tile0 + hi4 * 256 + lo4 + 16 * e]));
            fwd_round<Mk::F1>(x, tw1, p, pinv);
#pragma unroll
            for (int e = 0; e < 16; e++) grp[e * 17 + lo4] = x[e];
            ROW_GROUP_SYNC();
#pragma unroll
            for (int e = 0; e < 16; e++) x[e] = grp[lo4 * 17 + e];
            fwd_round<Mk::F2>(x, tw2, p, pinv);
#pragma unroll
            for (int e = 0; e < 16; e++) grp[lo4 * 17 + e] = canon_near<P51>(x[e], p, pinv);
            ROW_GROUP_SYNC();
            // canonical words out in the row-pair layout: 16 bytes per lane and store
#pragma unroll
            for (int s = 0; s < 8; s++) {
                const double *rr = grp + row_pair_lds(lo4, s);
                stream_store<NT>((ulonglong2 *)(dst + tile0) + row_pair_index(hi4, lo4, s), make_ulonglong2(d2u(rr[0]), d2u(rr[1])));
            }
        } else {
            {
                // all 16 words requested before the first is used: one memory latency per item, not sixteen
                // (row-pair layout: 16 bytes per lane and load)
                ulonglong2 raw[8];
                if (GAL) {
#pragma unroll
                    for (int s = 0; s < 8; s++) raw[s] = galois_pair_load(src, (unsigned)tile0 + hi4 * 256u + 32u * s + 2u * lo4, G->g[it], A.logN);
                } else {
#pragma unroll
                    for (int s = 0; s < 8; s++) raw[s] = stream_load<NT>((const ulonglong2 *)(src + tile0) + row_pair_index(hi4, lo4, s));
                }
                NTT_SCHED_FENCE();
#pragma unroll
                for (int s = 0; s < 8; s++) {
                    double *rr = grp + row_pair_lds(lo4, s);
                    rr[0] = u2d(raw[s].x);
                    rr[1] = u2d(raw[s].y);
                }
            }
            ROW_GROUP_SYNC();
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
#pragma unroll
            for (int e = 0; e < 16; e++) stream_store<NT>(&dst[tile0 + hi4 * 256 + lo4 + 16 * e], mid_store(x[e]));
        }
        ROW_GROUP_SYNC();
    }
}

// forward column pass of polynomials given as small signed integers (|coefficient| far below every modulus): same grid as
// ntt_v2_kernel; the residues are never written out limb by limb
template <bool NT>
__global__ __launch_bounds__(V2_THREADS) void ntt_v2_fwd_cols_small_kernel(NttV2Args A) {
    __shared__ double lds[16 * V2_GS];
    unsigned item_unused, li;
    const int t = resolve_limb(A.map, blockIdx.y, item_unused, li);
    if (t < 0) return;
    const bool p51 = is_p51(A.p51, t);
    switch (A.logN) {
        case 12: if (p51) ntt_v2_cols<false, 0, true, SRC_SMALL, false, NT>(A, lds, t, li); else ntt_v2_cols<false, 0, false, SRC_SMALL, false, NT>(A, lds, t, li); break;
        case 13: if (p51) ntt_v2_cols<false, 1, true, SRC_SMALL, false, NT>(A, lds, t, li); else ntt_v2_cols<false, 1, false, SRC_SMALL, false, NT>(A, lds, t, li); break;
        case 14: if (p51) ntt_v2_cols<false, 2, true, SRC_SMALL, false, NT>(A, lds, t, li); else ntt_v2_cols<false, 2, false, SRC_SMALL, false, NT>(A, lds, t, li); break;
        case 15: if (p51) ntt_v2_cols<false, 3, true, SRC_SMALL, false, NT>(A, lds, t, li); else ntt_v2_cols<false, 3, false, SRC_SMALL, false, NT>(A, lds, t, li); break;
        default: if (p51) ntt_v2_cols<false, 4, true, SRC_SMALL, false, NT>(A, lds, t, li); else ntt_v2_cols<false, 4, false, SRC_SMALL, false, NT>(A, lds, t, li); break;
    }
}

// forward column pass of an encoding's real coefficients (N >= 2^14, smaller rings: ntt_wg_fwd_real_kernel), same grid.  A kernel that rounds and writes
// every limb's residues before the transform costs two more limb transfers (and 64-bit divisions): 64 encodings of 24 primes at N = 2^16
// 862 -> 500 us for the rounding, the column and the row pass.
template <bool NT>
__global__ __launch_bounds__(V2_THREADS) void ntt_v2_fwd_cols_real_kernel(NttV2Args A) {
    __shared__ double lds[16 * V2_GS];
    unsigned item_unused, li;
    const int t = resolve_limb(A.map, blockIdx.y, item_unused, li);
    if (t < 0) return;
    const bool p51 = is_p51(A.p51, t);
    switch (A.logN) {
        case 14: if (p51) ntt_v2_cols<false, 2, true, SRC_REAL, false, NT>(A, lds, t, li); else ntt_v2_cols<false, 2, false, SRC_REAL, false, NT>(A, lds, t, li); break;
        case 15: if (p51) ntt_v2_cols<false, 3, true, SRC_REAL, false, NT>(A, lds, t, li); else ntt_v2_cols<false, 3, false, SRC_REAL, false, NT>(A, lds, t, li); break;
        default: if (p51) ntt_v2_cols<false, 4, true, SRC_REAL, false, NT>(A, lds, t, li); else ntt_v2_cols<false, 4, false, SRC_REAL, false, NT>(A, lds, t, li); break;
    }
}

// inverse row pass of a rotation's polynomial: same grid as ntt_v2_kernel, input read through the items' automorphisms
__global__ __launch_bounds__(V2_THREADS) void ntt_v2_inv_rows_gal_kernel(NttV2Args A, GaloisTab G) {
    __shared__ double lds[16 * V2_GS];
    unsigned item_unused, li;
    const int t = resolve_limb(A.map, blockIdx.y, item_unused, li);
    if (t < 0) return;
    if (is_p51(A.p51, t)) ntt_v2_rows<true, true, false, true>(A, lds, t, li, &G);
    else ntt_v2_rows<true, false, false, true>(A, lds, t, li, &G);
}

// grid: x = tile (N/4096), y = limb slot within an item, z = chunk of items (column pass: N >= 2^14, smaller rings go through ntt_wg_kernel)
template <bool INV, bool COLS, bool NT, bool F64 = false>
__global__ __launch_bounds__(V2_THREADS) void ntt_v2_kernel(NttV2Args A) {
    __shared__ double lds[16 * V2_GS];
    unsigned item_unused, li;
    const int t = resolve_limb(A.map, blockIdx.y, item_unused, li);
    if (t < 0) return;
    const bool p51 = is_p51(A.p51, t);
    if (!COLS) {
        if (p51) ntt_v2_rows<INV, true, NT>(A, lds, t, li);
        else ntt_v2_rows<INV, false, NT>(A, lds, t, li);
    } else {
        switch (A.logN) {
            case 14: if (p51) ntt_v2_cols<INV, 2, true, SRC_WORDS, F64, NT>(A, lds, t, li); else ntt_v2_cols<INV, 2, false, SRC_WORDS, F64, NT>(A, lds, t, li); break;
            case 15: if (p51) ntt_v2_cols<INV, 3, true, SRC_WORDS, F64, NT>(A, lds, t, li); else ntt_v2_cols<INV, 3, false, SRC_WORDS, F64, NT>(A, lds, t, li); break;
            case 16: if (p51) ntt_v2_cols<INV, 4, true, SRC_WORDS, F64, NT>(A, lds, t, li); else ntt_v2_cols<INV, 4, false, SRC_WORDS, F64, NT>(A, lds, t, li); break;
        }
    }
}
