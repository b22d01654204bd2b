// Multiply-accumulate of layers with many taps and many output channels on the matrix cores, by residues instead of digits.
//
// The digit kernels of mac_mfma.h spend 7 x 7 = 49 int8 products on each product of two 50-bit numbers.  Here both operands are
// replaced by their residues modulo 15 small numbers m_i <= 256, pairwise coprime, whose product M is 2^117.78: the sum
// S = sum_tap x*w of the integers 0 <= x < p and |w| <= p/2 (balanced) has |S| < 2^14 * 2^51 * 2^50 = 2^115 < M/5 for up to 2^14 taps and
// p < 2^51, so the 15 residues determine it: 15 int8 products instead of 49.
//     D_i = sum_tap (x mod m_i) * (w f_i mod m_i),   f_i = (M/m_i)^-1 mod m_i,   residues balanced, in [-128, 127]
// is an int32 (|D_i| <= 2^28) congruent to S (M/m_i)^-1, and S = sum_i D_i M/m_i - z M with z = rint(sum_i D_i / m_i).  Three
// neighbouring terms make one exact double, E_t = D_a m_b m_c + D_b m_a m_c + D_c m_a m_b (|E_t| < 2^46), so that
//     S mod p = sum_t E_t (M/M_t mod p) - z (M mod p),   z = rint(sum_t E_t / M_t),   M_t = m_a m_b m_c:
// five exact products and one for z through ONE accumulator (see rns_recombine).  z is exact: |S| / M < 0.15 stays 0.35 away from a tie, and the
// sum's rounding errors are below 2^-25.
//
// A residue of a word takes 2.25 vector instructions (t = rint(x/m) by one FP64 fma whose low mantissa bits are t; x - m t is
// needed modulo 256 only, so the low 16 bits of x and t go through packed 16-bit multiplies, two words at a time), 33 for all of them
// against 8 for the digits: it pays where many channels share them.
// Workgroup: 8 waves, 32 words x 128 channels, all taps.  Every thread turns 4 words of a 64-tap step into residues (B
// fragments in LDS, double-buffered, one barrier per step); wave v does the matrix work of moduli 2v and 2v + 1 for the whole
// tile, so that an A fragment is loaded by one wave only, straight into the registers of the matrix instruction, one step ahead.
// 3136 taps, 256 channels, 2^18 words of 8 primes: 6.7 ms, 8.9 with the digits.  What bounds it, from timings with parts left out: the matrix
// work alone takes 2.6 ms (1.3e15 products/s), with the A fragments 4.4 - 4.9 (96 GB from the L2s at 20 - 22 TB/s; 12 MB per prime, more than
// an L2 holds), words and residues alone 3.9; vector and matrix instructions of a SIMD's two waves overlap by a quarter only
// (8 matrix and 32 FP64 instructions take 103 ns, 58 and 74 apart).  Counters: matrix pipe 0.22, vector ALU 0.39 and LDS 0.28 of the cycles busy (two
// thirds of the LDS's in bank conflicts), 116 GB from the L2s with a hit rate of 0.89.  Slower: 64 words x 64 channels (7.2: twice the residues per product),
// 64 words x 128 channels in two halves of the moduli (7.1: half the A fragments, but every word twice), 1024 threads of
// half the tile each (7.2), 32x32x32 instructions (7.0), half of the waves with the residues first (7.3), A fragments half a step ahead (7.9).
#pragma once

#define MR_NM 15
#define MR_THREADS 512
#define MR_WORDS 32  // words of a workgroup
#define MR_CH 128    // channels
#define MR_CT (MR_CH / 16)
#define MR_WT (MR_WORDS / 16)
#define MR_AFRAG (MR_CT * 64)  // 16-byte fragment chunks per modulus and step
#define MR_BFRAG (MR_WT * 64)
#define MR_CRT 6     // doubles per prime: M/M_t mod p for the 5 groups of three moduli, and -M mod p, balanced

__host__ __device__ constexpr int mr_mod(int i) {
    constexpr int m[MR_NM] = {256, 255, 253, 251, 247, 241, 239, 233, 229, 227, 223, 217, 211, 199, 197};
    return m[i];
}
// f_i = (M/m_i)^-1 mod m_i
__host__ __device__ constexpr int mr_fold(int i) {
    const int m = mr_mod(i);
    int r = 1;
    for (int j = 0; j < MR_NM; j++)
        if (j != i) r = r * mr_mod(j) % m;
    for (int f = 1; f < m; f++)
        if (r * f % m == 1) return f;
    return 0;
}

#ifdef CKKSMI_EMULATE
// x - m*t in both 16-bit halves
static inline unsigned mr_submul16(unsigned x, unsigned t, unsigned m) {
    return (((x >> 16) - (t >> 16) * m) << 16) | (((x & 0xffffu) - (t & 0xffffu) * m) & 0xffffu);
}
#else
typedef unsigned short mr_us2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned mr_submul16(unsigned x, unsigned t, unsigned m) {
    const unsigned short n = (unsigned short)(0u - m);
    return __builtin_bit_cast(unsigned, __builtin_bit_cast(mr_us2, t) * mr_us2{n, n} + __builtin_bit_cast(mr_us2, x));
}
#endif

// A fragments [limb][step][channel group][modulus][CT][64 lanes] (one thread per 16 taps of one channel), the tap table and the constants of the recombination
__global__ __launch_bounds__(EW_THREADS) void mac_prepare_rns_kernel(const long long *w, v4i *afrag, TapEnt *taps, double *crt, const ModConst *modc, int level,
                                                                     int O, int C, int kh, int kw, int in_rows, int W, int Kb, int Mg) {
    const size_t idx = (size_t)blockIdx.x * EW_THREADS + threadIdx.x;
    const int K = C * kh * kw;
    if (idx < (size_t)Kb * 64) mm_tap_entry((int)idx, (int)idx, K, taps, (size_t)Kb * 64, level, kh, kw, in_rows, W);
    if (idx < (size_t)level) {
        const long long q = (long long)modc[idx].p;
        const double qinv = modc[idx].pinv;
        for (int t = 0; t < MR_CRT; t++) {  // the last one: all moduli
            long long r = t < MR_CRT - 1 ? 1 : -1;
            for (int j = 0; j < MR_NM; j++)
                if (j / 3 != t) r = mm_balanced(r * mr_mod(j), q, qinv);  // |r| < 2^50, times 256
            crt[idx * MR_CRT + t] = (double)r;
        }
    }
    if (idx >= (size_t)level * Kb * Mg * MR_AFRAG) return;
    size_t r = idx;
    const int lane = (int)(r % 64); r /= 64;
    const int ct = (int)(r % MR_CT); r /= MR_CT;
    const int mg = (int)(r % Mg); r /= Mg;
    const int kb = (int)(r % Kb); r /= Kb;
    const int i = (int)r;
    const long long q = (long long)modc[i].p;
    const double qinv = modc[i].pinv;
    const int m = mg * MR_CH + ct * 16 + lane % 16;
    double bal[16];
#pragma unroll
    for (int t = 0; t < 16; t++) {
        const int k = 64 * kb + 16 * (lane / 16) + t;
        bal[t] = (m < O && k < K) ? (double)mm_balanced(w[(size_t)m * K + k], q, qinv) : 0.0;
    }
    v4i *out = afrag + (((size_t)i * Kb + kb) * Mg + mg) * MR_NM * MR_AFRAG + (size_t)ct * 64 + lane;
#pragma unroll
    for (int j = 0; j < MR_NM; j++) {
        const double mod = mr_mod(j), inv = 1.0 / mod, f = mr_fold(j);
        v4i a;
#pragma unroll
        for (int c4 = 0; c4 < 4; c4++) {
            unsigned bytes = 0;
#pragma unroll
            for (int t = 0; t < 4; t++) {
                const double x = bal[4 * c4 + t];
                const double y = fma(-mod, rint(x * inv), x) * f;  // below 2^15
                bytes |= ((unsigned)(int)fma(-mod, rint(y * inv), y) & 0xffu) << (8 * t);
            }
            a[c4] = (int)bytes;
        }
        out[(size_t)j * MR_AFRAG] = a;
    }
}

// Residues of 4 words at 4 neighbouring taps, one dword per modulus.
// x < 2^51 and m >= 197: the quotient's error before rounding is below 2^-9.5, so |x - m t| <= m (1/2 + 2^-9.5) < 128.
__device__ __forceinline__ void mr_residues4(const u64d (&x)[4], unsigned (&res)[MR_NM]) {
    double xd[4];
#pragma unroll
    for (int t = 0; t < 4; t++) xd[t] = u2d(x[t]);
    const unsigned x01 = MM_PERM((unsigned)x[1], (unsigned)x[0], 0x05040100u), x23 = MM_PERM((unsigned)x[3], (unsigned)x[2], 0x05040100u);
#pragma unroll
    for (int i = 0; i < MR_NM; i++) {
        if (mr_mod(i) == 256) {
            res[i] = MM_PERM(x23, x01, 0x06040200u);
            continue;
        }
        unsigned u[4];
#pragma unroll
        for (int t = 0; t < 4; t++) u[t] = (unsigned)__double_as_longlong(fma(xd[t], 1.0 / mr_mod(i), 6755399441055744.0));
        const unsigned r01 = mr_submul16(x01, MM_PERM(u[1], u[0], 0x05040100u), (unsigned)mr_mod(i));
        const unsigned r23 = mr_submul16(x23, MM_PERM(u[3], u[2], 0x05040100u), (unsigned)mr_mod(i));
        res[i] = MM_PERM(r23, r01, 0x06040200u);
    }
}

// S mod p, canonical, from the 15 sums.  The accumulator starts at 3*2^48 p and stays within a quarter of it (|E_t| < 2^45.6,
// |z| < 2^25, constants below p/2), so what a step's rounding drops is at most 2^-53 * 15*2^46 p < p/8 and goes into l exactly.
__device__ __forceinline__ double mr_recombine(const int (&D)[MR_NM], const double *k, double p, double pinv) {
    double e[MR_NM / 3], z = 0.0;
#pragma unroll
    for (int t = 0; t < MR_NM / 3; t++) {
        const double a = mr_mod(3 * t), b = mr_mod(3 * t + 1), c = mr_mod(3 * t + 2);
        e[t] = fma((double)D[3 * t + 2], a * b, fma((double)D[3 * t + 1], a * c, (double)D[3 * t] * (b * c)));
        z = fma(e[t], 1.0 / (a * b * c), z);
    }
    ProductChain s = chain_first(844424930131968.0 * p, e[0], k[0]);
#pragma unroll
    for (int t = 1; t < MR_NM / 3; t++) chain_add(s, e[t], k[t]);
    chain_add(s, rint(z), k[MR_CRT - 1]);
    return canon(chain_value(s, p, pinv), p, pinv);
}

template <bool INTERIOR>
__device__ __forceinline__ void conv_mac_rns_body(const MacMfmaArgs &A, v4i *frag, unsigned mg, unsigned pos, unsigned wb, unsigned lc) {
    constexpr int BUF = MR_NM * MR_BFRAG;  // 16-byte chunks of a B buffer
    const unsigned N = 1u << A.logN;
    const unsigned tid = threadIdx.x, lane = tid & 63, wave = MM_UNIFORM(tid >> 6);
    const unsigned i = lc % (unsigned)A.level;
    const int oyl = (int)(pos / (unsigned)A.Wo), ox = (int)(pos % (unsigned)A.Wo);
    const int iy0 = (A.out_row0 + oyl) * A.stride - A.pad, ix0 = ox * A.stride - A.pad;
    const int origin = (iy0 - A.in_row0) * A.W + ix0;
    const unsigned twoL = 2u * (unsigned)A.level;

    // This thread's word and taps.  16 lanes take the words of one 16-word tile at four taps (128 bytes per tap), the next 16 lanes the
    // same words in the next k-group: a half wave writes its residues to 32 neighbouring chunks (512 bytes).
    const unsigned cw = wave % 2 * 16 + lane % 16, kg = wave / 2 % 2 * 2 + lane / 16 % 2, quad = wave / 4 * 2 + lane / 32;
    const u64d *inw = A.in + (size_t)lc * N + wb * MR_WORDS + cw;
    const TapEnt *tp = A.taps + (INTERIOR ? (size_t)A.Kb * 64 : 0) + 16 * kg + 4 * quad;
    // fragment (modulus, word tile): chunk 16*(tap/16) + word%16, byte tap%16
    unsigned *bdst = (unsigned *)frag + ((cw / 16 * 64 + kg * 16 + cw % 16) * 4 + quad);

    u64d x[4];
    unsigned mask = 0xf;
    TapEnt ent[4];  // of the step whose words are requested next
    auto entries = [&](int kb) {
#pragma unroll
        for (int t = 0; t < 4; t++) ent[t] = tp[(kb < A.Kb ? kb : A.Kb - 1) * 64 + t];
    };
    auto words = [&]() {
        unsigned real = 0;
#pragma unroll
        for (int t = 0; t < 4; t++) {
            const unsigned e = ent[t];
            unsigned row;
            if (INTERIOR) {
                row = e + (unsigned)origin * twoL;
            } else {
                real |= mm_tap_row(A, e, iy0, ix0, origin, row) ? 1u << t : 0u;
            }
            x[t] = inw[(size_t)row << A.logN];
        }
        mask = real;
    };
    auto residues = [&](int buf) {
        unsigned res[MR_NM];
        u64d y[4];
#pragma unroll
        for (int t = 0; t < 4; t++) y[t] = (INTERIOR || ((mask >> t) & 1u)) ? x[t] : 0ull;
        mr_residues4(y, res);
#pragma unroll
        for (int m = 0; m < MR_NM; m++) bdst[(buf * BUF + m * MR_BFRAG) * 4] = res[m];
    };

    // the wave's moduli: 2*wave and 2*wave + 1; the last wave has one
    const bool two = 2 * wave + 1 < MR_NM;
    const v4i *asrc = A.afrag + (((size_t)i * A.Kb * A.Mg + mg) * MR_NM + 2 * wave) * MR_AFRAG + lane;
    const size_t astep = (size_t)A.Mg * MR_NM * MR_AFRAG;
    v4i af[2][MR_CT], acc[2][MR_WT][MR_CT];
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
        for (int ct = 0; ct < MR_CT; ct++) {
            af[j][ct] = (j == 0 || two) ? asrc[j * MR_AFRAG + ct * 64] : v4i{0, 0, 0, 0};
#pragma unroll
            for (int wt = 0; wt < MR_WT; wt++) acc[j][wt][ct] = v4i{0, 0, 0, 0};
        }
    auto matrix = [&](int kb, int buf) {
        const v4i *an = asrc + (size_t)(kb + 1 < A.Kb ? kb + 1 : kb) * astep;
        const v4i *bs = frag + buf * BUF + 2 * wave * MR_BFRAG + lane;
#pragma unroll
        for (int j = 0; j < 2; j++) {
            if (j == 1 && !two) {
                MM_MFMA_ABSENT(MR_WT * MR_CT);
                break;
            }
            v4i b[MR_WT];
#pragma unroll
            for (int wt = 0; wt < MR_WT; wt++) b[wt] = bs[j * MR_BFRAG + wt * 64];
#pragma unroll
            for (int ct = 0; ct < MR_CT; ct++) {
#pragma unroll
                for (int wt = 0; wt < MR_WT; wt++) acc[j][wt][ct] = MM_MFMA(af[j][ct], b[wt], acc[j][wt][ct]);
                af[j][ct] = an[j * MR_AFRAG + ct * 64];
            }
        }
    };
    // Step kb: the matrix work of kb, then the residues of kb + 1, whose words were requested a step ago, then the words of kb + 2.
    // Memory operations complete in order, so the words come after the A fragments of the next step, which then don't wait for them.
    entries(0);
    words();
    entries(1);
    residues(0);
    words();
    entries(2);
    __syncthreads();
    for (int kb = 0; kb < A.Kb; kb++) {
        const int buf = kb & 1;
        matrix(kb, buf);
        residues(buf ^ 1);
        words();
        entries(kb + 3);
        __syncthreads();
    }

    // the 15 sums of an output word meet in LDS, 16 channels at a time (two buffers, one barrier each)
    const double p = A.modc[i].p, pinv = A.modc[i].pinv;
    const double *k = A.crt + i * MR_CRT;
    const size_t ctw = (size_t)2 * A.level * N, mstride = (size_t)A.out_rows * A.Wo * ctw;
    const unsigned ch = tid / MR_WORDS, word = tid % MR_WORDS;
    u64d *outp = A.out + ((size_t)oyl * A.Wo + ox) * ctw + (size_t)lc * N + wb * MR_WORDS + word;
#pragma unroll
    for (int c16 = 0; c16 < MR_CT; c16++) {
        int *sums = (int *)(frag + (c16 & 1) * BUF);  // [modulus][16 channels][32 words]
#pragma unroll
        for (int j = 0; j < 2; j++)
            if (j == 0 || two)
#pragma unroll
                for (int wt = 0; wt < MR_WT; wt++)
#pragma unroll
                    for (int r = 0; r < 4; r++) sums[((2 * wave + j) * 16 + lane / 16 * 4 + r) * MR_WORDS + wt * 16 + lane % 16] = acc[j][wt][c16][r];
        __syncthreads();
        const int m = (int)(mg * MR_CH + c16 * 16 + ch);
        if (m < A.O) {
            int D[MR_NM];
#pragma unroll
            for (int t = 0; t < MR_NM; t++) D[t] = sums[(t * 16 + ch) * MR_WORDS + word];
            outp[(size_t)m * mstride] = d2u(mr_recombine(D, k, p, pinv));
        }
    }
}

// grid and order of the workgroups as conv_mac_mfma_kernel
__global__ __launch_bounds__(MR_THREADS, 2) void conv_mac_rns_kernel(MacMfmaArgs A) {
    __shared__ v4i frag[2 * MR_NM * MR_BFRAG];
    const unsigned N = 1u << A.logN;
    const size_t per_xcd = A.total_wgs / 8;
    size_t v = (size_t)(blockIdx.x % 8u) * per_xcd + blockIdx.x / 8u;
    if (v >= A.real_wgs) return;  // uniform for the workgroup
    const unsigned mg = (unsigned)(v % (unsigned)A.Mg); v /= (unsigned)A.Mg;
    const unsigned pos = (unsigned)(v % A.positions); v /= A.positions;
    const unsigned wb = (unsigned)(v % (N / MR_WORDS)); v /= (N / MR_WORDS);
    const unsigned lc = (unsigned)v;
    if (mm_position(A, pos).interior)
        conv_mac_rns_body<true>(A, frag, mg, pos, wb, lc);
    else
        conv_mac_rns_body<false>(A, frag, mg, pos, wb, lc);
}
