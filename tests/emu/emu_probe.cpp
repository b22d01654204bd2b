// The library's device source on the CPU stand-in, with entry points into its launch sequences that no public call has.
#include "../../paper_1911_11377_amd/csrc/ckksmi_device.hip"

// A launch sequence that asks for a kernel which was not built.  which 0: a division with an addend in a form that takes none;
// 1: the register-tiled conversion from one source at N <= 2^13; 2: the on-chip key switch at a size it does not have
extern "C" int emu_probe_missing_kernel(ckksmi_ctx *c, int which) {
    Guard g(c);
    u64 word[2] = {0, 0};
    if (which == 0) launch_conv_final(c, 0, word, 0, c->divround[1], word, 0, word, 0, 0, word, 1, 1, nullptr);
    if (which == 1) launch_modup_cols(c, 1, word, 0, word, 1, 0, 1, &c->divround[1], 1.0, nullptr, c->d_fin_rescale);
    if (which == 2) {
        RowsInnerArgs R;
        KeyTab K;
        memset(&R, 0, sizeof(R));
        memset(&K, 0, sizeof(K));
        launch_inner_wg(c, R, K, word, 1, nullptr, nullptr);
    }
    return g.rc();
}

// Sum of K products as a conversion forms it (y canonical, w balanced, p < 2^50)
extern "C" double emu_probe_product_chain(const double *y, const double *w, int K, double p) {
    ProductChain c = chain_first(chain_origin(p), y[0], w[0]);
    for (int a = 1; a < K; a++) chain_add(c, y[a], w[a]);
    return chain_value(c, p, 1.0 / p);
}
extern "C" double emu_probe_chain_bound(int K) { return chain_bound(K); }

// The register rounds of a pass on 16 words, with their reductions: forward the two of a row pass whose results a pointwise step takes
// as they are, inverse the two of a row pass and the round that follows it in a column pass of 2^8 rows.  Returns the bound at the end.
template <bool P51>
static double probe_rounds(bool inverse, double (&x)[16], const double (&tw)[15], double p) {
    typedef RowMasks<P51, true> Mk;
    const WMul unused{0.0, 0.0};
    if (!inverse) {
        fwd_round<Mk::F1>(x, tw, p, 1.0 / p);
        fwd_round<Mk::F2>(x, tw, p, 1.0 / p);
        return LazyRange<P51>::ROWX;
    }
    inv_stages<0, INV_ROW1, P51>(x, tw, p, 1.0 / p, unused, unused);
    inv_stages<0, INV_ROW2, P51>(x, tw, p, 1.0 / p, unused, unused);
    inv_stages<0, INV_COL2, P51>(x, tw, p, 1.0 / p, unused, unused);
    return LazyRange<P51>::INV1;
}
extern "C" double emu_probe_lazy_rounds(int p51, int inverse, double *x, const double *tw, double p) {
    double xx[16], t[15];
    memcpy(xx, x, sizeof(xx));
    memcpy(t, tw, sizeof(t));
    const double b = p51 ? probe_rounds<true>(inverse != 0, xx, t, p) : probe_rounds<false>(inverse != 0, xx, t, p);
    memcpy(x, xx, sizeof(xx));
    return b;
}

// One inverse register round (an InvRound, from register stage S0 on) on 16 words; returns the bound of what it leaves.  x == nullptr: the bound alone
template <bool P51, InvRound B>
static double probe_inv_round(int S0, double *x, const double *tw, double ninv, double wlast, double p) {
    if (x) {
        double xx[16], t[15];
        memcpy(xx, x, sizeof(xx));
        memcpy(t, tw, sizeof(t));
        const WMul n{ninv, ninv / p}, w{wlast, wlast / p};
        switch (S0) {
            case 0: inv_stages<0, B, P51>(xx, t, p, 1.0 / p, n, w); break;
            case 1: inv_stages<1, B, P51>(xx, t, p, 1.0 / p, n, w); break;
            case 2: inv_stages<2, B, P51>(xx, t, p, 1.0 / p, n, w); break;
            case 3: inv_stages<3, B, P51>(xx, t, p, 1.0 / p, n, w); break;
            default: inv_stages<4, B, P51>(xx, t, p, 1.0 / p, n, w); break;
        }
        memcpy(x, xx, sizeof(xx));
    }
    return inv_exit<P51>(B);
}
template <bool P51>
static double probe_inv_named(int round, int S0, double *x, const double *tw, double ninv, double wlast, double p) {
    switch (round) {
        case INV_ROW1: return probe_inv_round<P51, INV_ROW1>(S0, x, tw, ninv, wlast, p);
        case INV_ROW2: return probe_inv_round<P51, INV_ROW2>(S0, x, tw, ninv, wlast, p);
        case INV_ROW2_12: return probe_inv_round<P51, INV_ROW2_12>(S0, x, tw, ninv, wlast, p);
        case INV_COL2: return probe_inv_round<P51, INV_COL2>(S0, x, tw, ninv, wlast, p);
        default: return probe_inv_round<P51, INV_COL1>(S0, x, tw, ninv, wlast, p);
    }
}
extern "C" double emu_probe_inv_round(int p51, int round, int S0, double *x, const double *tw, double ninv, double wlast, double p) {
    return p51 ? probe_inv_named<true>(round, S0, x, tw, ninv, wlast, p) : probe_inv_named<false>(round, S0, x, tw, ninv, wlast, p);
}

// canonical form of a word of at most 2.9p; one word's term of an inner product with a switching key, on top of a
extern "C" double emu_probe_canon_near(int p51, double x, double p) { return p51 ? canon_near<true>(x, p, 1.0 / p) : canon_near<false>(x, p, 1.0 / p); }
extern "C" double emu_probe_key_term(int p51, double k, double v, double a, double p) {
    double a1 = 0.0;
    if (p51) key_term<true>((u64d)k, (u64d)k, v, p, 1.0 / p, a, a1);
    else key_term<false>((u64d)k, (u64d)k, v, p, 1.0 / p, a, a1);
    return a;
}
extern "C" double emu_probe_key_factor(int p51) { return p51 ? LazyRange<true>::FACTOR : LazyRange<false>::FACTOR; }

// an encoding's coefficient as a residue; the magnitude that it reports
extern "C" double emu_probe_real_word(double v, double factor, double p, double *largest) { return real_word(v, factor, p, 1.0 / p, *largest); }
