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
