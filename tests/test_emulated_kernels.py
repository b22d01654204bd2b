"""The library's kernel sources, compiled against the CPU stand-in under tests/emu
and run fibre by fibre on tiny shapes with guard pages behind every buffer, compared
with the oracle.  This checks indexing and launch shapes on the CPU before a GPU ever
runs them; the parity claims themselves come from the GPU tests."""
import ctypes
import itertools

import numpy as np
import pytest

import parity_cases as pc
from paper_1911_11377_amd import ckksmi

# (logN, n_q, q_bits, k, special_bits, alpha)
TINY = (6, 3, 30, 1, 31, 1)
HYBRID = (5, 5, 40, 2, 41, 2)
HYBRID3 = (4, 7, 50, 3, 51, 3)
TWO_PASS = (13, 2, 50, 1, 51, 1)


@pytest.fixture(scope="module")
def be():
    return pc.EmuBackend()


@pytest.mark.parametrize("shape", [TINY, (2, 2, 20, 1, 21, 1), (9, 2, 50, 1, 51, 1), (12, 1, 40, 1, 41, 1), TWO_PASS,
                                   (14, 1, 50, 1, 51, 1), (16, 1, 50, 1, 51, 1), (16, 2, 30, 0, 31, 1)])
def test_emulated_ntt(be, shape):
    pc.case_ntt(be, shape, seed=100)


def test_emulated_inverse_of_hard_words(be):
    with be.tuned(64):
        pc.case_inverse_hard_words(be, seed=217)


@pytest.mark.parametrize("shape", [TINY, HYBRID3])
def test_emulated_elementwise(be, shape):
    pc.case_elementwise(be, shape, seed=101)


@pytest.mark.parametrize("shape", [TINY, HYBRID])
def test_emulated_rescale(be, shape):
    pc.case_rescale(be, shape, seed=102)


@pytest.mark.parametrize("shape,levels", [(TINY, [3, 1]), (HYBRID, [5, 4, 3]), (HYBRID3, [7, 5, 2])])
def test_emulated_relin_and_composite(be, shape, levels):
    pc.case_relin_and_composite(be, shape, seed=103, levels=levels)


def test_emulated_relin_small_workspace(be):
    pc.case_relin_and_composite(be, HYBRID, seed=104, batch=3, levels=[5], small_ws=True)


def test_emulated_two_pass_composite(be):
    pc.case_relin_and_composite(be, TWO_PASS, seed=105, batch=1, levels=[2])


@pytest.mark.parametrize("shape,level", [(TINY, 3), (HYBRID3, 5)])
def test_emulated_rotate(be, shape, level):
    pc.case_rotate(be, shape, seed=106, rotations=[1, 3, 7], batch=4, level=level)


def test_emulated_rotate_register_tiled_sizes(be):
    """2^12 <= N: no rotated copy is written; the inverse row pass and the fused inner product read c1 and c0 through the
    automorphism (rows of pairs); several items per workgroup, partial last digit"""
    pc.case_rotate(be, (12, 3, 50, 2, 51, 2), seed=126, rotations=[1, 3, 700], batch=3, level=3)
    with be.tuned(8):
        pc.case_rotate(be, (13, 2, 51, 1, 51, 1), seed=127, rotations=[5, 2047, 4095], batch=4, level=2)


def test_emulated_conv(be):
    pc.case_conv(be, TINY, seed=107, Cin=2, H=5, W=5, Oc=9, kh=3, stride=2, pad=0)
    pc.case_conv(be, TINY, seed=108, Cin=1, H=4, W=4, Oc=2, kh=3, stride=1, pad=1, level=2)


def test_emulated_conv_matrix_cores(be):
    """the three matrix-core kernels: strips shared by 2 x 2 and 1 x 4 positions, weight digits resident, weight digits
    streaming; full and quad steps, two channel groups (the second mostly empty), zero padding, a 51-bit prime, strips of rows"""
    pc.case_conv(be, (6, 2, 51, 0, 52, 1), seed=115, Cin=3, H=3, W=3, Oc=34, kh=5, stride=1, pad=2)     # 75 taps: full + quad step
    pc.case_conv(be, (6, 1, 50, 0, 51, 1), seed=116, Cin=4, H=5, W=5, Oc=8, kh=5, stride=1, pad=0, rows_check=False)    # 100 taps
    # 261 taps: more steps than stay in LDS, the streaming kernel; its FC part has 87 taps (two full steps)
    pc.case_conv(be, (6, 1, 50, 0, 51, 1), seed=117, Cin=29, H=3, W=3, Oc=8, kh=3, stride=1, pad=1, rows_check=False)
    # one output row of five positions: the four waves take 1 x 4 positions (two tiles, three waves without a position)
    pc.case_conv(be, (6, 1, 50, 0, 51, 1), seed=119, Cin=2, H=3, W=7, Oc=8, kh=3, stride=1, pad=0, fc_check=False)
    # stride 2 with padding, 5 x 5 outputs (waves without a position in both directions), strips of rows that end inside a
    # 2 x 2 block: the rows below the strip are neither read nor written
    pc.case_conv(be, (6, 1, 50, 0, 51, 1), seed=123, Cin=3, H=9, W=9, Oc=8, kh=3, stride=2, pad=1, fc_check=False)
    # a workgroup walks several tiles / positions: the double-buffered strip, the request for the next position's words
    with be.tuned(2):
        pc.case_conv(be, (6, 1, 50, 0, 51, 1), seed=120, Cin=3, H=7, W=6, Oc=8, kh=5, stride=1, pad=1, fc_check=False)    # 2 x 2 blocks, 20 positions
        pc.case_conv(be, (6, 1, 50, 0, 51, 1), seed=121, Cin=2, H=3, W=13, Oc=8, kh=3, stride=1, pad=0, rows_check=False, fc_check=False)    # 1 x 4 blocks, three tiles
        # 7 x 3 x 3 = 63 taps at stride 3: the window block (7*3*12 lines) is too wide to stage, weight digits resident, six positions
        pc.case_conv(be, (6, 1, 50, 0, 51, 1), seed=122, Cin=7, H=4, W=16, Oc=9, kh=3, stride=3, pad=1, fc_check=False)


def test_emulated_conv_residues(be):
    """the matrix-core kernel on residues: 449 taps end in a step of one tap, 385 in seven steps; ragged channel groups, padding with a strip
    of rows, 51-bit primes at the largest sum; its rule's other side (as many taps, too few channels) stays on digits"""
    with be.tuned(8):
        pc.case_conv_channels(be, (6, 2, 51, 0, 52, 1), 210, 449, 1, 1, 97, 1, 1, 0, residues=True)
        pc.case_conv_channels(be, (6, 1, 50, 0, 51, 1), 211, 43, 3, 3, 98, 3, 2, 1, residues=True, rows=(1, 2))
        pc.case_conv_channels(be, (6, 1, 51, 0, 52, 1), 212, 385, 1, 1, 193, 1, 1, 0, residues=True, extreme=True)
        pc.case_conv_channels(be, (6, 1, 50, 0, 51, 1), 213, 449, 1, 1, 96, 1, 1, 0, residues=False)
        pc.case_conv_channels(be, (6, 1, 50, 0, 51, 1), 214, 384, 1, 1, 97, 1, 1, 0, residues=False)


@pytest.mark.parametrize("layer", pc.PADDED_LAYERS)
def test_emulated_padded_layers_of_high_images(be, layer):
    """(with the bounds of the caller's buffers guarded)"""
    with be.tuned(8):
        pc.case_padded_layer(be, layer, seed=218)


def test_emulated_padded_layer_of_a_wide_image(be):
    pc.case_padded_layer(be, pc.WIDE_LAYER, seed=219)


def test_emulated_pooling(be):
    """(whole networks: the Table-1-like one below; the square-activation network runs on the GPU)"""
    pc.case_pool(be, TINY, seed=112, Cin=2, H=5, W=4, k=2)
    pc.case_pool(be, TINY, seed=113, Cin=1, H=3, W=3, k=3, level=2)
    pc.case_pool(be, TINY, seed=120, Cin=2, H=3, W=2, k=2, pad=1)


def test_emulated_table1_like_network(be):
    """the layer kinds of Table 1 with the degree-2 activation and a padded pooling (the full sequence runs on the GPU)"""
    pc.case_cnn(be, (6, 8, 50, 2, 51, 2), seed=121, topology="table1_tiny")


def test_emulated_item_loop_and_composite_at_2e16(be):
    """N = 2^16: both register-tiled passes, with workgroups looping over several items"""
    with be.tuned(16):
        pc.case_ntt(be, (16, 1, 50, 1, 51, 1), seed=109, batch=3)
        pc.case_ntt(be, (13, 2, 50, 1, 51, 1), seed=110, batch=3)
        pc.case_relin_and_composite(be, (16, 2, 50, 1, 51, 1), seed=111, batch=2, levels=[2])


def test_emulated_fused_hybrid_at_2e16(be):
    """N = 2^16 with 3-prime digits: fused ModUp / inner product / ModDown / rescale kernels, partial last digit"""
    with be.tuned(64):
        pc.case_relin_and_composite(be, (16, 4, 50, 3, 51, 3), seed=112, batch=2, levels=[4, 2])
        pc.case_rescale(be, (16, 3, 50, 0, 51, 1), seed=113, batch=2, levels=[3])


@pytest.mark.parametrize("logN", [12, 13, 14, 15])
def test_emulated_fused_path_other_sizes(be, logN):
    """2^12 <= N < 2^16: general column geometry (N1 = 16, 32, 64, 128), 40-, 50- and 51-bit primes"""
    with be.tuned(8):
        pc.case_ntt(be, (logN, 2, 50, 1, 51, 1), seed=116, batch=3)
        pc.case_relin_and_composite(be, (logN, 3, 50, 2, 51, 2), seed=117, batch=2, levels=[3, 2])
        pc.case_relin_and_composite(be, (logN, 2, 40, 1, 41, 1), seed=118, batch=1, levels=[2])


@pytest.mark.parametrize("shape,levels", [(TINY, [3, 2]), (HYBRID, [5, 4, 2]), (HYBRID3, [7, 5, 2])])
def test_emulated_merged_product_small_sizes(be, shape, levels):
    """one division by P*q_last, exact form: elementwise conversion with the double-precision overshoot"""
    pc.case_merged_product(be, shape, seed=121, levels=levels)
    if shape == HYBRID:
        pc.case_merged_product(be, shape, seed=122, batch=3, levels=[5], small_ws=True)


def test_emulated_merged_product_at_2e16(be):
    """the fused form: conversion kernel over {q_last, p_0, p_1, p_2} with the overshoot taken from the source registers"""
    with be.tuned(64):
        pc.case_merged_product(be, (16, 4, 50, 3, 51, 3), seed=123, batch=2, levels=[4, 2], expect_kernel="modup_cols_kernel<4, 4, 2>")


@pytest.mark.parametrize("logN", [13, 14, 15])
def test_emulated_merged_product_other_sizes(be, logN):
    with be.tuned(8):
        pc.case_merged_product(be, (logN, 3, 50, 2, 51, 2), seed=125, batch=2, levels=[3, 2])


@pytest.mark.parametrize("shape,level", [(TINY, 3), (HYBRID, 4), (HYBRID3, 5)])
def test_emulated_hoisted_rotations_small_sizes(be, shape, level):
    pc.case_rotate_hoisted(be, shape, seed=126, rotations=(1, 3, 6), level=level)
    if shape == HYBRID:
        pc.case_rotate_hoisted(be, shape, seed=127, rotations=(2, 5), level=5, small_ws=True)


def test_emulated_hoisted_rotations_at_2e13(be):
    """register-tiled sizes: shared ModUp through the fused conversion kernels, gathered inner product"""
    pc.case_rotate_hoisted(be, (13, 3, 50, 2, 51, 2), seed=128, rotations=(1, 100, 4095), batch=2, level=3)
    # more items than one workgroup stages (64 KiB of LDS: 32 digit rows), ragged last chunk; N = 256: a single run
    pc.case_rotate_hoisted(be, (9, 9, 40, 1, 41, 1), seed=129, rotations=(1, 77), batch=5, level=9)
    pc.case_rotate_hoisted(be, (8, 2, 40, 1, 41, 1), seed=130, rotations=(3,), batch=2, level=2)
    # more digits than the LDS-staged gather takes: the plain gather kernel; and a ring below 256 words
    pc.case_rotate_hoisted(be, (8, 17, 40, 1, 41, 1), seed=138, rotations=(2,), batch=1, level=17)


def test_emulated_sum_of_products(be):
    """lazy relinearisation: the tensor kernels accumulate the terms (elementwise kernel, and the one fused with the row pass)"""
    pc.case_sum_of_products(be, HYBRID, seed=131, terms=3, levels=[5, 2])
    pc.case_sum_of_products(be, (13, 3, 50, 2, 51, 2), seed=132, terms=4, batch=2, levels=[3])


def test_emulated_rotation_packed_layers(be):
    """single-image packing: a dense layer (every diagonal, two chunks of rotations) and a sparse convolution matrix"""
    from paper_1911_11377_amd import packed, workloads as wl
    pc.case_packed_layer(be, (6, 3, 40, 2, 41, 2), 134, wl.weights_float((32, 20), 134, "fc"))
    pc.case_packed_layer(be, (6, 3, 40, 2, 41, 2), 134, wl.weights_float((32, 20), 134, "fc"), max_rotations=7)  # five calls, ragged last
    w = wl.weights_float((2, 2, 3, 3), 135, "conv")
    pc.case_packed_layer(be, (7, 3, 40, 1, 41, 1), 135, packed.conv_matrix(w, 4, 4, 1))


@pytest.mark.parametrize("shape,log_scale", [(TINY, 30), ((2, 2, 20, 1, 21, 1), 12), ((12, 2, 50, 1, 51, 1), 40), ((13, 2, 50, 1, 51, 1), 45)])
def test_emulated_device_encode_and_encrypt(be, shape, log_scale):
    """one-pass and two-pass complex inverse transform, rounding, residues; encryption with supplied randomness"""
    pc.case_encode_encrypt_device(be, shape, seed=136, batch=2, log_scale=log_scale)
    if shape == TINY:
        pc.case_encode_encrypt_device(be, shape, seed=137, batch=3, level=2, log_scale=25, complex_slots=False, small_ws=True)
    if shape[0] == 12:
        # the fused encryption (column pass from the small coefficients, row pass forming the ciphertext): 51-bit primes,
        # workgroups looping over items, a level below the top, the batch swept in chunks
        with be.tuned(2):
            pc.case_encode_encrypt_device(be, (12, 3, 51, 1, 51, 1), seed=138, batch=3, level=2, log_scale=40, small_ws=True)
            pc.case_encode_encrypt_device(be, (12, 3, 51, 1, 51, 1), seed=139, batch=5, log_scale=40)


def test_emulated_device_sampler(be):
    pc.case_sample_device(be, TINY, seed=0x1234567890ABCDEF)
    pc.case_sample_device(be, (9, 2, 50, 1, 51, 1), seed=3, rows=2, sigma=1.5, first_index=0)


def test_emulated_variant_entry_points_refuse_bad_arguments(be):
    pc.case_variant_errors(be)


def test_emulated_misaligned_device_pointer_is_rejected(be):
    """device buffers must be 16-byte aligned (vector accesses of two words): an odd word offset is refused on the host"""
    shape = TINY
    ctx = be.context(*shape)
    N, level = 1 << shape[0], shape[1]
    a = be.empty(1 + 2 * level * N)
    out = be.empty(2 * (level - 1) * N)
    ws = be.ws(ctx.workspace_bytes(ckksmi.OP_RESCALE, level, 1))
    with pytest.raises(ckksmi.CkksmiError) as e:
        ctx.rescale(a[1:], out, level, 1, ws, stream=be.stream)
    assert e.value.code == ckksmi.EINVAL
    ctx.close()



FEW_PAIRS = (("qm1", "qm1"), ("half_lo", "half_hi"), ("alt", "qm1"), ("onehot", "alt_halves"))


@pytest.mark.parametrize("shape", [TINY, HYBRID, HYBRID3, (5, 9, 51, 2, 51, 2)])
def test_emulated_edge_values_generic_kernels(be, shape):
    """all-0, all-(q-1), (q-1)/2, (q+1)/2, alternating and one-hot residues, seeded key and all-(q-1) key, through every
    operation (generic kernels)"""
    pc.case_edge_values(be, shape, seed=140)


@pytest.mark.parametrize("shape,level,seeded", [((13, 24, 50, 3, 51, 3), 24, False), ((13, 15, 51, 3, 51, 3), 15, True)])
def test_emulated_edge_values_register_tiled_kernels(be, shape, level, seeded):
    """the same at a register-tiled size with 3-prime digits: 8 digits of 50-bit primes (eight terms meet in the fused inner
    product's accumulators before their one reduction; key of all q-1) and 5 digits of 51-bit primes (reduced every four
    terms; both keys).  Two operand pairs each: the GPU suite runs the full set."""
    pc.case_edge_values(be, shape, seed=142, level=level, conv=False, pairs=FEW_PAIRS[:2], seeded_key=seeded)


def test_emulated_edge_values_matrix_core_mac(be):
    pc.case_edge_values(be, (7, 2, 51, 0, 52, 1), seed=143)
    pc.case_edge_values(be, (7, 3, 50, 1, 51, 1), seed=144)


def test_emulated_activation_schedule_register_tiled(be):
    """x^2 then the degree-3 polynomial at N = 2^13 with 3-prime digits: the scalar rescale reads its input one level up and
    adds onto the output buffer; workspace carved by the call sequence; every item compared"""
    pc.case_activation(be, (13, 6, 50, 3, 51, 3), seed=145, level=6, batch=3, sample=[0, 1, 2])


def test_emulated_grouped_plaintext_products(be):
    pc.case_plain_mac(be, TINY, seed=160)
    pc.case_plain_mac(be, (5, 4, 50, 1, 51, 1), seed=161, n_ct=3, level=3)


def test_emulated_single_image_network_baby_and_giant_steps(be):
    """the same network with baby and giant steps: period 64 with two input ciphertexts (baby 8), period 128 with one"""
    pc.case_packed_network(be, (7, 8, 50, 2, 51, 2), seed=152, topology="single_image_tiny", max_rotations=5, bsgs=True)
    pc.case_packed_network(be, (8, 8, 50, 2, 51, 2), seed=153, topology="single_image_tiny", bsgs=True)


def test_emulated_single_image_network(be):
    """one image in the rotation-packed layout: strided convolution, activation, pooling merged into the next layer; with 64
    slots the input spans two ciphertexts (block matrix), with 128 one; rotations in calls of at most 5 in the first run"""
    pc.case_packed_network(be, (7, 8, 50, 2, 51, 2), seed=150, topology="single_image_tiny", max_rotations=5)
    pc.case_packed_network(be, (8, 8, 50, 2, 51, 2), seed=151, topology="single_image_tiny")


@pytest.mark.parametrize("logN,bits", [(12, 50), (13, 51), (14, 50), (15, 51), (16, 50), (16, 51)])
@pytest.mark.parametrize("tuned", [512, 8])
def test_emulated_one_source_division(be, logN, bits, tuned):
    """rescale, rescale of a scalar multiple (with a drop and an addend) on the kernel that keeps the converted limb on chip:
    every block size, coarse blocks (8 workgroups are enough) and fine ones (512), 50- and 51-bit reduction schedules"""
    shape = (logN, 3, bits, 0, 51, 1)
    with be.tuned(tuned):
        # (512: four limbs are a round at N = 2^16, two enough at 2^14; a level of 2 with one item has two)
        pc.case_rescale(be, shape, seed=140 + logN, batch=1 if logN > 14 or tuned > 8 else 5, levels=[3, 2],
                        **({"expect": ["conv_final_kernel"], "absent": ["modup_cols_kernel<%d, 1, 1>" % (logN - 12)]} if logN <= 14 or tuned == 8 else {}))


@pytest.mark.parametrize("shape,batch", [((12, 5, 51, 2, 51, 2), 2), ((12, 4, 50, 1, 51, 1), 9), ((12, 7, 50, 3, 51, 3), 1), ((13, 3, 50, 1, 51, 1), 3), ((12, 6, 50, 4, 51, 4), 1)])
def test_emulated_key_switch_on_chip(be, shape, batch):
    """lifted limbs that never leave their workgroup: digits cut short by the level, one to four sources, halves of a 2^13 ring, items
    that do not divide evenly over the XCDs; products, sums of products, relinearisation and rotations"""
    with be.tuned(64):
        level = shape[1]
        pc.case_relin_and_composite(be, shape, seed=170, batch=batch, levels=[level, level - 1], expect=["inner_wg_kernel"], absent=["rows_inner_kernel"])
        pc.case_rotate(be, shape, seed=171, rotations=[1, 1000], batch=batch, level=level - 1, expect=["inner_wg_kernel"], absent=["rows_inner_kernel"])
        pc.case_sum_of_products(be, shape, seed=172, terms=3, batch=1, levels=[level])


@pytest.mark.parametrize("shape,batch", [((12, 4, 51, 3, 51, 3), 2), ((12, 3, 50, 1, 51, 1), 1), ((13, 3, 51, 1, 51, 1), 2), ((14, 3, 50, 1, 51, 1), 1)])
def test_emulated_tail_on_chip(be, shape, batch):
    """ModDown followed by rescale without an intermediate: one to three special primes, whole rings and halves"""
    with be.tuned(64):
        pc.case_relin_and_composite(be, shape, seed=180, batch=batch, levels=[shape[1], 2], expect=["tail_sources_kernel", "conv_final_kernel"])


@pytest.mark.parametrize("shape,batch", [((12, 12, 50, 0, 51, 1), 9), ((13, 8, 51, 0, 52, 1), 9), ((12, 3, 50, 0, 51, 1), 17)])
def test_emulated_one_source_division_uneven_rows(be, shape, batch):
    """rows that do not divide evenly over the XCDs: few with many kept limbs (all taken in turn), few with few limbs and more of
    them (dealt to the XCDs, the last row of some missing)"""
    pc.case_rescale(be, shape, seed=150, batch=batch, levels=[shape[1]])


def test_emulated_division_route(be):
    """rescale and rescale of a scalar multiple at one size take the same kernels, also at N = 2^16"""
    with be.tuned(512):  # four kept limbs are enough
        pc.case_division_route(be, (16, 3, 50, 0, 51, 1), seed=155, batch=1, level=3, one_kernel=True)
        pc.case_division_route(be, (15, 3, 51, 0, 52, 1), seed=156, batch=1, level=3, one_kernel=True)
        pc.case_division_route(be, (15, 3, 51, 0, 52, 1), seed=157, batch=1, level=2, one_kernel=False)


def test_emulated_division_route_last_round(be):
    """N = 2^16: a last round of workgroups that is nearly empty keeps the pair of kernels; with a single kept limb a row also one
    that is half full"""
    with be.tuned(2048):  # sixteen kept limbs are a round
        pc.case_division_route(be, (16, 4, 50, 0, 51, 1), seed=158, batch=3, level=4, one_kernel=False, sample=[2])  # 18
    with be.tuned(512):  # four
        pc.case_division_route(be, (16, 2, 50, 0, 51, 1), seed=159, batch=3, level=2, one_kernel=False, sample=[2])  # 6
        pc.case_division_route(be, (16, 2, 50, 0, 51, 1), seed=160, batch=4, level=2, one_kernel=True, sample=[3])   # 8


def test_emulated_tail_route(be):
    """N = 2^14: ModDown followed by rescale goes on chip only with enough kept limbs a row"""
    with be.tuned(128):  # one row, three kept limbs
        pc.case_product_route(be, (14, 3, 50, 1, 51, 1), seed=185, batch=1, level=3, expect=["conv_final_kernel"], absent=["modup_cols_kernel<2, 2, 3>"])
        pc.case_product_route(be, (14, 3, 50, 1, 51, 1), seed=186, batch=1, level=2, expect=["modup_cols_kernel<2, 2, 3>"], absent=["conv_final_kernel"])


@pytest.mark.parametrize("shape,which", [((12, 3, 50, 1, 51, 1), 0), ((13, 3, 50, 1, 51, 1), 1), ((14, 3, 50, 1, 51, 1), 2)])
def test_emulated_missing_kernel_is_an_error(be, shape, which):
    """a launch sequence that asks for a kernel which was not built makes the call fail; the next call of the context runs"""
    ctx = be.context(*shape)
    assert be.lib.emu_probe_missing_kernel(ctx._h, which) == ckksmi.EUNSUPPORTED
    assert be.lib.emu_probe_missing_kernel(ctx._h, -1) == 0
    ctx.close()


def test_emulated_profile_names_the_kernels_that_run(be):
    """N = 2^12: the on-chip key switch and tail report their own kernels, the two-kernel forms theirs"""
    chip = ["inner_wg_kernel", "conv_final_kernel"]
    with be.tuned(64):
        pc.case_product_route(be, (12, 3, 50, 1, 51, 1), seed=190, batch=1, level=3, expect=chip + ["tensor_wg_kernel", "tail_sources_kernel"],
                              absent=["tensor_rows_kernel", "ntt_wg_kernel"])
        pc.case_rotate(be, (12, 3, 50, 1, 51, 1), seed=191, rotations=[1], batch=1, level=3, expect=chip + ["ntt_wg_inv_gal_kernel", "ntt_wg_kernel"],
                       absent=["ntt_v2_kernel<true, false>"])
    pc.case_product_route(be, (12, 3, 50, 3, 51, 3), seed=192, batch=1, level=3,
                          expect=["tensor_rows_kernel", "modup_cols_kernel<0, 3, 0>", "rows_inner_kernel", "modup_cols_kernel<0, 4, 3>", "rows_final_kernel"],
                          absent=chip + ["tensor_wg_kernel", "tail_sources_kernel"])


def test_emulated_merged_product_on_chip(be):
    """the accumulators of the on-chip key switch left as they are for the merged division"""
    with be.tuned(64):
        pc.case_product_route(be, (12, 3, 50, 1, 51, 1), seed=193, batch=2, level=3, merged=True, expect=["inner_wg_kernel", "modup_cols_kernel<0, 2, 2>"])


@pytest.mark.parametrize("logN,bits,tuned", [(14, 50, 1024), (15, 51, 512), (15, 50, 1024), (16, 51, 512)])
def test_emulated_rotation_division_on_chip(be, logN, bits, tuned):
    """ModDown with one special prime at the large rings, halves (512) and quarters (1024, N = 2^16) of a limb: a rotation, and two
    from a shared ModUp whose last step reads sigma(c0) through the automorphism"""
    names = {"expect": ["conv_final_kernel"], "absent": ["modup_cols_kernel<%d, 1, 1>" % (logN - 12)]}
    with be.tuned(tuned):
        pc.case_rotate(be, (logN, 2, bits, 1, 51, 1), seed=194, rotations=[5, 1000], batch=2, level=2, **names)
        pc.case_rotate_hoisted(be, (logN, 2, bits, 1, 51, 1), seed=195, rotations=(3, 700), batch=1, level=2, **names)


@pytest.mark.parametrize("shape", [(12, 9, 51, 1, 51, 1), (13, 9, 50, 1, 51, 1)])
def test_emulated_edge_values_on_chip(be, shape):
    """the on-chip key switch and tail on residues at the ends of [0, q), key of all q-1"""
    with be.tuned(64):
        pc.case_edge_values(be, shape, seed=196, conv=False, pairs=FEW_PAIRS[:2], seeded_key=False, expect=["inner_wg_kernel", "tail_sources_kernel"])


def _doubles(values):
    return (ctypes.c_double * len(values))(*[float(v) for v in values])


@pytest.mark.parametrize("terms", [2, 3, 4])
@pytest.mark.parametrize("bits", [40, 50])
def test_product_chain_is_exact_at_the_ends_of_its_range(be, terms, bits):
    """a conversion's sum of products with one reduction: an integer congruent to the exact sum and within its bound"""
    be.lib.emu_probe_product_chain.restype = be.lib.emu_probe_chain_bound.restype = ctypes.c_double
    rng = np.random.default_rng(bits + terms)
    for p in (2**bits - 27, 2 ** (bits - 1) + 9):
        half = p // 2
        ends = [(2**51 - 1, half), (2**51 - 1, -half), (2**51 - 1, half - 1), (0, half), (1, -1), (2**50 - 1, half)]
        cases = list(itertools.product(ends, repeat=terms))
        cases += [[(int(rng.integers(0, 2**51)), int(rng.integers(-half, half + 1))) for _ in range(terms)] for _ in range(500)]
        for c in cases:
            v = be.lib.emu_probe_product_chain(_doubles([y for y, _ in c]), _doubles([w for _, w in c]), terms, ctypes.c_double(p))
            assert v == int(v) and abs(v) <= be.lib.emu_probe_chain_bound(terms) * p
            assert (int(v) - sum(y * w for y, w in c)) % p == 0


def _exact_rounds(x, tw, p, inverse):
    """the rounds of emu_probe_lazy_rounds on integers"""
    x = list(x)
    for _ in range(3 if inverse else 2):
        for s in (range(3, -1, -1) if inverse else range(4)):
            span = 8 >> s
            for b in range(1 << s):
                for lo in range(2 * span * b, 2 * span * b + span):
                    u, v, w = x[lo], x[lo + span], tw[(1 << s) - 1 + b]
                    x[lo], x[lo + span] = ((u + v) % p, (u - v) * w % p) if inverse else ((u + v * w) % p, (u - v * w) % p)
    return x


@pytest.mark.parametrize("inverse", [0, 1])
@pytest.mark.parametrize("p51", [0, 1])
def test_lazy_rounds_stay_exact_from_the_ends_of_their_range(be, p51, inverse):
    """register rounds from words at their entry bound (the largest sums a pass can form), twiddles at +-p/2"""
    be.lib.emu_probe_lazy_rounds.restype = ctypes.c_double
    p = 2 ** (50 + p51) - 27
    entry = 1.25 if inverse else (2.5 if p51 else 3.5)
    top, half = int(entry * p) - 1, p // 2
    rng = np.random.default_rng(p51 * 2 + inverse)
    words = [[top] * 16, [-top] * 16, [top if i % 2 else -top for i in range(16)], [top if i < 8 else -top for i in range(16)]]
    words += [[int(v) for v in rng.integers(-top, top + 1, 16)] for _ in range(40)]
    words += [[int(v) for v in rng.choice([-top, top], 16)] for _ in range(40)]
    for x in words:
        for tw in ([half] * 15, [-half] * 15, [int(v) for v in rng.integers(-half, half + 1, 15)]):
            buf = _doubles(x)
            bound = be.lib.emu_probe_lazy_rounds(p51, inverse, buf, _doubles(tw), ctypes.c_double(p))
            assert all(v == int(v) and abs(v) <= bound * p for v in buf)
            assert [int(v) % p for v in buf] == _exact_rounds(x, tw, p, inverse)


INV_ROW1, INV_ROW2, INV_COL2, INV_COL1, INV_ROW2_12 = range(5)
# (round, first register stage) in the order in which a kernel runs them: a ring of 2^12 words in one workgroup, and as two passes; 2^13 .. 2^16
INV_CHAINS = [[(INV_ROW1, 0), (INV_ROW2_12, 0), (INV_COL1, 0)]] + [[(INV_ROW1, 0), (INV_ROW2, 0), (INV_COL2, 4 - Q), (INV_COL1, 0)] for Q in range(5)]


@pytest.mark.parametrize("chain", INV_CHAINS)
@pytest.mark.parametrize("p51", [0, 1])
def test_inverse_rounds_take_what_the_round_before_leaves(be, p51, chain):
    """every inverse round, the last one with its folded constants too, from words at the bound that the round before it declares: exact, and within
    its own bound.  (The words of a round come from 16 threads' rounds before it, so that all of them can be at the same register's bound.)"""
    probe = be.lib.emu_probe_inv_round
    probe.restype = ctypes.c_double
    p = 2 ** (50 + p51) - 27
    half, rng = p // 2, np.random.default_rng(p51)
    bound = 1.25  # a product of two canonical words
    for rnd, S0 in chain:
        top = int(bound * p)
        words = [[top] * 16, [-top] * 16, [top - 1] * 15 + [top], [top if i % 2 else -top for i in range(16)], [top if i < 8 else -top for i in range(16)]]
        words += [[int(v) for v in rng.choice([-top, 1 - top, top - 1, top], 16)] for _ in range(40)]
        words += [[top - int(v) for v in rng.integers(0, 2, 16)] for _ in range(40)]
        for x in words:
            for tw in ([half] * 17, [-half] * 17, [int(v) for v in rng.integers(-half, half + 1, 17)]):
                buf = _doubles(x)
                bound = probe(p51, rnd, S0, buf, _doubles(tw[:15]), ctypes.c_double(tw[15]), ctypes.c_double(tw[16]), ctypes.c_double(p))
                want = list(x)
                for s in range(3, S0 - 1, -1):
                    span = 8 >> s
                    for lo in (i for i in range(16) if not i & span):
                        u, v = want[lo] + want[lo + span], want[lo] - want[lo + span]
                        last = rnd == INV_COL1 and s == 0
                        want[lo], want[lo + span] = (u * tw[15], v * tw[16]) if last else (u, v * tw[(1 << s) - 1 + lo // (2 * span)])
                assert all(v == int(v) and abs(v) <= bound * p for v in buf)
                assert all((int(v) - w) % p == 0 for v, w in zip(buf, want))


@pytest.mark.parametrize("bits,p51", [(20, 0), (40, 0), (50, 0), (51, 1)])
def test_canonical_form_around_multiples_of_the_prime(be, bits, p51):
    """words at and next to every multiple of p up to 2.9p, where the quotient's floor changes, and at the ends of the range"""
    probe = be.lib.emu_probe_canon_near
    probe.restype = ctypes.c_double
    rng = np.random.default_rng(bits)
    for p in (2**bits - 27, 2**bits - 2**14 + 1, 2 ** (bits - 1) + 9, 2 ** (bits - 1) + 2**14 + 1):
        top = 29 * p // 10
        words = [k * p + d for k in range(-3, 4) for d in range(-9, 10)] + [k * p // 2 + d for k in range(-5, 6, 2) for d in (-1, 0, 1)]
        words += [top, -top] + [int(v) for v in rng.integers(-top, top + 1, 3000)]
        for x in words:
            if abs(x) <= top:
                assert probe(p51, ctypes.c_double(x), ctypes.c_double(p)) == x % p


@pytest.mark.parametrize("p51", [0, 1])
def test_key_products_stay_exact_at_the_ends_of_their_range(be, p51):
    """key words 0 .. p - 1 times words at the largest bound that a row pass leaves them at, on accumulators at what the terms before can sum to"""
    probe = be.lib.emu_probe_key_term
    probe.restype = be.lib.emu_probe_key_factor.restype = ctypes.c_double
    factor, term, terms = be.lib.emu_probe_key_factor(p51), 0.875 if p51 else 1.33, 4 if p51 else 5
    rng = np.random.default_rng(p51)
    for p in (2 ** (50 + p51) - 27, 2 ** (49 + p51) + 9):
        top = int(factor * p)
        vs = [top, -top, top - 1, 1 - top, p // 2, -(p // 2), 0] + [int(v) for v in rng.integers(-top, top + 1, 40)]
        ks = [p - 1, p - 2, p // 2, p // 2 + 1, 1, 0] + [int(v) for v in rng.integers(0, p, 40)]
        base = int((0.5 + (terms - 1) * term) * p)
        for k, v in itertools.product(ks, vs):
            for a in (0, base, -base):
                got = probe(p51, ctypes.c_double(k), ctypes.c_double(v), ctypes.c_double(a), ctypes.c_double(p))
                assert got == int(got) and abs(got) < 2**53 and abs(int(got) - a) <= term * p
                assert (int(got) - a - k * v) % p == 0


@pytest.mark.parametrize("bits,channels,size,kernel", pc.EXTREME_TAPS)
def test_digit_diagonals_at_their_largest(be, bits, channels, size, kernel):
    """every word p - 1, every weight +-(p - 1) / 2, output channels that end inside a channel group"""
    pc.case_conv_channels(be, (6, 1, bits, 0, bits + 1, 1), 420 + channels, channels, size, size + 1, 35, size, 1, 0, residues=False, extreme=True, kernel=kernel)


@pytest.mark.parametrize("digits,batch", [(1, 13), (2, 5), (3, 11), (4, 1), (5, 7), (6, 6), (7, 3), (8, 9), (9, 2)])
def test_shared_rotations_for_every_number_of_digits(be, digits, batch):
    """items that end inside a group of four and inside a workgroup's share, one and several rotations"""
    pc.case_rotate_hoisted(be, (8, digits, 40, 1, 41, 1), seed=440 + digits, rotations=[1, 5, 100], batch=batch)


@pytest.mark.parametrize("digits,batch", [c for c in pc.GATHERED_DIGITS if c[0] in (1, 3, 5, 6, 8, 9, 12, 16)])
def test_shared_rotations_several_per_workgroup(be, digits, batch):
    """the next rotation's key words are requested while this one's sums run, over several groups of items"""
    pc.case_several_rotations_per_workgroup(be, 8, 40, digits, batch)


def test_coefficients_become_residues_exactly(be):
    """the remainder of one floating-point reduction for coefficients up to 4e18, where the quotient by the smallest primes has 49 bits: at and next to
    multiples of p and of p / 2, as far as a double can be there"""
    probe = be.lib.emu_probe_real_word
    probe.restype = ctypes.c_double
    rng = np.random.default_rng(70)
    for p in (2**13 + 1, 12289, 40961, 2**20 + 7, 2**40 - 87, 2**50 - 27, 2**50 + 31, 2**51 - 129):
        near = [k * p // 2 + d for k in [1, 2, 3] + [int(x) for x in rng.integers(1, 8 * 10**18 // p, 1500)] for d in (-1, 0, 1)]
        for m in near + [int(x) for x in rng.integers(0, 4 * 10**18, 1500)] + [0, 4 * 10**18 - 512]:
            for v in (float(m), -float(m)):
                if abs(v) < 4e18:
                    largest = ctypes.c_double(0.0)
                    r = probe(ctypes.c_double(v), ctypes.c_double(1.0), ctypes.c_double(p), ctypes.byref(largest))
                    assert r == int(r) and abs(r) <= 0.63 * p and (int(r) - int(v)) % p == 0 and largest.value == abs(v)
    for v in (4e18, -5e18, float("inf"), float("-inf"), float("nan")):
        largest = ctypes.c_double(1.0)
        probe(ctypes.c_double(v), ctypes.c_double(1.0), ctypes.c_double(40961.0), ctypes.byref(largest))
        assert not largest.value < 4e18


@pytest.mark.parametrize("shape,batch", [((12, 2, 40, 0, 41, 1), 2), ((14, 1, 50, 0, 51, 1), 2), ((15, 1, 51, 0, 52, 1), 1)])
def test_encodings_that_are_too_large_are_refused(be, shape, batch):
    pc.case_encode_refusals(be, shape, batch)


def test_encodings_in_batches_and_one_by_one(be):
    """N = 2^14: 64 limbs take the whole-limb kernel, one item the two passes"""
    pc.case_encode_batch_against_singles(be, (14, 2, 50, 0, 51, 1), 32)


@pytest.mark.parametrize("logN,widths", [(12, w) for w in pc.MIXED_WIDTHS] + [(13, pc.MIXED_WIDTHS[0]), (14, pc.MIXED_WIDTHS[0])])
def test_chains_of_wide_and_narrow_primes(be, logN, widths):
    pc.case_mixed_widths(be, logN, widths, seed=480)
    if logN == 12:
        with be.tuned(8):  # converted limbs on chip
            pc.case_relin_and_composite(be, pc.mixed_shape(logN, *widths), seed=485, batch=2, levels=[len(widths[0])])


@pytest.mark.parametrize("bits,channels,size,kernel", pc.EXTREME_TAPS)
def test_digit_diagonals_at_extreme_digits(be, bits, channels, size, kernel):
    """words and weights of extreme digits, all taps alike; output channels that end inside a channel group"""
    pc.case_conv_channels(be, (6, 1, bits, 0, bits + 1, 1), 420 + channels, channels, size, size + 1, 35, size, 1, 0, residues=False, digits=True, kernel=kernel)
