"""What the compiler makes of the kernels that address memory through scalar_base (csrc/ntt_v2.h): the assembly for gfx950 of
one instance of each, compiled here without a GPU."""
import os
import re
import subprocess

import pytest

from paper_1911_11377_amd import build as lib_build

KERNELS = ["ntt_wg_kernel<false, 13>(NttV2Args)", "ntt_wg_kernel<true, 14>(NttV2Args)", "conv_final_kernel<14, 1, 1, 0>(ConvFinalArgs)",
           "conv_final_gal_kernel<14, 2, 1>(ConvFinalArgs, RowsFinalGal)", "tail_sources_kernel<13>(TailSourcesArgs)",
           "inner_wg_gal_kernel<12, 0, 3>(InnerWgArgs, KeyTab, GaloisTab)",
           # the streamed instances
           "ntt_wg_kernel<false, 13, true>(NttV2Args)", "ntt_wg_kernel<true, 14, true>(NttV2Args)", "conv_final_kernel<14, 1, 1, 0, true>(ConvFinalArgs)",
           "conv_final_gal_kernel<14, 2, 1, true>(ConvFinalArgs, RowsFinalGal)"]


@pytest.mark.skipif(not os.path.exists(lib_build.HIPCC), reason="no hipcc")
def test_scalar_bases_give_global_accesses(tmp_path):
    """no flat memory access (64-bit vector address each, waited for with the LDS) in any of these kernels"""
    src = tmp_path / "instances.hip"
    heads = ["ckksmi_internal.h", "kernels.h", "ntt_v2.h", "ks_fused.h", "ntt_wg.h", "ks_wg.h", "ks_inner_wg.h"]
    src.write_text("#include <hip/hip_runtime.h>\n" + "".join('#include "%s"\n' % h for h in heads)
                   + "".join("template __global__ void %s;\n" % k for k in KERNELS))
    out = tmp_path / "instances.s"
    flags = [f for f in lib_build.FLAGS if f not in ("-shared", "-fPIC", "-Wall")]
    subprocess.check_call([lib_build.HIPCC] + flags + ["--cuda-device-only", "-S", "-I", lib_build.CSRC, str(src), "-o", str(out)], stderr=subprocess.DEVNULL)
    kernel, flat, glob = None, {}, {}
    for line in out.read_text().splitlines():
        m = re.match(r"(_Z\d+(?:ntt_wg|conv_final|tail_sources|inner_wg)\w*):", line)
        if m:
            kernel = m.group(1)
            flat[kernel] = glob[kernel] = 0
        elif re.match(r"_Z\w+:", line):
            kernel = None
        elif kernel:
            flat[kernel] += bool(re.match(r"\s+flat_(load|store)", line))
            glob[kernel] += bool(re.match(r"\s+global_(load|store)", line))
    assert len(flat) == len(KERNELS), sorted(flat)
    assert not any(flat.values()), flat
    assert all(n >= 16 for n in glob.values()), glob


HEADS = ["ckksmi_internal.h", "kernels.h", "ntt_v2.h", "ks_fused.h", "ntt_wg.h", "ks_wg.h"]
needs_hipcc = pytest.mark.skipif(not os.path.exists(lib_build.HIPCC), reason="no hipcc")


def _assembly(tmp_path, kernels):
    """{mangled name: lines} of the instances, the compiler's own figures behind a kernel's end among them"""
    src, out = tmp_path / "instances.hip", tmp_path / "instances.s"
    src.write_text("#include <hip/hip_runtime.h>\n" + "".join('#include "%s"\n' % h for h in HEADS)
                   + "".join("template __global__ void %s;\n" % k for k in kernels))
    flags = [f for f in lib_build.FLAGS if f not in ("-shared", "-fPIC", "-Wall")]
    subprocess.check_call([lib_build.HIPCC] + flags + ["--cuda-device-only", "-S", "-I", lib_build.CSRC, str(src), "-o", str(out)], stderr=subprocess.DEVNULL)
    kernel, lines = None, {}
    for line in out.read_text().splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            kernel = m.group(1)
        if kernel:
            lines.setdefault(kernel, []).append(line)
    wanted = {k: v for k, v in lines.items() if any(re.match(r"_Z\d+%sI" % k2.split("<")[0], k) for k2 in kernels)}
    assert len(wanted) == len(kernels), sorted(lines)
    return wanted


def _count(lines, pattern):
    return sum(bool(re.match(pattern, line)) for line in lines)


@needs_hipcc
@pytest.mark.parametrize("digits", [9, 16])
def test_gathered_inner_product_has_no_conditions_on_digits(tmp_path, digits):
    """a rotation's key words and an item's staged words are read in straight-line code, whatever the number of digits (with a condition for
    every digit: 137 branches)"""
    (lines,) = _assembly(tmp_path, ["inner_product_hoisted_tile_kernel<8192, %d>(HoistArgs)" % digits]).values()
    assert _count(lines, r"\s+global_load_dwordx4") >= 16 + 2 * digits
    assert _count(lines, r"\s+s_cbranch") <= 48 and _count(lines, r"\s+scratch_") == 0


@needs_hipcc
def test_kept_limbs_are_streamed_where_that_was_faster(tmp_path):
    """word pairs are requested past the caches by the last pass of limbs that the call wrote, not by the one for the caller's words or for scalar multiples"""
    code = _assembly(tmp_path, ["rows_final_kernel<true, false, true>(RowsFinalArgs)", "rows_final_kernel<true, false, false>(RowsFinalArgs)",
                                "rows_final_scalar_kernel<true>(RowsFinalArgs, ScalarTab)"])
    streamed = sorted(("scalar" if "scalar" in k else "plain", _count(v, r"\s+global_load_dwordx4 .* nt")) for k, v in code.items())
    assert streamed == [("plain", 0), ("plain", 16), ("scalar", 0)], streamed  # 8 each for p < 2^50 and p < 2^51


@needs_hipcc
def test_tail_sources_leave_room_for_two_workgroups(tmp_path):
    """N = 2^13: the words in flight do not take the registers of the compute unit's second workgroup (512 threads each: four waves per SIMD)"""
    (lines,) = _assembly(tmp_path, ["tail_sources_kernel<13>(TailSourcesArgs)"]).values()
    occupancy = [int(m.group(1)) for m in (re.match(r"; Occupancy: (\d+)", line) for line in lines) if m]
    assert occupancy == [4], occupancy


@needs_hipcc
def test_forward_transforms_end_as_was_faster(tmp_path):
    """whole limbs from N = 2^13 on: the results are reduced before the exchange, in streamed transforms made canonical behind it (a floor each, for p < 2^50);
    neither spills"""
    code = _assembly(tmp_path, ["ntt_wg_kernel<false, %d, %s>(NttV2Args)" % (n, nt) for n in (12, 13, 14) for nt in ("false", "true")])
    floors = {re.search(r"Li(1\d)ELb([01])", k).groups(): _count(v, r"\s+v_floor_f64") for k, v in code.items()}
    assert floors == {("12", "0"): 16, ("12", "1"): 16, ("13", "0"): 0, ("13", "1"): 16, ("14", "0"): 0, ("14", "1"): 16}, floors
    assert not any(_count(v, r"\s+scratch_") for v in code.values())


@needs_hipcc
def test_last_passes_address_their_words_as_was_faster(tmp_path):
    """the transformed words of a division without an addend come from scalar bases, those of scalar multiples by addresses of their own"""
    code = _assembly(tmp_path, ["rows_final_kernel<false, false, false>(RowsFinalArgs)", "rows_final_scalar_kernel<false>(RowsFinalArgs, ScalarTab)"])
    scalar = {("scalar" if "scalar" in k else "plain"): _count(v, r"\s+global_load_dwordx2 v\S+ v\d+, s\[") for k, v in code.items()}
    assert scalar["plain"] - scalar["scalar"] >= 32, scalar  # 16 each for p < 2^50 and p < 2^51
