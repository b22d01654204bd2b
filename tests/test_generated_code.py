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
