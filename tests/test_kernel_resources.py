"""The row sort runs at the register limit of a 1024-thread workgroup (128 VGPRs): a small change can push the
compiler over it, and the kernel then spills into scratch memory and runs several times slower without any test
failing.  This test compiles the clustering kernels for gfx950 (no GPU needed) and reads the compiler's
resource remarks."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def resource_remarks(source):
    from paper_2412_04180_amd import _build

    src = os.path.join(_build.CSRC, source)
    flags = [f for f in _build.HIPCC_FLAGS if f != "-shared"]
    cmd = [HIPCC] + flags + ["--cuda-device-only", "-c", "-Rpass-analysis=kernel-resource-usage", "-I",
                             os.path.join(ROOT, "include"), "-I", _build.CSRC, "-x", "hip", src, "-o", os.devnull]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-2000:]
    return r


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_sort_kernel_variants_for_rows_up_to_12288_keep_their_keys_in_registers():
    r = resource_remarks("skim_cluster.hip")
    found = 0
    for variant in ("sort_kernelILi8ELb1E", "sort_kernelILi12ELb1E", "sort_kernelILi8ELb0E", "sort_kernelILi12ELb0E"):
        m = re.search(r"Function Name: \S*" + variant + r".*?LDS Size", r.stdout, re.S)
        assert m, f"no resource remarks for {variant}"
        scratch = int(re.search(r"ScratchSize \[bytes/lane\]: (\d+)", m.group(0)).group(1))
        vgprs = int(re.search(r"VGPRs: (\d+)", m.group(0)).group(1))
        assert scratch == 0, f"{variant} spills {scratch} bytes per lane into scratch memory"
        assert vgprs <= 128
        found += 1
    assert found == 4
    # the iterations: at most three doubles a lane, parked around what only rare rows execute, and the wavefronts they are written for
    found = list(re.finditer(r"Function Name: \S*lloyd_iter_kernelILb[01]ELb([01])ELi([048])ELi[124]E.*?LDS Size", r.stdout, re.S))
    assert len(found) == 12
    for m in found:
        scratch = int(re.search(r"ScratchSize \[bytes/lane\]: (\d+)", m.group(0)).group(1))
        occupancy = int(re.search(r"Occupancy \[waves/SIMD\]: (\d+)", m.group(0)).group(1))
        assert scratch <= 24, m.group(0)[:120]
        assert occupancy == (4 if m.group(2) != "0" else 2 if m.group(1) == "1" else 3)


def scratch_inside_mfma_loops(source, kernel):
    """Scratch instructions between the first and the last MFMA of every instantiation of a kernel, by its mangled name."""
    from paper_2412_04180_amd import _build

    flags = [f for f in _build.HIPCC_FLAGS if f != "-shared"]
    r = subprocess.run([HIPCC] + flags + ["-Wno-inline-asm", "--cuda-device-only", "-S", "-I", os.path.join(ROOT, "include"), "-I", _build.CSRC,
                                          "-x", "hip", os.path.join(_build.CSRC, source), "-o", "-"],
                       stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    found = {}
    for m in re.finditer(r"^(\S*\d" + kernel + r"(?:I\S*)?E?Ev?P\S*):.*?s_endpgm", r.stdout, re.S | re.M):
        lines = m.group(0).splitlines()
        mfma = [i for i, line in enumerate(lines) if "v_mfma" in line]
        assert mfma, m.group(1)
        found[m.group(1)] = sum("scratch_" in line for line in lines[mfma[0]:mfma[-1]])
    return found


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_hessian_kernel_for_wide_layers_does_not_spill():
    """Two wavefronts per SIMD, 128 accumulator registers each: a reload from scratch memory inside the MFMA loop
    waits behind every tile load in flight (the memory counter is in-order).  All three ways of summing the chunks."""
    r = resource_remarks("skim_hessian.hip")
    found = list(re.finditer(r"Function Name: \S*xtx_big_kernel.*?LDS Size", r.stdout, re.S))
    assert len(found) == 3, "resource remarks for xtx_big_kernel"
    for m in found:
        scratch = int(re.search(r"ScratchSize \[bytes/lane\]: (\d+)", m.group(0)).group(1))
        occupancy = int(re.search(r"Occupancy \[waves/SIMD\]: (\d+)", m.group(0)).group(1))
        assert scratch == 0, f"xtx_big_kernel spills {scratch} bytes per lane into scratch memory"
        assert occupancy == 2


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_contraction_kernels_do_not_spill_in_their_stage_loops():
    """The same holds for the contraction with H.  The kernels around it: the gradient kernel keeps a row in registers, the row kernel
    is held to 64 of them where two of its workgroups share a compute unit (three for labels from bounds do not fit)."""
    r = resource_remarks("skim_loss.hip")
    for kernel, limit, count in (("grad_rows_kernel", 0, 3), ("row_prep_kernel", 12, 24), ("hmax_kernel", 0, 1)):
        found = list(re.finditer(r"Function Name: \S*\d" + kernel + r".*?LDS Size", r.stdout, re.S))
        assert len(found) == count, kernel
        for m in found:
            assert int(re.search(r"ScratchSize \[bytes/lane\]: (\d+)", m.group(0)).group(1)) <= limit, m.group(0)[:120]
    for kernel, limit in (("dwh_kernel", 0), ("dwh_loss_kernel", 0)):
        m = re.search(r"Function Name: \S*\d" + kernel + r".*?LDS Size", r.stdout, re.S)
        assert m, f"no resource remarks for {kernel}"
        assert int(re.search(r"ScratchSize \[bytes/lane\]: (\d+)", m.group(0)).group(1)) <= limit
        assert int(re.search(r"Occupancy \[waves/SIMD\]: (\d+)", m.group(0)).group(1)) == 2
        inside = scratch_inside_mfma_loops("skim_loss.hip", kernel)
        assert len(inside) == 1 and not any(inside.values()), inside
