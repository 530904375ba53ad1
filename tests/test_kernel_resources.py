"""Register budget of the compiled convolution kernels (host-side check, no GPU).

The LDS-patch kernel keeps 4..16 accumulator tiles, a weight ring and the patch
prefetch in registers at two or three waves per SIMD.  A change that pushes a
variant over its budget does not fail any numerical test -- the compiler spills
to scratch memory and the layer just gets several times slower -- so the spill
counts the compiler reports are pinned here.
"""
import functools
import os
import re
import subprocess
import tempfile

import pytest

from paper_1908_05033_amd import build as B

CSRC = os.path.join(os.path.dirname(B.__file__), "csrc")
MAX_SPILLED_VGPRS = 40            # whole kernel
MAX_SCRATCH_BYTES = 4 * MAX_SPILLED_VGPRS + 16     # per lane: an array in scratch memory is no spill to the compiler
MAX_SCRATCH_IN_MFMA_BLOCK = 48    # scratch instructions in a basic block that issues MFMAs


@functools.lru_cache(maxsize=None)
def _device_asm(src):
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, "k.s")
        flags = [f for f in B.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
        cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags + ["-S", "--cuda-device-only", "-o", out, src]
        proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        assert proc.returncode == 0, proc.stdout[-2000:]
        return open(out).read()


@pytest.mark.parametrize("source", ["conv_patch_c4r3.hip", "conv_patch_c4r1.hip", "conv_patch_c2r3.hip", "conv_patch_c2r1.hip",
                                    "conv_patch_c3r3.hip", "conv_patch_c3r1.hip",
                                    "conv_simple.hip", "conv_fc.hip", "conv_wq.hip", "quantize_act.hip",
                                    "conv_split.hip", "soft_quantize.hip"])
def test_kernels_stay_inside_their_register_budget(source):
    asm = _device_asm(os.path.join(CSRC, source))
    kernels = re.findall(r"\.name:\s+(\S+).*?\.vgpr_count:\s+(\d+).*?\.vgpr_spill_count:\s+(\d+)", asm, re.S)
    assert kernels, "no kernel metadata found in the device assembly"
    over = [(n, int(v), int(s)) for n, v, s in kernels if int(s) > MAX_SPILLED_VGPRS]
    assert not over, "kernels spilling more than %d registers: %s" % (MAX_SPILLED_VGPRS, over[:5])
    scratch = re.findall(r"\.name:\s+(\S+).*?\.private_segment_fixed_size:\s+(\d+)", asm, re.S)
    assert len(scratch) == len(kernels)
    over = [(n, int(b)) for n, b in scratch if int(b) > MAX_SCRATCH_BYTES]
    assert not over, "kernels with more than %d bytes of scratch a lane: %s" % (MAX_SCRATCH_BYTES, over[:5])
    # no variant may spill inside the blocks that feed the matrix cores
    hot = []
    for fn in re.split(r"\n(?=_Z\S+:)", asm):
        name = fn.split(":", 1)[0]
        for block in re.split(r"\n\.LBB\d+_\d+:", fn):
            ins = [l.split()[0] for l in block.splitlines() if l.startswith("\t") and not l.startswith("\t.")]
            if sum("mfma" in i for i in ins) >= 8:
                n_scratch = sum(i.startswith("scratch_") for i in ins)
                if n_scratch > MAX_SCRATCH_IN_MFMA_BLOCK:
                    hot.append((name, n_scratch))
    assert not hot, "scratch traffic inside MFMA blocks: %s" % hot[:5]


def test_split_k_workgroups_share_a_cu():
    """Eight waves per workgroup: two workgroups fit a CU (four waves per SIMD) up to 128 registers.
    Layers whose waves have one chunk each yield many short workgroups and need that; the variant
    that prefetches a next chunk (LONG) may take more."""
    asm = _device_asm(os.path.join(CSRC, "conv_fc.hip"))
    kernels = re.findall(r"\.name:\s+(\S+).*?\.vgpr_count:\s+(\d+)", asm, re.S)
    short = [(n, int(v)) for n, v in kernels if not re.search(r"conv_fc_kernelILi\dELb1E", n)]
    assert short and all(v <= 128 for _, v in short), short


def test_general_epilogue_leaves_the_waves_per_simd():
    """Kernels that form their results through the per-lane functions of conv_epilogue.h: four 2-bit workgroups of the
    split-K kernel, in the variant for many tiles, share a compute unit up to 64 registers (as many as its LDS allows), and the simple kernel
    runs five waves per SIMD up to 96."""
    asm = _device_asm(os.path.join(CSRC, "conv_fc.hip"))
    short = re.findall(r"\.name:\s+\S*conv_fc_kernelILi2ELb0ELi0E\S*.*?\.vgpr_count:\s+(\d+)", asm, re.S)
    assert len(short) == 1 and int(short[0]) <= 64, short
    asm = _device_asm(os.path.join(CSRC, "conv_simple.hip"))
    simple = re.findall(r"\.name:\s+\S*conv_simple_kernel\S*.*?\.vgpr_count:\s+(\d+)", asm, re.S)
    assert len(simple) == 3 and all(int(v) <= 96 for v in simple), simple


def test_few_tile_workgroups_share_a_cu():
    """Split-K kernel for few output tiles: two workgroups of eight waves share a CU up to 128 registers.  Its variants
    with the tap sums of l_a != 0 and with nine steps of 4 bits in flight may take twice as many."""
    asm = _device_asm(os.path.join(CSRC, "conv_split.hip"))
    kernels = re.findall(r"\.name:\s+\S*conv_split_kernelILi(\d)ELi(\d)ELi(\d)E\S*.*?\.vgpr_count:\s+(\d+)", asm, re.S)
    assert len(kernels) == 18
    over = [k for k in kernels if int(k[3]) > (256 if k[2] == "1" or k[:2] == ("4", "9") else 128)]
    assert not over, over


def test_small_tiles_of_strided_layers_run_three_waves_per_simd():
    """The 128x64 tile with eight fetch units per thread and more, one wave group: layers of one channel block run the
    variant of which three workgroups are resident per compute unit, up to 168 registers."""
    asm = _device_asm(os.path.join(CSRC, "conv_patch_c4r3.hip"))
    kernels = re.findall(r"\.name:\s+(\S*conv_patch_kernelILi4ELi3ELi4ELi1ELi1ELi2ELi(?:8|12)ELi3ELi3ELi1E\S*).*?\.vgpr_count:\s+(\d+)",
                         asm, re.S)
    assert len(kernels) == 8 and all(int(v) <= 168 for _, v in kernels), kernels


def test_two_backward_workgroups_share_a_cu():
    """The backward training quantizer's workgroups are 16 waves and large tensors launch two per compute unit:
    both are resident up to 64 registers."""
    asm = _device_asm(os.path.join(CSRC, "soft_quantize.hip"))
    kernels = re.findall(r"\.name:\s+(\S*soft_bwd\S*).*?\.vgpr_count:\s+(\d+)", asm, re.S)
    assert kernels and all(int(v) <= 64 for _, v in kernels), kernels


def test_1x1_stages_do_not_wait_for_the_next_weights():
    """FP4 variants of 1x1 layers with two wave groups: a stage ends with its barrier.  A wait for
    global memory behind it is one for the weights of the next stage, fetched a moment before."""
    asm = _device_asm(os.path.join(CSRC, "conv_patch_c2r1.hip"))
    seen, late = 0, []
    for m in re.finditer(r"\n(_Z\S*conv_patch_kernel(?:ILi2ELi1E)(?:Li\d+E){7}Li2EL\S+):", asm):
        body = asm[m.start():asm.index("s_endpgm", m.start())]
        for block in re.split(r"\n(?=\.LBB\d+_\d+:)", body):
            label = block.split(":")[0].strip()
            if "mfma" not in block or "s_barrier" not in block or not re.search(r"s_cbranch\S+ " + re.escape(label) + r"\b", block):
                continue
            seen += 1
            if "vmcnt" in block[block.rindex("s_barrier"):]:
                late.append(m.group(1))
    assert seen >= 16 and not late, (seen, late[:3])
