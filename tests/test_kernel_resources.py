"""What the compiler made of kernels whose time is a chain of memory round trips: scratch memory would lengthen it."""
import re
import subprocess

from paper_2605_14513_amd import build as hb


def scratch_of(source):
    """Bytes of scratch a lane of every kernel of a source file."""
    flags = [f for f in hb.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    asm = subprocess.run(["/opt/rocm/bin/hipcc", *flags, "--offload-device-only", "-S", "-o", "-", f"{hb.CSRC}/{source}"],
                         stdout=subprocess.PIPE, stderr=subprocess.DEVNULL, check=True, text=True).stdout
    names = re.findall(r"^\s*\.amdhsa_kernel (\S+)", asm, re.M)
    sizes = re.findall(r"^\s*\.amdhsa_private_segment_fixed_size (\d+)", asm, re.M)
    assert names and len(names) == len(sizes)
    return dict(zip(names, map(int, sizes)))


def test_drift_kernels_use_no_scratch_memory():
    sizes = scratch_of("drift.hip")
    assert not any(sizes.values()), sizes


def test_band_error_kernels_use_no_scratch_memory():
    sizes = scratch_of("ebc.hip")
    assert not any(sizes.values()), sizes


def test_attention_kernels_use_no_scratch_memory():
    """But the merged shares at D = 128 (mode 4), which keep up to four registers there while they add up parts, behind the MFMA
    stream.  (Not for the time: a reload whose wait also waits for the loads in flight towards LDS would stall that stream.)"""
    sizes = {n: b for n, b in scratch_of("block_sparse_attn.hip").items() if b}
    assert all(re.search(r"attn_kernelILi128ELi(64|128)ELb[01]ELNS_8AttnModeE4E", n) and b <= 16 for n, b in sizes.items()), sizes
