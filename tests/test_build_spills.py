"""What the built trace kernels spill to memory, from the metadata of the library's own gfx950 code.

A ray's state through an RK4 step is 29 doubles (Y, the accumulated and the stage's state and derivative, z): 232
bytes a lane that the pair loops of the kernels with 128 registers may push out.  The FP32 sums hold 40 floats of
compensated moments beside them, and the expansion's coordinates: 512 bytes.  The kernels of few rays have the registers to keep
everything."""
import os
import re
import subprocess

import pytest

from paper_1110_4894_amd import build as libbuild

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _scratch(tmp_path):
    """{kernel name: bytes of scratch per lane} of every gfx950 kernel in the library."""
    if not os.path.exists(libbuild.LIB):
        pytest.skip("librt.so is not built")
    fat = tmp_path / "fat"
    subprocess.run([libbuild.llvm_tool("llvm-objcopy"), "--dump-section=.hip_fatbin=" + str(fat), libbuild.LIB,
                    str(tmp_path / "copy")], check=True)
    data = fat.read_bytes()
    starts = [m.start() for m in re.finditer(MAGIC, data)]
    out = {}
    for i, at in enumerate(starts):
        one, co = tmp_path / ("fat%d" % i), tmp_path / ("co%d" % i)
        one.write_bytes(data[at:starts[i + 1] if i + 1 < len(starts) else len(data)])
        subprocess.run([libbuild.llvm_tool("clang-offload-bundler"), "--unbundle", "--type=o",
                        "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--input=" + str(one), "--output=" + str(co)],
                       check=True)
        notes = subprocess.run([libbuild.llvm_tool("llvm-readobj"), "--notes", str(co)], check=True,
                               capture_output=True, text=True).stdout
        for name, size in re.findall(r"\.name:\s+(\S*kernel\S*)\n(?:.*\n)*?\s*\.private_segment_fixed_size:\s+(\d+)", notes):
            out[name] = int(size)
    return out


def test_trace_kernels_spill_little(tmp_path):
    scratch = _scratch(tmp_path)
    fp64 = {k: v for k, v in scratch.items() if "trace_kernelILb1" in k}
    fp32 = {k: v for k, v in scratch.items() if "trace_kernelILb0" in k}
    few = {k: v for k, v in scratch.items() if "trace_few_kernel" in k}
    assert fp64 and fp32 and few
    assert max(fp64.values()) <= 232, fp64
    assert max(fp32.values()) <= 512, fp32
    assert max(few.values()) == 0, few
