"""The attention kernels' entry table is written to LDS by some waves and read
by all: in the code as compiled, every kernel meets a barrier between its
first LDS write (the table) and its first LDS read.  Read from the assembly,
because a run shows a missing barrier only when the writing wave happens to be
late."""
import os
import re
import subprocess

import pytest

from paper_2606_10671_amd import build


def lds_ops(name):
    """{kernel: its LDS instructions and barriers, in order} of one source, as build() compiles it."""
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    src = os.path.join(build.PKG, "csrc", name)
    cmd = [build.HIPCC, *flags, "-I", os.path.join(build.ROOT, "include"), "--cuda-device-only", "-S", src, "-o", "-"]
    text = subprocess.run(cmd, capture_output=True, text=True, check=True, timeout=300).stdout
    kernels = re.findall(r"^\s*\.amdhsa_kernel (\S+)", text, re.M)
    return {k: re.findall(r"^\s+(ds_\w+|s_barrier|buffer_load\S* .* lds|global_load_lds\w*)",
                          text[text.index(f"\n{k}:"):text.index(".Lfunc_end", text.index(f"\n{k}:"))], re.M)
            for k in kernels}


@pytest.mark.parametrize("source,count", [("attend_bf16.hip", 4), ("attend_f32.hip", 4)])
def test_entry_table_is_read_behind_a_barrier(source, count):
    ops = {k: o for k, o in lds_ops(source).items() if any(x.startswith("ds_write") for x in o)}
    assert len(ops) == count, sorted(ops)
    for kernel, seq in ops.items():
        write = next(i for i, x in enumerate(seq) if x.startswith("ds_write"))
        read = next(i for i, x in enumerate(seq) if x.startswith("ds_read"))
        assert write < read, (kernel, seq[:8])
        assert "s_barrier" in seq[write:read], (kernel, seq[:8])
