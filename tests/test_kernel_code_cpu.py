"""What the fused inner kernels that leave their partial results to the merge must not hold, read from the code objects built
here: a wavefront by itself meets nobody (no barrier), and no value is canonicalised in front of a maximum (NaN handling that
only the quantiser needs)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BUILT = os.path.join(ROOT, "paper_2602_23200_amd", "_build", "attention_inner.o")
LLVM = "/opt/rocm/llvm/bin"


def test_merge_keeping_kernels_carry_no_work_group_code(tmp_path):
    tools = [shutil.which(t, path=LLVM) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-objdump")]
    if not all(tools) or not os.path.exists(BUILT):
        pytest.skip("no object file built here, or no ROCm binutils")
    fat, code = str(tmp_path / "fat"), str(tmp_path / "code")
    subprocess.run([tools[0], "--dump-section", f".hip_fatbin={fat}", BUILT], check=True)
    subprocess.run([tools[1], "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={fat}", f"--output={code}", "--unbundle"],
                   check=True)
    listing = subprocess.run([tools[2], "-d", "--no-show-raw-insn", code], check=True, stdout=subprocess.PIPE, text=True).stdout
    name, alone, canonical = None, {}, {}
    for line in listing.splitlines():
        head = re.match(r"^[0-9a-f]+ <(.*)>:", line)
        if head:
            name = head.group(1) if "attention_inner_kernel" in head.group(1) else None
            one = name and re.search(r"Lb1EEEv", name)           # (the last template argument: one wavefront a work-group)
            if one:
                alone[name] = 0
            if name:
                canonical[name] = 0
        elif name:
            if name in alone and "s_barrier" in line:
                alone[name] += 1
            if re.search(r"v_(pk_)?max(_num)?_f(16|32)(_e32|_e64)? v\d+, (v\d+), \5\b", line):
                canonical[name] += 1
    assert len(alone) >= 24 and len(canonical) > len(alone)
    assert not any(alone.values()), {k: v for k, v in alone.items() if v}
    assert not any(canonical.values()), {k: v for k, v in canonical.items() if v}
