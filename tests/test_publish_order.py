"""A block's completion flag is set after its bytes are stored, to the compiler
too (no GPU needed): in the compiled decoder the wait for a wave's stores, which
is no memory operation, stands between two release fences wherever a flag is
stored after it."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FENCE = 'fence syncscope("workgroup") release'


def test_flags_are_stored_behind_fences(tmp_path):
    if not (os.path.exists(HIPCC) or shutil.which("hipcc")):
        pytest.skip("hipcc not available")
    from paper_2606_18900_amd.build import FLAGS
    out = tmp_path / "kernels.ll"
    subprocess.run([HIPCC] + [f for f in FLAGS if f not in ("-fPIC", "-Wall")] +
                   ["-x", "hip", "--cuda-device-only", "-S", "-emit-llvm",
                    os.path.join(ROOT, "paper_2606_18900_amd", "csrc", "kernels.hip"), "-o", str(out)],
                   check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    bodies = re.findall(r"^define amdgpu_kernel void @\S*k_decode.*?^}", out.read_text(), re.S | re.M)
    assert len(bodies) == 2                           # one archive, and up to four
    for body in bodies:
        ins = [l.strip() for l in body.splitlines()]
        flags = [i for i, l in enumerate(ins) if l.startswith("store atomic i32") and 'syncscope("agent")' in l]
        assert len(flags) == 2                        # by wave 0 alone, and after the workgroup's stores
        for i in flags:
            w = max(k for k in range(i) if re.search(r"s\.waitcnt\(i32 3952\)", ins[k]))     # vmcnt(0)
            assert ins[w - 1].startswith(FENCE) and ins[w + 1].startswith(FENCE), ins[w - 2:w + 3]
