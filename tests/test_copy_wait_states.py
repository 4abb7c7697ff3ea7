"""The direct copies to LDS are inline assembly, in front of which the compiler
inserts no wait states: a copy must come at least five of them after a vector
instruction (v_readlane, v_readfirstlane) that wrote a register of its
descriptor, and its descriptor must be in scalar registers at all.  Read from
the built kernels' own code."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BUILD = os.path.join(ROOT, "paper_2409_02227_amd", "_build")
LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
COPY = re.compile(r"buffer_load_dwordx4 v\d+, ([sv])\[(\d+):(\d+)\], 0 offen lds")
WRITE = re.compile(r"(?:v_readlane_b32|v_readfirstlane_b32) s(\d+),")


@pytest.mark.parametrize("unit", ["kernels_d_bf16", "kernels_bf16", "kernels_d_fp8", "kernels_fp8",
                                  "kernels_joint_bf16", "kernels_joint_fp8", "kernels_f32", "kernels_joint_f32"])
def test_wait_states_before_copies(tmp_path, unit):
    obj = os.path.join(BUILD, unit + ".o")
    tools = [os.path.join(LLVM, t) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-objdump")]
    if not os.path.exists(obj) or not all(shutil.which(t) for t in tools):
        pytest.skip("no built kernel objects or LLVM tools")
    fat, dev = str(tmp_path / "fat"), str(tmp_path / "dev.o")
    subprocess.run([tools[0], f"--dump-section=.hip_fatbin={fat}", obj, os.devnull], check=True)
    subprocess.run([tools[1], "--unbundle", "--type=o", f"--input={fat}", f"--output={dev}",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
    text = subprocess.run([tools[2], "-d", "--no-show-raw-insn", dev], check=True, capture_output=True, text=True).stdout
    last, copies = [], 0
    for line in text.splitlines():
        ins = line.split("//")[0].strip()
        if not line.startswith(("\t", " ")) or not ins:
            continue
        m = COPY.match(ins)
        if m:
            copies += 1
            assert m.group(1) == "s", ins
            waits = 0
            for prev in reversed(last):
                if waits >= 5:
                    break
                w = WRITE.match(prev)
                assert not (w and int(m.group(2)) <= int(w.group(1)) <= int(m.group(3))), (unit, prev, ins, waits)
                nop = re.match(r"s_nop (\d+)", prev)
                waits += int(nop.group(1)) + 1 if nop else 1
        last = (last + [ins])[-8:]
    assert copies > 50
