"""The direct copies to LDS are inline assembly, in front of which the compiler
inserts no wait states: on every path to a copy, five of them lie between it
and a vector instruction that wrote a scalar register of its descriptor, and
one between it and a write of M0; and its descriptor must be in scalar
registers at all.  Rings of several stages count the copies in flight, so their
kernels may issue no other vector memory instruction in the loop: they use no
scratch memory.  Read from the built kernels' own code."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BUILD = os.path.join(ROOT, "paper_2409_02227_amd", "_build")
LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
COPY = re.compile(r"buffer_load_dwordx4 v\d+, ([sv])\[(\d+):(\d+)\], 0 offen lds")
LINE = re.compile(r"\s+(\S.*?)\s*// ([0-9A-F]{8,}):")
SCALAR = re.compile(r"s(?:(\d+)|\[(\d+):(\d+)\])$")


def scalar_range(operand):
    m = SCALAR.match(operand)
    return None if not m else (int(m.group(1)),) * 2 if m.group(1) else (int(m.group(2)), int(m.group(3)))


def vector_writes(ins):
    """Scalar registers that a vector instruction writes: its first operand, or
    the second of those that return a carry or a scale flag."""
    name, _, rest = ins.partition(" ")
    if not name.startswith("v_"):
        return []
    ops = [o.strip() for o in re.split(r",(?![^\[]*\])", rest)]
    dst = ops[:2] if "_co_" in name or "div_scale" in name else ops[:1]
    return [r for r in map(scalar_range, dst) if r]


def instructions(text):
    return [(int(m.group(2), 16), m.group(1)) for m in map(LINE.match, text.splitlines()) if m]


def predecessors(code):
    """Indices of the instructions that may run just before each one."""
    index = {addr: i for i, (addr, _) in enumerate(code)}
    pred = [[] for _ in code]
    for i, (addr, ins) in enumerate(code):
        if i + 1 < len(code) and not re.match(r"s_(branch|endpgm|setpc_b64)\b", ins):
            pred[i + 1].append(i)
        m = re.match(r"s_c?branch\w* (\d+)$", ins)
        if m:
            off = int(m.group(1))
            pred[index[addr + 4 + 4 * (off - 65536 if off >= 32768 else off)]].append(i)
        if ins.startswith("s_setpc_b64"):  # a far branch: s_getpc, s_add_u32 of the distance, s_addc, s_setpc
            regs = scalar_range(ins.split()[1])
            j = next(j for j in range(i, i - 8, -1) if code[j][1].startswith("s_getpc_b64 s[%d:%d]" % regs))
            lo = next(x for _, x in code[j + 1:i] if x.startswith("s_add_u32 s%d, s%d, 0x" % (regs[0], regs[0])))
            dist = int(lo.split()[-1], 16)
            pred[index[code[j + 1][0] + (dist - (1 << 32) if dist >= 1 << 31 else dist)]].append(i)
    return pred


def check_copies(text):
    """The copies of a listing; fails on one that comes too early after a write on any path."""
    code = instructions(text)
    pred = predecessors(code)
    copies = 0
    for i, (addr, ins) in enumerate(code):
        m = COPY.match(ins)
        if not m:
            continue
        copies += 1
        assert m.group(1) == "s", ins
        lo, hi = int(m.group(2)), int(m.group(3))
        seen, todo = set(), [(p, 0) for p in pred[i]]
        while todo:
            j, waits = todo.pop()
            if waits >= 5 or (j, waits) in seen:
                continue
            seen.add((j, waits))
            prev = code[j][1]
            for a, b in vector_writes(prev):
                assert b < lo or hi < a, (hex(addr), prev, ins, waits)
            assert waits >= 1 or not re.match(r"\w+ m0,", prev), (hex(addr), prev, ins)
            nop = re.match(r"s_nop (\d+)", prev)
            todo += [(p, waits + (int(nop.group(1)) + 1 if nop else 1)) for p in pred[j]]
    return copies


@pytest.mark.parametrize("unit", [f"kernels_{family}{dt}" for dt in ("bf16", "f16", "fp8", "f32")
                                  for family in ("d_", "", "joint_") if (family, dt) != ("d_", "f32")])
def test_wait_states_before_copies(tmp_path, unit):
    obj = os.path.join(BUILD, unit + ".o")
    tools = [os.path.join(LLVM, t) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-objdump", "llvm-readelf")]
    if not os.path.exists(obj) or not all(shutil.which(t) for t in tools):
        pytest.skip("no built kernel objects or LLVM tools")
    fat, dev = str(tmp_path / "fat"), str(tmp_path / "dev.o")
    subprocess.run([tools[0], f"--dump-section=.hip_fatbin={fat}", obj, os.devnull], check=True)
    subprocess.run([tools[1], "--unbundle", "--type=o", f"--input={fat}", f"--output={dev}",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
    text = subprocess.run([tools[2], "-d", "--no-show-raw-insn", dev], check=True, capture_output=True, text=True).stdout
    assert check_copies(text) > 50
    if unit.startswith(("kernels_d_", "kernels_joint_")):  # the others have two stages and wait for every copy
        notes = subprocess.run([tools[3], "--notes", dev], check=True, capture_output=True, text=True).stdout
        scratch = [int(x) for x in re.findall(r"\.private_segment_fixed_size:\s*(\d+)", notes)]
        assert len(scratch) > 0 and set(scratch) == {0}, (unit, scratch)


COPY_LINE = "buffer_load_dwordx4 v1, s[4:7], 0 offen lds"


def listing(*lines):
    return "\n".join("\t%s  // %08X: 00" % (ins, 4 * i) for i, ins in enumerate(lines))


@pytest.mark.parametrize("lines,ok", [
    (["v_readlane_b32 s4, v9, 1", "s_nop 3", COPY_LINE], False),
    (["v_readlane_b32 s4, v9, 1", "s_nop 4", COPY_LINE], True),
    (["v_cmp_lt_i32_e64 s[6:7], v1, v2", "s_nop 0", COPY_LINE], False),
    (["v_cmp_lt_i32_e64 s[8:9], v1, v2", "s_nop 0", COPY_LINE], True),
    (["v_add_co_u32_e64 v2, s[2:5], v1, v3", "s_nop 0", COPY_LINE], False),
    (["s_mov_b32 m0, s9", COPY_LINE], False),
    # a loop whose tail writes the descriptor of the copy at its head
    (["s_nop 4", "s_nop 0", COPY_LINE, "v_readlane_b32 s7, v9, 1", "s_cbranch_scc0 65532"], False),
    (["s_nop 4", "s_nop 0", COPY_LINE, "v_readlane_b32 s7, v9, 1", "s_nop 3", "s_cbranch_scc0 65531"], True),
])
def test_the_check_finds_early_copies(lines, ok):
    if ok:
        assert check_copies(listing(*lines)) == 1
    else:
        with pytest.raises(AssertionError):
            check_copies(listing(*lines))
