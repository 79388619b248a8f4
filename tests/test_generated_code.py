"""What the compiler has to leave alone around the instruction of its own that loads operand tiles into LDS, checked in the
machine code of this build: wait states before the descriptor's scalar registers, M0, and no vector-memory operation
that the counted waits do not know of."""
import os
import re
import subprocess

import pytest

from paper_2309_03824_amd import build

OBJ = os.path.join(build.OBJ, "mfma_gemm2.hip.o")
LLVM = "/opt/rocm/llvm/bin/"
WAIT_STATES = 5      # between a vector instruction's write of a scalar register and a vector-memory read of it


def listing(tmp_path):
    """{kernel: [(address, mnemonic, operands, branch target)]}"""
    if not os.path.exists(OBJ):
        os.makedirs(build.OBJ, exist_ok=True)
        build._compile(os.path.join(build.CSRC, "mfma_gemm2.hip"))
    bundle, code = str(tmp_path / "bundle"), str(tmp_path / "code")
    subprocess.run([LLVM + "llvm-objcopy", "--dump-section", ".hip_fatbin=" + bundle, OBJ, str(tmp_path / "rest.o")], check=True)
    subprocess.run([LLVM + "clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--input=" + bundle,
                    "--output=" + code], check=True)
    text = subprocess.run([LLVM + "llvm-objdump", "-d", "--mcpu=gfx950", code], check=True, capture_output=True, text=True).stdout
    return parse(text)


def parse(text):
    kernels, start, rows = {}, 0, None
    for line in text.splitlines():
        head = re.match(r"([0-9a-f]+) <(\w+)>:", line)
        if head:
            start, rows = int(head.group(1), 16), kernels.setdefault(head.group(2), [])
            continue
        m = re.match(r"\s+(\w+)\s*(.*?)\s*// ([0-9A-F]+):[0-9A-F ]+(?:<\w+(?:\+0x([0-9a-f]+))?>)?", line)
        if m and rows is not None:
            branch = "branch" in m.group(1)
            rows.append((int(m.group(3), 16), m.group(1), m.group(2), start + int(m.group(4) or "0", 16) if branch else None))
    return kernels


def scalar_registers(text):
    regs = set()
    for a, b, c in re.findall(r"\bs(?:\[(\d+):(\d+)\]|(\d+))", text):
        regs |= {int(c)} if c else set(range(int(a), int(b) + 1))
    return regs


def faults(rows):
    """Addresses of the LDS loads whose descriptor a vector instruction may have written too few states before."""
    at = {r[0]: i for i, r in enumerate(rows)}
    before = [[] for _ in rows]
    for i, (_, op, _, target) in enumerate(rows):
        if i + 1 < len(rows) and op not in ("s_branch", "s_endpgm", "s_setpc_b64"):
            before[i + 1].append(i)
        if target is not None:
            before[at[target]].append(i)
    bad = []
    for i, (addr, op, args, _) in enumerate(rows):
        if not (op.startswith("buffer_load") and args.endswith(" lds")):
            continue
        desc, todo, seen = scalar_registers(args), [(p, 0) for p in before[i]], {}
        while todo:
            j, states = todo.pop()
            if states >= WAIT_STATES or seen.get(j, WAIT_STATES) <= states:
                continue
            seen[j] = states
            _, op_j, args_j, _ = rows[j]
            # (a carry or scale result stands second)
            results = args_j.split(",")[:2 if re.search("_co_|div_scale|mad_[ui]64", op_j) else 1]
            if op_j.startswith("v_") and scalar_registers(",".join(results)) & desc:
                bad.append(addr)
                break
            todo += [(p, states + 1 + (int(args_j, 0) if op_j == "s_nop" else 0)) for p in before[j]]
    return bad


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    return listing(tmp_path_factory.mktemp("code"))


def test_descriptors_are_settled_before_the_loads_that_use_them(kernels):
    loads = sum(op.startswith("buffer_load") and args.endswith(" lds") for rows in kernels.values() for _, op, args, _ in rows)
    assert loads > 1000
    assert not {k: [hex(a) for a in faults(rows)] for k, rows in kernels.items() if faults(rows)}


def m0_writes(kernels):
    """The loads that M0 is written for; nothing else touches it."""
    writes = 0
    for k, rows in kernels.items():
        for i, (_, op, args, _) in enumerate(rows):
            if re.search(r"\bm0\b", args):
                assert op == "s_mov_b32" and args.startswith("m0, s"), (k, op, args)
                assert rows[i + 1][1] == "s_nop" and rows[i + 2][2].endswith(" lds"), (k, rows[i:i + 3])
                writes += 1
    return writes


def test_m0_belongs_to_the_loads(kernels):
    assert m0_writes(kernels) > 1000


def test_nothing_is_spilled(kernels):
    # (a spill's store or reload would count among "all but the newest n" loads)
    assert not [k for k, rows in kernels.items() if any(op.startswith("scratch_") for _, op, _, _ in rows)]


def test_the_scan_sees_a_late_write():
    def code(*lines):
        text = "0000000000001000 <k>:\n" + "".join(f"\t{l} // {0x1000 + 4 * i:012X}: BF800000\n" for i, l in enumerate(lines))
        return parse(text)["k"]

    load = "buffer_load_dwordx4 v1, s[4:7], 0 offen lds"
    assert faults(code("v_readfirstlane_b32 s5, v0", "s_mov_b32 m0, s9", "s_nop 0", load))
    assert faults(code("v_cmp_gt_u32_e64 s[6:7], v0, v2", "s_nop 3", load))
    assert not faults(code("v_readfirstlane_b32 s5, v0", "s_nop 4", load))
    assert not faults(code("v_readfirstlane_b32 s8, v0", load))
    # round a loop: the write stands behind the load, before the branch back to it
    loop = code("s_nop 7", load, "v_readlane_b32 s4, v0, 1", "s_branch 0")
    loop[3] = loop[3][:3] + (0x1004,)
    assert faults(loop)
