"""Wait states behind matrix instructions in the built library: whatever way leads from an MFMA to the first other instruction that touches
its result (behind a loop, over a branch taken or not), at least as many instructions lie between as its passes ask for.  The compiler puts
them in; nothing in hardware waits.  The machine code is read here, so no GPU is needed."""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2304_11745_amd import build

OBJDUMP = next((p for p in (shutil.which("llvm-objdump"), "/opt/rocm/llvm/bin/llvm-objdump") if p and os.path.exists(p)), None)
# wait states before a vector instruction may read or overwrite the result: passes + 2, bf16 (8 passes) on gfx950 two more
NEEDED = {"v_mfma_f32_32x32x16_bf16": 12, "v_mfma_f32_32x32x2_f32": 18, "v_mfma_f32_16x16x4_f32": 10}
REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def registers(text):
    out = set()
    for kind, lo, hi, one in REG.findall(text):
        out.update((kind, i) for i in (range(int(lo), int(hi) + 1) if lo else [int(one)]))
    return out


def functions(listing):
    """{name: [(instruction, operands, index of the branch's target or None)]} of a disassembly."""
    out, code, at, name = {}, [], {}, None

    def close():
        if name is not None:
            out[name] = [(op, args, at.get(to)) for op, args, to in code]
    base = 0
    for line in listing.splitlines():
        head = re.match(r"^([0-9a-f]+) <(.+)>:$", line)
        if head:
            close()
            base, name, code, at = int(head.group(1), 16), head.group(2), [], {}
            continue
        ins = re.match(r"^\t(\S+) ?(.*?)\s*// ([0-9A-F]+):[^<]*(?:<(.+)>)?$", line)
        if not ins or name is None:
            continue
        op, args, addr, to = ins.groups()
        at[int(addr, 16)] = len(code)
        off = re.match(re.escape(name) + r"(?:\+0x([0-9a-f]+))?$", to) if to else None
        code.append((op, args, base + int(off.group(1) or "0", 16) if off else None))
    close()
    return out


def shortest(code, start, limit):
    """Fewest wait states between the MFMA at `start` and an instruction other than an MFMA that touches its result (or a call, which may);
    `limit` if there are as many on every way.  Every way that branches allow counts, also those that their conditions rule out."""
    result = registers(code[start][1].split(", ")[0])
    best, seen, todo = limit, {}, [(start + 1, 0)]
    while todo:
        i, waits = todo.pop()
        while i < len(code) and waits < best and waits < seen.get(i, limit):
            seen[i] = waits
            op, args, to = code[i]
            if op.startswith("v_mfma"):
                if registers(args.split(", ")[0]) & result:
                    break                              # the chain goes on; the next MFMA's own distance counts
            elif op.startswith(("s_swappc", "s_setpc")) or (not op.startswith("s_") and registers(args) & result):
                best = waits
                break
            if op == "s_endpgm":
                break
            waits += int(args, 0) + 1 if op == "s_nop" else 1
            if op.startswith(("s_cbranch", "s_branch")):
                assert to is not None, (op, args)
                if op == "s_branch":
                    i = to
                    continue
                todo.append((to, waits))
            i += 1
    return best


LOOP = """
0000000000001000 <k>:
	v_mfma_f32_32x32x16_bf16 a[0:15], v[20:23], v[24:27], a[0:15]// 000000001000: D3B78000 04023114
	s_cbranch_scc1 65533                                       // 000000001008: BF85FFFD <k>
	s_cbranch_scc0 2                                           // 00000000100C: BF840002 <k+0x18>
	s_nop 15                                                   // 000000001010: BF80000F
	v_accvgpr_read_b32 v1, a0                                  // 000000001014: D3D84001 18000100
	s_nop {0}                                                    // 000000001018: BF800008
	v_accvgpr_read_b32 v0, a15                                 // 00000000101C: D3D84000 1800010F
	s_endpgm                                                   // 000000001024: BF810000
"""


@pytest.mark.parametrize("nops,waits", [(8, 11), (9, 12), (0, 3), (15, 18)])
def test_the_distance_is_that_of_the_shortest_way(nops, waits):
    code = functions(LOOP.format(nops))["k"]
    assert len(code) == 8 and shortest(code, 0, 40) == waits


@pytest.mark.skipif(OBJDUMP is None, reason="llvm-objdump not found")
def test_results_of_matrix_instructions_are_waited_for(tmp_path):
    lib = shutil.copy(build.LIB, tmp_path)                        # the code objects are unpacked beside it
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, timeout=120)
    checked, kernels, short = 0, set(), []
    for obj in sorted(glob.glob(str(tmp_path / "*gfx950"))):
        listing = subprocess.run([OBJDUMP, "-d", obj], check=True, capture_output=True, text=True, timeout=120).stdout
        for name, code in functions(listing).items():
            for i, (op, _, _) in enumerate(code):
                if not op.startswith("v_mfma"):
                    continue
                assert op in NEEDED, f"{op} in {name}: how long its result takes is not in the table"
                checked += 1
                kernels.add(name)
                got = shortest(code, i, NEEDED[op])
                if got < NEEDED[op]:
                    short.append((name, i, op, got))
    assert not short, short[:10]
    for kernel in ("igemm_kernel", "igemm_dma_kernel", "slices_kernel", "rowgemm_kernel", "conv3_kernel", "attention_kernel", "expand_dw_kernel", "stem_kernel"):
        assert any(kernel in k for k in kernels), kernel
    assert checked > 1000
