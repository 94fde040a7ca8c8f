"""Host-only check of the built library's own code: the 256 x 256 tiles write their MFMAs as asm, around which the compiler puts no wait
states.  Every path to an MFMA has to leave two of them behind a vector instruction that writes one of its operands, and every path from
an MFMA to an instruction that reads or writes its result nineteen (a 16-pass MFMA's, the longest there is); no kernel may use scratch."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2509_14279_amd import build as b

BIN = "/opt/rocm/llvm/bin"
BEFORE, AFTER = 2, 19
REGISTERS = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")
LINE = re.compile(r"^\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):")
NO_RESULT = ("v_cmp", "v_readlane", "v_readfirstlane", "v_nop")      # (of vector registers)


def registers(text):
    return {(m[1], r) for m in REGISTERS.finditer(text) for r in range(int(m[2] or m[4]), int(m[3] or m[4]) + 1)}


class Instruction:
    def __init__(self, name, operands, address):
        self.name, self.address = name, address
        self.mfma = name.startswith("v_mfma")
        first, _, rest = operands.partition(",")
        self.all = registers(operands)
        self.first, self.rest = registers(first), registers(rest)
        self.valu_result = self.first if name.startswith("v_") and not self.mfma and not name.startswith(NO_RESULT) else set()
        self.states = int(operands, 0) + 1 if name == "s_nop" else 1
        self.target = None
        if "branch" in name:
            offset = int(operands.split()[0])
            self.target = address + 4 + 4 * (offset - 65536 if offset >= 32768 else offset)
        self.falls_through = name not in ("s_branch", "s_endpgm", "s_setpc_b64")


def kernels(listing):
    """name -> instructions, of a disassembled code object"""
    out, body = {}, None
    for line in listing.splitlines():
        head = re.match(r"^[0-9a-f]{16} <(.+)>:$", line)
        if head:
            body = out.setdefault(head[1], [])
        elif body is not None:
            m = LINE.match(line)
            if m:
                body.append(Instruction(m[1], m[2], int(m[3], 16)))
    return out


def violations(body):
    at = {i.address: n for n, i in enumerate(body)}
    behind = [[n - 1] if n and body[n - 1].falls_through else [] for n in range(len(body))]
    for n, i in enumerate(body):
        if i.target is not None:
            behind[at[i.target]].append(n)

    def hit(n, states, bad):
        """whether fewer than `states` wait states lie between instruction n and one before it that is `bad`"""
        stack, seen = [(p, states) for p in behind[n]], {}
        while stack:
            p, left = stack.pop()
            if left <= 0 or seen.get(p, 0) >= left:
                continue
            seen[p] = left
            if bad(body[p]):
                return True
            stack += [(q, left - body[p].states) for q in behind[p]]
        return False

    found = []
    for n, i in enumerate(body):
        if i.mfma:
            if hit(n, BEFORE, lambda p: p.valu_result & i.rest):
                found.append((i.name, hex(i.address), "operand just written"))
            # (an accumulator passed on whole is forwarded; any other use of a result by an MFMA would need waits)
            if hit(n, AFTER, lambda p: p.mfma and p.first & i.all and p.first != i.first):
                found.append((i.name, hex(i.address), "another MFMA's result"))
        elif any(k == "a" for k, _ in i.all):
            if hit(n, AFTER, lambda p: p.mfma and p.first & i.all):
                found.append((i.name, hex(i.address), "result in the making"))
    return found


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    obj = os.path.join(b.OBJ, "gemm_bf16.o")
    if not os.path.exists(obj) or not os.path.exists(os.path.join(BIN, "llvm-objdump")):
        pytest.skip("the library was not built here")
    d = tmp_path_factory.mktemp("code")
    shutil.copy(obj, d / "o")
    subprocess.run([os.path.join(BIN, "llvm-objdump"), "--offloading", "o"], cwd=d, check=True, capture_output=True)
    part = next(f for f in os.listdir(d) if "gfx950" in f)
    text = subprocess.run([os.path.join(BIN, "llvm-objdump"), "-d", part], cwd=d, check=True, capture_output=True, text=True).stdout
    notes = subprocess.run([os.path.join(BIN, "llvm-readelf"), "--notes", part], cwd=d, check=True, capture_output=True, text=True).stdout
    return kernels(text), notes


def test_no_scratch(code):
    sizes = re.findall(r"\.private_segment_fixed_size:\s*(\d+)", code[1])
    assert len(sizes) >= 20 and set(sizes) == {"0"}


def test_wait_states(code):
    tiles = {k: v for k, v in code[0].items() if any(i.mfma for i in v)}
    assert len(tiles) >= 20 and all("gemm_bf16" in k for k in tiles)
    for name, body in tiles.items():
        assert sum(i.mfma for i in body) >= 64 * 2
        assert violations(body) == [], name


# planted in the listing: a move in front of an MFMA, a read behind one, one behind a loop's end
@pytest.mark.parametrize("lines,bad", [
    (["v_mov_b32_e32 v4, v9", "v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]"], True),
    (["v_mov_b32_e32 v4, v9", "s_nop 1", "v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]"], False),
    (["v_accvgpr_write_b32 a2, v9", "v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]"], True),
    (["v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]", "s_nop 15", "v_accvgpr_read_b32 v1, a3"], True),
    (["v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]", "s_nop 15", "s_nop 2", "v_accvgpr_read_b32 v1, a3"], False),
    (["v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]", "v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]"], False),
    (["v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]", "v_mfma_f32_16x16x32_bf16 a[4:7], v[4:7], v[8:11], a[2:5]"], True),
    (["v_accvgpr_read_b32 v1, a3", "s_nop 15", "s_nop 15", "v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]", "s_cbranch_scc1 65531"], True),
])
def test_the_check_sees(lines, bad):
    body = [Instruction(x.split()[0], x.partition(" ")[2], 4 * n) for n, x in enumerate(lines)]
    assert bool(violations(body)) == bad
