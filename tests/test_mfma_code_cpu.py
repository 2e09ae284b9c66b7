"""The tiled GEMM's matrix instructions are assembly that the compiler does not know as such: it keeps no distance between them and
what it writes or reads around them.  What it made of them is read back from the built library and checked against the wait states
that the hardware asks for -- on every path through every kernel, so that a copy of an accumulator or of an operand that another
compiler puts next to one is found here."""
import re
import shutil
import struct
import subprocess

import pytest

from paper_2505_14468_amd.build import LIB_PATH

LLVM = "/opt/rocm/llvm/bin/"
FAR = 32  # wait states that are as good as any number
MFMA_TO_ACCESS = 10  # an MFMA of this file, then anything else that reads or writes its accumulator (bf16: 8)
VALU_TO_MFMA = 2  # a vector instruction's result, then an MFMA that reads it
M0_TO_LDS_LOAD = 1

pytestmark = pytest.mark.skipif(not shutil.which(LLVM + "llvm-objdump"), reason="no disassembler")


def code_objects(path, tmp):
    """The gfx950 code objects of the library's fat binaries."""
    fat = tmp / "fat"
    subprocess.run([LLVM + "llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", path, str(tmp / "copy")], check=True)
    data, magic, out = fat.read_bytes(), b"__CLANG_OFFLOAD_BUNDLE__", []
    at = data.find(magic)
    while at >= 0:
        n = struct.unpack_from("<Q", data, at + len(magic))[0]
        pos = at + len(magic) + 8
        for _ in range(n):
            off, size, tl = struct.unpack_from("<QQQ", data, pos)
            triple = data[pos + 24:pos + 24 + tl].decode()
            pos += 24 + tl
            if triple.endswith("gfx950"):
                out.append(data[at + off:at + off + size])
        at = data.find(magic, at + 1)
    return out


class Instr:
    """One instruction: mnemonic, what it reads and writes of the vector, accumulator and M0 registers, wait states it counts for."""

    def __init__(self, addr, text, target):
        self.addr, self.text, self.target = addr, text, target
        self.op = text.split()[0]
        ops = text[len(self.op):].split(",")
        self.mfma = self.op.startswith("v_mfma")
        self.valu = self.op.startswith("v_") and not self.mfma
        self.states = int(ops[0], 0) + 1 if self.op == "s_nop" else 1
        reg = lambda s: [(k, i) for k, a, b, c in re.findall(r"\b([av])(?:(\d+)|\[(\d+):(\d+)\])", s) for i in
                         (range(int(b), int(c) + 1) if b else [int(a)])]
        self.regs = {r for o in ops for r in reg(o)}
        self.dst = set(reg(ops[0])) if self.op.startswith("v_") else set()
        self.srcs = {r for o in ops[1:3] for r in reg(o)} if self.mfma else set()  # (A and B)
        self.writes_m0 = self.op.startswith("s_") and ops[0].strip() == "m0"
        self.names_m0 = re.search(r"\bm0\b", text) is not None
        self.lds_load = self.op.startswith("buffer_load") and re.search(r"\blds\b", text) is not None


def kernels(obj):
    text = subprocess.run([LLVM + "llvm-objdump", "-d", "--mcpu=gfx950", str(obj)], check=True, stdout=subprocess.PIPE, text=True).stdout
    for name, body in re.findall(r"^[0-9a-f]+ <(\S*gemm_tile_kernel\S*)>:\n(.*?)(?=^[0-9a-f]+ <|\Z)", text, re.S | re.M):
        code = []
        base = None
        for line in body.splitlines():
            m = re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+):", line)
            if not m or m[1].startswith("."):
                continue
            addr = int(m[2], 16)
            base = addr if base is None else base
            t = re.search(r"<\S+\+0x([0-9a-f]+)>", line) if "branch" in m[1] else None
            target = base + int(t[1], 16) if t else (base if "branch" in m[1] else None)
            code.append(Instr(addr, m[1], target))
        yield name, code


def before(code):
    """Index -> indexes of the instructions that can run right before it."""
    index = {x.addr: i for i, x in enumerate(code)}
    prev = [[] for _ in code]
    for i, x in enumerate(code):
        if x.target is not None:
            prev[index[x.target]].append(i)
        if i + 1 < len(code) and x.op not in ("s_branch", "s_endpgm", "s_setpc_b64"):
            prev[i + 1].append(i)
    return prev


def states_since(code, prev, hit):
    """For every instruction, the fewest wait states since one for which hit() is true, on any path (FAR: none, or that many)."""
    following = [[] for _ in code]
    for i, ps in enumerate(prev):
        for p in ps:
            following[p].append(i)
    since = [FAR] * len(code)
    work = list(range(len(code)))
    while work:
        i = work.pop()
        new = min([FAR] + [0 if hit(code[p]) else since[p] + code[p].states for p in prev[i]])
        if new < since[i]:
            since[i] = new
            work += following[i]
    return since


def writers(code, prev, i, states):
    """Instructions whose results an instruction could read with fewer than `states` wait states in between."""
    seen, work, out = set(), [(p, 0) for p in prev[i]], []
    while work:
        p, passed = work.pop()
        if passed >= states or (p, passed) in seen:
            continue
        seen.add((p, passed))
        out.append(code[p])
        work += [(q, passed + code[p].states) for q in prev[p]]
    return out


def faults(code):
    prev = before(code)
    since_mfma = states_since(code, prev, lambda x: x.mfma)
    out = []
    for i, x in enumerate(code):
        if not x.mfma and any(k == "a" for k, _ in x.regs) and since_mfma[i] < MFMA_TO_ACCESS:
            out.append(("accumulator touched next to an MFMA", x.text, since_mfma[i]))
        if x.mfma and any(w.valu and w.dst & x.regs for w in writers(code, prev, i, VALU_TO_MFMA)):
            out.append(("operand written next to its MFMA", x.text))
        if x.names_m0 and not (x.writes_m0 and x.op == "s_add_i32"):
            out.append(("M0 used for something else", x.text))
        if x.lds_load and any(w.writes_m0 for w in writers(code, prev, i, M0_TO_LDS_LOAD)):
            out.append(("M0 written right in front of a load", x.text))
        if x.op.startswith("scratch_"):
            out.append(("registers spilled", x.text))
    return out


@pytest.fixture(scope="module")
def tiled(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("code")
    found = {}
    for k, data in enumerate(code_objects(LIB_PATH, tmp)):
        if b"gemm_tile_kernel" in data:
            obj = tmp / f"object_{k}"
            obj.write_bytes(data)
            found.update(kernels(obj))
    return found


def test_wait_states_of_every_tiled_kernel(tiled):
    assert len(tiled) == 21  # eight tiles of both types, bf16 with three and fp32 with two that split K
    for name, code in tiled.items():
        assert sum(x.mfma for x in code) >= 40 and sum(x.lds_load for x in code) >= 6, name
        assert not faults(code), (name, faults(code)[:3])


PLAIN = ["v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]", "s_nop 9", "v_accvgpr_read_b32 v9, a2", "s_endpgm"]


@pytest.mark.parametrize("code,what", [
    (PLAIN, None),
    ([PLAIN[0], "s_nop 8", *PLAIN[2:]], "accumulator touched"),
    (["v_mov_b32_e32 v5, v8", *PLAIN], "operand written"),
    (["v_mov_b32_e32 v5, v8", "s_nop 0", *PLAIN], "operand written"),
    (["v_mov_b32_e32 v5, v8", "s_nop 1", *PLAIN], None),
    (["v_accvgpr_write_b32 a3, v8", "s_nop 0", *PLAIN], "operand written"),
    (["s_add_i32 m0, s0, 16", "buffer_load_dwordx4 v1, s[0:3], s4 offen lds", "s_endpgm"], "M0 written"),
    (["s_add_i32 m0, s0, 16", "s_nop 0", "buffer_load_dwordx4 v1, s[0:3], s4 offen lds", "s_endpgm"], None),
    (["s_mov_b32 m0, s1", "s_endpgm"], "M0 used"),
    (["scratch_store_dword off, v1, s2", "s_endpgm"], "registers spilled"),
    ([PLAIN[0], "s_cbranch_scc1 3", "s_nop 15", "s_endpgm", "v_accvgpr_read_b32 v9, a0", "s_endpgm"], "accumulator touched"),
])
def test_the_check_finds_what_it_looks_for(code, what):
    seq = [Instr(4 * i, t, 16 if "cbranch" in t else None) for i, t in enumerate(code)]
    got = faults(seq)
    assert (got == []) if what is None else any(what in f[0] for f in got), got
