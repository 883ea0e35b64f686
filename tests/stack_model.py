"""A host model of the pruned-stack recursion's machine code (split_stack.h): the
header's own macro text is preprocessed, assembled and disassembled, and its
instructions run on one wave of 64 lanes with every memory access checked.

Besides the values, the model keeps what a GPU would not report: loads that
have not been waited for (reading or overwriting their registers fails), masks
read by a vector instruction sooner than the hardware delivers them, the branch
condition VCCZ, which a write of vcc_lo alone leaves as it was, registers read
before anything wrote them, and the number of instructions."""
import os
import re
import subprocess

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_05179_amd", "csrc")
LLVM = "/opt/rocm/llvm/bin"
TOOLS = [os.path.join(LLVM, t) for t in ("clang", "llvm-mc", "llvm-objdump")]

ALL = (1 << 64) - 1
OPERANDS = {"m": "v0", "ov": "v1", "L": "v2", "vq": "v3", "va": "v4", "ta": "v5", "tb": "v6", "tc": "v7", "vQ": "v8",
            "vn": "v9", "row": "v10", "col": "v11", "tab": "s[0:1]", "n": "s2", "f0": "s3", "Q": "s4", "base": "s5",
            "baseh": "s6", "out": "s7", "outh": "s8", "step": "s9", "steph": "s10", "ab": "s[12:13]"}
TAB, AB, PERM, OUT = 0x1_0000_0000, 0x2_0000_0000, 0x3_0000_0000, 0x4_0000_0000  # where the model's buffers lie


class Fault(AssertionError):
    pass


def source(ring, src, out):
    """The asm text of one variant, operands and unique labels put in."""
    use = '#include "split_stack.h"\nMARK SPLIT_STACK_ASM(%d, SPLIT_STACK_START_%s, SPLIT_STACK_STEP_%s, SPLIT_STACK_COLD_%s, ' % (
        ring, src, src, src)
    use += "SPLIT_STACK_BEGIN_%s, SPLIT_STACK_PUT_%s, SPLIT_STACK_NEXT_%s) MARK\n" % (out, out, out)
    text = subprocess.run([TOOLS[0], "-E", "-P", "-xc++", "-I", os.path.join(ROOT, "tests", "sanitize", "host_hip"), "-I",
                           os.path.join(ROOT, "include"), "-I", CSRC, "-"],
                          input=use, capture_output=True, text=True, check=True).stdout
    body = text[text.index("MARK") + 4:text.rindex("MARK")]
    asm = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', body)).encode().decode("unicode_escape")
    asm = re.sub(r"%\[(\w+)\]", lambda m: OPERANDS[m.group(1)], asm)
    return asm.replace("%=", "0").replace("%%", "%")


def assemble(asm, tmp):
    """[(address, mnemonic, operands, branch target or None)] by address."""
    src, obj = os.path.join(tmp, "stack.s"), os.path.join(tmp, "stack.o")
    with open(src, "w") as f:
        f.write(".text\n" + asm + "\ns_endpgm\n")
    arch = ["--triple=amdgcn-amd-amdhsa", "--mcpu=gfx950"]
    subprocess.run([TOOLS[1], *arch, "--filetype=obj", "-o", obj, src], check=True, capture_output=True)
    out = subprocess.run([TOOLS[2], "-d", "--mcpu=gfx950", obj], check=True, capture_output=True, text=True).stdout
    code = []
    for line in out.splitlines():
        m = re.match(r"\s+(\w+)(?:\s+(.*?))?\s*// ([0-9A-F]+):((?: [0-9A-F]{8})+)", line)
        if not m:
            continue
        op, args, addr, words = m.group(1), m.group(2) or "", int(m.group(3), 16), m.group(4).split()
        target = None
        if op.startswith(("s_cbranch", "s_branch")):
            simm = int(words[0], 16) & 0xFFFF
            target = addr + 4 + 4 * (simm - 0x10000 if simm & 0x8000 else simm)
        code.append((addr, op, [a.strip() for a in args.split(",")] if args else [], target))
    return code


def _reg(a):
    """('v'|'s', first, count) of a register operand, else None."""
    if a in ("vcc", "vcc_lo", "vcc_hi", "exec"):
        return (a, 0, 1)
    m = re.match(r"([vs])\[(\d+):(\d+)\]$", a)
    if m:
        return m.group(1), int(m.group(2)), int(m.group(3)) - int(m.group(2)) + 1
    m = re.match(r"([vs])(\d+)$", a)
    return (m.group(1), int(m.group(2)), 1) if m else None


def _const(a):
    floats = {"2.0": 0x40000000, "-2.0": 0xC0000000}
    if a in floats:
        return floats[a]
    try:
        return int(a, 0) & 0xFFFFFFFF
    except ValueError:
        return None


class Wave:
    """One run.  lds: bytes; tab: int32 [entries, 2]; ab: int32 [n, 2]; perm:
    uint32 words; rows x lanes of the value table come back in `table`."""

    def __init__(self, code, lanes, lds=b"", tab=None, ab=None, perm=None, table=None):
        self.code, self.index = code, {c[0]: i for i, c in enumerate(code)}
        self.v = np.zeros((256, 64), np.uint32)
        self.vdef = np.zeros(256, bool)
        self.s = [None] * 104
        self.vcc, self.vccz, self.exec, self.scc = 0, True, (1 << lanes) - 1, 0
        self.lanes = np.array([bool(self.exec >> i & 1) for i in range(64)])
        self.lds, self.tab, self.ab, self.perm, self.table = np.frombuffer(lds, np.uint8), tab, ab, perm, table
        self.lgkm, self.vm = {}, {}  # registers in flight
        self.mask_at = {}  # scalar register -> step at which a vector instruction wrote it
        self.step = 0

    # -- registers
    def _landed(self, kind, i):
        if (kind, i) in self.lgkm or (kind, i) in self.vm:
            raise Fault("%s%d touched while a load into it is in flight" % (kind, i))

    def rs(self, a):
        r = _reg(a)
        if r is None:
            return _const(a)
        kind, i, n = r
        if kind == "vcc":
            return self.vcc
        if kind == "exec":
            return self.exec
        v = 0
        for k in range(n):
            self._landed("s", i + k)
            if self.s[i + k] is None:
                raise Fault("s%d read before it is written" % (i + k))
            v |= self.s[i + k] << (32 * k)
        return v

    def ws(self, a, val):
        kind, i, n = _reg(a)
        if kind == "vcc":
            self.vcc, self.vccz = val & ALL, (val & ALL) == 0
            return
        if kind == "vcc_lo":  # leaves VCCZ as it was
            self.vcc = (self.vcc & ~0xFFFFFFFF) | (val & 0xFFFFFFFF)
            return
        if kind == "exec":
            self.exec = val & ALL
            return
        for k in range(n):
            self._landed("s", i + k)
            self.s[i + k] = val >> (32 * k) & 0xFFFFFFFF
            self.mask_at.pop(i + k, None)

    def rv(self, a):
        r = _reg(a)
        if r is not None and r[0] == "v":
            self._landed("v", r[1])
            if not self.vdef[r[1]]:
                raise Fault("v%d read before it is written" % r[1])
            return self.v[r[1]].copy()
        val = self.rs(a)
        if val is None:
            raise Fault("operand " + a)
        if r is not None and r[0] == "s":
            self._mask_ready(r)
        return np.full(64, val & 0xFFFFFFFF, np.uint32)

    def _mask_ready(self, r):
        for k in range(r[2]):
            if self.step - self.mask_at.get(r[1] + k, -99) < 3:
                raise Fault("s%d read by a vector instruction %d after the one that wrote it" %
                            (r[1] + k, self.step - self.mask_at[r[1] + k]))

    def active(self):
        return np.array([bool(self.exec >> i & 1) for i in range(64)]) if self.exec != ALL else np.ones(64, bool)

    def wv(self, a, val):
        kind, i, n = _reg(a)
        assert kind == "v" and n == 1
        self._landed("v", i)
        act = self.active()
        self.v[i][act] = val.astype(np.uint32)[act]
        self.vdef[i] = True

    # -- memory
    def smem(self, addr):
        if addr % 4:
            raise Fault("scalar load at %#x" % addr)
        for base, words in ((TAB, self.tab), (AB, self.ab)):
            if words is not None and base <= addr < base + (1 << 30) or words is not None and base - 64 <= addr < base:
                k = (addr - base) // 4
                flat = words.reshape(-1)
                if not 0 <= k < flat.size:
                    raise Fault("scalar load of word %d of %d" % (k, flat.size))
                return int(flat[k]) & 0xFFFFFFFF
        raise Fault("scalar load at %#x" % addr)

    def lds_at(self, addr, size):
        act = self.active()
        a = addr.astype(np.int64)
        if act.any() and (a[act].min() < 0 or a[act].max() + size > self.lds.size or (a[act] % size).any()):
            raise Fault("LDS read outside the tile")
        out = np.zeros(64, np.uint32)
        view = self.lds if size == 1 else self.lds.view(np.int16)
        out[act] = view[a[act] // size].astype(np.int32).astype(np.uint32)
        return out

    def run(self, limit):
        pc = 0
        while True:
            addr, op, a, target = self.code[pc]
            pc += 1
            self.step += 1
            if self.step > limit:
                raise Fault("more than %d instructions" % limit)
            if op == "s_endpgm":
                if self.lgkm or self.vm:
                    raise Fault("loads in flight at the end")
                return
            jump = self.one(op, a)
            if jump:
                if target not in self.index:
                    raise Fault("branch to %#x" % target)
                pc = self.index[target]

    def one(self, op, a):
        i32 = lambda x: x.view(np.int32)  # noqa: E731
        op = re.sub(r"_e(32|64)$", "", op)
        if op in ("s_nop",):
            return False
        if op == "s_waitcnt":
            text = " ".join(a)
            if "lgkmcnt(0)" in text:
                self.lgkm.clear()
            if "vmcnt(0)" in text:
                self.vm.clear()
            return False
        # control
        if op == "s_branch":
            return True
        if op.startswith("s_cbranch_"):
            c = op[10:]
            return {"vccz": self.vccz, "vccnz": not self.vccz, "scc0": not self.scc, "scc1": bool(self.scc),
                    "execz": self.exec == 0, "execnz": self.exec != 0}[c]
        # scalar
        if op.startswith("s_load_dword"):
            n = int(op[len("s_load_dwordx"):] or 1) if op != "s_load_dword" else 1
            base, off = self.rs(a[1]), self.rs(a[2])
            _, i, _ = _reg(a[0])
            words = [self.smem(base + off + 4 * k) for k in range(n)]
            for k in range(n):
                self._landed("s", i + k)
                self.s[i + k] = words[k]
                self.lgkm[("s", i + k)] = True
            return False
        if op in ("s_mov_b32", "s_mov_b64", "s_movk_i32"):
            self.ws(a[0], self.rs(a[1]))
            return False
        if op.startswith("s_cmp_"):
            x, y = self.rs(a[0]), self.rs(a[1])
            self.scc = int(x == y if "_eq_" in op else x != y)
            return False
        if op == "s_or_b64" or op == "s_or_b32":
            r = self.rs("vcc" if a[1] == "vcc_lo" else a[1]) | self.rs(a[2])
            self.ws(a[0], r)
            self.scc = int(r != 0)
            return False
        if op in ("s_add_u32", "s_addc_u32", "s_sub_u32"):
            x, y = self.rs(a[1]), self.rs(a[2])
            r = x - y if op == "s_sub_u32" else x + y + (self.scc if op == "s_addc_u32" else 0)
            self.scc = int(r < 0 or r > 0xFFFFFFFF)
            self.ws(a[0], r & 0xFFFFFFFF)
            return False
        if op == "s_ashr_i32":
            x = self.rs(a[1])
            r = ((x - (1 << 32) if x >> 31 else x) >> (self.rs(a[2]) & 31)) & 0xFFFFFFFF
            self.ws(a[0], r)
            self.scc = int(r != 0)
            return False
        if op == "s_lshl_b32":
            r = self.rs(a[1]) << (self.rs(a[2]) & 31) & 0xFFFFFFFF
            self.ws(a[0], r)
            self.scc = int(r != 0)
            return False
        # vector
        m = re.match(r"v_cmp(x?)_(le|gt)_i32$", op)
        if m:
            x, y = i32(self.rv(a[1])), i32(self.rv(a[2]))
            bits = (x <= y if m.group(2) == "le" else x > y) & self.active()
            val = sum(1 << int(i) for i in np.flatnonzero(bits))
            self.ws(a[0], val)
            r = _reg(a[0])
            if r[0] == "s":
                for k in range(r[2]):
                    self.mask_at[r[1] + k] = self.step
            if m.group(1):
                self.exec = val
            return False
        if op == "v_cndmask_b32":
            r = _reg(a[3])
            if r[0] == "s":
                self._mask_ready(r)
            mask = self.rs(a[3])
            sel = np.array([bool(mask >> i & 1) for i in range(64)])
            self.wv(a[0], np.where(sel, self.rv(a[2]), self.rv(a[1])))
            return False
        if op in ("v_min_i32", "v_min3_i32"):
            r = i32(self.rv(a[1]))
            for x in a[2:]:
                r = np.minimum(r, i32(self.rv(x)))
            self.wv(a[0], r.view(np.uint32))
            return False
        if op == "v_mov_b32":
            self.wv(a[0], self.rv(a[1]))
            return False
        if op == "v_add_u32":
            self.wv(a[0], self.rv(a[1]) + self.rv(a[2]))
            return False
        if op == "v_and_b32":
            self.wv(a[0], self.rv(a[1]) & self.rv(a[2]))
            return False
        if op == "v_lshl_add_u32":
            self.wv(a[0], (self.rv(a[1]) << self.rv(a[2])) + self.rv(a[3]))
            return False
        if op == "v_dot4_u32_u8":
            x, y, r = self.rv(a[1]), self.rv(a[2]), self.rv(a[3])
            for k in range(4):
                r = r + (x >> np.uint32(8 * k) & np.uint32(255)) * (y >> np.uint32(8 * k) & np.uint32(255))
            self.wv(a[0], r)
            return False
        if op in ("ds_read_u8", "ds_read_i16"):
            self.wv(a[0], self.lds_at(self.rv(a[1].split()[0]), 1 if op.endswith("u8") else 2))
            self.lgkm[("v", _reg(a[0])[1])] = True
            return False
        if op == "global_load_dword":
            base = self.rs(a[2].split()[0])
            off = int(a[2].split("offset:")[1]) if "offset:" in a[2] else 0
            where = base + off + self.rv(a[1]).astype(np.int64) - PERM
            act = self.active()
            if (where[act] < 0).any() or (where[act] // 4 >= self.perm.size).any() or (where[act] % 4).any():
                raise Fault("load outside the tour-ordered copy")
            out = np.zeros(64, np.uint32)
            out[act] = self.perm[where[act] // 4]
            self.wv(a[0], out)
            self.vm[("v", _reg(a[0])[1])] = True
            return False
        if op == "global_store_dword":
            where = self.rs(a[2].split()[0]) + self.rv(a[0]).astype(np.int64) - OUT
            act = self.active()
            flat = self.table.reshape(-1)
            if (where[act] < 0).any() or (where[act] // 4 >= flat.size).any() or (where[act] % 4).any():
                raise Fault("store outside the value table")
            flat[where[act] // 4] = i32(self.rv(a[1]))[act]
            return False
        raise Fault("unknown instruction " + op)
