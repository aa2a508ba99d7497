"""What the hand-scheduled loads and matrix instructions of the grouped products rely on, looked up in the machine code that the library
holds: their waits are written by hand, and the compiler, which takes an inline assembly statement for complete where it ends,
is free to move registers around them.  Followed along every path of the control flow graph:

  base       no memory instruction uses a scalar register that the vector unit has written less than five wait states before
  acc        nothing but another MFMA touches the result of an MFMA before it is written
  in_flight  no register that a load has yet to write is read, written or moved before a wait that covers the load
  m0         every write to M0 (the LDS address of the direct loads) is used by such a load before the next write
  settled    between the last write of a direct load's scalar base by the vector unit and the load, the scalar unit writes the base

CPU only: it reads the library as built, and plants each mistake in a few lines of text to see that it is found."""
import functools
import os
import re
import struct
import subprocess

import pytest

from paper_2604_00785_amd import binding as B

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
MEMORY = ("global_", "buffer_", "scratch_", "flat_")


def _code_objects(path):
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        place = at + len(MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", data, place - 8)[0]):
            start, size, n = struct.unpack_from("<QQQ", data, place)
            if size and b"gfx950" in data[place + 24:place + 24 + n]:
                yield data[at + start:at + start + size]
            place += 24 + n
        at = data.find(MAGIC, at + 1)


def _parse(text):
    """{kernel: [(address, instruction)]} of a disassembly."""
    kernels, cur = {}, None
    for line in text.splitlines():
        m = re.match(r"[0-9a-f]+ <(\S+)>:", line)
        if m:
            cur = kernels.setdefault(m.group(1), [])
            continue
        m = re.match(r"\s+(\S.*?)\s*// ([0-9A-F]{12}):", line)
        if m and cur is not None:
            cur.append((int(m.group(2), 16), m.group(1)))
    return kernels


@functools.lru_cache(None)
def kernels():
    B.load()
    found = {}
    for i, obj in enumerate(_code_objects(B.LIB_PATH)):
        path = "/tmp/moe_code_%d_%d.o" % (os.getpid(), i)
        with open(path, "wb") as f:
            f.write(obj)
        out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", path], capture_output=True, text=True, check=True).stdout
        os.remove(path)
        found.update({n: Kernel(code) for n, code in _parse(out).items() if "grouped_gemm" in n})
    return found


def _registers(text, kind):
    regs = set()
    for m in re.finditer(r"(?<![a-z_0-9])%s\[(\d+):(\d+)\]|(?<![a-z_0-9])%s(\d+)\b" % (kind, kind), text):
        regs |= {int(m.group(3))} if m.group(3) else set(range(int(m.group(1)), int(m.group(2)) + 1))
    return frozenset(regs)


class Kernel:
    """One kernel's instructions with what the checks ask of each, and the paths between them."""

    def __init__(self, code):
        self.code = code
        self.text = [x for _, x in code]
        self.op = [x.split()[0] for x in self.text]
        self.first = [x.split(None, 1)[1].split(",")[0] if " " in x else "" for x in self.text]
        self.v, self.s, self.a = ([_registers(x, k) for x in self.text] for k in "vsa")
        self.s_out = [_registers(x, "s") for x in self.first]
        self.memory = [o.startswith(MEMORY) for o in self.op]
        index = {a: i for i, (a, _) in enumerate(code)}
        self.next = []
        for i, (a, x) in enumerate(code):
            m = re.match(r"(s_branch|s_cbranch_\w+) (\d+)", x)
            if self.op[i] == "s_endpgm":
                self.next.append(())
            elif m:
                off = int(m.group(2))
                to = index.get(a + 4 + 4 * (off - 65536 if off >= 32768 else off))
                self.next.append(tuple(j for j in ((to,) if m.group(1) == "s_branch" else (to, i + 1)) if j is not None and j < len(code)))
            else:
                self.next.append((i + 1,) if i + 1 < len(code) else ())
        # flags that the compiler keeps in a scalar pair (all ones or zero) to lead control flow past a block: a path that carries
        # their values does not take both arms of a branch, or none
        self.flags = {m.group(1) for x in self.text for m in [re.match(r"s_and(?:n2)?_b64 vcc, exec, (s\[\d+:\d+\])", x)] if m}

        self.joins = {j for i, to in enumerate(self.next) for j in to if to != (i + 1,)}

    def known_at(self, i):
        """The flags that instruction i's own straight stretch of code sets in front of it."""
        start = i
        while start > 0 and start not in self.joins:
            start -= 1
        known = ()
        for j in range(start, i):
            known = self.step(j, known)[1]
        return known

    def step(self, i, known):
        """Where control may go from instruction i, and the flags known there ({register pair or "vcc": all ones?} as sorted pairs)."""
        x, op = self.text[i], self.op[i]
        if op in ("s_cbranch_vccz", "s_cbranch_vccnz", "s_cbranch_execnz"):
            # (the lanes that a branch on exec looks at are all there unless exec has just been changed, at the end of a divergent loop)
            value = dict(known).get("vcc") if "vcc" in op else None if any("exec" in self.first[j] for j in range(max(i - 3, 0), i)) else True
            if value is not None and len(self.next[i]) == 2:
                return (self.next[i][0] if value == op.endswith("nz") else self.next[i][1],), known
            return self.next[i], known
        if not op.startswith(("s_", "v_cmp")) or op.startswith(("s_nop", "s_wait", "s_barrier", "s_cmp", "s_bitcmp")):
            if not (op.startswith("v_readlane") or op.startswith("v_readfirstlane")):
                return self.next[i], known
        k = dict(known)
        m = re.match(r"s_mov_b64 (s\[\d+:\d+\]|vcc), (0|-1)$", x)
        n = re.match(r"s_and(n2)?_b64 vcc, exec, (s\[\d+:\d+\])$", x)
        if m and (m.group(1) in self.flags or m.group(1) == "vcc"):
            k[m.group(1)] = m.group(2) == "-1"
        elif n:
            value = k.get(n.group(2))
            k.pop("vcc", None)
            if value is not None:
                k["vcc"] = value != bool(n.group(1))
        else:
            if "vcc" in self.first[i] or op.startswith("v_cmp") and "_e32" in op:
                k.pop("vcc", None)
            for f in list(k):
                if f != "vcc" and _registers(f, "s") & self.s_out[i]:
                    k.pop(f)
        return self.next[i], tuple(sorted(k.items()))


def _states(text):
    """Wait states that an instruction takes."""
    return 1 + int(text.split()[1], 0) if text.startswith("s_nop") else 1


def _vector_writes_scalar(k, i):
    op = k.op[i]
    return op.startswith(("v_readlane", "v_readfirstlane")) or op.startswith("v_cmp") and "_e64" in op


def _scalar_writes(k, i):
    op = k.op[i]
    return op.startswith("s_") and not op.startswith(("s_nop", "s_branch", "s_cbranch", "s_wait", "s_barrier", "s_cmp", "s_bitcmp", "s_endpgm"))


def base(k):
    bad = []
    for i in range(len(k.code)):
        if not _vector_writes_scalar(k, i):
            continue
        todo, seen = [(j, 0, k.s_out[i]) for j in k.next[i]], set()
        while todo:
            j, waited, regs = todo.pop()
            if waited >= 5 or not regs or (j, waited, regs) in seen:
                continue
            seen.add((j, waited, regs))
            if k.memory[j] and k.s[j] & regs:
                bad.append((hex(k.code[i][0]), k.text[i], hex(k.code[j][0]), k.text[j]))
                continue
            if _scalar_writes(k, j):
                regs = regs - k.s_out[j]
            todo += [(n, waited + _states(k.text[j]), regs) for n in k.next[j]]
    return bad


def acc(k):
    bad = []
    for i in range(len(k.code)):
        if not k.op[i].startswith("v_mfma"):
            continue
        regs = _registers(k.first[i], "a")
        todo, seen = [(j, 0) for j in k.next[i]], {}
        while todo:
            j, waited = todo.pop()
            if waited >= 18 or seen.get(j, 99) <= waited:
                continue
            seen[j] = waited
            if k.op[j].startswith("v_mfma"):
                waited += 4
            else:
                if k.a[j] & regs:
                    bad.append((hex(k.code[i][0]), k.text[i], hex(k.code[j][0]), k.text[j]))
                    continue
                waited += _states(k.text[j])
            todo += [(n, waited) for n in k.next[j]]
    return bad


def in_flight(k):
    waits = {}
    for i, x in enumerate(k.text):
        if x.startswith("s_waitcnt"):
            v, g = re.search(r"vmcnt\((\d+)\)", x), re.search(r"lgkmcnt\((\d+)\)", x)
            waits[i] = (int(v.group(1)) if v else None, int(g.group(1)) if g else None)
    bad = []
    for i in range(len(k.code)):
        vector = k.op[i].startswith("global_load_dword") or k.op[i].startswith("buffer_load")
        if not (vector or k.op[i].startswith(("ds_read", "ds_bpermute"))):
            continue
        regs = _registers(k.first[i], "v")
        # (place, younger requests of the same kind, flags known): requests complete in order
        to, known = k.step(i, k.known_at(i))
        todo, seen = [(j, 0, known) for j in to], {}
        while todo:
            j, younger, known = todo.pop()
            if seen.get((j, known), 99) <= younger:
                continue
            seen[j, known] = younger
            if j in waits:
                allowed = waits[j][0 if vector else 1]
                if allowed is not None and allowed <= younger:
                    continue
            elif k.op[j].startswith(("v_", "ds_")) or k.memory[j]:
                used = k.v[j]
                if not vector and k.op[j].startswith("ds_read"):      # LDS reads return in order: writing the same register again is fine
                    used = _registers(k.text[j].split(",", 1)[1], "v")
                if used & regs:
                    bad.append((hex(k.code[i][0]), k.text[i], hex(k.code[j][0]), k.text[j], younger))
                    break
            younger += k.memory[j] if vector else k.op[j].startswith("ds_")
            to, known = k.step(j, known)
            todo += [(n, min(younger, 64), known) for n in to]
    return bad


def m0(k):
    bad = []
    for i in range(len(k.code)):
        if k.first[i].strip() != "m0":
            continue
        to, known = k.step(i, k.known_at(i))
        todo, seen = [(j, known) for j in to], set()
        while todo:
            j, known = todo.pop()
            if (j, known) in seen or k.op[j].startswith("global_load_lds"):
                continue
            seen.add((j, known))
            if k.first[j].strip() == "m0" or k.op[j] == "s_endpgm":
                bad.append((hex(k.code[i][0]), k.text[i], hex(k.code[j][0]), k.text[j]))
                continue
            to, known = k.step(j, known)
            todo += [(n, known) for n in to]
    return bad


def settled(k):
    bad = []
    for i in range(len(k.code)):
        if not _vector_writes_scalar(k, i):
            continue
        todo, seen = [(j, k.s_out[i]) for j in k.next[i]], set()
        while todo:
            j, regs = todo.pop()
            if not regs or (j, regs) in seen:
                continue
            seen.add((j, regs))
            if k.op[j].startswith("global_load_lds") and k.s[j] & regs:
                bad.append((hex(k.code[i][0]), k.text[i], hex(k.code[j][0]), k.text[j]))
                continue
            if _scalar_writes(k, j) or _vector_writes_scalar(k, j):
                regs = regs - k.s_out[j]
            todo += [(n, regs) for n in k.next[j]]
    return bad


CHECKS = [base, acc, in_flight, m0, settled]


@pytest.mark.parametrize("check", CHECKS, ids=lambda c: c.__name__)
def test_grouped_products(check):
    assert len(kernels()) >= 12
    for name, k in kernels().items():
        assert any(o.startswith("v_mfma") for o in k.op) and any(o.startswith("global_load_lds") for o in k.op), name
        bad = check(k)
        assert not bad, (name, len(bad), bad[:4])


def _text(*lines):
    return "\n".join(["0000 <planted>:"] + ["\t%s // %012X:" % (x, 4 * i) for i, x in enumerate(lines)])


@pytest.mark.parametrize("check,wrong,right", [
    (base, ["v_readlane_b32 s4, v1, 3", "s_nop 3", "global_load_lds_dwordx4 v2, s[4:5] offset:16"],
     ["v_readlane_b32 s4, v1, 3", "s_nop 4", "global_load_lds_dwordx4 v2, s[4:5] offset:16"]),
    (base, ["v_readfirstlane_b32 s5, v1", "global_load_dword v3, v2, s[4:5]"],
     ["v_readfirstlane_b32 s5, v1", "s_mov_b64 s[4:5], s[4:5]", "global_load_dword v3, v2, s[4:5]"]),
    (acc, ["v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]", "s_nop 7", "v_accvgpr_read_b32 v9, a2"],
     ["v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]", "s_nop 15", "s_nop 3", "v_accvgpr_read_b32 v9, a2"]),
    (in_flight, ["global_load_dword v3, v2, s[4:5]", "global_load_lds_dwordx4 v8, s[6:7]", "s_waitcnt vmcnt(2)", "v_mov_b32_e32 v5, v3"],
     ["global_load_dword v3, v2, s[4:5]", "global_load_lds_dwordx4 v8, s[6:7]", "s_waitcnt vmcnt(1)", "v_mov_b32_e32 v5, v3"]),
    (in_flight, ["ds_read_b128 v[4:7], v1", "s_cbranch_vccz 1", "s_waitcnt lgkmcnt(0)", "v_mov_b32_e32 v9, v6"],
     ["ds_read_b128 v[4:7], v1", "s_mov_b64 vcc, -1", "s_cbranch_vccz 1", "s_waitcnt lgkmcnt(0)", "v_mov_b32_e32 v9, v6"]),
    (m0, ["s_mov_b32 m0, s3", "s_mov_b32 m0, s7", "global_load_lds_dwordx4 v8, s[6:7]"],
     ["s_mov_b32 m0, s3", "global_load_lds_dwordx4 v8, s[6:7]", "s_mov_b32 m0, s7", "global_load_lds_dwordx4 v8, s[6:7]"]),
    (settled, ["v_readlane_b32 s4, v1, 3"] + ["v_mov_b32_e32 v3, v4"] * 9 + ["global_load_lds_dwordx4 v2, s[4:5]"],
     ["v_readlane_b32 s4, v1, 3", "s_add_u32 s4, s4, s8", "global_load_lds_dwordx4 v2, s[4:5]"]),
], ids=lambda c: getattr(c, "__name__", ""))
def test_a_planted_mistake_is_found(check, wrong, right):
    assert check(Kernel(_parse(_text(*wrong, "s_endpgm"))["planted"]))
    assert not check(Kernel(_parse(_text(*right, "s_endpgm"))["planted"]))
