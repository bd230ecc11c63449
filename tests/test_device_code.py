"""What the compiler made of the kernels, read from the built library's disassembly (no GPU).  Three things that no
source line shows and that have gone wrong, and one that the sources have to say:

* The result of a matrix instruction may be read by a vector instruction only some wait states later, and the hardware
  does not hold the reader back.  The compiler counts them, but not along every path where branches meet: the
  SwiGLU products of one row tile read an accumulator two instructions after its last product and lost what that
  product had added.
* A register parked in the accumulation registers must not be fetched back where no lane is active: behind the exit of
  a loop that masks lanes off, before the mask is restored, the copy does nothing.
* A kernel whose vector registers do not fit keeps some of them in memory.  The attention variants of eight wavefronts per
  workgroup, two of which have to fit a SIMD, did when a request fetched more ahead than was left for it.
* Inline assembly that sets m0 says so to the compiler."""
import os
import re
import shutil
import struct
import subprocess

import pytest

OBJDUMP = next((p for p in ("/opt/rocm/llvm/bin/llvm-objdump", shutil.which("llvm-objdump")) if p and os.path.exists(p)), None)
# An XDL product of four passes (16x16x32 bf16): passes + 3.
WAIT_STATES = 7


class Code:
    """One function: its instructions as (mnemonic, operands, index of the branch target or None)."""

    def __init__(self, name, lines):
        self.name, self.ins, at, targets = name, [], {}, []
        for line in lines:
            text, _, note = line.partition("//")
            parts = text.split(None, 1)
            addr = re.match(r"\s*([0-9A-Fa-f]+):", note)
            if not parts or not addr:
                continue
            at[int(addr.group(1), 16)] = len(self.ins)
            to = re.search(r"<[^>]*?(?:\+0x([0-9a-f]+))?>", note) if parts[0].startswith(("s_branch", "s_cbranch")) else None
            targets.append(int(to.group(1) or "0", 16) if to else None)
            self.ins.append((parts[0], [o.strip() for o in parts[1].split(",")] if len(parts) > 1 else []))
        base = min(at) if at else 0
        self.to = [None if t is None else at.get(base + t) for t in targets]


def _functions(text):
    for part in re.split(r"\n(?=[0-9a-f]{8,} <)", text):
        m = re.match(r"[0-9a-f]+ <([^>]+)>:", part)
        if m:
            yield Code(m.group(1), part.split("\n")[1:])


def _objects(tmp_path_factory):
    from paper_2411_00853_amd import build
    lib = build.build_library()
    data, out, at = open(lib, "rb").read(), [], 0
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        p = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + n] and size:
                out.append(data[at + off:at + off + size])
            p += 24 + n
        at += 24
    folder = tmp_path_factory.mktemp("code")
    for i, elf in enumerate(out):
        path = folder / ("%d.elf" % i)
        path.write_bytes(elf)
        yield str(path)


def _tool(name, *args):
    return subprocess.run([os.path.join(os.path.dirname(OBJDUMP), name), *args], capture_output=True, text=True, check=True).stdout


@pytest.fixture(scope="module")
def objects(tmp_path_factory):
    if OBJDUMP is None:
        pytest.skip("no llvm-objdump")
    return list(_objects(tmp_path_factory))


@pytest.fixture(scope="module")
def kernels(objects):
    return [k for o in objects for k in _functions(_tool("llvm-objdump", "-d", o)) if k.ins]


def _regs(operand):
    operand = operand.lstrip("-|")
    m = re.match(r"([va])\[(\d+):(\d+)\]", operand)
    if m:
        return {m.group(1) + str(i) for i in range(int(m.group(2)), int(m.group(3)) + 1)}
    m = re.match(r"([va]\d+)\b", operand)
    return {m.group(1)} if m else set()


def _vector(op):
    return op.startswith(("v_", "ds_", "global_", "buffer_", "scratch_", "flat_"))


def _is_store(op):
    return op.startswith(("ds_write", "global_store", "buffer_store", "scratch_store", "flat_store"))


def fewest_wait_states(code):
    """(wait states, product, reader) of the closest read of a product's result by another kind of vector
    instruction, over all paths; None if there is none within 24."""
    best = None
    for i, (op, a) in enumerate(code.ins):
        if not op.startswith("v_mfma"):
            continue
        seen, paths = {}, [(i + 1, 0, frozenset(_regs(a[0])))]
        while paths:
            j, waited, live = paths.pop()
            while j is not None and j < len(code.ins) and waited < 24 and live and seen.get(j, 99) > waited:
                seen[j] = waited
                o, b = code.ins[j]
                if o.startswith("v_mfma"):
                    live = live - _regs(b[0])
                elif _vector(o) and b:
                    read = set().union(*(_regs(x) for x in (b if _is_store(o) else b[1:])))
                    if read & live and (best is None or waited < best[0]):
                        best = (waited, "%s %s" % (op, ", ".join(a)), "%s %s" % (o, ", ".join(b)))
                    if not _is_store(o):
                        live = live - _regs(b[0])
                if o == "s_endpgm":
                    break
                waited += int(b[0], 0) + 1 if o == "s_nop" else 1
                if o == "s_branch":
                    j = code.to[j]
                    continue
                if o.startswith("s_cbranch") and code.to[j] is not None:
                    paths.append((code.to[j], waited, live))
                j += 1
    return best


def copies_without_lanes(code):
    """Copies to or from accumulation registers that a branch taken because no lane is active leads to, before the
    mask is restored."""
    mask = re.compile(r"s_\w+ exec,")
    text = ["%s %s" % (op, ", ".join(a)) for op, a in code.ins]
    found = []
    for n, (op, _) in enumerate(code.ins):
        if op != "s_cbranch_execz" or code.to[n] is None:
            continue
        if not any("saveexec" in t or mask.match(t) for t in text[max(0, n - 4):n]):
            continue
        for t in text[code.to[n]:]:
            if mask.match(t) or "saveexec" in t or t.startswith(("s_endpgm", "s_branch", "s_cbranch")):
                break
            if "accvgpr" in t:
                found.append(t)
    return found


def test_matrix_results_are_waited_for(kernels):
    users = [k for k in kernels if any(op.startswith("v_mfma") for op, _ in k.ins)]
    assert len(users) > 200     # attention and projection variants
    early = [(k.name, w) for k in users if (w := fewest_wait_states(k)) and w[0] < WAIT_STATES]
    assert not early


def test_no_register_is_fetched_back_without_lanes(kernels):
    assert [(k.name, c) for k in kernels if (c := copies_without_lanes(k))] == []


def test_no_kernel_keeps_vector_registers_in_memory(objects):
    found = [m for o in objects for m in re.findall(r"\.name:\s+(_Z\S+).*?\.vgpr_spill_count:\s+(\d+)",
                                                    _tool("llvm-readelf", "--notes", o), re.S)]
    assert len(found) > 300
    assert [(n, count) for n, count in found if count != "0"] == []


def undeclared_m0(text):
    """Inline assembly that writes m0 without naming it among the registers it changes."""
    found = []
    for asm in re.findall(r"\basm\s+volatile\s*\((.*?)\)\s*;", text, re.S):
        if re.search(r"\bs_\w+\s+m0\b", asm) and not re.search(r'"m0"', asm.rsplit(":", 1)[-1]):
            found.append(asm)
    return found


def test_assembly_names_m0_where_it_sets_it():
    # (nothing else in a kernel that fetches into LDS uses it today; a compiler that kept something there would lose it)
    from paper_2411_00853_amd import build
    sources = [os.path.join(build.CSRC, f) for f in sorted(os.listdir(build.CSRC))]
    assert sum("s_mov_b32 m0" in open(f).read() for f in sources) > 0
    assert [(f, a) for f in sources for a in undeclared_m0(open(f).read())] == []


def _listing(lines):
    return Code("f", ["%s // %012X: 00000000%s" % (l, 0x100 + 8 * i, "" if to is None else " <f+0x%x>" % (8 * to))
                      for i, (l, to) in enumerate(lines)])


def test_the_checks_find_what_they_look_for():
    mfma = ("v_mfma_f32_16x16x32_bf16 a[4:7], v[0:3], v[4:7], a[4:7]", None)
    read, nops, end = ("v_accvgpr_read_b32 v2, a5", None), ("s_nop 6", None), ("s_endpgm", None)
    assert fewest_wait_states(_listing([mfma, nops, read, end]))[0] == 7
    # the wait stands on the way through, not on the branch past it
    assert fewest_wait_states(_listing([mfma, ("s_cbranch_execnz 1", 3), nops, read, end]))[0] == 1
    assert fewest_wait_states(_listing([mfma, ("v_accvgpr_write_b32 a5, 0", None), read, end])) is None
    assert undeclared_m0('asm volatile("s_mov_b32 m0, %0" ::"s"(x) : "memory");')
    assert not undeclared_m0('asm volatile("s_mov_b32 m0, %0" ::"s"(x) : "memory", "m0");')
    save, skip = ("s_and_saveexec_b64 s[0:1], vcc", None), ("s_cbranch_execz 2", 3)
    restore, back = ("s_or_b64 exec, exec, s[0:1]", None), ("v_accvgpr_read_b32 v9, a1", None)
    assert copies_without_lanes(_listing([save, skip, nops, back, restore, end]))
    assert not copies_without_lanes(_listing([save, skip, nops, restore, back, end]))
