"""Static check of the MFMA data hazards around hand-written (inline asm) matrix instructions.

The kernels issue their steady-state MFMAs as volatile asm statements, which the compiler's
hazard recogniser does not see as matrix instructions.  Two rules that it would otherwise
enforce with s_nop are therefore checked here on the generated gfx950 assembly:

  A. a vector-ALU write of a register must be at least 2 wait states old when an MFMA reads
     that register as one of its A/B/C operands;
  B. the result of an 8-pass MFMA (32x32x16 bf16) must be at least 11 wait states old when
     any instruction other than an MFMA touches it (16-pass 32x32x2 f32: 19).

The direct-to-LDS loads (asm as well) take their LDS target from M0, and several of them share
one M0 value set by an asm statement the compiler knows nothing about:

  C. in a function that contains such loads, no instruction outside the asm statements may
     write M0.

Wait states are counted like the compiler does: one per instruction, N+1 for `s_nop N`;
an intervening MFMA counts as its own pass count because it occupies the matrix pipe that
long.  Only hazards with an asm MFMA on one side are reported (compiler-emitted MFMAs are
already covered by the compiler).  The scan follows every path of a function, taken branches and
the back edges of loops among them: the steps of the pinned loops end with MFMAs whose results the
next trip's first vector instructions read.

The register counts of the kernels are read from the same listing (kernel_registers): two workgroups
of 256 threads share a compute unit where a kernel stays within 256.

Run as a module to check the library sources:  python -m paper_2409_04431_amd.isa_check
"""
import functools
import os
import re
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

from .build import CSRC, HIPCC_FLAGS, SOURCES

_REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+))")
_PASSES = {"v_mfma_f32_32x32x16_bf16": 8, "v_mfma_f32_32x32x2_f32": 16, "v_mfma_f32_32x32x2f32": 16}
_AFTER_MFMA = {8: 11, 16: 19}


def _regs(operand):
    """Set of ('v'|'a', index) named by one operand string."""
    out = set()
    for m in _REG.finditer(operand):
        kind = m.group(1)
        if m.group(4) is not None:
            out.add((kind, int(m.group(4))))
        else:
            out.update((kind, i) for i in range(int(m.group(2)), int(m.group(3)) + 1))
    return out


class Inst:
    __slots__ = ("op", "dst", "src", "in_asm", "text", "line", "succ")

    def __init__(self, text, in_asm, line):
        self.text, self.in_asm, self.line, self.succ = text, in_asm, line, ()
        parts = text.split(None, 1)
        self.op = parts[0]
        ops = [o.strip() for o in parts[1].split(",")] if len(parts) > 1 else []
        writes_first = self.op.startswith(("v_", "ds_read", "global_load", "buffer_load", "scratch_load")) \
            and not self.op.startswith(("v_cmp", "v_cmpx", "global_load_lds"))
        self.dst = _regs(ops[0]) if (ops and writes_first) else set()
        self.src = set()
        for o in (ops[1:] if writes_first else ops):
            self.src |= _regs(o)

    @property
    def is_mfma(self):
        return self.op.startswith("v_mfma")

    @property
    def is_valu(self):
        return self.op.startswith("v_") and not self.is_mfma

    def wait_states(self):
        if self.op == "s_nop":
            return int(self.text.split()[1], 0) + 1
        if self.is_mfma:
            return _PASSES.get(self.op, 4)
        return 1


def _link(insts, labels):
    """Set every instruction's successors (indices into `insts`)."""
    for i, ins in enumerate(insts):
        nxt = [i + 1] if i + 1 < len(insts) and ins.op not in ("s_branch", "s_endpgm") else []
        if ins.op == "s_branch" or ins.op.startswith("s_cbranch"):
            target = labels[ins.text.split()[1]]
            if target < len(insts):
                nxt.append(target)
        ins.succ = tuple(nxt)
    return insts


def parse_functions(asm_text):
    """Yield (name, [Inst]) for every function of an AMDGPU assembly listing."""
    name, insts, labels, in_asm, in_metadata = None, [], {}, False, False
    for ln, raw in enumerate(asm_text.splitlines(), 1):
        line = raw.strip()
        if line in (".amdgpu_metadata", ".end_amdgpu_metadata"):
            in_metadata = line == ".amdgpu_metadata"
        if in_metadata:
            continue
        if line.startswith(";;#ASMSTART"):
            in_asm = True
            continue
        if line.startswith(";;#ASMEND"):
            in_asm = False
            continue
        m = re.match(r"^([A-Za-z_.][\w$.]*):", line)
        if m:
            label = m.group(1)
            if label.startswith(".Lfunc_end") or not label.startswith(".L"):
                if name and insts:
                    yield name, _link(insts, labels)
                name, insts, labels = None if label.startswith(".L") else label, [], {}
            else:
                labels[label] = len(insts)
            continue
        if not line or line.startswith((";", ".", "//")):
            continue
        code = line.split(";")[0].strip()
        if code and name is not None:
            insts.append(Inst(code, in_asm, ln))
    if name and insts:
        yield name, _link(insts, labels)


def kernel_registers(asm_text):
    """{kernel: vector registers (both kinds) it takes}, from the descriptors of a listing."""
    return {m.group(1): int(m.group(2))
            for m in re.finditer(r"^\s*\.amdhsa_kernel (\S+)\n(?:.*\n)*?\s*\.amdhsa_next_free_vgpr (\d+)", asm_text, re.M)}


def _reach(insts, i, need):
    """(instruction, wait states since instruction i) for what runs on some path within `need` of them."""
    best, todo = {}, [(j, 0) for j in insts[i].succ]
    while todo:
        j, ws = todo.pop()
        if ws >= need or best.get(j, need) <= ws:
            continue
        best[j] = ws
        todo.extend((k, ws + insts[j].wait_states()) for k in insts[j].succ)
    return [(insts[j], ws) for j, ws in sorted(best.items())]


def check_function(insts):
    """Return a list of (rule, message) violations."""
    bad = []
    for i, ins in enumerate(insts):
        if ins.is_valu and ins.dst:
            for n, ws in _reach(insts, i, 2):
                if n.is_mfma and n.in_asm and (ins.dst & n.src):
                    bad.append(("A", f"line {ins.line}: '{ins.text}' feeds '{n.text}' (line {n.line}) after {ws} wait states"))
        elif ins.is_mfma and ins.in_asm:
            for n, ws in _reach(insts, i, _AFTER_MFMA[_PASSES.get(ins.op, 8)]):
                if not n.is_mfma and ((n.src | n.dst) & ins.dst):
                    bad.append(("B", f"line {n.line}: '{n.text}' touches the result of '{ins.text}' (line {ins.line}) after {ws} wait states"))
                    break
                if n.is_mfma and (n.dst & ins.dst) and n.dst != ins.dst:
                    bad.append(("B", f"line {n.line}: '{n.text}' partly overlaps the result of '{ins.text}' (line {ins.line})"))
                    break
    # Rule C
    if any(i.in_asm and i.op.startswith("global_load_lds") for i in insts):
        for ins in insts:
            if not ins.in_asm and re.match(r"^s_\w+\s+m0\b", ins.text):
                bad.append(("C", f"line {ins.line}: '{ins.text}' writes M0 outside the asm statements"))
    return bad


def check_text(asm_text):
    out = []
    for name, insts in parse_functions(asm_text):
        for rule, msg in check_function(insts):
            out.append(f"{name}: rule {rule}: {msg}")
    return out


@functools.lru_cache(maxsize=1)
def compile_to_asm(extra_flags=()):
    """Device-only assembly of the library sources with the product's flags."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = [f for f in HIPCC_FLAGS if f not in ("-fPIC", "-shared")]
    with tempfile.TemporaryDirectory() as td:
        def one(s):
            out = os.path.join(td, s + ".s")
            cmd = [hipcc] + flags + list(extra_flags) + ["--cuda-device-only", "-S", "-o", out, os.path.join(CSRC, s)]
            res = subprocess.run(cmd, capture_output=True, text=True)
            if res.returncode != 0:
                raise RuntimeError("hipcc failed:\n" + res.stderr)
            with open(out) as f:
                return f.read()
        with ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 1, 16)) as pool:
            texts = list(pool.map(one, SOURCES))
    return "\n".join(texts)


if __name__ == "__main__":
    problems = check_text(compile_to_asm())
    for p in problems:
        print(p)
    print(f"{len(problems)} hazard(s)")
    sys.exit(1 if problems else 0)
